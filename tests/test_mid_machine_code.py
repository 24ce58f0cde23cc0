"""What hipcc makes of the small-tile kernels that read token rows in whole lines (units), run lane by lane on the CPU: every
address lies in its buffer, the direct loads of a wave bring every token piece and weight fragment of its units once, in order
and to their slots, nothing is read from LDS before it has landed or requested again before it has been read, for waves with
every number of units and of fragments in the last one.  Tests of results cannot show these: a pointer that a compiler loses on
one path through the loop (it has happened) sends loads to addresses that a GPU answers with a fault."""
import os
import struct
import subprocess
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from paper_2603_08185_amd import build
from tests import _isa

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
FILES = ("gemm_mid.hip", "gemm_mid_mx.hip", "grouped_mid.hip")


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    """{mangled name: lines} of all small-tile kernels, {mangled name: resource figures}, what the compiler had to say"""
    tmp = tmp_path_factory.mktemp("asm")

    def one(f):
        out = str(tmp / (f + ".s"))
        said = subprocess.run([HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, f), "-o", out], check=True,
                              capture_output=True, text=True).stderr
        return open(out).read(), said

    lines, meta, said = {}, {}, ""
    with ThreadPoolExecutor(len(FILES)) as pool:
        for text, err in pool.map(one, FILES):
            lines.update(_isa.kernels(text))
            meta.update(_isa.metadata(text))
            said += err
    return lines, meta, said


def _named(table, part):
    found = [k for k in table if part in k]
    assert len(found) == 1, (part, found)
    return found[0]


# form, kernel, waves, fragments of a unit, stages of the ring, bytes of a stage and of a wave's region
FORMS = {
    "int8": ("int", "serq_mid_kernelILi8ELi2EE", 4, 2, 3, 6144, 18432),
    "mxfp4": ("mx", "serq_mx_mid_kernel", 4, 4, 2, 8192, 17408),
    "g128 int8, 4 waves": ("g128", "serq_g128_mid_kernelILi8ELb1ELi4E", 4, 2, 3, 6400, 19200),
    "g128 int8, 8 waves": ("g128", "serq_g128_mid_kernelILi8ELb1ELi8E", 8, 2, 3, 6400, 19200),
}


def _call(form, M, N, K, r, abits=8):
    """Kernel arguments, buffers and tiles of a layer call (MidParams, MxMidParams, G128Args + tiles)."""
    NB, KB, T, LF = N // 32, K // 64, (K // 64 + 3) // 4, (r + 63) // 64
    row = K // 2 if form == "mx" or abits == 4 else K
    size = {"Xq": M * row, "Wq": NB * KB * 1024}
    if form == "int":
        size.update(scale=4 * M, wscale=4 * N, Rp=N * r * 2, rscale=4 * N)
    elif form == "g128":
        size.update(scale=4 * M, zero=4 * M, gsc=N * K // 64, wsum=4 * N, Rp=N * r * 2)
    else:
        size.update(xsc=T * (M + M % 2) * 8, wsc=NB * T * 256, Rq=NB * LF * 1024, rsc=NB * ((LF + 3) // 4) * 256)
    buf, at = {}, 0x7F0000000000
    for k, n in size.items():                              # a megabyte and more between two of them
        buf[k] = (at, n)
        at += (n + (1 << 20) & -(1 << 20)) + (1 << 20)
    p = {k: v[0] for k, v in buf.items()}
    tm, tn = (M + 63) // 64, (N + 63) // 64
    if form == "int":
        arg = struct.pack("<QQQQQiiQiii4xQi4xqQqiii", p["Xq"], p["scale"], p["Wq"], p["wscale"], p["Rp"], 0, r, p["rscale"], M, N, K,
                          at, 1, N, 0, 0, tm, tn, tm)
    elif form == "g128":
        arg = struct.pack("<QQQQQQQiiiiiiQi4xqiii", p["Xq"], p["scale"], p["zero"], p["Wq"], p["gsc"], p["wsum"], p["Rp"], 0, 0, r, M, N, K,
                          at, 1, N, tm, tn, tm)
    else:
        arg = struct.pack("<QQQQQQiiiii4xQi4xqiii", p["Xq"], p["xsc"], p["Wq"], p["wsc"], p["Rq"], p["rsc"], 0, r, M, N, K,
                          at, 1, N, tm, tn, tm)
    return arg + bytes(16), buf, tm, tn


def _units(form, waves, FU, KB, w):
    """(first fragment, fragments) of the units of wave w: whole ones go round, the rest in pieces of half a unit if that is enough."""
    full, per = KB // (FU * waves), FU
    left = KB - full * FU * waves
    if form != "g128" and left <= FU // 2 * waves:
        per = FU // 2
    first = full * FU * waves + w * per
    out = [((w + waves * u) * FU, FU) for u in range(full)]
    return out + [(first, min(per, KB - first))] if first < KB else out


def _check(asm, name, M, N, K, r=32, start=None):
    """start: (n, instructions that a direct load may take on average among a wave's first n)"""
    form, kernel, waves, FU, NS, stage, region = FORMS[name]
    lines, meta, _ = asm
    kernel = _named(lines, kernel)
    prog = _isa.program(lines[kernel])
    arg, buf, tm, tn = _call(form, M, N, K, r)
    KB, row, per = K // 64, K // 2 if form == "mx" else K, 8 // FU
    lane = np.arange(64)
    for wg in sorted({0, tm * tn - 1}):                    # the first tile, and the last one: ragged rows, one channel block
        # (workgroups are dealt to eight XCDs, each with a run of tiles; tiles run along the tokens first)
        n, x = tm * tn, wg % 8
        tile = x * (n // 8) + min(x, n % 8) + wg // 8
        m0, nb0 = tile % tm * 64, tile // tm * 2
        nbt = min(2, N // 32 - nb0)
        for w in range(waves):
            where = (name, M, N, K, "workgroup", wg, "wave", w)
            try:
                wave = _isa.Wave(prog, arg, wg, w, buf, meta[kernel]["group_segment_fixed_size"])
                loads = wave.run()
            except _isa.Fault as e:
                raise AssertionError((*where, str(e))) from None
            # a wait that is not counted by hand empties the ring
            assert not loads or not any(loads[0].at < t < loads[-1].at for t in wave.own_waits), where
            assert start is None or loads[start[0] - 1].at - loads[0].at <= (start[0] - 1) * start[1], where
            codes = [ld for ld in loads if ld.buf in ("Xq", "Wq")]
            units = _units(form, waves, FU, KB, w)
            assert len(codes) == len(units) * 2 * (4 + FU), where
            scales = iter([ld for ld in loads if ld not in codes])
            it = iter(codes)
            for u, (f0, have) in enumerate(units):
                for h in range(2):
                    for k in range(4 + FU):
                        ld = next(it)
                        at = (*where, "unit", u, "half", h, "load", k)
                        assert ld.lds == w * region + (2 * u + h) % NS * stage + 1024 * k, at
                        assert ld.size == 16, at
                        if k < 4:
                            r_ = m0 + 32 * h + 8 * k + lane // 8
                            c = (lane % 8) ^ (4 * (k % 2) + lane // 16)
                            want = r_ * row + 16 * (f0 * per + c)
                            real = (r_ < M) & (c < have * per)   # (for any other piece all that is in bounds will do)
                            assert ld.buf == "Xq" and (ld.off[real].astype(np.int64) == want[real]).all(), at
                        else:
                            blk = nb0 + (h if nbt > 1 else 0)
                            want = (blk * KB + f0 + min(k - 4, have - 1)) * 1024 + 16 * lane
                            assert ld.buf == "Wq" and (ld.off.astype(np.int64) == want).all(), at
                    if form == "g128":                 # the 32 scales of the group and of this half's block
                        ld, blk = next(scales), nb0 + (h if nbt > 1 else 0)
                        assert ld.lds == w * region + (2 * u + h) % NS * stage + 6144 and ld.size == 4, (*where, u, h)
                        assert (ld.off.astype(np.int64) == (blk * (K // 128) + f0 // 2) * 64 + 4 * (lane % 16)).all(), (*where, u, h)
                    elif form == "mx" and h == 0:      # of the scale tile: 64 of each block, of two token rows a lane
                        ld, T, tile_ = next(scales), (KB + 3) // 4, f0 // 4
                        blk = nb0 + (lane // 16 if nbt > 1 else 0)
                        rows = np.minimum(lane % 32, (min(64, M - m0) - 1) // 2)
                        want = np.where(lane < 32, (blk * T + tile_) * 256 + lane % 16 * 16, (tile_ * (M + M % 2) + m0) * 8 + rows * 16)
                        assert ld.lds == w * region + NS * stage and ld.size == 16, (*where, u)
                        assert (ld.off.astype(np.int64) == want).all(), (*where, u)
            assert next(scales, None) is None, where


# 0 to 13 units per wave, both parities, and every number of fragments in a last one
@pytest.mark.parametrize("name", FORMS)
def test_loads(asm, name):
    form, _, waves, FU = FORMS[name][:4]
    step = 2 if form == "g128" else 1                      # fragments of 64 channels; whole groups of 128
    one = FU * waves                                       # fragments of a round of whole units
    frags = {step * n for n in range(1, one // step + 1)}                       # up to a round
    frags |= {one * u + left for u in (2, 3, 4, 6) for left in (0, step, one // 2, one // 2 + 1, one - 1) if left % step == 0}
    frags |= {one * u for u in (1, 5, 7, 8, 12, 13)}
    for n in sorted(frags):
        _check(asm, name, 109, 96, 64 * n)
    for left in (0, step, one - step):                     # a last tile of one row, and of nine
        _check(asm, name, 65, 64, 64 * (one + left))
        _check(asm, name, 73, 64, 64 * (one + left))


# the first loads of a wave, of whole units and of ones that lack fragments, pick no pieces and fragments lane by lane (picking
# takes 11 to 14 instructions a load)
@pytest.mark.parametrize("name", FORMS)
def test_start(asm, name):
    form, _, waves, FU = FORMS[name][:4]
    for u in (1, 2, 3, 4):
        _check(asm, name, 109, 96, 64 * FU * waves * u, start=(12, 10))
    if form != "g128":
        _check(asm, name, 109, 96, 64 * FU * waves // 2, start=(4 + FU, 10))    # (the first half of a unit)
        _check(asm, name, 109, 96, 64 * (FU * waves - 1), start=(4 + FU, 10))


# the kernels that read 4-bit tokens in steps: nothing out of bounds or out of turn, and every fragment is fetched
@pytest.mark.parametrize("form,kernel,waves", [("int", "serq_mid_kernelILi4ELi2EE", 4), ("g128", "serq_g128_mid_kernelILi4ELb1ELi4E", 4),
                                               ("g128", "serq_g128_mid_kernelILi4ELb1ELi8E", 8)])
def test_step_loads(asm, form, kernel, waves):
    lines, meta, _ = asm
    kernel = _named(lines, kernel)
    prog = _isa.program(lines[kernel])
    for KB in (1, 2, 3, 7, 8, 9, 16, 17, 31, 34, 63, 64, 86):
        if form == "g128" and KB % 2:
            continue
        M, N, K = 109, 96, 64 * KB
        arg, buf, tm, tn = _call(form, M, N, K, 32, 4)
        for wg in (0, tm * tn - 1):
            seen = set()
            for w in range(waves):
                for ld in _isa.Wave(prog, arg, wg, w, buf, meta[kernel]["group_segment_fixed_size"]).run():
                    if ld.buf == "Wq":
                        seen.add(int(ld.off[0]) // 1024)
            nb0 = 0 if wg == 0 else 2                  # (the last tile has one channel block)
            assert seen == set(range(nb0 * KB, min(nb0 + 2, N // 32) * KB)), (kernel, K, wg)


def test_registers_suffice(asm):
    for name, m in asm[1].items():
        assert m["private_segment_fixed_size"] == 0 and m["vgpr_spill_count"] == 0 and m["sgpr_spill_count"] == 0, (name, m)


def test_no_warnings(asm):
    assert "warning:" not in asm[2], asm[2]
