"""Tiled kernels: every count of main tiles around the ring's depth with every remainder, and more tiles, of different widths, than
compute units.  (A workgroup takes one tile.)"""
import numpy as np
import pytest
import torch

import workloads
from oracle import serq_oracle as orc
from paper_2603_08185_amd import binding as serq
from tests._util import DT, assert_y_close, f32, f64, oracle_pack

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _spec(abits, M, K, N, r, in_dtype="bf16", out_dtype="bf16"):
    return workloads.LayerSpec(f"tiles_a{abits}_M{M}_K{K}_N{N}_r{r}", 9, abits, M, K, N, r, in_dtype, out_dtype, 3, 20.0, 60.0)


def _int(spec, rform, coltiles=0):
    L = workloads.make_layer(spec)
    pk_o = oracle_pack("int", spec, L)
    pk = serq.pack_weights(L["W"].to(DEV), L["s"].to(DEV), 0)
    Xhat = workloads.permute_channels(L["X"], pk_o["perm"])
    Xq_o, sc_o = orc.quantize_act(f32(Xhat), pk_o["s_inv"], spec.abits)
    Xq, sc = serq.quantize_act(Xhat.to(DEV), pk.s_inv, spec.abits)
    fl = serq.flags(serq.PATH_MFMA, coltiles=coltiles)
    acc = serq.gemm_i32(Xq, spec.abits, pk.Wq, spec.M, spec.N, spec.K, flags_=fl)
    assert np.array_equal(acc.cpu().numpy(), orc.gemm_i32(Xq_o, pk_o["Wq"])), spec.name
    kw = dict(Rp=None, r=0)
    Y64 = orc.linear(Xq_o, sc_o, pk_o["Wq"], pk_o["wscale"], np.zeros((0, spec.N)))
    if spec.r and rform == "i4":
        kw = dict(Rp=serq.pack_lowrank_q4(L["R"].to(DEV)), r=spec.r, r_dtype=serq.I4)
        Rq, rs = orc.quantize_lowrank(f32(L["R"]))
        Y64 = orc.linear_q4r(Xq_o, sc_o, pk_o["Wq"], pk_o["wscale"], Rq, rs)
    elif spec.r:
        kw = dict(Rp=serq.pack_lowrank(L["R"].to(DEV)), r=spec.r, r_dtype=DT[spec.in_dtype])
        Y64 = orc.linear(Xq_o, sc_o, pk_o["Wq"], pk_o["wscale"], f64(L["R"]))
    # the output is a column slice of a wider buffer whose other columns and whose rows behind the last token must stay as they are
    big = torch.full((spec.M + 3, spec.N + 16), 7.0, dtype=DT[spec.out_dtype], device=DEV)
    Y = serq.linear(Xq, sc, spec.abits, pk.Wq, pk.wscale, spec.M, spec.N, spec.K, Y=big[:spec.M, 8:8 + spec.N], flags_=fl, **kw)
    assert_y_close(Y, Y64, spec.name)
    assert bool((big[spec.M:] == 7).all()) and bool((big[:, :8] == 7).all()) and bool((big[:, 8 + spec.N:] == 7).all())


def _mx(spec, coltiles=0):
    L = workloads.make_layer(spec)
    pk_o = oracle_pack("mx", spec, L)
    pk = serq.mx_pack_weights(L["W"].to(DEV), L["s"].to(DEV), spec.r)
    Xhat = workloads.permute_channels(L["X"], pk_o["perm"])
    Xc, Xe = orc.mx_quantize_act(f32(Xhat), pk_o["s_inv"])
    Xq, xsc = serq.mx_quantize_act(Xhat.to(DEV), pk.s_inv)
    Y64 = orc.mx_linear(Xc, Xe, pk_o["Wc"], pk_o["We"], pk_o.get("Rc"), pk_o.get("Re"))
    big = torch.full((spec.M + 3, spec.N + 16), 7.0, dtype=DT[spec.out_dtype], device=DEV)
    Y = serq.mx_linear(Xq, xsc, pk.Wq, pk.wsc, spec.M, spec.N, spec.K, Rq=pk.Rq, rsc=pk.rsc, r=spec.r,
                       Y=big[:spec.M, 8:8 + spec.N], flags_=serq.flags(serq.PATH_MFMA, coltiles=coltiles))
    assert_y_close(Y, Y64, spec.name)
    assert bool((big[spec.M:] == 7).all()) and bool((big[:, :8] == 7).all()) and bool((big[:, 8 + spec.N:] == 7).all())


# main tiles of 128 (W4A8) or 256 channels in rings of three or two: none whole to seven, with every remainder
@pytest.mark.parametrize("n", list(range(1, 15)) + [17, 20, 23, 24, 28, 31])
def test_tile_counts(n):
    K = 64 * n
    out_dtype = "bf16" if n % 3 else "fp32"
    for abits, r, rform in ((8, 0, ""), (8, 48, "bf16"), (4, 64, "i4"), (4, 16, "bf16"), (4, 0, "")):
        if r + 63 < K or r == 0 or (rform == "bf16" and r <= K):
            _int(_spec(abits, 260, K, 288, r, out_dtype=out_dtype), rform)
    for r in (0, 32, 96):
        if 64 * ((r + 63) // 64) <= K:
            _mx(_spec(4, 260, K, 288, r, out_dtype=out_dtype))


# 9 token tiles x 30, 41, 13 column tiles (30: of two blocks and of one; 41: one each; 13: four and three) on 256 compute units,
# and 17 x 41: workgroups in up to three rounds, the first tiles of a round beside the last ones of the round before
@pytest.mark.parametrize("out_dtype", ["bf16", "fp16", "fp32"])
@pytest.mark.parametrize("M,coltiles", [(2100, 30), (2049, 41), (2100, 13), (4200, 41)])
@pytest.mark.parametrize("K,r", [(64, 32), (320, 0), (576, 64), (1344, 128)])
def test_more_tiles_than_compute_units(M, coltiles, K, r, out_dtype):
    dt = "fp16" if out_dtype == "fp16" else "bf16"
    for abits, rform in ((8, dt), (4, "i4" if M == 2049 else dt)):
        rr = r if rform != "i4" or 64 * ((r + 63) // 64) <= K else 0
        _int(_spec(abits, M, K, 1312, rr, in_dtype=dt, out_dtype=out_dtype), rform, coltiles=coltiles)
    _mx(_spec(4, M, K, 1312, r if K > 64 else 0, in_dtype=dt, out_dtype=out_dtype), coltiles=coltiles)
