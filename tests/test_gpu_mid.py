"""The kernels for batches between decode and prefill (64 x 64 tiles, K shared by the waves of a workgroup), which AUTO takes
for these sizes: against the oracle, and against the tiled kernels.  And which of the two AUTO takes."""
import pytest
import torch

from paper_2603_08185_amd import binding as serq
from tests import test_gpu_grouped as grouped
from tests import test_gpu_mx as mx
from tests import test_gpu_parity as parity

pytestmark = pytest.mark.gpu

# one token past the decode range, ragged last token tile, one / two / an odd number of channel blocks; K from a single
# fragment (one wave has work) over odd fragment counts to rings that wrap
SHAPES = [
    (33, 64, 32, 16),
    (64, 192, 64, 0),
    (65, 576, 96, 48),
    (100, 1088, 288, 128),
    (200, 4160, 160, 144),       # two chunks of the rank-r term, the second ragged
    (129, 2560, 1056, 320),
    (333, 6144, 64, 64),
    (70, 8256, 4096, 32),        # half of the compute units and a long K
    (70, 8256, 4096, 208),       # ... and a second chunk of the rank-r term, whose operands replace the first one's
    (400, 1024, 5152, 208),      # three tiles for the busiest compute unit
    (1100, 4096, 96, 32),        # 8-bit token codes beyond 4 MiB: token tiles in bands, 6 + 6 + 6
    (2100, 4096, 96, 32),        # 4-bit ones too: 7 + 7 + 7 + 7 + 5
]


@pytest.mark.parametrize("abits", [4, 8])
@pytest.mark.parametrize("in_dtype,out_dtype", [("bf16", "bf16"), ("fp16", "fp32"), ("fp16", "fp16")])
@pytest.mark.parametrize("M,K,N,r", SHAPES)
def test_integer_layer(abits, in_dtype, out_dtype, M, K, N, r):
    spec = parity._small_spec(abits, M, K, N, r, in_dtype=in_dtype, out_dtype=out_dtype)
    mode = "random" if r else "none"
    Y, _, _ = parity._run_layer(spec, R_mode=mode)          # (also the exact integer sums of gemm_i32)
    Yt, _, _ = parity._run_layer(spec, R_mode=mode, path=serq.PATH_MFMA, check_pack=False)
    # the same integer sums, the same order of the rank-r products: the same bits as the tiled kernel
    assert torch.equal(Y, Yt)


@pytest.mark.parametrize("abits", [4, 8])
@pytest.mark.parametrize("out_dtype", ["fp16", "fp32"])
@pytest.mark.parametrize("M,K,N,r", [s for s in SHAPES if s[3]])
def test_integer_layer_q4r(abits, out_dtype, M, K, N, r):
    parity._run_layer_q4r(parity._small_spec(abits, M, K, N, r, in_dtype="fp16", out_dtype=out_dtype))


# 8-bit tokens, four waves, 512 channels a round: 1 to 7 units per wave (both parities, every length of the loop's end), last
# units of one fragment and of two, waves with and without one
@pytest.mark.parametrize("K", [320, 512, 1024, 1600, 2048, 2624, 2880, 3072, 3584])
def test_integer_units(K):
    spec = parity._small_spec(8, 45, K, 96, 32, in_dtype="fp16", out_dtype="fp32")
    Y, _, _ = parity._run_layer(spec, R_mode="random")
    Yt, _, _ = parity._run_layer(spec, R_mode="random", path=serq.PATH_MFMA, check_pack=False)
    assert torch.equal(Y, Yt)


def test_salient_block_offset():
    for abits in (4, 8):
        parity._run_layer_q4r(parity._small_spec(abits, 70, 768, 96, 160), s_begin=416)


# K: one group (one wave has work), 9 groups, 33 groups (a ragged last round of the ring); two tiles per compute unit
# (workgroups of four waves) with 21 groups, so that their ring comes to its steady state; token tiles in bands
@pytest.mark.parametrize("abits", [4, 8])
@pytest.mark.parametrize("in_dtype,out_dtype", [("bf16", "bf16"), ("fp16", "fp32"), ("fp16", "fp16")])
@pytest.mark.parametrize("M,K,N,r", [(33, 128, 32, 16), (65, 1152, 96, 0), (100, 4224, 288, 128), (200, 2560, 160, 144),
                                     (129, 384, 1056, 320), (333, 6144, 64, 64), (400, 1152, 5152, 208),
                                     (300, 2688, 4096, 144), (2100, 4096, 96, 32)])
def test_g128_layer(abits, in_dtype, out_dtype, M, K, N, r):
    spec = grouped._spec(abits, M, K, N, r, in_dtype=in_dtype, out_dtype=out_dtype)
    Y, _, _ = grouped._run(spec, R_mode="residual" if r else "none")
    Yb, _, _ = grouped._run(spec, R_mode="residual" if r else "none")
    assert torch.equal(Y, Yb)                               # fixed summation order


# 8-bit tokens, eight waves (one tile per compute unit at most): eight groups of 128 channels a round, 0 to 6 units per wave
@pytest.mark.parametrize("K", [512, 1024, 1152, 2048, 3072, 4096, 5120, 6144])
def test_g128_units(K):
    grouped._run(grouped._spec(8, 45, K, 96, 32, in_dtype="fp16", out_dtype="fp32"), R_mode="residual")


# 8-bit tokens, four waves (265 tiles): four groups a round, 1 to 9 units per wave, some waves with one more than the others.
# (That AUTO takes the small-tile kernel here is shown below, at both ends of the range.)
@pytest.mark.parametrize("K", [512, 640, 1024, 1920, 2048, 2560, 3072, 3712, 4608])
def test_g128_units_four_waves(K):
    grouped._run(grouped._spec(8, 300, K, 3360, 160, in_dtype="fp16", out_dtype="fp32"), R_mode="residual")


def test_g128_layer_variants():
    for abits in (4, 8):
        spec = grouped._spec(abits, 70, 768, 96, 160, out_dtype="fp32")
        grouped._run(spec, asym=False)                      # symmetric codes, no zero points
        grouped._run(spec, R_mode="random", s_begin=416)    # salient block elsewhere, not on a group boundary


# K: one fragment; two; a last scale tile that is dealt in halves, alone in a wave and behind others; several compensation fragments
@pytest.mark.parametrize("in_dtype,out_dtype", [("bf16", "bf16"), ("fp16", "fp32"), ("fp16", "fp16")])
@pytest.mark.parametrize("M,K,N,r", [(33, 64, 32, 32), (65, 128, 96, 0), (100, 448, 64, 96), (200, 4416, 288, 128),
                                     (129, 2688, 1056, 640), (333, 6144, 64, 64), (64, 4160, 160, 256),
                                     (400, 1088, 5152, 352), (2100, 4096, 96, 32)])
def test_mx_layer(in_dtype, out_dtype, M, K, N, r):
    spec = mx._spec(M, K, N, r, in_dtype=in_dtype, out_dtype=out_dtype)
    Y, Y64, _ = mx._run_mx(spec)
    Yb, _, _ = mx._run_mx(spec)
    assert torch.equal(Y, Yb)                               # fixed summation order
    mx._run_mx(spec, path=serq.PATH_MFMA)


# four waves, 1024 channels a round: 0 to 7 units per wave, last units of 1 to 4 fragments (of 3, the one that lacks a fragment of its
# second half: K = 704 alone, 1984 and 4800 behind others), some in the second half of a scale tile
@pytest.mark.parametrize("K", [512, 704, 1024, 1600, 1984, 2048, 3072, 3520, 4096, 4800, 5120, 6144, 7168])
def test_mx_units(K):
    mx._run_mx(mx._spec(45, K, 96, 32, in_dtype="fp16", out_dtype="fp32"))


def test_mx_salient_block_offset():
    mx._run_mx(mx._spec(70, 1344, 96, 160, out_dtype="fp32"), s_begin=768)


# ---- which kernel AUTO takes -----------------------------------------------------------------------------------------------
# The tiled kernels leave a trace where they cut K: the parked tiles in the workspace, behind the decode path's words.  Their
# results are those of PATH_MFMA bit for bit, which the fp32 sums of the small-tile kernels are not.
DEV = "cuda:0"


def _codes(n, seed):
    return torch.randint(0, 256, (n,), dtype=torch.uint8, device=DEV, generator=torch.Generator(device=DEV).manual_seed(seed))


def _trace(ws, words):
    ws[words:] = 0x55
    return lambda: bool((ws[words:] != 0x55).any())


@pytest.mark.parametrize("abits,M,N,K,sliced", [
    (8, 512, 4096, 8192, False), (8, 512, 4096, 28672, True),        # two tiles per compute unit: the larger tiles from a long K on
    (8, 256, 4096, 28672, False),                                    # one tile per compute unit
    (8, 384, 4096, 17408, False), (8, 192, 8192, 15616, False),
    (8, 192, 11008, 4096, False), (8, 192, 11008, 11008, False), (8, 192, 11008, 14336, True),      # three
    (8, 512, 2560, 28672, False),                                    # never slices that a wider layer's decode words could lie in
    (4, 512, 4096, 28672, False), (4, 256, 11008, 28672, False)])
def test_auto_takes_the_cheaper_kernel(abits, M, N, K, sliced):
    X = torch.randn((M, K), device=DEV, generator=torch.Generator(device=DEV).manual_seed(1)).bfloat16()
    Xq, scale = serq.quantize_act(X, None, abits)
    Wq, wscale = _codes(N * K // 2, 2), torch.rand(N, device=DEV) + 0.5
    ws = serq.workspace(M, N, K, 0, abits, DEV)
    words = serq.lib().serq_workspace_bytes(1, N, K, 0, abits)
    touched = _trace(ws, words)
    Y = serq.linear(Xq, scale, abits, Wq, wscale, M, N, K, ws=ws)
    assert touched() == sliced and not ws[:words].any()
    Yt = serq.linear(Xq, scale, abits, Wq, wscale, M, N, K, ws=ws, flags_=serq.flags(serq.PATH_MFMA))
    assert touched() == (ws.numel() > words) and torch.equal(Y, Yt)
    assert torch.equal(Y, serq.linear(Xq, scale, abits, Wq, wscale, M, N, K))      # nothing to park in


@pytest.mark.parametrize("M,N,K,sliced", [(512, 4096, 8192, False), (512, 4096, 28672, True), (256, 4096, 28672, False),
                                          (256, 11008, 4096, False), (256, 11008, 20480, True)])
def test_auto_takes_the_cheaper_mx_kernel(M, N, K, sliced):
    X = torch.randn((M, K), device=DEV, generator=torch.Generator(device=DEV).manual_seed(1)).bfloat16()
    Xq, xsc = serq.mx_quantize_act(X, None)
    Wq = _codes(N * K // 2, 2)
    wsc = 96 + _codes(serq.lib().serq_mx_weight_scale_bytes(N, K), 3) % 48      # far apart: the fp32 sums round
    ws = serq.mx_workspace(M, N, K, DEV)
    words = serq.lib().serq_mx_workspace_bytes(1, N, K)
    touched = _trace(ws, words)
    Y = serq.mx_linear(Xq, xsc, Wq, wsc, M, N, K, out_dtype=torch.float32, ws=ws)
    assert touched() == sliced
    Yt = serq.mx_linear(Xq, xsc, Wq, wsc, M, N, K, out_dtype=torch.float32, ws=ws, flags_=serq.flags(serq.PATH_MFMA))
    assert touched() == (ws.numel() > words)                # (the tiled kernel cuts K wherever it has asked for room)
    assert torch.equal(Y, Yt) == sliced


@pytest.mark.parametrize("abits,M,N,K,r,tiled", [
    (8, 256, 4096, 1024, 0, False), (8, 512, 4096, 1024, 0, True), (8, 512, 4096, 1024, 128, False),
    (8, 768, 4096, 1024, 0, True), (8, 768, 4096, 4096, 128, False), (4, 512, 4096, 4096, 0, False), (4, 768, 4096, 512, 0, True),
    (8, 300, 3360, 512, 160, False), (8, 300, 3360, 4608, 160, False),
    (8, 192, 8096, 5120, 0, False), (8, 128, 14144, 13440, 64, False), (8, 128, 15968, 6144, 128, False)])
def test_auto_takes_the_cheaper_g128_kernel(abits, M, N, K, r, tiled):
    g = torch.Generator(device=DEV).manual_seed(1)
    X = torch.randn((M, K), device=DEV, generator=g).bfloat16()
    Xq, scale, zero = serq.quantize_act_asym(X, None, abits)
    Wq, gs = _codes(N * K // 2, 2), torch.exp(8 * torch.rand(N * K // 128, device=DEV, generator=g) - 8).half()   # sums that round
    wsum = torch.randn(N, device=DEV, generator=g)
    Rp = serq.pack_lowrank(torch.randn((r, N), device=DEV, generator=g).bfloat16()) if r else None
    Y, Yt = (serq.g128_linear(Xq, scale, zero, abits, Wq, gs.view(torch.uint8), wsum, M, N, K, Rp=Rp, r=r,
                              r_dtype=torch.bfloat16, out_dtype=torch.float32, flags_=serq.flags(path))
             for path in (serq.PATH_AUTO, serq.PATH_MFMA))
    assert torch.equal(Y, Yt) == tiled
