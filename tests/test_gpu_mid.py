"""The kernels for batches between decode and prefill (64 x 64 tiles, K shared by the waves of a workgroup), which AUTO takes
for these sizes: against the oracle, and against the tiled kernels."""
import pytest
import torch

from paper_2603_08185_amd import binding as serq
from tests import test_gpu_grouped as grouped
from tests import test_gpu_mx as mx
from tests import test_gpu_parity as parity

pytestmark = pytest.mark.gpu

# one token past the decode range, ragged last token tile, one / two / an odd number of channel blocks; K from a single
# fragment (seven waves idle) over odd fragment counts to rings that wrap
SHAPES = [
    (33, 64, 32, 16),
    (64, 192, 64, 0),
    (65, 576, 96, 48),
    (100, 1088, 288, 128),
    (200, 4160, 160, 144),       # two chunks of the rank-r term, the second ragged
    (129, 2560, 1056, 320),
    (333, 6144, 64, 64),
    (70, 8256, 4096, 32),        # half of the compute units and a long K: eight waves for 8-bit tokens
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


def test_salient_block_offset():
    for abits in (4, 8):
        parity._run_layer_q4r(parity._small_spec(abits, 70, 768, 96, 160), s_begin=416)


# K: one group (seven waves idle), 9 groups, 33 groups (a ragged last round of the ring)
@pytest.mark.parametrize("abits", [4, 8])
@pytest.mark.parametrize("in_dtype,out_dtype", [("bf16", "bf16"), ("fp16", "fp32"), ("fp16", "fp16")])
@pytest.mark.parametrize("M,K,N,r", [(33, 128, 32, 16), (65, 1152, 96, 0), (100, 4224, 288, 128), (200, 2560, 160, 144),
                                     (129, 384, 1056, 320), (333, 6144, 64, 64), (400, 1152, 5152, 208),
                                     (2100, 4096, 96, 32)])
def test_g128_layer(abits, in_dtype, out_dtype, M, K, N, r):
    spec = grouped._spec(abits, M, K, N, r, in_dtype=in_dtype, out_dtype=out_dtype)
    Y, _, _ = grouped._run(spec, R_mode="residual" if r else "none")
    Yb, _, _ = grouped._run(spec, R_mode="residual" if r else "none")
    assert torch.equal(Y, Yb)                               # fixed summation order


def test_g128_layer_variants():
    for abits in (4, 8):
        spec = grouped._spec(abits, 70, 768, 96, 160, out_dtype="fp32")
        grouped._run(spec, asym=False)                      # symmetric codes, no zero points
        grouped._run(spec, R_mode="random", s_begin=416)    # salient block elsewhere, not on a group boundary


# K: one fragment; a last scale tile of 1, 2 and 3 fragments, alone in its wave and behind others; several compensation fragments
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


def test_mx_salient_block_offset():
    mx._run_mx(mx._spec(70, 1344, 96, 160, out_dtype="fp32"), s_begin=768)
