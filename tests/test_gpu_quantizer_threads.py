"""The quantisers choose their threads per row by the row length and the number of rows: bit-exact against the oracle on both
sides of every limit (rows of 1024 / 1032 / 1536 / 1544 / 2048 / 2056 pieces of 16 bytes, batches of 512 and 513 rows)."""
import numpy as np
import pytest
import torch

from oracle import serq_oracle as orc
from paper_2603_08185_amd import binding as serq

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("M", [3, 512, 513])
@pytest.mark.parametrize("K", [2112, 4096, 4160, 8192, 8256, 12288, 12352, 16384, 16448])
def test_codes_match_the_oracle(M, K):
    g = torch.Generator().manual_seed(M + K)
    X = torch.randn((M, K), generator=g)
    X[:, K - 1] *= 40                                  # the last piece of the row decides the scale
    X = X.to(torch.bfloat16)
    s_inv = torch.rand(K, generator=g) + 0.5
    rows = [0, M // 2, M - 1]
    Xo = X[rows].float().numpy()
    Xd, sd = X.to(DEV), s_inv.to(DEV)
    for abits in (4, 8):
        Xq, sc = serq.quantize_act(Xd, sd, abits)
        c, s = orc.quantize_act(Xo, s_inv.numpy(), abits)
        assert np.array_equal(serq.unpack_act(Xq, abits, M, K).cpu().numpy()[rows], c)
        assert np.array_equal(sc.cpu().numpy()[rows], s)
        Xq, sc, z = serq.quantize_act_asym(Xd, sd, abits)
        c, s, zo = orc.quantize_act_asym(Xo, s_inv.numpy(), abits)
        assert np.array_equal(serq.unpack_act(Xq, abits, M, K).cpu().numpy()[rows], c)
        assert np.array_equal(sc.cpu().numpy()[rows], s) and np.array_equal(z.cpu().numpy()[rows], zo)
    Xq, xs = serq.mx_quantize_act(Xd, sd)
    c, e = serq.mx_unpack_act(Xq, xs, M, K)
    co, eo = orc.mx_quantize_act(Xo, s_inv.numpy())
    assert np.array_equal(c.cpu().numpy()[rows], co) and np.array_equal(e.cpu().numpy()[rows], eo)
