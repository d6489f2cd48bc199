"""The 4-bit kernel that takes four tiles per scan (k_int4_quad.hip: columns up
to 2^20) on the GPU, bit for bit against the int8 oracle on the same codes.

The shapes put its edges in play: last quads of one to four tiles, half tiles
(K % 32 == 16), waves with no, one, two and several quads, grids on both sides
of one row block per CU (16 or 8 waves), full and empty tiles, batches of 1 to
16 rows, and the largest sums on both sides of the 2^20 columns from where the
other kernel runs."""
import numpy as np
import pytest

import synth
from tests._helpers import to_dev
from tests.test_gpu_int4 import _assert_equal, _pack4

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spl():
    import paper_2405_03594_amd as spl

    spl.lib()
    return spl


def _run(spl, Xq, sx, W4, sw, N):
    import torch

    M = Xq.shape[0]
    acc = torch.full((M + 1, N), 77, dtype=torch.int32, device="cuda")
    Y = torch.full((M + 1, N), 7.0, dtype=torch.float16, device="cuda")
    spl.sparse_linear_int4(to_dev(Xq, "i8"), torch.from_numpy(sx).cuda(), W4, torch.from_numpy(sw).cuda(), out=Y[:M],
                           acc_out=acc[:M])
    assert (acc[M] == 77).all() and (Y[M] == 7.0).all(), "written past the outputs"
    return acc[:M].cpu().numpy(), Y[:M].cpu().view(torch.int16).numpy().view(np.uint16)


@pytest.mark.parametrize("N,K,s", [(5, 32, 0.5), (33, 80, 0.6), (17, 112, 0.0), (40, 128, 0.7), (20, 144, 0.7),
                                   (100, 2048, 0.5), (31, 4112, 0.7), (16, 6208, 0.3), (48, 13824, 0.7),
                                   (8208, 208, 0.7), (8300, 2080, 0.6), (24, 1024, 1.0), (4112, 1040, 0.6),
                                   (4112, 3088, 0.6), (4090, 3088, 0.6)])
def test_int4_quad(orc, spl, N, K, s):
    Wq, mask, sw = synth.int4_weight_full_range(930 + N, N, K, s)
    W4 = _pack4(spl, Wq, mask)
    Xq, sx = synth.int8_activations(931 + K, 16, K)
    p = orc.pack(Wq, "i8", mask)
    for M in (1, 4, 5, 9, 16):
        acc_ref, y_ref = orc.linear_i8(Xq[:M], sx[:M], p, sw)
        acc, y = _run(spl, Xq[:M], sx[:M], W4, sw, N)
        _assert_equal(acc, acc_ref, f"acc N={N} K={K} s={s} M={M}")
        _assert_equal(y, y_ref, f"Y N={N} K={K} s={s} M={M}")


@pytest.mark.parametrize("N", [1, 8208])
@pytest.mark.parametrize("K", [(1 << 20) - 16, 1 << 20, (1 << 20) + 16])
def test_int4_quad_largest_sums(spl, N, K):
    """Every product of the live rows is 1024, the largest there is; of 8208 rows (8 waves) only 16 have values."""
    import torch

    W8 = torch.zeros((N, K), dtype=torch.int8, device="cuda")   # up to 8.6 GB
    rows = min(N, 16)
    W8[:rows] = -8
    W4 = spl.pack_int4(spl.pack_sparse(W8))
    Xq = np.full((2, K), -128, dtype=np.int8)
    Xq[1, ::2] = 127
    sx, sw = np.ones(2, np.float32), np.ones(N, np.float32)
    acc, _ = _run(spl, Xq, sx, W4, sw, N)
    ref = np.zeros((2, N), np.int64)
    ref[:, :rows] = -8 * Xq.astype(np.int64).sum(axis=1)[:, None]
    assert ref.max() < 2**31
    _assert_equal(acc, ref.astype(np.int32), f"acc N={N} K={K}")
