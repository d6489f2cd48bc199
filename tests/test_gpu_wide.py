"""The streaming kernel of several batch fragments (k_wide.hip: AUTO batches of
2..128 rows, the gated half up to 112, int8 from 17 rows, from 12 on small grids) on the GPU vs the
oracle: fp16/bf16 within the parity tolerance, int8 bit for bit.

The shapes put its edges in play: grids of up to one, below and above 3.5 row
blocks per CU (one or two row blocks and 4, 8 or 16 waves per workgroup; an odd
number of row blocks for the pairs), every staged-row group
count and both sides of each, a batch split over two workgroups, a last chunk
of one tile, columns past K, full tiles off a 16-byte boundary (129 value
pieces), an all-pruned matrix, and ranges longer than one offsets window."""
import numpy as np
import pytest

import synth
from tests._helpers import assert_close, from_dev_f64, to_dev

pytestmark = pytest.mark.gpu

BATCHES = [2, 3, 4, 8, 9, 16, 17, 24, 25, 32, 33, 40, 41, 48, 49, 56, 57, 64, 65, 97, 128]


@pytest.fixture(scope="module")
def spl():
    import paper_2405_03594_amd as spl

    spl.lib()
    return spl


def _weight(seed, N, K, dtype, s):
    """s < 0: everything kept but the first entry of each row block's first tile, so that full tiles follow at
    odd offsets."""
    W, mask = synth.weight(seed, N, K, dtype, max(s, 0.0))
    if s < 0:
        mask = np.ones_like(mask)
        mask[::16, 0] = 0
    return W, mask


def _packed(spl, W, mask, dtype):
    import torch

    return spl.pack_sparse(to_dev(W, dtype), torch.from_numpy(mask).cuda())


# 8192 < N: 513 row blocks (two per CU of 256); 16384 < N: 1025 (four, an odd number); 2100: 132, more than one
# workgroup per CU in two splits; 4800: 300, more than one per CU, below 3.5 in two splits; 10232, 10250 and 16376,
# 16390: both sides of 640 and 1024, from where on 2 rows, and 3, take the decode kernel (at 70% pruned)
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("N,K,s", [(1, 8, 0.5), (33, 96, 0.7), (100, 1000, 0.5), (48, 160, -1.0), (17, 264, 1.0),
                                   (40, 2088, 0.7), (8200, 72, 0.6), (16390, 136, 0.6), (16390, 64, -1.0),
                                   (2100, 200, 0.6), (4800, 136, 0.6), (10232, 72, 0.7), (10250, 72, 0.7),
                                   (16376, 72, 0.7), (16390, 72, 0.7)])
def test_wide_linear(orc, spl, dtype, N, K, s):
    W, mask = _weight(900 + N + K, N, K, dtype, s)
    X = synth.activations(901 + K, max(BATCHES), K, dtype)
    ref = orc.linear_f64(X, orc.pack(W, dtype, mask))
    Wc, Xd = _packed(spl, W, mask, dtype), to_dev(X, dtype)
    for M in BATCHES:
        Y = spl.sparse_linear(Xd[:M].contiguous(), Wc)
        assert_close(from_dev_f64(Y), ref[:M], f"{dtype} N={N} K={K} s={s} M={M}")


def test_wide_long_rows(orc, spl):
    """Wave ranges longer than the 63 tiles of one offsets window (16 and 8 waves)."""
    N, K = 16, 40008
    W, mask = _weight(77, N, K, "bf16", 0.7)
    X = synth.activations(78, 64, K, "bf16")
    ref = orc.linear_f64(X, orc.pack(W, "bf16", mask))
    Wc, Xd = _packed(spl, W, mask, "bf16"), to_dev(X, "bf16")
    for M in (3, 33, 64):
        assert_close(from_dev_f64(spl.sparse_linear(Xd[:M].contiguous(), Wc)), ref[:M], f"M={M}")


@pytest.mark.parametrize("M", [2, 33, 128])
def test_wide_group(orc, spl, M):
    """Tasks of different shapes, one of them all pruned, in one launch; nothing is written past an output."""
    import torch

    shapes = [(100, 1000, 0.7), (48, 2056, 0.5), (17, 264, 1.0), (64, 4096, 0.7), (33, 512, -1.0)]
    mats, refs, Xs, outs = [], [], [], []
    for i, (N, K, s) in enumerate(shapes):
        W, mask = _weight(300 + i, N, K, "bf16", s)
        X = synth.activations(400 + i, M, K, "bf16")
        mats.append(_packed(spl, W, mask, "bf16"))
        Xs.append(to_dev(X, "bf16"))
        refs.append(orc.linear_f64(X, orc.pack(W, "bf16", mask)))
        outs.append(torch.full((M + 1, N), 7.0, dtype=torch.bfloat16, device="cuda"))
    spl.sparse_linear_group(Xs, mats, [o[:M] for o in outs])
    for i, (o, ref) in enumerate(zip(outs, refs)):
        assert_close(from_dev_f64(o[:M]), ref, f"task {i}")
        assert (o[M] == 7.0).all(), f"task {i}: written past its output"


# 1024 and 1032 columns, 55% and 70% pruned: both sides of where up to 16 rows take the decode kernel; 7160 .. 8192
# rows: of where more than 64 rows are expanded in place
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("N,K,s", [(40, 72, 0.7), (100, 1000, 0.5), (8200, 96, 0.6),
                                   (2100, 1096, 0.6), (4800, 1096, 0.6), (33, 1024, 0.7), (33, 1024, 0.55), (33, 1032, 0.7),
                                   (7160, 72, 0.6), (7170, 72, 0.6), (8192, 72, 0.6)])
def test_wide_gated(orc, spl, dtype, N, K, s):
    (Wg, mg), (Wu, mu) = (_weight(600 + i + N, N, K, dtype, s) for i in range(2))
    X = synth.activations(602 + K, 112, K, dtype)
    ref = orc.silu_mul_f64(X, orc.pack(Wg, dtype, mg), orc.pack(Wu, dtype, mu))
    g, u, Xd = _packed(spl, Wg, mg, dtype), _packed(spl, Wu, mu, dtype), to_dev(X, dtype)
    for M in (1, 2, 8, 9, 16, 17, 32, 33, 41, 64, 65, 112):
        Y = spl.sparse_linear_silu_mul(Xd[:M].contiguous(), g, u)
        assert_close(from_dev_f64(Y), ref[:M], f"{dtype} N={N} K={K} M={M}")


@pytest.mark.parametrize("N,K,s", [(33, 112, 0.7), (64, 2064, 0.5), (48, 160, 0.0), (8200, 80, 0.6), (16390, 144, 0.6),
                                   (2100, 144, 0.6), (4800, 80, 0.6)])
def test_wide_int8(orc, spl, N, K, s):
    import torch

    Wq, mask, sw = synth.int8_weight(800 + N, N, K, s)
    if s == 0.0:
        mask[::16, 0] = 0
    Xq, sx = synth.int8_activations(801 + K, 127, K)
    p = orc.pack(Wq, "i8", mask)
    Wc = _packed(spl, Wq, mask, "i8")
    Xd, sxd, swd = to_dev(Xq, "i8"), torch.from_numpy(sx).cuda(), torch.from_numpy(sw).cuda()
    for M in (8, 9, 11, 12, 15, 16, 17, 24, 32, 33, 48, 64, 65, 127):
        acc_ref, y_ref = orc.linear_i8(Xq[:M], sx[:M], p, sw)
        acc = torch.empty((M, N), dtype=torch.int32, device="cuda")
        Y = spl.sparse_linear_int8(Xd[:M].contiguous(), sxd[:M].contiguous(), Wc, swd, acc_out=acc)
        assert np.array_equal(acc.cpu().numpy(), acc_ref), f"sums N={N} K={K} M={M}"
        assert np.array_equal(Y.cpu().view(torch.int16).numpy().view(np.uint16), y_ref), f"Y N={N} K={K} M={M}"
