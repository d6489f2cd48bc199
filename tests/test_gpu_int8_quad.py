"""The int8 kernel that takes four tiles per scan (k_int8_quad.hip: batches of
up to 16 rows) on the GPU, bit for bit against the oracle.

The shapes put its edges in play: last quads of one to four tiles, half tiles
(K % 32 == 16), waves with no, one, two and several quads, grids of up to one
row block per CU (16 waves, 8 where K has fewer than 16 quads), up to and above
three per CU (8 and 4 waves), and full and empty tiles.  Up to one row block per
CU AUTO keeps this kernel to 8 rows (11 past 3072 columns, 15 past 4096)."""
import numpy as np
import pytest

import synth
from tests._helpers import to_dev
from tests.test_gpu_int4 import _assert_equal

pytestmark = pytest.mark.gpu
MS = (1, 4, 5, 8, 9, 11, 16)


@pytest.fixture(scope="module")
def spl():
    import paper_2405_03594_amd as spl

    spl.lib()
    return spl


def _bits(Y):
    import torch

    return Y.cpu().view(torch.int16).numpy().view(np.uint16)


@pytest.mark.parametrize("N,K,s", [(5, 32, 0.5), (33, 80, 0.6), (17, 112, 0.0), (40, 128, 0.7), (20, 144, 0.7),
                                   (100, 2048, 0.5), (31, 4112, 0.7), (16, 6208, 0.3), (48, 13824, 0.7),
                                   (8208, 208, 0.7), (8300, 2080, 0.6), (24, 1024, 1.0), (4112, 2064, 0.6), (33, 3088, 0.6), (12300, 144, 0.6),
                                   (16390, 144, 0.6), (16390, 2064, 0.6)])
def test_int8_quad(orc, spl, N, K, s):
    import torch

    Wq, mask, sw = synth.int8_weight(940 + N, N, K, s)
    W8 = spl.pack_sparse(to_dev(Wq, "i8"), torch.from_numpy(mask).cuda())
    Xq, sx = synth.int8_activations(941 + K, 16, K)
    p = orc.pack(Wq, "i8", mask)
    for M in MS:
        acc_ref, y_ref = orc.linear_i8(Xq[:M], sx[:M], p, sw)
        acc = torch.full((M + 1, N), 77, dtype=torch.int32, device="cuda")
        Y = torch.full((M + 1, N), 7.0, dtype=torch.float16, device="cuda")
        spl.sparse_linear_int8(to_dev(Xq[:M], "i8"), torch.from_numpy(sx[:M]).cuda(), W8, torch.from_numpy(sw).cuda(),
                               out=Y[:M], acc_out=acc[:M])
        assert (acc[M] == 77).all() and (Y[M] == 7.0).all(), "written past the outputs"
        _assert_equal(acc[:M].cpu().numpy(), acc_ref, f"acc N={N} K={K} s={s} M={M}")
        _assert_equal(_bits(Y[:M]), y_ref, f"Y N={N} K={K} s={s} M={M}")


@pytest.mark.parametrize("M", MS)
def test_int8_quad_group(orc, spl, M):
    """Matrices of different shapes, one of them all pruned, with activations of their own, in one launch."""
    import torch

    shapes = [(100, 1008, 0.7), (48, 2064, 0.5), (17, 272, 1.0), (8200, 4096, 0.7), (33, 512, 0.0)]
    args, refs = [], []
    for i, (N, K, s) in enumerate(shapes):
        Wq, mask, sw = synth.int8_weight(950 + i, N, K, s)
        Xq, sx = synth.int8_activations(960 + i, M, K)
        refs.append(orc.linear_i8(Xq, sx, orc.pack(Wq, "i8", mask), sw)[1])
        args.append((to_dev(Xq, "i8"), torch.from_numpy(sx).cuda(),
                     spl.pack_sparse(to_dev(Wq, "i8"), torch.from_numpy(mask).cuda()), torch.from_numpy(sw).cuda()))
    outs = spl.sparse_linear_int8_group(*[list(a) for a in zip(*args)])
    for i, (y, ref) in enumerate(zip(outs, refs)):
        _assert_equal(_bits(y), ref, f"task {i} M={M}")


@pytest.mark.parametrize("M", (1, 8, 16))
def test_int8_quad_large_group(orc, spl, M):
    """More than three row blocks per CU in one launch (4 waves), both tasks with a last partial block."""
    import torch

    args, refs = [], []
    for i, (N, K, s) in enumerate([(9000, 144, 0.6), (8200, 272, 0.5)]):
        Wq, mask, sw = synth.int8_weight(970 + i, N, K, s)
        Xq, sx = synth.int8_activations(980 + i, M, K)
        refs.append(orc.linear_i8(Xq, sx, orc.pack(Wq, "i8", mask), sw)[1])
        args.append((to_dev(Xq, "i8"), torch.from_numpy(sx).cuda(),
                     spl.pack_sparse(to_dev(Wq, "i8"), torch.from_numpy(mask).cuda()), torch.from_numpy(sw).cuda()))
    for i, (y, ref) in enumerate(zip(spl.sparse_linear_int8_group(*[list(a) for a in zip(*args)]), refs)):
        _assert_equal(_bits(y), ref, f"task {i} M={M}")


def test_int8_quad_every_selector(spl):
    """All 16 patterns of 4 columns at every count before them, from every byte alignment of the first value."""
    import torch

    g = torch.Generator(device="cuda").manual_seed(7)
    N, K = 512, 4096                                 # 4 M patterns of 16 columns: every one of the 65536 is likely
    pat = torch.randint(0, 1 << 16, (N, K // 16), generator=g, device="cuda")
    mask = ((pat[..., None] >> torch.arange(16, device="cuda")) & 1).bool().view(N, K)
    W = torch.randint(-127, 128, (N, K), generator=g, device="cuda", dtype=torch.int8)
    W[W == 0] = 1
    X = torch.randint(-127, 128, (16, K), generator=g, device="cuda", dtype=torch.int8)
    W8 = spl.pack_sparse(W, mask.to(torch.uint8))
    ref = X.cpu().double() @ (W * mask).cpu().double().t()
    for M in MS:
        acc = torch.empty((M, N), dtype=torch.int32, device="cuda")
        spl.sparse_linear_int8(X[:M], torch.ones(M, device="cuda"), W8, torch.ones(N, device="cuda"), acc_out=acc)
        assert torch.equal(acc.cpu().double(), ref[:M]), f"M={M}"
