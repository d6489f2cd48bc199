"""Products through decoded fragments (k_gemm.hip: AUTO batches past the
streaming kernels, given scratch memory) on the GPU vs the oracle: fp16/bf16
within the parity tolerance, int8 bit for bit, the input gradient through W's
decoded transpose.

The shapes put its edges in play: rows past the last 16-row block and past a
workgroup's tile, outputs whose rows are not whole 16-byte pieces, columns
short of a stage, one to six stages (the loop takes four at a time), the last
batch row of a tile and the first of the next, and each workgroup tile (64 x
128 for the small grids; the larger ones are chosen by the grids below on a
device of 256 CUs).  Calls too small to gain are expanded in place, so that
narrow matrices are run as groups of four (int8: two); every test asserts that
its calls are offered scratch."""
import ctypes

import numpy as np
import pytest

import synth
from tests._helpers import assert_close, from_dev_f64, to_dev

pytestmark = pytest.mark.gpu

BATCHES = [129, 200, 257]


@pytest.fixture(scope="module")
def spl():
    import paper_2405_03594_amd as spl

    spl.lib()
    return spl


def _packed(spl, W, mask, dtype):
    import torch

    return spl.pack_sparse(to_dev(W, dtype), torch.from_numpy(mask).cuda())


def _group_scratch(spl, Xs, mats, outs):
    views = [m.view() for m in mats]
    tasks = (spl._SparseTask * len(mats))(*[spl._SparseTask(x.data_ptr(), ctypes.pointer(v), o.data_ptr())
                                            for x, v, o in zip(Xs, views, outs)])
    return spl.lib().spl_sparse_linear_group_scratch_bytes(tasks, len(mats), Xs[0].shape[0])


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("N,K,s", [(1, 8, 0.5), (16, 64, 0.7), (40, 72, 0.5), (72, 136, 0.0), (130, 200, 0.7),
                                   (300, 320, 0.7), (33, 1000, 0.5), (17, 264, 1.0)])
def test_frag_linear(orc, spl, dtype, N, K, s):
    import torch

    W, mask = synth.weight(40 + N + K, N, K, dtype, s)
    X = synth.activations(41 + K, max(BATCHES), K, dtype)
    ref = orc.linear_f64(X, orc.pack(W, dtype, mask))
    Wc, Xd = _packed(spl, W, mask, dtype), to_dev(X, dtype)
    for M in BATCHES:
        x = Xd[:M].contiguous()
        outs = [torch.full((M + 1, N), 7.0, dtype=Xd.dtype, device="cuda") for _ in range(4)]
        assert _group_scratch(spl, [x] * 4, [Wc] * 4, outs) > 0 or Wc.nnz == 0
        spl.sparse_linear_group([x] * 4, [Wc] * 4, [o[:M] for o in outs])
        for out in outs:
            assert_close(from_dev_f64(out[:M]), ref[:M], f"{dtype} N={N} K={K} M={M}")
            assert (out[M] == 7.0).all(), "written past the output"


# 16 x 16 tiles of 128 x 256 fill 256 CUs once; 256 of 128 x 128 leave one per CU; both on whole and ragged stages
@pytest.mark.parametrize("N,M,K", [(2048, 4096, 1536), (2040, 4090, 1536), (2048, 2048, 1600), (2048, 2048, 1608)])
def test_frag_tiles(spl, N, M, K):
    import torch

    W, mask = synth.weight(50 + K, N, K, "bf16", 0.7)
    X, Wc = to_dev(synth.activations(51 + K, M, K, "bf16"), "bf16"), _packed(spl, W, mask, "bf16")
    assert _group_scratch(spl, [X], [Wc], [X]) > 0
    dense = to_dev(W, "bf16").double() * torch.from_numpy(mask).cuda()
    ref = X.double() @ dense.t().contiguous()
    assert_close(from_dev_f64(spl.sparse_linear(X, Wc)), ref.cpu().numpy(), f"N={N} M={M} K={K}")


def test_frag_group_and_scratch_limits(orc, spl):
    """A group of different shapes (one all pruned) in one launch; too little, misaligned or no scratch gives the
    plain call; batches of the streaming kernels ask for none."""
    import torch

    L, M = spl.lib(), 150
    mats, Xs, refs = [], [], []
    for i, (N, K, s) in enumerate([(100, 1000, 0.7), (17, 264, 1.0), (64, 512, 0.5)]):
        W, mask = synth.weight(60 + i, N, K, "f16", s)
        X = synth.activations(70 + i, M, K, "f16")
        mats.append(_packed(spl, W, mask, "f16"))
        Xs.append(to_dev(X, "f16"))
        refs.append(orc.linear_f64(X, orc.pack(W, "f16", mask)))
    for Y, ref in zip(spl.sparse_linear_group(Xs, mats), refs):
        assert_close(from_dev_f64(Y), ref, "group")
    views = [m.view() for m in mats]
    outs = [torch.empty((M, m.rows), dtype=torch.float16, device="cuda") for m in mats]
    tasks = (spl._SparseTask * 3)(*[spl._SparseTask(x.data_ptr(), ctypes.pointer(v), o.data_ptr())
                                    for x, v, o in zip(Xs, views, outs)])
    need = L.spl_sparse_linear_group_scratch_bytes(tasks, 3, M)
    assert need == (7 * 32 + 4 * 16) * 1024      # 7 and 4 row blocks of 32 and 16 fragments; nothing for no values
    assert L.spl_sparse_linear_group_scratch_bytes(tasks, 3, 128) == 0
    plain = spl.sparse_linear_group(Xs, mats, algo="prefill")
    buf = torch.empty((need + 256,), dtype=torch.uint8, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    for ptr, have in ((0, need), (buf.data_ptr(), need - 1), (buf.data_ptr() + 16, need)):
        for o in outs:
            o.zero_()
        assert L.spl_sparse_linear_group_scratch(tasks, 3, M, ptr, have, stream) == 0
        assert all(torch.equal(o, p) for o, p in zip(outs, plain))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("N,K,s", [(20, 1608, 0.7), (70, 1736, 0.5), (264, 1664, 0.6)])
def test_frag_gated(orc, spl, dtype, N, K, s):
    (Wg, mg), (Wu, mu) = (synth.weight(80 + i + N, N, K, dtype, s) for i in range(2))
    X = synth.activations(82 + K, max(BATCHES), K, dtype)
    ref = orc.silu_mul_f64(X, orc.pack(Wg, dtype, mg), orc.pack(Wu, dtype, mu))
    g, u, Xd = _packed(spl, Wg, mg, dtype), _packed(spl, Wu, mu, dtype), to_dev(X, dtype)
    for M in [113] + BATCHES:
        assert spl.lib().spl_sparse_linear_silu_mul_scratch_bytes(M, ctypes.byref(g.view()), ctypes.byref(u.view())) > 0
        assert_close(from_dev_f64(spl.sparse_linear_silu_mul(Xd[:M].contiguous(), g, u)), ref[:M],
                     f"{dtype} N={N} K={K} M={M}")


@pytest.mark.parametrize("N,K,M,s", [(33, 112, 129, 0.7), (130, 144, 200, 0.0), (64, 640, 257, 0.5),
                                     (2048, 256, 4096, 0.7), (2040, 144, 2050, 0.7)])
def test_frag_int8(orc, spl, N, K, M, s):
    import torch

    Wq, mask, sw = synth.int8_weight(90 + N, N, K, s)
    Xq, sx = synth.int8_activations(91 + K, M, K)
    acc_ref, y_ref = orc.linear_i8(Xq, sx, orc.pack(Wq, "i8", mask), sw)
    n = 1 if N > 1000 else 2                    # one small matrix is expanded in place
    accs = [torch.empty((M, N), dtype=torch.int32, device="cuda") for _ in range(n)]
    Xd, sxd, swd, Wc = to_dev(Xq, "i8"), torch.from_numpy(sx).cuda(), torch.from_numpy(sw).cuda(), _packed(spl, Wq, mask,
                                                                                                          "i8")
    Ys = spl.sparse_linear_int8_group([Xd] * n, [sxd] * n, [Wc] * n, [swd] * n, acc_outs=accs)
    view = Wc.view()
    tasks = (spl._Int8Task * n)(*[spl._Int8Task(Xd.data_ptr(), sxd.data_ptr(), ctypes.pointer(view), swd.data_ptr(),
                                                y.data_ptr(), None) for y in Ys])
    assert spl.lib().spl_sparse_linear_int8_group_scratch_bytes(tasks, n, M) > 0
    for acc, Y in zip(accs, Ys):
        assert np.array_equal(acc.cpu().numpy(), acc_ref)
        assert np.array_equal(Y.cpu().view(torch.int16).numpy().view(np.uint16), y_ref)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("N,K,M,s", [(8, 8, 1, 0.5), (40, 72, 7, 0.7), (264, 40, 130, 0.0), (72, 1000, 257, 0.6),
                                     (512, 520, 300, 0.7)])
def test_frag_input_grad(orc, spl, dtype, N, K, M, s):
    W, mask = synth.weight(95 + N, N, K, dtype, s)
    dY = synth.activations(96 + K, M, N, dtype)
    Wc = _packed(spl, W, mask, dtype)
    assert spl.lib().spl_sparse_input_grad_scratch_bytes(M, ctypes.byref(Wc.view())) > 0
    dX = from_dev_f64(spl.sparse_input_grad(to_dev(dY, dtype), Wc))
    assert_close(dX, orc.input_grad_f64(dY, dtype, orc.pack(W, dtype, mask)), f"{dtype} N={N} K={K} M={M}")


def test_frag_graph_replays_and_streams(spl):
    """Scratch from the graph's pool, and from another stream's pool, gives the eager result."""
    import torch

    W, mask = synth.weight(7, 512, 2048, "bf16", 0.7)
    Wc, X = _packed(spl, W, mask, "bf16"), to_dev(synth.activations(8, 300, 2048, "bf16"), "bf16")
    eager = spl.sparse_linear(X, Wc)
    assert _group_scratch(spl, [X], [Wc], [eager]) > 0
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    other = torch.empty_like(eager)
    spl.sparse_linear(X, Wc, out=other, stream=side)
    side.synchronize()
    assert torch.equal(other, eager)
    out = torch.empty_like(eager)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        spl.sparse_linear(X, Wc, out=out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager)
        assert torch.equal(spl.sparse_linear(X, Wc), eager)
