"""The one-row kernel (k_row.hip: AUTO at M = 1, linear groups and the gated
half) on the GPU vs the oracle, within the parity tolerance.

The shapes put its edges in play: grids of up to one, of one to three and of
more row blocks per CU (16, 8 or 4 waves; 8 from six to nine with 4096 columns
and more), a last quad of one to three tiles, columns past K, ranges longer than
one offsets window, an all-pruned matrix, densities on both sides of the two-quad chunk (50%), full quads off a
16-byte boundary (257 value pieces), and nearly full tiles, whose upper windows
end in the next row's or the next column group's first dword."""
import pytest

from tests._helpers import assert_close, from_dev_f64, to_dev
from tests.test_gpu_wide import _packed, _weight
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spl():
    import paper_2405_03594_amd as spl

    spl.lib()
    return spl


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("N,K,s", [(1, 8, 0.5), (33, 96, 0.7), (100, 1000, 0.5), (48, 1160, -1.0), (17, 264, 1.0),
                                   (40, 2088, 0.45), (64, 4096, 0.02), (33, 40008, 0.7), (16, 70000, 0.1),
                                   (4128, 520, 0.7), (8200, 72, 0.0), (12300, 136, 0.6), (24580, 136, 0.6), (24580, 4104, 0.9), (16390, 136, 0.6), (16390, 2056, 0.7)])
def test_row_linear(orc, spl, dtype, N, K, s):
    W, mask = _weight(70 + N + K, N, K, dtype, s)
    X = synth.activations(71 + K, 1, K, dtype)
    ref = orc.linear_f64(X, orc.pack(W, dtype, mask))
    Wc, Xd = _packed(spl, W, mask, dtype), to_dev(X, dtype)
    assert_close(from_dev_f64(spl.sparse_linear(Xd, Wc)), ref, f"{dtype} N={N} K={K} s={s}")
    assert_close(from_dev_f64(spl.sparse_linear(Xd, Wc, algo="decode")), ref, f"decode {dtype} N={N} K={K} s={s}")


def test_row_group(orc, spl):
    """Tasks of different shapes, one of them all pruned, in one launch; nothing is written past an output."""
    import torch

    shapes = [(100, 1000, 0.7), (48, 2056, 0.5), (17, 264, 1.0), (8200, 4096, 0.7), (33, 512, -1.0)]
    mats, refs, Xs, outs = [], [], [], []
    for i, (N, K, s) in enumerate(shapes):
        W, mask = _weight(30 + i, N, K, "bf16", s)
        X = synth.activations(40 + i, 1, K, "bf16")
        mats.append(_packed(spl, W, mask, "bf16"))
        Xs.append(to_dev(X, "bf16"))
        refs.append(orc.linear_f64(X, orc.pack(W, "bf16", mask)))
        outs.append(torch.full((2, N), 7.0, dtype=torch.bfloat16, device="cuda"))
    spl.sparse_linear_group(Xs, mats, [o[:1] for o in outs])
    for i, (o, ref) in enumerate(zip(outs, refs)):
        assert_close(from_dev_f64(o[:1]), ref, f"task {i}")
        assert (o[1] == 7.0).all(), f"task {i}: written past its output"


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("N,K,s", [(40, 72, 0.7), (100, 1000, 0.5), (8200, 96, 0.6), (4112, 4104, 0.05)])
def test_row_gated(orc, spl, dtype, N, K, s):
    (Wg, mg), (Wu, mu) = (_weight(60 + i + N, N, K, dtype, s) for i in range(2))
    X = synth.activations(62 + K, 1, K, dtype)
    ref = orc.silu_mul_f64(X, orc.pack(Wg, dtype, mg), orc.pack(Wu, dtype, mu))
    Y = spl.sparse_linear_silu_mul(to_dev(X, dtype), _packed(spl, Wg, mg, dtype), _packed(spl, Wu, mu, dtype))
    assert_close(from_dev_f64(Y), ref, f"{dtype} N={N} K={K}")


def test_row_propagates_nonfinite(spl):
    """An infinite activation against pruned weights is NaN in every row, and a NaN stays one, as in the decode
    kernel; an infinite weight leaves the other rows alone."""
    import torch

    W = torch.ones(64, 256, device="cuda").bfloat16()
    mask = torch.rand(64, 256, device="cuda") > 0.5
    mask[5, 7] = True
    X = torch.ones(1, 256, device="cuda").bfloat16()
    W[5, 7] = float("inf")
    Wc = spl.pack_sparse(W, mask)
    y, d = spl.sparse_linear(X, Wc), spl.sparse_linear(X, Wc, algo="decode")
    assert torch.isinf(y[0, 5]) and torch.isfinite(y[0]).sum() == 63
    assert torch.equal(y, d)                         # sums of at most 256 ones: exact
    X[0, 130] = float("inf")
    y, d = spl.sparse_linear(X, Wc), spl.sparse_linear(X, Wc, algo="decode")
    assert torch.equal(torch.isnan(y), torch.isnan(d)) and torch.equal(torch.isinf(y), torch.isinf(d))
