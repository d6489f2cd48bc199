"""Activations that are not finite, through every kernel that AUTO picks: an
infinity or NaN reaches exactly the outputs that the masked dense product
sends it to (0 x inf is NaN), and no other batch row.  An all-pruned matrix
gives NaN in such rows up to 32 batch rows and +0 above, whichever kernel runs."""
import pytest

import synth
from tests._helpers import to_dev

pytestmark = pytest.mark.gpu

BATCHES = [1, 2, 5, 17, 32, 33, 64, 113, 128, 129, 300]


@pytest.fixture(scope="module")
def spl():
    import paper_2405_03594_amd as spl

    spl.lib()
    return spl


def _case(spl, N, K, s, M, dtype):
    import torch

    W, mask = synth.weight(5 + N, N, K, dtype, s)
    X = to_dev(synth.activations(6 + K, M, K, dtype), dtype)
    X[0, 3] = float("inf")
    X[M // 2, K - 1] = float("-inf")
    X[M - 1, K // 2] = float("nan")
    return spl.pack_sparse(to_dev(W, dtype), torch.from_numpy(mask).cuda()), to_dev(W, dtype), torch.from_numpy(mask).cuda(), X


def _same_kind(Y, ref, what):
    import torch

    assert torch.equal(torch.isnan(Y), torch.isnan(ref)), what
    inf = torch.isinf(ref)
    assert torch.equal(torch.isinf(Y), inf) and torch.equal(Y[inf].float(), ref[inf]), what


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("N,K,s", [(33, 136, 0.5), (2050, 1608, 0.7)])
def test_nonfinite_linear(spl, dtype, N, K, s):
    import torch

    for M in BATCHES:
        Wc, W, mask, X = _case(spl, N, K, s, M, dtype)
        d = (W.float() * mask.float()).cpu()
        ref = torch.stack([(x[None, :] * d).sum(dim=1) for x in X.float().cpu()]).cuda()   # 0 x inf is NaN
        _same_kind(spl.sparse_linear(X, Wc), ref, f"{dtype} N={N} K={K} M={M}")


@pytest.mark.parametrize("M", BATCHES)
def test_nonfinite_all_pruned(spl, M):
    import torch

    Wc, _, _, X = _case(spl, 40, 136, 1.0, M, "bf16")
    assert Wc.nnz == 0
    Y = spl.sparse_linear(X, Wc).float()
    bad = torch.zeros(M, dtype=torch.bool, device="cuda")
    if M <= 32:
        bad[[0, M // 2, M - 1]] = True
    assert torch.isnan(Y[bad]).all(), f"M={M}"
    assert (Y[~bad] == 0).all() and not torch.signbit(Y[~bad]).any(), f"M={M}"
