"""Infinities in the training kernels stay where arithmetic puts them.

The sparse products take a row's entries four at a time: the lanes past the
row's end belong to no entry and must not bring in row i of the vectors, which
0 * inf would turn into a NaN.  The backward pass takes 16 rows at a time: the
rows past n repeat no activation.  Both against the oracle's plain sums, entry
by entry: the same infinities and NaNs, and the finite values within the
bounds of the finite cases (1e-10 for dL/dP, 1e-3 for the gradients through
the bf16 roundings).
"""
import numpy as np
import pytest

from tests.test_gpu_spai import S, bits_bf16, random_params, split_grad, to_device  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def same(got, ref, tol):
    """Equal infinities and NaNs; the finite part within tol of its norm."""
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    inf = np.isinf(ref)
    assert np.array_equal(inf, np.isinf(got)) and np.array_equal(got[inf], ref[inf])
    f = np.isfinite(ref)
    assert f.any() and np.linalg.norm(got[f] - ref[f]) <= tol * np.linalg.norm(ref[f])


def off_diagonal(n, reach):
    """Negative entries at distance 1 .. reach (an odd one only), no diagonal."""
    import scipy.sparse as sp
    from _helpers import csr_from_scipy
    offs = [d for k in range(1, reach + 1, 2) for d in (-k, k)]
    rng = np.random.default_rng(n)
    return csr_from_scipy(sp.diags([-1.0 - rng.random(n - abs(d)) for d in offs], offs))


@pytest.mark.parametrize("reach", [1, 5])
@pytest.mark.parametrize("K", [3, 32])
def test_row_ends_bring_in_no_infinity(S, dev, reach, K):
    """Rows of 2 and of 6 entries: the last batch is half empty.  One vector
    holds -inf in one row.  With A < 0 < P no sum meets opposite infinities,
    and with odd distances only, rows of the other parity stay finite."""
    import paper_2009_12101_amd as cbg
    n, at = 41, 20
    print(f"row ends reach={reach} K={K}", flush=True)
    A = off_diagonal(n, reach)
    rng = np.random.default_rng(K)
    V = S.fl32(0.1 + rng.random((K, n))).astype(np.float16).astype(np.float64)
    V[K // 2, at] = -np.inf
    pv = S.fl32(0.1 + rng.random(A.nnz))
    L, dP = S.loss_and_grad_p(A, pv, V)
    assert L == np.inf and np.isfinite(dP[A.row_ptr[at]:A.row_ptr[at + 1]]).all()
    Ad = cbg.DeviceCSR.from_host(A, dev)
    Vd = torch.from_numpy(V.T.astype(np.float16).copy().view(np.int16)).to(dev)
    loss, got = cbg.spai_grad_p(Ad, cbg.csr_transpose_values(Ad),
                                torch.from_numpy(pv.astype(np.float32)).to(dev), Vd, 1.0 / K)
    assert loss.item() == np.inf
    same(got.cpu().numpy(), dP, 1e-10)


@pytest.mark.parametrize("n", [1, 17, 47])
@pytest.mark.parametrize("where", ["F", "H1", "H2"])
def test_rows_past_n_repeat_no_activation(S, dev, n, where):
    """One column of the last row's features or activations is infinite, the
    last tile is ragged, and every activation of that row is positive: the
    column's gradients are infinite, not NaN, and the others stay finite."""
    import paper_2009_12101_amd as cbg
    print(f"backward {where} n={n}", flush=True)
    rng = np.random.default_rng(n)
    prm = random_params(S, 9)
    X = {"F": S.bf16(rng.standard_normal((n, 64))), "H1": S.bf16(0.1 + rng.random((n, 64))),
         "H2": S.bf16(0.1 + rng.random((n, 64)))}
    X[where][n - 1, 5] = np.inf
    dO = S.bf16(rng.standard_normal((n, 32)) * 1e-2)
    ref = S.backward(X["F"], X["H1"], X["H2"], prm["W2"], prm["W3"], dO)
    assert sum(np.isinf(r).sum() for r in ref.values()) >= 32
    assert not any(np.isnan(r).any() for r in ref.values())
    _, weights = to_device(prm, dev)
    args = [bits_bf16(t).to(dev) for t in (X["F"], X["H1"], X["H2"], dO)] + [weights]
    got = split_grad(cbg.mlp_backward(*args).cpu().numpy())
    for k in ref:
        same(got[k], ref[k], 1e-3)
