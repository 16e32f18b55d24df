"""The training kernels at the shapes where their tiles and lanes run out.

* Loss and dL/dP for K = 1 .. 32 vectors (32 has a form of its own with
  16-byte loads; 32 vectors at an odd address take the general one), on rows
  of a stencil and on irregular rows (empty, one entry, more than a batch),
  against the oracle: 1e-12 and 1e-10, the bounds of the existing parity
  test of these sums.
* The backward pass at row counts around its 16-row tiles and with more tiles
  than waves in a block, inputs at odd addresses included, against the
  oracle: 1e-5 for W3 and b3 (fp32 accumulation), 1e-3 for the others
  (through the bf16 roundings), as in the existing parity test.
* One whole evaluation with K = 17 equals the separate calls: the loss to
  1e-12, the gradient to the 1e-3 of the bf16 roundings.
"""
import numpy as np
import pytest

from tests.test_gpu_spai import (NPARAM, S, bits_bf16, random_params, split_grad,  # noqa: F401
                                 to_device, unit_vectors)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def irregular_symmetric(n, seed):
    """A structurally symmetric pattern with rows of 0 to about 40 entries."""
    import scipy.sparse as sp
    from _helpers import csr_from_scipy
    rng = np.random.default_rng(seed)
    B = sp.random(n, n, density=4.0 / n, random_state=seed).tolil()
    B[5, rng.choice(n, 35, replace=False)] = 1.0
    B = sp.csr_matrix(B)
    M = B + B.T + sp.diags(np.where(np.arange(n) % 9 == 4, 0.0, 5.0))
    M = sp.csr_matrix(M)
    keep = np.arange(n) % 9 != 4                   # those rows and columns: empty
    M = sp.diags(keep.astype(float)) @ M @ sp.diags(keep.astype(float))
    M = sp.csr_matrix(M)
    M.eliminate_zeros()
    M.data = rng.standard_normal(M.nnz)
    return csr_from_scipy(M)


def odd_address(t):
    """The same values one element further on in memory than an aligned start."""
    b = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    b[1:] = t.reshape(-1)
    return b[1:].view(t.shape)


@pytest.mark.parametrize("pattern", ["stencil", "irregular"])
@pytest.mark.parametrize("K,odd", [(1, False), (8, False), (17, False), (31, False), (32, False),
                                   (32, True)])
def test_grad_p_vector_counts(S, dev, pattern, K, odd):
    import paper_2009_12101_amd as cbg
    from paper_2009_12101_amd import problems as P
    A = P.lognormal27(7, 2) if pattern == "stencil" else irregular_symmetric(203, 1)
    print(f"grad_p {pattern} K={K} odd={odd} n={A.n}", flush=True)
    V = S.fl32(unit_vectors(A.n, K, 4)).astype(np.float16).astype(np.float64)
    pv = S.fl32(np.random.default_rng(6).standard_normal(A.nnz) * 0.2)
    L, dP = S.loss_and_grad_p(A, pv, V)
    Ad = cbg.DeviceCSR.from_host(A, dev)
    Vd = torch.from_numpy(V.T.astype(np.float16).copy().view(np.int16)).to(dev)
    loss, got = cbg.spai_grad_p(Ad, cbg.csr_transpose_values(Ad),
                                torch.from_numpy(pv.astype(np.float32)).to(dev),
                                odd_address(Vd) if odd else Vd, 1.0 / K)
    assert abs(loss.item() - L) <= 1e-12 * L
    assert np.linalg.norm(got.cpu().numpy() - dP) <= 1e-10 * np.linalg.norm(dP)


@pytest.mark.parametrize("n,odd", [(1, False), (15, False), (16, False), (17, False), (65, True),
                                   (1331, False), (16411, False)])
def test_backward_row_counts(S, dev, n, odd):
    import paper_2009_12101_amd as cbg
    print(f"backward n={n} odd={odd}", flush=True)
    rng = np.random.default_rng(n)
    prm = random_params(S, 9)
    F = S.bf16(rng.standard_normal((n, 64)))
    H1, H2, _ = S.forward(F, prm["W1"], prm["b1"], prm["W2"], prm["b2"], prm["W3"], prm["b3"])
    dO = S.bf16(rng.standard_normal((n, 32)) * 1e-2)
    ref = S.backward(F, H1, H2, prm["W2"], prm["W3"], dO)
    _, weights = to_device(prm, dev)
    args = [bits_bf16(t).to(dev) for t in (F, H1, H2, dO)] + [weights]
    if odd:
        args = [odd_address(t) for t in args]
    got = split_grad(cbg.mlp_backward(*args).cpu().numpy())
    for k in ref:
        tol = 1e-5 if k in ("W3", "b3") else 1e-3
        assert np.linalg.norm(got[k] - ref[k]) <= tol * np.linalg.norm(ref[k]), k


def test_evaluation_equals_its_parts(S, dev):
    import paper_2009_12101_amd as cbg
    from paper_2009_12101_amd import problems as P
    A, K = P.lognormal27(9, 3), 17
    params, weights = to_device(random_params(S, 12), dev)
    Ad = cbg.DeviceCSR.from_host(A, dev)
    t, feat = cbg.csr_transpose_values(Ad), cbg.spai_features(Ad, A.grid)
    V = unit_vectors(A.n, K, 30).astype(np.float16)
    Vd = torch.from_numpy(V.T.copy().view(np.int16)).to(dev)
    loss = torch.zeros(1, dtype=torch.float64, device=dev)
    grad = torch.zeros(NPARAM, dtype=torch.float64, device=dev)
    cbg.spai_loss_grad(Ad, t, A.grid, feat, weights, params, Vd, 0.5, loss, grad)
    O, h1, h2 = cbg.mlp_forward(feat, weights, params, keep_activations=True)
    loss2, dP = cbg.spai_grad_p(Ad, t, cbg.spai_assemble(Ad, A.grid, O), Vd, 0.5)
    grad2 = cbg.mlp_backward(feat, h1, h2, cbg.spai_grad_o(Ad, A.grid, dP), weights)
    assert abs(loss.item() - loss2.item()) <= 1e-12 * loss2.item()
    g, g2 = split_grad(grad.cpu().numpy()), split_grad(grad2.cpu().numpy())
    for k in g:
        assert np.linalg.norm(g[k] - g2[k]) <= 1e-3 * np.linalg.norm(g2[k]), k
