"""The multi-dot and the update at the edges of their tiles and chunks.

Rows: one below, at and one above whole tiles (2048 and 4096 rows), a single
row, odd remainders.  Stored vectors: one, one more or less than a batch and
than a ring of batches, and counts whose multi-dot splits into several
chunks.  The entries of the basis beyond n (up to the leading dimension)
hold all-ones codes, which decode to NaN in the float formats: a kernel that
let them in would show it.  Compared with the oracle within the FP64 bounds
of a dot and of an update, |err| <= c * terms * 2^-53 * sum|terms|.
"""
import numpy as np
import pytest

from tests.test_gpu_kernels import U, _basis

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.mark.parametrize("fmt", ["fp64", "fp32", "fp16", "int16", "e4m3"])
@pytest.mark.parametrize("n,j", [(1, 5), (2047, 3), (2049, 17), (4095, 9), (4096, 16), (4097, 8),
                                 (12289, 33), (40961, 15)])
def test_tile_edges(orc, dev, fmt, n, j):
    import paper_2009_12101_amd as cbg
    print(f"tile edges {fmt} n={n} j={j}", flush=True)
    ld = (n + 15) // 16 * 16
    raw, dec, scales = _basis(orc, fmt, n, j, ld, seed=n + j)
    raw.view(np.uint8).reshape(j, -1)[:, n * raw.itemsize:] = 0xFF
    w = np.random.default_rng(n).standard_normal(n)
    Vd = torch.from_numpy(raw.view(np.uint8).reshape(-1)).to(dev)
    sd = torch.from_numpy(scales).to(dev)
    wd = torch.from_numpy(w).to(dev)
    h = cbg.multidot(fmt, Vd, ld, sd, n, j, wd).cpu().numpy()
    ho = dec @ w
    assert np.all(np.abs(h - ho) <= 4 * n * U * (np.abs(dec) @ np.abs(w)) + 1e-300)
    norms = cbg.update(fmt, Vd, ld, sd, n, j, torch.from_numpy(ho).to(dev), wd).cpu().numpy()
    w2 = wd.cpu().numpy()
    bound = 4 * (j + 1) * U * (np.abs(w) + np.abs(ho) @ np.abs(dec))
    assert np.all(np.abs(w2 - (w - ho @ dec)) <= bound)
    assert abs(norms[0] - np.linalg.norm(w2)) <= 1e-13 * norms[0]
    assert norms[1] == np.abs(w2).max()


@pytest.mark.parametrize("fmt", ["fp64", "fp32", "fp16", "e4m3"])
@pytest.mark.parametrize("nx", [1, 3, 45, 46, 90, 91, 128, 129, 181, 182])
def test_small_step_edges(orc, dev, fmt, nx):
    """Steps whose folds run inside the update (up to eight tiles) and the
    first sizes beyond: one ragged tile, tile counts of 1, 2, 4, 8 and 9 for
    2048 and 4096 rows.  Three steps with Jacobi, before stored entries can
    round differently, against the oracle's Fig. 1: residuals and x to 1e-12."""
    import paper_2009_12101_amd as cbg
    from paper_2009_12101_amd import problems as P
    A = P.poisson2d(nx)
    print(f"small step {fmt} n={A.n}", flush=True)
    b = P.rhs_uniform(A.n, nx)
    kw = dict(restart=10, fmt=fmt, tol=0.0, maxiter=3 if nx > 1 else 1, precond="jacobi")
    o = orc.gmres(A, b, **kw)
    r = cbg.solve(cbg.DeviceCSR.from_host(A, dev), torch.from_numpy(b).to(dev), **kw)
    assert r.iterations == o["iterations"]
    assert np.linalg.norm(r.x.cpu().numpy() - o["x"]) <= 1e-12 * np.linalg.norm(o["x"])
    assert np.allclose(r.hist, o["hist"], rtol=1e-12, atol=1e-15)


@pytest.mark.parametrize("m", [1, 8, 63, 64, 65, 127, 129, 200])
def test_back_substitution_sizes(orc, dev, m):
    """Whole cycles of m steps around the back substitution's row counts (64
    per register): x and the residuals of one fp64 cycle against the oracle."""
    import paper_2009_12101_amd as cbg
    from paper_2009_12101_amd import problems as P
    A = P.convdiff7(12)
    b = P.rhs_uniform(A.n, m)
    steps = min(m, 60)                   # the system converges soon after
    kw = dict(restart=m, fmt="fp64", tol=0.0, maxiter=steps)
    o = orc.gmres(A, b, **kw)
    r = cbg.solve(cbg.DeviceCSR.from_host(A, dev), torch.from_numpy(b).to(dev), **kw)
    assert r.iterations == o["iterations"]
    assert np.linalg.norm(r.x.cpu().numpy() - o["x"]) <= 1e-8 * np.linalg.norm(o["x"])


@pytest.mark.parametrize("first", [1791, 1792, 1793, 2048, 2049, 3071, 3072, 3073, 5000])
def test_spmv_product_buffer_edges(orc, dev, first):
    """CSR SpMV of 64-row blocks around one batch per thread (7 x 256) and
    the product buffer (3072): the first block holds `first` entries, the
    others 20 a row.  |err| <= (entries + 1) * 2^-53 * sum |a x| per row."""
    import scipy.sparse as sp
    from paper_2009_12101_amd.problems import CSR
    import paper_2009_12101_amd as cbg
    n = 64 * 40 + 17
    rng = np.random.default_rng(first)
    per = np.full(n, 20)
    per[:64] = first // 64
    per[:first % 64] += 1
    rp = np.concatenate([[0], np.cumsum(per)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in per]).astype(np.int32)
    A = sp.csr_matrix((rng.standard_normal(rp[-1]), ci, rp), shape=(n, n))
    x = rng.standard_normal(n)
    Ad = cbg.DeviceCSR.from_host(CSR(n, rp, ci, A.data), dev, sell=False)
    y = cbg.spmv(Ad, torch.from_numpy(x).to(dev)).cpu().numpy()
    bound = (per + 1) * 2.0 ** -53 * (abs(A) @ abs(x))
    ref = np.array([np.sum((A.data[a:b] * x[A.indices[a:b]]).astype(np.longdouble))
                    for a, b in zip(rp[:-1], rp[1:])], dtype=np.float64)
    assert np.all(np.abs(y - ref) <= bound)
