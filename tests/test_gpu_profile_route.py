"""prof_spmv_bytes counts the SpMV kernel that was timed.

Steps 13-14 run in a pass of their own, after which the step's SpMV is the
plain product, or inside the SpMV's gather, which also reads w, divides it
and stores v_j.  The three ways to ask for it (pass, gather, the solver's own
choice) give the same iterates, so the solver's choice must report the bytes
of one of the other two: of the gather on small systems whose rows are known
to be short (a sliced-ELL copy of at most 32 diagonals), of the pass on larger
ones and on rows that may be long, which a division per entry slows down.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def spmv_bytes(dev, A, how, sell=True, **kw):
    import paper_2009_12101_amd as cbg
    from paper_2009_12101_amd import problems as P
    b = torch.from_numpy(P.rhs_uniform(A.n, 5)).to(dev)
    r = cbg.solve(cbg.DeviceCSR.from_host(A, dev, sell=sell), b, restart=16, tol=0.0, maxiter=16,
                  normalise=how, profile="spmv", **kw)
    assert r.iterations == r.prof_spmv_launches == 16
    return r.prof_spmv_bytes


@pytest.mark.parametrize("nx,own", [(11, "gather"), (40, "gather"), (41, "pass")])
@pytest.mark.parametrize("fmt,precond", [("fp16", "none"), ("fp64", "jacobi"), ("e4m3", "jacobi")])
def test_bytes_of_the_launched_kernel(dev, nx, own, fmt, precond):
    from paper_2009_12101_amd import problems as P
    print(f"profile route {nx} {fmt} {precond}", flush=True)
    A = P.lognormal27(nx, 4)
    kw = dict(fmt=fmt, precond=precond)
    by = {how: spmv_bytes(dev, A, how, **kw) for how in ("pass", "gather", "auto")}
    assert by["pass"] < by["gather"]
    assert by["auto"] == by[own]


def diagonals(n, count):
    """`count` diagonals at distances 0, 3, 6, ... above and below."""
    import scipy.sparse as sp
    from tests._helpers import csr_from_scipy
    offs = [0] + [s * 3 * k for k in range(1, count) for s in (1, -1)]
    rng = np.random.default_rng(count)
    return csr_from_scipy(sp.diags([4.0 * (d == 0) + rng.uniform(-1, 1, n - abs(d)) / count
                                    for d in offs[:count]], offs[:count]))


def one_long_row(n):
    """Tridiagonal, and a row with an entry in every third column."""
    import scipy.sparse as sp
    from tests._helpers import csr_from_scipy
    M = sp.diags([np.full(n - 1, -1.0), np.full(n, 4.0), np.full(n - 1, -1.0)],
                 [-1, 0, 1]).tolil()
    M[n // 2, ::3] = 0.01
    M[n // 2, n // 2] = 4.0
    return csr_from_scipy(M.tocsr())


@pytest.mark.parametrize("system,sell,own", [
    ("diag31", True, "gather"), ("diag32", True, "gather"), ("diag33", True, "pass"),
    ("diag31", False, "pass"), ("long_row", False, "pass"), ("long_row", True, "pass")])
def test_rows_that_may_be_long_keep_the_pass(dev, system, sell, own):
    A = one_long_row(3000) if system == "long_row" else diagonals(3000, int(system[4:]))
    print(f"profile route {system} sell={sell}", flush=True)
    kw = dict(fmt="fp16", precond="jacobi", sell=sell)
    by = {how: spmv_bytes(dev, A, how, **kw) for how in ("pass", "gather", "auto")}
    assert by["pass"] < by["gather"]
    assert by["auto"] == by[own]
