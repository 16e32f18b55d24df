"""prof_spmv_bytes counts the SpMV kernel that was timed.

Steps 13-14 run in a pass of their own, after which the step's SpMV is the
plain product, or inside the SpMV's gather, which also reads w, divides it
and stores v_j.  The three ways to ask for it (pass, gather, the solver's own
choice) give the same iterates, so the solver's choice must report the bytes
of one of the other two: of the gather on small systems, of the pass on
larger ones.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def spmv_bytes(dev, A, how, **kw):
    import paper_2009_12101_amd as cbg
    from paper_2009_12101_amd import problems as P
    b = torch.from_numpy(P.rhs_uniform(A.n, 5)).to(dev)
    r = cbg.solve(cbg.DeviceCSR.from_host(A, dev), b, restart=16, tol=0.0, maxiter=16,
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
