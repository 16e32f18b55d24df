"""Back substitution over whole cycles of m columns.

The kernel keeps 64 rows per register and lane (one, two, four or eight of
them by the restart length) and eight columns in flight: cycles that end one
before, at and one after a register's last row, and lengths of the widest
form.  2D Poisson on 160 x 160 is far from converged after 300 steps, so every
cycle reaches its m.  fp64 basis against the oracle's Fig. 1, with the bounds
of the longest restart's test (residuals 1e-9, x 1e-8), and once more with a
restart longer than the cycle, where the last registers hold no column.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from tests._helpers import FIG1


@pytest.fixture(scope="module")
def system():
    from paper_2009_12101_amd import problems as P
    A = P.poisson2d(160)
    return A, P.rhs_uniform(A.n, 3)


@pytest.mark.parametrize("m,steps", [(63, 63), (64, 64), (65, 65), (127, 127), (128, 128),
                                     (129, 129), (200, 200), (256, 256), (257, 257), (300, 300),
                                     (300, 1), (256, 129), (128, 64)])
def test_whole_cycles(orc, system, m, steps):
    import paper_2009_12101_amd as cbg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    A, b = system
    print(f"back substitution m={m} steps={steps}", flush=True)
    kw = dict(restart=m, fmt="fp64", tol=0.0, maxiter=steps)
    o = orc.gmres(A, b, variant=FIG1, **kw)
    r = cbg.solve(cbg.DeviceCSR.from_host(A, dev), torch.from_numpy(b).to(dev), **kw)
    assert o["iterations"] == r.iterations == steps and o["cycle_len"][0] == steps
    assert np.allclose(r.hist, o["hist"], rtol=1e-9, atol=0)
    assert np.linalg.norm(r.x.cpu().numpy() - o["x"]) <= 1e-8 * np.linalg.norm(o["x"])
