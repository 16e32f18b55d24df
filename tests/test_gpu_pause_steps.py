"""The first hard step before, at and after the points where the host looks.

A diagonal with c tight clusters makes step c of the first cycle hard: the
cycle pauses there, and the host, which enqueues ahead and looks after 8 and 16
steps, runs the second pass and resumes.  Whatever was queued behind the
pause must have left no trace: one fp64 cycle of 28 steps has an orthonormal
basis and the residuals of the oracle's Fig. 1, with the bounds of the
near-breakdown tests (1e-12; 1e-6 on residuals above 1e-13 of the first).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from tests._helpers import FIG1
from tests.test_gpu_hard_steps import csr_diagonal


@pytest.mark.parametrize("c", [2, 7, 8, 9, 12, 15, 16, 17, 18])
def test_first_hard_step(orc, c):
    import paper_2009_12101_amd as cbg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    print(f"pause at step {c}", flush=True)
    n, m = 40 * c, 28
    rng = np.random.default_rng(c)
    A = csr_diagonal(np.tile(np.arange(1.0, c + 1), 40) * (1 + 1e-7 * rng.standard_normal(n)),
                     f"clusters_{c}")
    b = np.ones(n)
    kw = dict(restart=m, fmt="fp64", tol=0.0, maxiter=m)
    ref = orc.gmres(A, b, variant=FIG1, **kw)
    ws = torch.empty(cbg.workspace_bytes(n, m, "fp64"), dtype=torch.uint8, device=dev)
    r = cbg.solve(cbg.DeviceCSR.from_host(A, dev), torch.from_numpy(b).to(dev), workspace=ws, **kw)
    assert r.iterations == ref["iterations"] == m and r.breakdowns == ref["breakdowns"] == 0
    assert r.explicit_steps >= 1
    off, _ = cbg.workspace_basis(n, m, "fp64")
    ld = cbg.basis_ld(n)
    V = ws[off:off + m * ld * 8].view(torch.float64).reshape(m, ld)[:, :n].cpu().numpy()
    assert np.linalg.norm(np.eye(m) - V @ V.T) <= 1e-12
    k = int(np.sum(ref["hist"] > 1e-13 * ref["hist"][0]))
    assert np.allclose(r.hist[:k], ref["hist"][:k], rtol=1e-6, atol=0)
