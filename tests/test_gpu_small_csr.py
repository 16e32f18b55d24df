"""Small steps on the CSR arrays, where the SpMV leaves many partials.

Small steps fold the SpMV's partials of omega^2 = ||A M^-1 v||^2 inside the
update.  Without a sliced-ELL copy the SpMV runs one block per 64 rows (one
per 32 rows beyond 60 entries a row on average): up to 448 partials on the
largest small step (14,336 rows of fp64), and 512 or 1024 on a step of eight
tiles.  Below, at and above the 64 that a lane of each of the four waves takes
at once (256 partials), on the last small step and beyond it.

A lost partial shows in step 7's test and in t1^2 = omega^2 - h^T h - h^T u:
three steps, before stored entries can round differently, follow the oracle's
Fig. 1 with residuals and x to 1e-12 and the same count of
re-orthogonalisations; none of them is hard (t1 stays above 0.2 omega on these
systems), and they take the same forms as on the sliced-ELL copy, which has a
quarter of the partials.
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


def random_rows(n, mean, seed):
    """n rows of mean / 2 to 3 mean / 2 entries: a positive diagonal, the other
    columns within 200 of it, off-diagonal rows about as long as the diagonal.
    The rows of the last partial of the first wave's quarter are 30 times the
    others, so that omega^2 hangs on that partial."""
    from paper_2009_12101_amd.problems import CSR
    rng = np.random.default_rng(seed)
    per = rng.integers(mean // 2, mean + mean // 2 + 1, n)
    rp = np.concatenate([[0], np.cumsum(per)]).astype(np.int32)
    rows = 32 if mean > 60 else 64
    heavy = -(-(-(-n // rows)) // 4) - 1
    cols, vals = [], []
    for i, k in enumerate(per):
        lo, hi = max(0, i - 200), min(n, i + 201)
        c = rng.choice(np.delete(np.arange(lo, hi), i - lo), k - 1, replace=False)
        c = np.sort(np.append(c, i))
        v = rng.uniform(-6.0, 6.0, k) / np.sqrt(k)
        v[c == i] = 1.0 + 9.0 * rng.random()
        cols.append(c)
        vals.append(30.0 * v if i // rows == heavy else v)
    return CSR(n, rp, np.concatenate(cols).astype(np.int32), np.concatenate(vals))


SYSTEMS = {
    # 27-point rows, 64 rows a block: 244 and 275 partials, then 512
    "stencil_25": lambda P: P.lognormal27(25, 4),
    "stencil_26": lambda P: P.lognormal27(26, 4),
    "stencil_32": lambda P: P.lognormal27(32, 4),
    # uneven rows, 64 rows a block: 256, 260, 313, 512 and (not small) 516
    "rows26_16384": lambda P: random_rows(16384, 26, 1),
    "rows26_16385": lambda P: random_rows(16385, 26, 2),
    "rows26_20000": lambda P: random_rows(20000, 26, 3),
    "rows26_32768": lambda P: random_rows(32768, 26, 4),
    "rows26_32769": lambda P: random_rows(32769, 26, 5),
    # the last small step of the 4-byte and of the 16-bit formats, and beyond
    "rows26_6144": lambda P: random_rows(6144, 26, 12),
    "rows26_6145": lambda P: random_rows(6145, 26, 13),
    "rows26_8192": lambda P: random_rows(8192, 26, 14),
    "rows26_8193": lambda P: random_rows(8193, 26, 15),
    # long rows, 32 rows a block: 256, 264, 448, (not small) 456, 512 and 1024
    "rows70_8192": lambda P: random_rows(8192, 70, 6),
    "rows70_8448": lambda P: random_rows(8448, 70, 7),
    "rows70_14336": lambda P: random_rows(14336, 70, 10),
    "rows70_14592": lambda P: random_rows(14592, 70, 11),
    "rows70_16384": lambda P: random_rows(16384, 70, 8),
    "rows70_32768": lambda P: random_rows(32768, 70, 9),
}


@pytest.mark.parametrize("system,fmt,precond", [
    ("stencil_25", "fp16", "none"), ("stencil_26", "fp16", "none"),
    ("stencil_26", "e4m3", "jacobi"), ("stencil_32", "fp16", "none"),
    ("stencil_32", "int16", "jacobi"),
    ("rows26_16384", "fp16", "none"), ("rows26_16385", "fp16", "none"),
    ("rows26_20000", "bf16", "none"), ("rows26_32768", "e4m3", "none"),
    ("rows26_32769", "fp16", "none"),
    ("rows26_6144", "fp32", "none"), ("rows26_6144", "int32", "none"),
    ("rows26_6145", "fp32", "none"), ("rows26_6145", "int32", "jacobi"),
    ("rows26_8192", "fp16", "none"), ("rows26_8192", "int16", "none"),
    ("rows26_8193", "fp16", "none"), ("rows26_8193", "fp16s", "none"),
    ("rows70_8192", "fp64", "none"), ("rows70_8448", "fp64", "none"),
    ("rows70_14336", "fp64", "none"), ("rows70_14336", "fp64", "jacobi"),
    ("rows70_14592", "fp64", "none"), ("rows70_16384", "fp64", "jacobi"), ("rows70_16384", "fp32", "none"),
    ("rows70_32768", "fp16", "none"), ("rows70_32768", "fp16", "jacobi")])
def test_omega_counts_every_partial(orc, dev, system, fmt, precond):
    import paper_2009_12101_amd as cbg
    from paper_2009_12101_amd import problems as P
    A = SYSTEMS[system](P)
    print(f"small CSR steps {system} {fmt} {precond} n={A.n}", flush=True)
    b = P.rhs_uniform(A.n, 3)
    kw = dict(restart=10, fmt=fmt, tol=0.0, maxiter=3, precond=precond)
    o = orc.gmres(A, b, **kw)
    bd = torch.from_numpy(b).to(dev)
    r = cbg.solve(cbg.DeviceCSR.from_host(A, dev, sell=False), bd, **kw)
    assert r.iterations == o["iterations"]
    assert r.reorths == o["reorths"]
    assert r.explicit_steps == 0
    assert np.linalg.norm(r.x.cpu().numpy() - o["x"]) <= 1e-12 * np.linalg.norm(o["x"])
    assert np.allclose(r.hist, o["hist"], rtol=1e-12, atol=1e-15)
    s = cbg.solve(cbg.DeviceCSR.from_host(A, dev, sell=True), bd, **kw)
    assert s.reorths == r.reorths and s.explicit_steps == 0
