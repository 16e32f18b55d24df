"""What this framework is asked to do, as cases that can be timed and checked.

A case is a dict of plain values; its "kind" says which entry points it goes
through:

* solve: cbg.solve, the restarted method, as the benchmark (to a tolerance),
  the restart sweep and the training-vector generator (a fixed number of
  Arnoldi steps, tol = 0) call it; with pc = "learned" the stored
  preconditioner is built from the matrix first, inside the pass;
* train: one LearnedSPAI.step (forward, loss, backward, Adam) over a batch;
* build: the learned preconditioner's stored form from a matrix;
* spmv: y = A x (and ||y||) alone;
* orth: the multi-dot and the update (or the update with the re-dot) alone;
* dots: the multi-dot in its form for callers that do not allocate;
* codec: a vector stored through the accessor and read back.

The systems are the repository's own stencil families (problems.py), built
on the GPU from the case's sizes and the seed, and irregular rows (4 to 82
entries, the range of the paper's matrices) for which no sliced-ELL copy is
kept.
"""
from __future__ import annotations

import math

import torch

import paper_2009_12101_amd as cbg
from paper_2009_12101_amd.spai import Instance, LearnedSPAI

DEV = "cuda"
BYTES = cbg.FORMAT_BYTES
CODE_TYPE = {"fp64": torch.float64, "fp32": torch.float32, "fp16": torch.int16,
             "bf16": torch.int16, "e4m3": torch.uint8, "int32": torch.int32,
             "int16": torch.int16, "fp16s": torch.int16}
MAX_PADDING = 0.25          # DeviceCSR.from_host's limit for the sliced-ELL copy
NF, NH, NO = 64, 64, 32     # the network's layers
NPARAM = NF * NH + NH + NH * NH + NH + NH * NO + NO


def listed():
    return [
        # the small correctness system, solved to the tolerance: every kernel is
        # a few microseconds, the whole call is launches and their latency
        dict(name="poisson2d_64_tol", kind="solve", system="poisson2d", nx=64, ny=64, nz=1,
             fmt="fp64", pc="none", restart=100, steps=340, tol=1e-10),
        # a small system of the smoke check's size, short restarts, Jacobi
        dict(name="convdiff7_16_jacobi", kind="solve", system="convdiff7", nx=16, ny=16, nz=16,
             fmt="fp16", pc="jacobi", restart=30, steps=60, tol=0.0),
        # the cycle that supplies the preconditioner's training vectors
        dict(name="lognormal27_64_fp64", kind="solve", system="lognormal27", nx=64, ny=64, nz=64,
             fmt="fp64", pc="none", restart=100, steps=100, tol=0.0),
        # one cycle of the 7-point benchmark configuration
        dict(name="convdiff7_128_fp16", kind="solve", system="convdiff7", nx=128, ny=128, nz=128,
             fmt="fp16", pc="none", restart=100, steps=100, tol=0.0),
        # one cycle of the headline configuration, its preconditioner's build
        # included
        dict(name="lognormal27_160_learned", kind="solve", system="lognormal27", nx=160, ny=160,
             nz=160, fmt="fp16", pc="learned", restart=200, steps=200, tol=0.0),
        # a ragged grid with the fixed-point basis and Jacobi
        dict(name="lognormal27_95_int16", kind="solve", system="lognormal27", nx=95, ny=81, nz=70,
             fmt="int16", pc="jacobi", restart=50, steps=50, tol=0.0),
        # block-Jacobi (its set-up is part of the solve) with an fp32 basis
        dict(name="convdiff7_101_bj", kind="solve", system="convdiff7", nx=101, ny=90, nz=83,
             fmt="fp32", pc="block_jacobi", restart=40, steps=40, tol=0.0),
        # a training step at the training set's size
        dict(name="train_64", kind="train", nx=64, ny=64, nz=64, vectors=32, batch=2),
        # inference of the preconditioner on the held-out system
        dict(name="build_128", kind="build", nx=128, ny=128, nz=128),
        # a general sparse matrix, on the CSR arrays
        dict(name="spmv_irregular", kind="spmv", system="irregular", n=1000003, norm=True),
        # the orthogonalisation pair as a program with its own loop calls it
        dict(name="orth_bf16", kind="orth", fmt="bf16", n=1000003, j=50, redot=False),
        # a vector into its compressed form and back
        dict(name="codec_fp16", kind="codec", fmt="fp16", n=2097152),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, lo, hi):
    """An uneven grid of about _log(lo, hi) points."""
    n = _log(rng, lo, hi)
    nx = max(3, int(round(n ** (1 / 3) * rng.uniform(0.7, 1.4))))
    ny = max(3, int(round((n / nx) ** 0.5 * rng.uniform(0.8, 1.25))))
    return dict(nx=nx, ny=ny, nz=max(3, int(round(n / (nx * ny)))))


def draw(rng):
    kind = rng.choice(["solve"] * 6 + ["train", "build", "spmv", "spmv", "orth", "orth", "dots",
                                       "codec"])
    if kind == "solve":
        system = rng.choice(["convdiff7", "lognormal27"])
        # few steps on the coarse formats: a run's rounding travels through all
        # the steps that follow
        fmt = rng.choice(["fp64", "fp64", "fp32", "fp16", "fp16", "bf16", "int32", "int16"])
        m = rng.randint(15, 100 if BYTES[fmt] >= 4 else 50)
        pc = rng.choice(["none", "jacobi", "block_jacobi"] +
                        (["learned"] if system == "lognormal27" else []))
        return dict(kind=kind, system=system, **_grid(rng, 2000, 1500000), fmt=fmt, pc=pc,
                    restart=m, steps=m if BYTES[fmt] < 4 else m * rng.randint(1, 2), tol=0.0)
    if kind == "train":
        return dict(kind=kind, **_grid(rng, 4000, 262144), vectors=rng.choice([8, 17, 32]),
                    batch=rng.randint(1, 4))
    if kind == "build":
        return dict(kind=kind, **_grid(rng, 4000, 4000000))
    if kind == "spmv":
        system = rng.choice(["irregular", "convdiff7", "lognormal27"])
        size = dict(n=_log(rng, 2000, 2000000)) if system == "irregular" else \
            _grid(rng, 2000, 4000000)
        return dict(kind=kind, system=system, **size, norm=rng.random() < 0.5)
    fmt = rng.choice(sorted(BYTES))
    if kind == "orth":
        return dict(kind=kind, fmt=fmt, n=_log(rng, 3000, 2000000), j=_log(rng, 2, 120),
                    redot=rng.random() < 0.25)
    if kind == "dots":
        return dict(kind=kind, fmt=fmt, n=_log(rng, 3000, 500000), j=_log(rng, 2, 120))
    return dict(kind=kind, fmt=fmt, n=_log(rng, 3000, 4000000))


# ---------------------------------------------------------------- systems

def _offsets(system):
    if system == "poisson2d":
        return [(0, -1, 0), (0, 0, -1), (0, 0, 0), (0, 0, 1), (0, 1, 0)]
    if system == "convdiff7":
        return [(-1, 0, 0), (0, -1, 0), (0, 0, -1), (0, 0, 0), (0, 0, 1), (0, 1, 0), (1, 0, 0)]
    return [(dz, dy, dx) for dz in (-1, 0, 1) for dy in (-1, 0, 1) for dx in (-1, 0, 1)]


def _gen(seed, salt):
    return torch.Generator(device=DEV).manual_seed(1000003 * (seed % 2 ** 31) + salt)


class Stencil:
    """One value per row and stencil offset: val (offsets, n), 0 where the
    neighbour is outside the grid (mask false)."""

    def __init__(self, case, seed):
        system = case.get("system", "lognormal27")
        nx, ny, nz = self.grid = (case["nx"], case["ny"], case["nz"])
        n = self.n = nx * ny * nz
        offs = _offsets(system)
        i = torch.arange(n, device=DEV)
        x, y, z = i % nx, (i // nx) % ny, i // (nx * ny)
        self.shift = [dz * nx * ny + dy * nx + dx for dz, dy, dx in offs]
        self.mask = torch.stack([(x + dx >= 0) & (x + dx < nx) & (y + dy >= 0) & (y + dy < ny) &
                                 (z + dz >= 0) & (z + dz < nz) for dz, dy, dx in offs])
        self.val = torch.empty((len(offs), n), dtype=torch.float64, device=DEV)
        c = self.centre = offs.index((0, 0, 0))
        if system == "lognormal27":
            kap = torch.exp(torch.randn(n, dtype=torch.float64, device=DEV,
                                        generator=_gen(seed, 1)))
            self.val[c] = 1e-2
            for p, s in enumerate(self.shift):
                if p != c:
                    nb = torch.where(self.mask[p], self.at(i, s), i)
                    w = torch.sqrt(kap * kap[nb])
                    self.val[c] += w
                    self.val[p] = -w
        else:
            bh = 10.0 / (nx + 1) if system == "convdiff7" else 0.0
            for p, s in enumerate(self.shift):
                self.val[p] = -(1.0 + bh) if s < 0 else -1.0
            self.val[c] = 6.0 + 3.0 * bh if system == "convdiff7" else 4.0
        self.val *= self.mask

    def at(self, i, s):
        return torch.clamp(i + s, 0, self.n - 1)

    def csr(self):
        m = self.mask.t().contiguous()
        cols = torch.arange(self.n, device=DEV)[:, None] + torch.tensor(self.shift, device=DEV)
        rp = torch.zeros(self.n + 1, dtype=torch.int32, device=DEV)
        rp[1:] = torch.cumsum(m.sum(dim=1), 0)
        ci = cols.to(torch.int32)[m]
        return cbg.DeviceCSR(self.n, int(ci.numel()), rp, ci, self.val.t().contiguous()[m])

    def moved(self, v, s):
        """Row i of v at row i + s (rows outside [0, n) repeat an end)."""
        return v[self.at(torch.arange(self.n, device=DEV), s)]

    def times(self, v, val=None):
        """A v for v (n,) or (n, k)."""
        out = torch.zeros_like(v)
        for a, s in zip(self.val if val is None else val, self.shift):
            out += (a if v.dim() == 1 else a[:, None]) * self.moved(v, s)
        return out


def _irregular(case, seed):
    """Rows of 4 to 82 entries at sorted, irregularly spaced columns."""
    n, g = case["n"], _gen(seed, 2)
    lens = torch.exp(torch.empty(n, dtype=torch.float64, device=DEV).uniform_(
        math.log(4.0), math.log(83.0), generator=g)).to(torch.int64).clamp_(4, min(82, n))
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rp[1:] = torch.cumsum(lens, 0)
    nnz = int(rp[-1])
    row = torch.repeat_interleave(torch.arange(n, device=DEV), lens)
    gap = torch.randint(1, max(2, min(200, n // 83)), (nnz,), device=DEV, generator=g)
    run = torch.cumsum(gap, 0)
    run = run - run[rp[:-1]][row]
    span = run[rp[1:] - 1]
    first = torch.minimum(torch.clamp(torch.arange(n, device=DEV) - span // 2, min=0),
                          n - 1 - span)
    col = (first[row] + run).to(torch.int32)
    val = torch.randn(nnz, dtype=torch.float64, device=DEV, generator=g)
    return cbg.DeviceCSR(n, nnz, rp.to(torch.int32), col, val)


def _vector(n, seed, salt, unit=False):
    v = torch.randn(n, dtype=torch.float64, device=DEV, generator=_gen(seed, salt))
    return v / v.norm() if unit else v


def _rhs(n, seed):
    return torch.rand(n, dtype=torch.float64, device=DEV, generator=_gen(seed, 3)) * 2.0 - 1.0


def _params(seed):
    """The network as it is in the middle of training: the initial weights
    with a small random last layer and small biases (corrections of a few
    percent of the Jacobi rows)."""
    model = LearnedSPAI(DEV, seed)
    z = torch.randn(NPARAM, dtype=torch.float32, device=DEV, generator=_gen(seed, 4))
    w3 = NF * NH + NH + NH * NH + NH
    model.params[w3:] = 0.002 * z[w3:]
    model.params[NF * NH:NF * NH + NH] = 0.02 * z[NF * NH:NF * NH + NH]
    cbg.spai_round_weights(model.params, model.weights)
    return model


def _training_vectors(n, K, seed, k):
    V = torch.randn((n, K), dtype=torch.float64, device=DEV, generator=_gen(seed, 100 + k))
    return (V / V.norm(dim=0)).to(torch.float16)


# ---------------------------------------------------------------- prepare

def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case)
    if kind in ("solve", "build", "spmv"):
        irregular = case.get("system") == "irregular"
        A = _irregular(case, seed) if irregular else Stencil(case, seed).csr()
        s["A"] = A.build_sell(max_padding=MAX_PADDING)
    if kind == "solve":
        s["b"] = _rhs(A.n, seed)
        pc = "stencil" if case["pc"] == "learned" else case["pc"]
        s["ws"] = torch.empty(cbg.workspace_bytes(A.n, case["restart"], case["fmt"], pc),
                              dtype=torch.uint8, device=DEV)
    if kind == "build" or case.get("pc") == "learned":
        s["model"] = _params(seed)
        s["codes"] = torch.empty(27 * cbg.basis_ld(A.n), dtype=torch.int16, device=DEV)
        s["sws"] = torch.empty(cbg.spai_workspace_bytes(A.n, A.nnz, 0), dtype=torch.uint8,
                               device=DEV)
    if kind == "spmv":
        s["x"] = _vector(A.n, seed, 5)
        s["y"] = torch.empty_like(s["x"])
    if kind == "train":
        s["model"] = _params(seed)
        s["batch"] = []
        for k in range(case["batch"]):
            A = Stencil(case, 16 * seed + k).csr().build_sell(max_padding=MAX_PADDING)
            V = _training_vectors(A.n, case["vectors"], seed, k)
            s["batch"].append(Instance(A, (case["nx"], case["ny"], case["nz"]),
                                       cbg.csr_transpose_values(A),
                                       cbg.spai_features(A, (case["nx"], case["ny"], case["nz"])),
                                       V.view(torch.int16)))
        nnz = max(i.A.nnz for i in s["batch"])
        s["sws"] = torch.empty(cbg.spai_workspace_bytes(A.n, nnz, case["vectors"]),
                               dtype=torch.uint8, device=DEV)
    if kind in ("orth", "dots"):
        n, j, fmt = case["n"], case["j"], case["fmt"]
        ld = s["ld"] = cbg.basis_ld(n)
        V = torch.zeros((j, ld), dtype=CODE_TYPE[fmt], device=DEV)
        s["scales"] = torch.empty(j, dtype=torch.float64, device=DEV)
        for k in range(j):
            cbg.encode(fmt, _vector(n, seed, 1000 + k, unit=True), out=V[k],
                       scale=s["scales"][k:k + 1])
        s["V"] = V.view(-1)
        s["w0"] = _vector(n, seed, 6)
        s["w"] = s["w0"].clone()
        s["h"] = torch.empty(j, dtype=torch.float64, device=DEV)
        s["ws"] = torch.empty(cbg.kernel_workspace_bytes(n, j), dtype=torch.uint8, device=DEV)
    if kind == "codec":
        s["v"] = _vector(case["n"], seed, 7, unit=True)
        s["q"] = torch.empty(case["n"], dtype=CODE_TYPE[case["fmt"]], device=DEV)
        s["ws"] = torch.empty(cbg.kernel_workspace_bytes(case["n"], 0), dtype=torch.uint8,
                              device=DEV)
    return s


# ---------------------------------------------------------------- run

def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "solve":
        more = {}
        pc = c["pc"]
        if pc == "learned":
            s["model"].build_stencil(s["A"], (c["nx"], c["ny"], c["nz"]), ws=s["sws"],
                                     out=s["codes"])
            pc = "stencil"
            more = dict(p_stencil=s["codes"], grid=(c["nx"], c["ny"], c["nz"]))
        r = cbg.solve(s["A"], s["b"], restart=c["restart"], fmt=c["fmt"], tol=c["tol"],
                      maxiter=c["steps"] if c["tol"] == 0.0 else 10000, precond=pc,
                      workspace=s["ws"], hist=c["tol"] == 0.0, **more)
        return dict(x=r.x, hist=r.hist) if c["tol"] == 0.0 else dict(x=r.x)
    if kind == "train":
        m = s["model"]
        m.step(s["batch"], ws=s["sws"])
        return dict(loss=m.loss, params=m.params, m1=m.m1, m2=m.m2)
    if kind == "build":
        return s["model"].build_stencil(s["A"], (c["nx"], c["ny"], c["nz"]), ws=s["sws"],
                                        out=s["codes"])
    if kind == "spmv":
        return cbg.spmv(s["A"], s["x"], s["y"], want_norm=c["norm"])
    if kind == "dots":
        return cbg.multidot_noalloc(c["fmt"], s["V"], s["ld"], s["scales"], c["n"], c["j"],
                                    s["w"], s["h"])
    if kind == "orth":
        s["w"].copy_(s["w0"])            # the loop's next vector
        h = cbg.multidot(c["fmt"], s["V"], s["ld"], s["scales"], c["n"], c["j"], s["w"],
                         h=s["h"], ws=s["ws"])
        if c["redot"]:
            u, norms = cbg.update_redot(c["fmt"], s["V"], s["ld"], s["scales"], c["n"], c["j"],
                                        h, s["w"], ws=s["ws"])
            return dict(h=h, w=s["w"], u=u, norms=norms)
        norms = cbg.update(c["fmt"], s["V"], s["ld"], s["scales"], c["n"], c["j"], h, s["w"],
                           ws=s["ws"])
        return dict(h=h, w=s["w"], norms=norms)
    q, scale = cbg.encode(c["fmt"], s["v"], out=s["q"], ws=s["ws"])
    return dict(q=q, scale=scale, v=cbg.decode(c["fmt"], q, scale))


# ---------------------------------------------------------------- work

def _entries(c):
    system = c.get("system", "lognormal27")
    if system == "irregular":
        return c["n"], int(26.0 * c["n"])
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    n = nx * ny * nz
    if system == "lognormal27":
        return n, (3 * nx - 2) * (3 * ny - 2) * (3 * nz - 2)
    if system == "convdiff7":
        return n, 7 * n - 2 * (nx * ny + ny * nz + nx * nz)
    return n, 5 * n - 2 * (nx + ny)


def work(c):
    kind = c["kind"]
    if kind in ("orth", "dots", "codec"):
        n, bs = c["n"], BYTES[c["fmt"]]
        if kind == "codec":
            return dict(bytes=n * (16 + 2 * bs), flops=n)
        j = c["j"]
        if kind == "dots":
            return dict(bytes=j * n * bs + 8 * n, flops=2 * j * n)
        # the dots need all of the basis before the update can begin
        return dict(bytes=2 * j * n * bs + 40 * n, flops=(6 if c["redot"] else 4) * j * n)
    n, nnz = _entries(c)
    matrix = 12 * nnz + 4 * n
    mlp = 2 * n * (NF * NH + NH * NH + NH * NO)
    if kind == "spmv":
        return dict(bytes=matrix + 16 * n, flops=2 * nnz)
    if kind == "build":
        return dict(bytes=matrix + 54 * n, flops=mlp)
    if kind == "train":
        K = c["vectors"]
        # A, A^T's values, the features and the vectors once; three sparse
        # products over K vectors and their gradient, the network both ways
        per = matrix + 8 * nnz + 2 * NF * n + 2 * K * n
        return dict(bytes=c["batch"] * per, flops=c["batch"] * (8 * nnz * K + 3 * mlp))
    bs, m = BYTES[c["fmt"]], c["restart"]
    total, flops = 0.0, 0.0
    for j in (k % m + 1 for k in range(c["steps"])):
        pre = {"none": 0, "jacobi": 8 * n, "block_jacobi": 8 * n, "learned": 62 * n}[c["pc"]]
        total += matrix + pre + 16 * n + 2 * j * n * bs + n * bs
        flops += 2 * nnz + 6 * j * n
    if c["pc"] == "learned":
        total += matrix + 54 * n
        flops += mlp
    return dict(bytes=total, flops=flops)


# ---------------------------------------------------------------- exact

def _bf16(v):
    return v.to(torch.bfloat16).to(torch.float64)


def _network(S, params):
    """(F, H1, H2, O, weights): the features and layers as the network is
    defined, with its bf16 rounding points, in 64 bits otherwise."""
    d = S.val[S.centre]
    F = torch.zeros((S.n, NF), dtype=torch.float64, device=DEV)
    off = torch.zeros_like(d)
    for p, s in enumerate(S.shift):
        F[:, p] = S.val[p] / d
        F[:, 32 + p] = torch.where(S.mask[p], S.moved(d, s) / d, 0.0)
        if p != S.centre:
            off += S.val[p].abs()
    F[:, 27] = (d - off) / d
    F = _bf16(F.to(torch.float32))
    P = params.to(torch.float64)
    o, W = 0, []
    for a, b in ((NF, NH), (NH, NH), (NH, NO)):
        W.append((_bf16(P[o:o + a * b]).view(a, b), P[o + a * b:o + a * b + b]))
        o += a * b + b
    H1 = _bf16(torch.relu(F @ W[0][0] + W[0][1]))
    H2 = _bf16(torch.relu(H1 @ W[1][0] + W[1][1]))
    return F, H1, H2, H2 @ W[2][0] + W[2][1], W


def _inverse(S, case, seed):
    """M^-1 as a function, in 64 bits (block-Jacobi: the blocks' inverses as
    they are before storage)."""
    d = S.val[S.centre]
    if case["pc"] == "none":
        return lambda v: v
    if case["pc"] == "jacobi":
        return lambda v: v / d
    if case["pc"] == "learned":
        o = _network(S, _params(seed).params)[3][:, :len(S.shift)].t()
        o = o.to(torch.float16).to(torch.float64) * S.mask
        o[S.centre] += 1.0
        return lambda v: S.times(v, o) / d
    bs = 4
    nb = -(-S.n // bs)
    D = torch.zeros((nb * bs, bs), dtype=torch.float64, device=DEV)
    D[S.n:] = torch.eye(bs, dtype=torch.float64, device=DEV)[
        torch.arange(S.n, nb * bs, device=DEV) % bs]
    i = torch.arange(S.n, device=DEV)
    for p, s in enumerate(S.shift):
        k = i % bs + s
        ok = S.mask[p] & (k >= 0) & (k < bs)
        D[i[ok], k[ok]] = S.val[p][ok]
    D = D.view(nb, bs, bs)
    X = torch.eye(bs, dtype=torch.float64, device=DEV).repeat(nb, 1, 1)
    for c in range(bs):                  # the diagonal dominates: no pivoting
        piv = D[:, c, c].clone()[:, None]
        D[:, c], X[:, c] = D[:, c] / piv, X[:, c] / piv
        for r in range(bs):
            if r != c:
                f = D[:, r, c].clone()[:, None]
                D[:, r], X[:, r] = D[:, r] - f * D[:, c], X[:, r] - f * X[:, c]

    def apply(v):
        u = torch.zeros(nb * bs, dtype=torch.float64, device=DEV)
        u[:S.n] = v
        return (X * u.view(nb, 1, bs)).sum(dim=2).view(-1)[:S.n]
    return apply


def _gmres(S, b, inverse, restart, steps):
    """Restarted GMRES in 64 bits (two Gram-Schmidt passes a step, least
    squares by Givens rotations): x and the relative residual of each step."""
    x, nb, hist = torch.zeros_like(b), float(b.norm()), []
    left = steps
    while left > 0:
        m = min(restart, left)
        left -= m
        r = b - S.times(x)
        beta = float(r.norm())
        V = torch.empty((m + 1, S.n), dtype=torch.float64, device=DEV)
        V[0] = r / beta
        R = torch.zeros((m, m), dtype=torch.float64)
        g, rot = [beta], []
        for j in range(m):
            w = S.times(inverse(V[j]))
            h = torch.zeros(j + 1, dtype=torch.float64, device=DEV)
            for _ in range(2):
                u = (V[:j + 1] * w).sum(dim=1) if S.n * (j + 1) < 2 ** 26 else V[:j + 1] @ w
                h += u
                w = w - u @ V[:j + 1]
            t = float(w.norm())
            V[j + 1] = w / t if t else w
            col = h.tolist()
            for k, (c, sn) in enumerate(rot):
                col[k], col[k + 1] = c * col[k] + sn * col[k + 1], -sn * col[k] + c * col[k + 1]
            rr = math.hypot(col[j], t)
            rot.append((col[j] / rr, t / rr))
            R[:j, j], R[j, j] = torch.tensor(col[:j], dtype=torch.float64), rr
            g.append(-t / rr * g[j])
            g[j] *= col[j] / rr
            hist.append(abs(g[j + 1]) / nb)
        y = torch.linalg.solve_triangular(R, torch.tensor(g[:m], dtype=torch.float64)[:, None],
                                          upper=True)[:, 0]
        x = x + inverse(y.to(DEV) @ V[:m])
    return x, torch.tensor(hist, dtype=torch.float64)


def _exact_training(case, seed):
    model = _params(seed)
    grad, loss = torch.zeros(NPARAM, dtype=torch.float64, device=DEV), 0.0
    scale = 1.0 / (case["vectors"] * case["batch"])
    for k in range(case["batch"]):
        S = Stencil(case, 16 * seed + k)
        V = _training_vectors(S.n, case["vectors"], seed, k).to(torch.float64)
        F, H1, H2, O, W = _network(S, model.params)
        d = S.val[S.centre]
        o = O[:, :27].t().clone()
        o[S.centre] += 1.0
        R = S.times(S.times(V, (o / d * S.mask).to(torch.float32).to(torch.float64))) - V
        loss = loss + scale * float((R * R).sum())
        # A^T: the entry (c, i) for the slot of (i, c)
        last = len(S.shift) - 1
        t = torch.stack([torch.where(S.mask[p], S.moved(S.val[last - p], s), 0.0)
                         for p, s in enumerate(S.shift)])
        G = 2.0 * scale * S.times(R, t)
        dO = torch.zeros((S.n, NO), dtype=torch.float64, device=DEV)
        for p, s in enumerate(S.shift):
            dO[:, p] = torch.where(S.mask[p], (G * S.moved(V, s)).sum(dim=1) / d, 0.0)
        dO = _bf16(dO)
        d2 = _bf16((dO @ W[2][0].t()) * (H2 > 0))
        d1 = _bf16((d2 @ W[1][0].t()) * (H1 > 0))
        grad += torch.cat([(F.t() @ d1).reshape(-1), d1.sum(0), (H1.t() @ d2).reshape(-1),
                           d2.sum(0), (H2.t() @ dO).reshape(-1), dO.sum(0)])
    m1, m2 = 0.1 * grad, 0.001 * grad * grad
    step = 1e-3 * (m1 / 0.1) / (torch.sqrt(m2 / 0.001) + 1e-8)
    return dict(loss=torch.tensor([loss], dtype=torch.float64),
                params=model.params.to(torch.float64) - step, m1=m1, m2=m2)


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        S = Stencil(case, seed)
        b, inv = _rhs(S.n, seed), _inverse(S, case, seed)
        if case["tol"] == 0.0:
            x, hist = _gmres(S, b, inv, case["restart"], case["steps"])
            return dict(x=x, hist=hist)
        # far past the tolerance: the solution
        return dict(x=_gmres(S, b, inv, 300, 300)[0])
    if kind == "train":
        return _exact_training(case, seed)
    if kind == "build":
        return None                      # float16 codes, held as whole numbers
    if kind == "spmv":
        x = _vector(_entries(case)[0], seed, 5)
        if case["system"] == "irregular":
            A = _irregular(case, seed)
            row = torch.repeat_interleave(torch.arange(A.n, device=DEV),
                                          (A.row_ptr[1:] - A.row_ptr[:-1]).to(torch.int64))
            y = torch.zeros_like(x).index_add_(0, row, A.val * x[A.col_idx.to(torch.int64)])
        else:
            y = Stencil(case, seed).times(x)
        return (y, y.norm().reshape(1)) if case["norm"] else y
    if kind == "codec":
        return dict(q=None, scale=None, v=_vector(case["n"], seed, 7, unit=True))
    n, j, fmt = case["n"], case["j"], case["fmt"]
    if fmt == "e4m3":
        return None                      # 4 significant bits: the stored vectors are others
    V = torch.stack([_vector(n, seed, 1000 + k, unit=True) for k in range(j)])
    w = _vector(n, seed, 6)
    h = (V * w).sum(dim=1)
    if kind == "dots":
        return h
    w = w - h @ V
    out = dict(h=h, w=w, norms=torch.stack([w.norm(), w.abs().max()]))
    if case["redot"]:
        # what the first pass leaves is of the size of a 16-bit vector's rounding
        out["u"] = (V * w).sum(dim=1) if BYTES[fmt] >= 4 else None
    return out
