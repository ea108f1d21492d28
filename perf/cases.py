"""Workloads of the framework's public entry points, for timing and checking.

``listed()`` names the cases, ``draw(rng)`` gives one more of the same
ranges, ``prepare(case, seed)`` builds what a program holds before the call
(operator, blocks), ``run(state)`` makes the call, ``work(case)`` counts the
bytes and operations it cannot do without and ``exact(case, seed)`` computes
the same outputs with plain torch in FP64.

Sizes are those of this repository's workloads: boxes of 2 bohr cells of
order 2..7 (mostly 4, 5 and 6) up to 24^3 cells at p = 6 (2,985,984 nodes),
blocks of 1 to 256 columns, filter degrees up to 30.
"""
import math

import numpy as np
import torch

import paper_2203_07820_amd as lib
import workloads

PREC = {"f64": lib.F64, "f32": lib.F32, "bf16": lib.BF16, "c128": lib.C128, "c64": lib.C64}
DTYPE = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.float32,
         "c128": torch.complex128, "c64": torch.complex64}


def listed():
    return [
        # one H~X on a full column block at production size: the Rayleigh-Ritz
        # product of every pass, and the unit every filter step is made of
        {"name": "apply_f64_p6_24", "kind": "apply", "p": 6, "nc": 24, "atoms": 64, "ncols": 128, "prec": "f64"},
        # the same in single precision (the mixed-precision filter's step)
        {"name": "apply_f32_p6_24", "kind": "apply", "p": 6, "nc": 24, "atoms": 64, "ncols": 128, "prec": "f32"},
        # bf16 products, the first pass of the precision schedule
        {"name": "apply_bf16_p6_12", "kind": "apply", "p": 6, "nc": 12, "atoms": 16, "ncols": 128, "prec": "bf16"},
        # the largest Bloch operator of the k-point workload
        {"name": "apply_c128_p5_20", "kind": "apply", "p": 5, "nc": 20, "atoms": 48, "ncols": 128, "prec": "c128"},
        # the Chebyshev filter of one column block, the bulk of a pass
        {"name": "filter_f64_p6_24", "kind": "filter", "p": 6, "nc": 24, "atoms": 64, "ncols": 128, "m": 30,
         "block": 128, "prec": "f64"},
        # the filter of a mid-size box, wanted and buffer columns in one ragged block
        {"name": "filter_f64_p5_12", "kind": "filter", "p": 5, "nc": 12, "atoms": 16, "ncols": 160, "m": 30,
         "block": 160, "prec": "f64"},
        # many small Bloch problems in one batched filter
        {"name": "batch_c128_p5_small", "kind": "batch", "p": 5, "nprob": 16, "mix": 1, "m": 20, "prec": "c128"},
        # one whole pass of a small problem: launches and latency
        {"name": "pass_f64_p4_4", "kind": "pass", "p": 4, "nc": 4, "atoms": 2, "ncols": 32, "m": 20, "prec": "f64"},
        # the spectrum's upper bound at the start of a solve: one vector, one product after another
        {"name": "bounds_f64_p5_12", "kind": "bounds", "p": 5, "nc": 12, "atoms": 16, "ncols": 1, "prec": "f64"},
        # Cholesky-Gram-Schmidt of a whole subspace at production size
        {"name": "ortho_f64_p6_24", "kind": "ortho", "p": 6, "nc": 24, "atoms": 0, "ncols": 256, "prec": "f64"},
        # spectrum-splitting Rayleigh-Ritz of an SCF step
        {"name": "split_f64_p5_12", "kind": "split", "p": 5, "nc": 12, "atoms": 16, "ncols": 160, "nfr": 32,
         "prec": "f64"},
        # the electron density at the Gauss points of every cell
        {"name": "density_p6_12", "kind": "density", "p": 6, "nc": 12, "atoms": 16, "ncols": 192, "points": "gauss",
         "prec": "f64"},
    ]


def _loguni(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["apply"] * 5 + ["filter"] * 3 + ["batch", "pass", "bounds", "ortho", "split", "density"])
    p = rng.choice([2, 3, 4, 4, 5, 5, 5, 6, 6, 6, 7])
    # nodes per side up to 144, at least 2 cells per side
    nc = max(2, _loguni(rng, 8, 144) // p)
    M = (nc * p) ** 3
    c = {"kind": kind, "p": p, "nc": nc, "atoms": max(1, min(64, nc ** 3 // 100 + rng.randint(0, 3)))}
    if kind == "apply":
        c["prec"] = rng.choice(["f64", "f64", "f64", "f32", "f32", "bf16", "c128", "c128", "c64"])
        c["ncols"] = _loguni(rng, 1, min(256 if M < 1e6 else 128, M))
    elif kind == "filter":
        c["prec"] = rng.choice(["f64", "f64", "c128"])
        c["ncols"] = _loguni(rng, 1, min(256 if M < 1e6 else 64, M))
        c["m"] = rng.randint(2, 30)
        c["block"] = rng.choice([c["ncols"], max(1, c["ncols"] // 2), 64])
    elif kind == "batch":
        c = {"kind": kind, "p": rng.choice([4, 5, 5]), "nprob": _loguni(rng, 2, 16), "mix": rng.randint(2, 999),
             "m": rng.randint(5, 20), "prec": rng.choice(["f64", "c128"])}
    elif kind == "pass":
        c["nc"] = rng.randint(3, 6)
        c["p"] = rng.choice([3, 4, 5])
        c["atoms"] = rng.randint(1, 4)
        c["ncols"] = rng.randint(12, 48)
        c["m"] = rng.randint(8, 20)
        c["prec"] = rng.choice(["f64", "c128"])
    elif kind == "bounds":
        c["ncols"] = 1
        c["prec"] = rng.choice(["f64", "c128"])
    else:
        c["ncols"] = _loguni(rng, 8, min(256, M // 8))
        c["prec"] = rng.choice(["f64", "f64", "c128"])
        if kind == "split":
            c["nfr"] = max(1, c["ncols"] // rng.randint(3, 10))
        if kind == "density":
            c["points"] = rng.choice(["gauss", "nodes"])
    return c


# ---- inputs -----------------------------------------------------------------
def _system(nc, p, atoms, seed, cplx, index=0):
    L = 2.0 * nc
    s = workloads.make_system(L, nc, p, atoms, seed=seed % (2 ** 31) + index, d_min=min(1.0, L / 4),
                              has_proj=atoms > 0)
    return s.with_k(workloads.kpoints_mp4(L)[(seed + index) % 4]) if cplx else s


def _is_complex(c):
    return c["prec"] in ("c128", "c64")


def _batch_shapes(c):
    rng = np.random.default_rng(c["mix"])
    return [(int(rng.integers(3, 7)), int(rng.integers(2, 7)), int(rng.integers(16, 49))) for _ in range(c["nprob"])]


def _systems(c, seed):
    cplx = _is_complex(c)
    if c["kind"] == "batch":
        return [_system(nc, c["p"], na, seed, cplx, i) for i, (nc, na, _) in enumerate(_batch_shapes(c))]
    return [_system(c["nc"], c["p"], c["atoms"], seed, cplx)]


def _block(s, ncols, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(s.M, ncols, dtype=dtype, device="cuda", generator=g)


def _subspace_block(s, ncols, dtype, seed):
    """A block as a filter leaves it: columns mixed from directions of uneven weight."""
    X = _block(s, ncols, dtype, seed)
    g = torch.Generator(device="cuda").manual_seed(seed + 1)
    R = torch.linalg.qr(torch.randn(ncols, ncols, dtype=dtype, device="cuda", generator=g))[0]
    w = torch.logspace(0, -2, ncols, dtype=torch.float64, device="cuda")
    return (X * w) @ R


def _blocks(c, systems, seed):
    dt = DTYPE[c["prec"]]
    if c["kind"] == "batch":
        return [_block(s, n, dt, seed + 7 * i) for i, (s, (_, _, n)) in enumerate(zip(systems, _batch_shapes(c)))]
    if c["kind"] in ("ortho", "split"):
        return [_subspace_block(systems[0], c["ncols"], dt, seed)]
    return [_block(systems[0], c["ncols"], dt, seed)]


def _interval(s):
    """(a, b, aL) of the filter: b bounds the spectrum from above."""
    f = _Fe(s)
    b = 1.05 * 1.5 * f.kmax * f.mmax ** 2 + 10.0
    return 0.1 * b, b, -5.0


def _weights(c, seed):
    return np.random.default_rng(seed).uniform(0.0, 2.0, c["ncols"])


def prepare(case, seed):
    c = case
    systems = _systems(c, seed)
    ctx = lib.Context(0)
    st = {"case": c, "ctx": ctx, "ops": [lib.Operator(ctx, s) for s in systems], "X0": _blocks(c, systems, seed),
          "prec": PREC[c["prec"]]}
    k = c["kind"]
    if k == "apply":
        st["Y"] = torch.empty_like(st["X0"][0])
    elif k != "bounds" and k != "density":
        # calls that work in place get a fresh copy of the block each time
        st["X"] = [torch.empty_like(x) for x in st["X0"]]
        st["iv"] = [_interval(s) for s in systems]
    if k == "split":
        st["fr"] = torch.empty(systems[0].M, c["nfr"], dtype=st["X0"][0].dtype, device="cuda")
    if k == "density":
        s = systems[0]
        st["w"] = _weights(c, seed)
        st["rho"] = torch.empty(s.M if c["points"] == "nodes" else s.E * s.mcell, dtype=torch.float64, device="cuda")
    return st


def run(state):
    c, k, op, X0 = state["case"], state["case"]["kind"], state["ops"][0], state["X0"]
    if k == "apply":
        op.apply(X0[0], state["Y"], prec=state["prec"])
        return state["Y"]
    if k == "bounds":
        return torch.tensor(op.bounds(20, X0[0][:, 0]), dtype=torch.float64)
    if k == "density":
        op.density(X0[0], state["w"], state["rho"], points=lib.RHO_NODES if c["points"] == "nodes" else lib.RHO_GAUSS)
        return state["rho"]
    for x, x0 in zip(state["X"], X0):
        x.copy_(x0)
    X = state["X"][0]
    if k == "filter":
        a, b, aL = state["iv"][0]
        op.filter(X, c["m"], a, b, aL, prec=state["prec"], block=c["block"])
        return X
    if k == "batch":
        a, b, aL = zip(*state["iv"])
        state["ctx"].filter_batched(state["ops"], state["X"], c["m"], a, b, aL, state["prec"], use_graph=True)
        return state["X"]
    if k == "pass":
        a, b, aL = state["iv"][0]
        th, r = op.one_pass(X, c["ncols"], c["m"], c["ncols"], a, b, aL, filter_prec=state["prec"])
        return {"theta": th, "resid": r, "X": X}
    if k == "ortho":
        op.orthonormalize(X)
        return X
    th = op.rayleigh_ritz_split(X, c["nfr"], state["fr"])
    return {"theta": th, "X": X, "fr": state["fr"]}


# ---- the work a pass cannot do without ----------------------------------------
def _hx_work(M, E, p, natoms, ncols, prec, steps):
    """`steps` products H~X: the block read once and written once each, the
    previous iterate read from the second step on; the cell products as the
    tensor products of 1D matrices that they are (7 passes per cell), the
    projectors on the nodes within 6 w of their atom."""
    cplx = prec in ("c128", "c64")
    es = {"f64": 8, "f32": 4, "bf16": 4, "c128": 16, "c64": 8}[prec]
    q = p + 1
    cf = 4 if cplx else 1
    nodes = natoms * 4.19 * (6 * 1.15) ** 3 * (p / 2.0) ** 3   # box of 2 bohr cells
    nodes = min(nodes, natoms * M)
    fl = cf * ncols * (7 * 2.0 * q * E * q ** 3 + 2 * 8.0 * nodes) + 3.0 * M * ncols * (2 if cplx else 1)
    return {"bytes": (2.0 * steps + max(0, steps - 1)) * M * ncols * es, "flops": steps * fl}


def work(case):
    c, k = case, case["kind"]
    if k == "batch":
        tot = {"bytes": 0.0, "flops": 0.0}
        for nc, na, n in _batch_shapes(c):
            w = _hx_work((nc * c["p"]) ** 3, nc ** 3, c["p"], na, n, c["prec"], c["m"])
            tot = {q: tot[q] + w[q] for q in tot}
        return tot
    M, E, N = (c["nc"] * c["p"]) ** 3, c["nc"] ** 3, c["ncols"]
    cplx = _is_complex(c)
    es, cf = (16 if cplx else 8), (4.0 if cplx else 1.0)
    hx = lambda steps: _hx_work(M, E, c["p"], c["atoms"], N, c["prec"], steps)
    if k == "apply":
        return hx(1)
    if k == "filter":
        return hx(c["m"])
    if k == "bounds":
        return hx(20)
    if k == "ortho":   # X^H X (half), X L^-H (triangular)
        return {"bytes": 3.0 * M * N * es, "flops": cf * 2.0 * M * N * N}
    if k == "density":
        q = c["p"] + 1
        out = M if c["points"] == "nodes" else E * q ** 3
        fl = 3.0 * M * N if c["points"] == "nodes" else N * E * (6.0 * q ** 4 + 2.0 * q ** 3)
        return {"bytes": 1.0 * M * N * es + 8.0 * out, "flops": fl * (2 if cplx else 1)}
    h = hx(1)
    if k == "pass":    # filter, X^H X, X L^-H, W = H X, X^H W, X Q, W Q
        f = hx(c["m"])
        return {"bytes": f["bytes"] + h["bytes"] + 6.0 * M * N * es,
                "flops": f["flops"] + h["flops"] + cf * 7.0 * M * N * N}
    # split: W = H X, X^H X, X^H W, X Q_fr, X L^-H
    return {"bytes": h["bytes"] + 4.0 * M * N * es + 1.0 * M * c["nfr"] * es,
            "flops": h["flops"] + cf * (3.0 * M * N * N + 2.0 * M * N * c["nfr"])}


# ---- the same outputs in FP64 with plain torch ---------------------------------
class _Fe:
    """1D tables of the mesh, scaled by the lumped mass (numpy)."""

    def __init__(self, s):
        p, nc, h = s.p, s.ncell, s.L / s.ncell
        q = p + 1
        P = np.polynomial.legendre.Legendre.basis(p)
        xi = np.concatenate([[-1.0], np.sort(P.deriv().roots().real), [1.0]])
        for _ in range(3):   # Newton steps on P_p'
            xi[1:-1] -= P.deriv()(xi[1:-1]) / P.deriv(2)(xi[1:-1])
        xi = 0.5 * (xi - xi[::-1])
        w = 2.0 / (p * q * P(xi) ** 2)
        gx, gw = np.polynomial.legendre.leggauss(q)
        l, dl = np.zeros((q, q)), np.zeros((q, q))     # [point, basis]
        for a in range(q):
            f = np.polynomial.Polynomial([1.0])
            for b in range(q):
                if b != a:
                    f = f * np.polynomial.Polynomial([-xi[b], 1.0]) / (xi[a] - xi[b])
            l[:, a], dl[:, a] = f(gx), f.deriv()(gx)
        K = (2.0 / h) * dl.T @ (gw[:, None] * dl)
        Mc = (h / 2.0) * l.T @ (gw[:, None] * l)
        G = l.T @ (gw[:, None] * dl)
        d = 1.0 / np.sqrt(np.where((np.arange(q) == 0) | (np.arange(q) == p), w * h, w * h / 2.0))
        n = nc * p
        self.n, self.q, self.p, self.nc = n, q, p, nc
        idx = [[(c * p + a) % n for a in range(q)] for c in range(nc)]
        self.K, self.M, self.S = np.zeros((n, n)), np.zeros((n, n)), np.zeros((n, n))
        self.I = np.zeros((nc * q, n))                  # nodes (coefficients of D X) -> Gauss points
        for c, ix in enumerate(idx):
            at = np.ix_(ix, ix)
            np.add.at(self.K, at, d[:, None] * K * d)
            np.add.at(self.M, at, d[:, None] * Mc * d)
            np.add.at(self.S, at, d[:, None] * (0.5 * (G - G.T)) * d)
            np.add.at(self.I, np.ix_(range(c * q, c * q + q), ix), l)
        self.x = np.array([c * h + (1.0 + xi[a]) * h / 2.0 for c in range(nc) for a in range(p)])
        self.d = np.tile(d[:p], nc)
        self.kmax = float(np.linalg.eigvalsh(self.K)[-1])
        self.mmax = float(np.linalg.eigvalsh(self.M)[-1])


def _axis(A, X, axis):
    """A (n_out x n) applied along one axis of X (nz, ny, nx, cols)."""
    nz, ny, nx, c = X.shape
    if axis == 0:
        return torch.matmul(A, X.reshape(nz, -1)).reshape(A.shape[0], ny, nx, c)
    if axis == 1:
        return torch.matmul(A, X.reshape(nz, ny, nx * c)).reshape(nz, A.shape[0], nx, c)
    return torch.matmul(A, X.reshape(nz * ny, nx, c)).reshape(nz, ny, A.shape[0], c)


class _Ham:
    """H~ of a system on blocks (M x cols) of FP64 / complex128 on the GPU."""

    def __init__(self, s):
        f = self.f = _Fe(s)
        n = f.n
        k = np.asarray(s.k, dtype=np.float64)
        self.dt = torch.complex128 if s.is_complex else torch.float64
        put = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda().to(self.dt)
        self.M1 = put(f.M)
        # axis 0, 1, 2 of a block are z, y, x
        self.B = [put(0.5 * f.K - 1j * k[2 - ax] * f.S if s.is_complex else 0.5 * f.K) for ax in range(3)]
        V = np.zeros((n, n, n)) + 0.5 * float(k @ k)
        for R, Z, sg in zip(s.pos, s.Z, s.s):
            K = int(math.ceil(10 * sg / s.L)) + 1
            g = [sum(np.exp(-(f.x - R[i] - j * s.L) ** 2 / (2 * sg * sg)) for j in range(-K, K + 1)) for i in range(3)]
            V -= Z * g[2][:, None, None] * g[1][None, :, None] * g[0][None, None, :]
        self.V = torch.from_numpy(V.reshape(-1, 1)).cuda()
        self.proj = [self._projector(s, a) for a in range(s.natoms)] if s.has_proj else []

    def _projector(self, s, a):
        f, R, w, L = self.f, s.pos[a], s.w[a], s.L
        rc = 6.0 * w
        K = int(math.ceil(rc / L)) + 1
        ns = 1.0 / math.sqrt(math.pi ** 1.5 * w ** 3)
        npr = 1.0 / math.sqrt(math.pi ** 1.5 * w ** 5 / 2.0)
        n = f.n
        near = [[(j, np.nonzero(np.abs(f.x - R[i] - j * L) <= rc)[0]) for j in range(-K, K + 1)] for i in range(3)]
        near = [[(j, ix) for j, ix in e if ix.size] for e in near]
        ids, vals = [], []
        for jz, iz in near[2]:
            for jy, iy in near[1]:
                for jx, ix in near[0]:
                    dz, dy, dx = np.meshgrid(f.x[iz] - R[2] - jz * L, f.x[iy] - R[1] - jy * L,
                                             f.x[ix] - R[0] - jx * L, indexing="ij")
                    r2 = dx * dx + dy * dy + dz * dz
                    ok = r2 <= rc * rc
                    if not ok.any():
                        continue
                    node = ix[None, None, :] + n * (iy[None, :, None] + n * iz[:, None, None])
                    sc = 1.0 / (f.d[iz][:, None, None] * f.d[iy][None, :, None] * f.d[ix][None, None, :])
                    g = np.exp(-r2 / (2 * w * w)) * sc
                    if s.is_complex:
                        ph = (s.k[2] * (f.x[iz] - jz * L)[:, None, None] + s.k[1] * (f.x[iy] - jy * L)[None, :, None]
                              + s.k[0] * (f.x[ix] - jx * L)[None, None, :])
                        g = g * np.exp(-1j * ph)
                    v = np.stack([ns * g, npr * dx * g, npr * dy * g, npr * dz * g], axis=-1)
                    ids.append(node[ok])
                    vals.append(v[ok])
        ids, vals = np.concatenate(ids), np.concatenate(vals)
        u, inv = np.unique(ids, return_inverse=True)
        C = np.zeros((u.size, 4), dtype=vals.dtype)
        np.add.at(C, inv, vals)
        h = np.array([s.h_s[a], s.h_p[a], s.h_p[a], s.h_p[a]])
        return (torch.from_numpy(u).cuda(), torch.from_numpy(C).cuda().to(self.dt),
                torch.from_numpy(h).cuda().to(self.dt)[:, None])

    def __call__(self, X):
        n = self.f.n
        X4 = X.reshape(n, n, n, -1)
        a = _axis(self.M1, X4, 2)
        c = _axis(self.M1, a, 1)
        Y = _axis(self.B[0], c, 0)
        del c
        d = _axis(self.B[1], a, 1)
        del a
        d += _axis(self.M1, _axis(self.B[2], X4, 2), 1)
        Y += _axis(self.M1, d, 0)
        del d
        Y = Y.reshape(X.shape)
        Y += self.V * X
        for u, C, h in self.proj:
            Y.index_add_(0, u, C @ (h * (C.conj().T @ X[u])))
        return Y


def _filter(H, X, m, a, b, aL):
    e, c = (b - a) / 2, (b + a) / 2
    s1 = s = e / (aL - c)
    prev, cur = X, (H(X) - c * X) * (s1 / e)
    for _ in range(2, m + 1):
        sn = 1.0 / (2.0 / s1 - s)
        prev, cur = cur, (H(cur) - c * cur) * (2.0 * sn / e) - (s * sn) * prev
        s = sn
    return cur


# products with tall blocks go by ranges of rows
def _gram(X, Y):
    return sum(X[i:i + 2 ** 18].conj().T @ Y[i:i + 2 ** 18] for i in range(0, X.shape[0], 2 ** 18))


def _rotate(X, Z):
    return torch.cat([X[i:i + 2 ** 18] @ Z for i in range(0, X.shape[0], 2 ** 18)])


def _chol_inv(X):
    """L^-1 with X^H X = L L^H (N x N)."""
    L = torch.linalg.cholesky(_gram(X, X))
    return torch.linalg.solve_triangular(L, torch.eye(L.shape[0], dtype=L.dtype, device=L.device), upper=False)


def _lanczos(H, v):
    v = v / torch.linalg.norm(v)
    f = H(v)
    al = [torch.sum(v.conj() * f).real]
    f = f - al[0] * v
    be = []
    for _ in range(1, 20):
        be.append(torch.linalg.norm(f))
        prev, v = v, f / be[-1]
        f = H(v) - be[-1] * prev
        al.append(torch.sum(v.conj() * f).real)
        f = f - al[-1] * v
    T = np.diag([float(x) for x in al]) + np.diag([float(x) for x in be], 1) + np.diag([float(x) for x in be], -1)
    ev = np.linalg.eigvalsh(T)
    return torch.tensor([ev[-1] + float(torch.linalg.norm(f)), ev[0]], dtype=torch.float64)


def exact(case, seed):
    c, k = case, case["kind"]
    systems = _systems(c, seed)
    wide = torch.complex128 if _is_complex(c) else torch.float64
    X = [x.to(wide) for x in _blocks(c, systems, seed)]
    s = systems[0]
    if k == "apply":
        if c["prec"] == "bf16":
            return None   # the products of bf16-rounded operands are the path's own definition
        return _Ham(s)(X[0])
    if k == "bounds":
        return _lanczos(_Ham(s), X[0])
    if k == "filter":
        return _filter(_Ham(s), X[0], c["m"], *_interval(s))
    if k == "batch":
        return [_filter(_Ham(t), x, c["m"], *_interval(t)) for t, x in zip(systems, X)]
    if k == "ortho":
        return _rotate(X[0], _chol_inv(X[0]).conj().T.contiguous())
    if k == "density":
        f = _Fe(s)
        w = torch.from_numpy(_weights(c, seed)).cuda()
        d = torch.from_numpy(f.d).cuda()
        D = (d[:, None, None] * d[None, :, None] * d[None, None, :]).reshape(-1, 1)
        if c["points"] == "nodes":
            return ((D * X[0]).abs() ** 2) @ w
        n, q, nc = f.n, f.q, f.nc
        I = torch.from_numpy(f.I).cuda().to(wide)
        rho = 0.0
        for c0 in range(0, c["ncols"], 32):
            Y = (D * X[0][:, c0:c0 + 32]).reshape(n, n, n, -1)
            for ax in range(3):
                Y = _axis(I, Y, ax)
            rho = rho + (Y.abs() ** 2) @ w[c0:c0 + 32]
        return rho.reshape(nc, q, nc, q, nc, q).permute(0, 2, 4, 1, 3, 5).reshape(-1)
    H = _Ham(s)
    if k == "pass":
        Y = _filter(H, X[0], c["m"], *_interval(s))
        Y = _rotate(Y, _chol_inv(Y).conj().T.contiguous())
        W = H(Y)
        A = _gram(Y, W)
        th, Q = torch.linalg.eigh(0.5 * (A + A.conj().T))
        r = torch.linalg.norm(W @ Q - (Y @ Q) * th, dim=0)
        return {"theta": th, "resid": r, "X": None}   # Ritz vectors have a free phase
    Li = _chol_inv(X[0])
    Z = Li.conj().T.contiguous()
    A = Li @ _gram(X[0], H(X[0])) @ Z
    th = torch.linalg.eigvalsh(0.5 * (A + A.conj().T))
    return {"theta": th, "X": _rotate(X[0], Z), "fr": None}
