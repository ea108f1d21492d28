"""The dense cell kernel where it is the only one that can run: operators with
the per-cell quadrature potential (each cell has its own matrix) and BF16
products.  Batched filters in every launch shape, and deterministic assembly by
colour classes.  (Operators whose cells share one matrix take the
tensor-product kernel in both, whatever shape is loaded.)

Tolerances as in the tests of the same calls on nodal-potential operators:
filters of degree 8 against the oracle 1e-11 (FP64, complex128), 1e-4 (FP32),
5e-5 (complex64), against the same block filtered alone 1e-12 and 2e-5; the two
assemblies 1e-13 of max|Y|, 1e-5 in single precision."""
import numpy as np
import pytest
import scipy.sparse.linalg as spla

import workloads
from oracle import chfsi as ochfsi
from oracle import dhm

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2203_07820_amd as lib  # noqa: E402

K = (0.1, -0.2, 0.3)
PREC = {"f64": lib.F64, "f32": lib.F32, "c128": lib.C128, "c64": lib.C64}
DTYPE = {"f64": np.float64, "f32": np.float32, "bf16": np.float32, "c128": np.complex128, "c64": np.complex64}


@pytest.fixture()
def ctx():
    c = lib.Context(0)
    yield c
    c.close()


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def _relerr(a, b):
    return float(np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-300))


def _bits(a):
    a = np.ascontiguousarray(a)
    return a.view(np.uint64 if a.dtype.itemsize % 8 == 0 else np.uint32)


# ---- batched filters ----------------------------------------------------------
def _refs(systems, cols, cplx):
    """Oracle filters (degree 8) of every problem."""
    out = []
    for q, s in enumerate(systems):
        H = dhm.assemble_quadrature(s)
        lmax = float(spla.eigsh(H, k=1, which="LA", return_eigenvectors=False)[0])
        iv = (0.05 * lmax, 1.05 * lmax, -0.1 * lmax)
        X = workloads.start_block(s.M, cols[q], seed=300 + q, complex_=cplx)
        out.append((X, iv, ochfsi.cheb_filter(lambda v: H @ v, X, 8, *iv)))
    return out


@pytest.fixture(scope="module")
def kpoint_batch():
    systems = []
    for nc, na, seed in [(2, 2, 21), (3, 3, 22)]:
        base = workloads.small_system(nc, 5, na, seed=seed, has_proj=True)
        systems += [base.with_k(k) for k in workloads.kpoints_mp4(base.L)]
    return systems, _refs(systems, [24, 9, 40, 17, 33, 48, 12, 29], True)


@pytest.fixture(scope="module")
def real_batch():
    systems = [workloads.small_system(nc, 3, na, seed=seed, has_proj=True) for nc, na, seed in
               [(2, 2, 11), (3, 3, 12), (4, 2, 13)]]
    return systems, _refs(systems, [20, 37, 9], False)


def _filter_batch(ctx, tmp_path, batch, p, prec, block, grid, contiguous, col_tile):
    systems, refs = batch
    P = PREC[prec]
    path = tmp_path / "tune.json"
    path.write_text('[\n{"key": "gfx950:p%d:prec%d:B%d", "grid_per_cu": %d, "contiguous": %d, "col_tile": %d, '
                    '"ms": 1.0}\n]\n' % (p, P, block, grid, contiguous, col_tile))
    ctx.load_tuning(str(path))
    ops = [lib.Operator(ctx, s, potential="quadrature") for s in systems]
    a, b, aL = zip(*[r[1] for r in refs])
    tol, alone = {"f64": (1e-11, 1e-12), "c128": (1e-11, 1e-12), "f32": (1e-4, 2e-5), "c64": (5e-5, 2e-5)}[prec]
    for graph in (False, True):
        Xd = [_dev(r[0]) for r in refs]
        ctx.filter_batched(ops, Xd, 8, a, b, aL, P, block=block, use_graph=graph)
        for q, op in enumerate(ops):
            got = _host(Xd[q])
            assert _relerr(got, refs[q][2]) < tol, (q, graph)
            if not graph:
                Xi = _dev(refs[q][0])
                op.filter(Xi, 8, *refs[q][1], prec=P, block=block)
                assert _relerr(got, _host(Xi)) < alone, q


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("col_tile,block", [(64, 16), (32, 16), (64, 40), (32, 40)])
@pytest.mark.parametrize("grid,contiguous", [(0, 1), (1, 1), (1, 0), (2, 1), (2, 0), (4, 1), (4, 0)])
def test_batched_every_launch_shape(ctx, tmp_path, kpoint_batch, grid, contiguous, col_tile, block, prec):
    _filter_batch(ctx, tmp_path, kpoint_batch, 5, prec, block, grid, contiguous, col_tile)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("col_tile", [64, 32])
@pytest.mark.parametrize("grid", [0, 2])
def test_batched_real_launch_shapes(ctx, tmp_path, real_batch, grid, col_tile, prec):
    _filter_batch(ctx, tmp_path, real_batch, 3, prec, 40, grid, 1, col_tile)


def test_batch_with_one_quadrature_operator(ctx):
    # one such operator makes the whole batch take the dense kernel
    sys_ = [workloads.small_system(nc, 4, 2, seed=nc, has_proj=True) for nc in (2, 3, 4)]
    ops = [lib.Operator(ctx, s, potential="quadrature" if i == 1 else "nodal") for i, s in enumerate(sys_)]
    X0 = [workloads.start_block(s.M, 20 + i, seed=40 + i) for i, s in enumerate(sys_)]
    want = [_dev(X) for X in X0]
    for op, X in zip(ops, want):
        op.filter(X, 7, 20.0, 80.0, -1.0, block=16)
    for graph in (False, True):
        Xd = [_dev(X) for X in X0]
        ctx.filter_batched(ops, Xd, 7, [20.0] * 3, [80.0] * 3, [-1.0] * 3, lib.F64, block=16, use_graph=graph)
        for X, W in zip(Xd, want):
            assert _relerr(_host(X), _host(W)) < 1e-11


# ---- deterministic assembly -----------------------------------------------------
# odd sides (27 colour classes) and even ones (8), real and complex
CASES = [
    (3, 3, 2, (0, 0, 0), 11),
    (2, 5, 2, (0, 0, 0), 12),
    (4, 4, 3, (0, 0, 0), 13),
    (3, 4, 2, K, 14),
    (2, 4, 2, K, 15),
]


def _case(ctx, case, potential="quadrature"):
    nc, p, na, k, seed = case
    s = workloads.small_system(nc, p, na, seed=seed, has_proj=True, k=k)
    return s, lib.Operator(ctx, s, potential=potential)


def _apply(op, X, prec):
    Y = torch.zeros_like(X)
    op.apply(X, Y, prec=prec)
    return _host(Y)


@pytest.mark.parametrize("single", [False, True])
@pytest.mark.parametrize("case", CASES)
def test_deterministic_products(ctx, case, single):
    s, op = _case(ctx, case)
    prec = ("c64" if single else "c128") if op.is_complex else ("f32" if single else "f64")
    Xh = workloads.start_block(op.M, min(70, op.M), seed=5, complex_=op.is_complex).astype(DTYPE[prec])
    X = _dev(Xh)
    Ya = _apply(op, X, PREC[prec])
    ctx.set_deterministic(True)
    Y1, Y2 = _apply(op, X, PREC[prec]), _apply(op, X, PREC[prec])
    Y3 = torch.zeros_like(X)
    ctx.check(ctx.lib.chfsi_apply_noalloc(op.h, lib._tptr(X), lib._tptr(Y3), X.shape[1], X.shape[1], PREC[prec]))
    Y3 = _host(Y3)
    assert np.array_equal(_bits(Y1), _bits(Y2))
    assert np.array_equal(_bits(Y1), _bits(Y3))
    assert _relerr(Y1, Ya) < (1e-5 if single else 1e-13)
    H = dhm.assemble_quadrature(s)
    assert _relerr(Y1, H @ Xh.astype(np.complex128 if op.is_complex else np.float64)) < (2e-5 if single else 1e-12)


@pytest.mark.parametrize("case", [CASES[0], CASES[2], CASES[3]])
def test_deterministic_filter_and_batch(ctx, case):
    _, op = _case(ctx, case)
    _, other = _case(ctx, (2, case[1], 2, case[3], 16))
    ops = [op, other]
    X0 = [workloads.start_block(o.M, 30, seed=6 + i, complex_=op.is_complex) for i, o in enumerate(ops)]
    b = 1.1 * max(float(o.bounds(steps=20, seed=1)[0]) for o in ops)
    P = lib.C128 if op.is_complex else lib.F64
    plain = _dev(X0[0])
    op.filter(plain, 6, 0.2 * b, b, -1.0)
    ctx.set_deterministic(True)
    runs = []
    for batched in (False, False, True):
        Xd = [_dev(x) for x in X0]
        if batched:
            ctx.filter_batched(ops, Xd, 6, [0.2 * b] * 2, [b] * 2, [-1.0] * 2, P, use_graph=True)
        else:
            for o, x in zip(ops, Xd):
                o.filter(x, 6, 0.2 * b, b, -1.0)
        runs.append([_host(x) for x in Xd])
    for r in runs[1:]:
        for x, y in zip(runs[0], r):
            assert np.array_equal(_bits(x), _bits(y))
    assert _relerr(runs[0][0], _host(plain)) < 1e-11


def test_one_nonzero_contribution_per_node_is_bitwise_equal_to_atomic(ctx):
    # no projectors; X nonzero only at the interior nodes of one cell: every
    # other cell's product is exactly zero, so the order cannot matter
    nc, p = 3, 4
    op = lib.Operator(ctx, workloads.small_system(nc, p, 2, seed=15, has_proj=False), potential="quadrature")
    n = nc * p
    rows = [((p + a) % n) + n * (((2 * p + b) % n) + n * c) for c in range(1, p) for b in range(1, p)
            for a in range(1, p)]
    X = np.zeros((op.M, 50))
    X[rows, :] = workloads.start_block(len(rows), 50, seed=8)
    Xd = _dev(X)
    Ya = _apply(op, Xd, lib.F64)
    ctx.set_deterministic(True)
    Yd = _apply(op, Xd, lib.F64)
    assert np.count_nonzero(Ya) > 0
    assert np.array_equal(_bits(Ya), _bits(Yd))


@pytest.mark.parametrize("case", [CASES[0], CASES[2]])
def test_deterministic_bf16(ctx, case):
    _, op = _case(ctx, case, potential="nodal")
    X = _dev(workloads.start_block(op.M, 64, seed=7).astype(np.float32))
    Ya = _apply(op, X, lib.BF16)
    ctx.set_deterministic(True)
    Y1, Y2 = _apply(op, X, lib.BF16), _apply(op, X, lib.BF16)
    assert np.array_equal(_bits(Y1), _bits(Y2))
    assert _relerr(Y1, Ya) < 1e-5
