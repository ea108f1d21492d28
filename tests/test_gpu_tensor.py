"""H~X by the tensor-product kernel and the nonlocal update that follows it,
where their tiles end: boxes of 1 to 7 cells per side against x tiles of 2 to
4 cells, columns around the 16 (FP64) and 32 (FP32) of a lane group and the
32 of an update wave, odd leading dimensions, degrees of both parities (the
filter's two buffers), and boxes whose cells hold more than 4 atoms.

Tolerances relative to the largest entry: a filter step sums, per entry, 3(p+1)
products of 1D factors plus at most a few projectors per atom, each bounded by
the growth of the step itself, so 1e-12 for one FP64 product and 1e-11 for a
filter; single precision has 5e8 times the unit roundoff, 2e-5 and 1e-4.
"""
import ctypes

import numpy as np
import pytest

import workloads
from oracle import chfsi as ochfsi
from oracle import fe

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2203_07820_amd as lib  # noqa: E402

K = (0.1, -0.2, 0.15)


@pytest.fixture(scope="module")
def ctx():
    c = lib.Context(0)
    yield c
    c.close()


def _relerr(got, want):
    return float(np.max(np.abs(got - want)) / np.max(np.abs(want)))


def _run(ctx, nc, p, atoms, k, ncols, ld, single, m):
    s = workloads.small_system(nc, p, atoms, seed=10 * nc + p, has_proj=atoms > 0, k=k)
    op = lib.Operator(ctx, s)
    H = fe.assemble(fe.build_operator(s))
    cplx = op.is_complex
    dt = {(False, False): np.float64, (False, True): np.float32,
          (True, False): np.complex128, (True, True): np.complex64}[cplx, single]
    prec = {(False, False): lib.F64, (False, True): lib.F32, (True, False): lib.C128, (True, True): lib.C64}[cplx, single]
    ncols = min(ncols, op.M)
    X = workloads.start_block(op.M, ncols, seed=7, complex_=cplx).astype(dt)
    buf = torch.full((op.M, ld), 3.0, dtype=torch.from_numpy(X).dtype, device="cuda")
    buf[:, :ncols] = torch.from_numpy(X).cuda()
    out = torch.full_like(buf, 5.0)
    ctx.check(ctx.lib.chfsi_apply(op.h, lib._tptr(buf), lib._tptr(out), ncols, ld, prec))
    torch.cuda.synchronize()
    Xr = X.astype(np.complex128 if cplx else np.float64)
    Y = out.cpu().numpy()
    assert _relerr(Y[:, :ncols], H @ Xr) < (2e-5 if single else 1e-12)
    assert np.all(Y[:, ncols:] == 5)
    if single:
        return
    b = float(abs(H).sum(axis=1).max())   # an upper bound of the spectrum
    want = ochfsi.cheb_filter(lambda v: H @ v, Xr, m, 0.3 * b, b, -1.0)
    ctx.check(ctx.lib.chfsi_filter(op.h, lib._tptr(buf), ncols, ld, m, 0.3 * b, b, -1.0, prec, 0))
    torch.cuda.synchronize()
    Y = buf.cpu().numpy()
    assert _relerr(Y[:, :ncols], want) < 1e-11
    assert np.all(Y[:, ncols:] == 3)


# every order, real and complex, on boxes that end inside an x tile
@pytest.mark.parametrize("p,nc", [(p, nc) for p in range(2, 8) for nc in (1, 2, 3, 5) if p * nc <= 18])
@pytest.mark.parametrize("k", [(0, 0, 0), K])
def test_tiles(ctx, p, nc, k):
    for single in (False, True):
        _run(ctx, nc, p, 1 if nc > 1 else 0, k, 5, 7, single, 2 + nc % 2)


@pytest.mark.parametrize("ncols,ld", [(1, 1), (15, 15), (16, 17), (17, 64), (31, 31), (33, 35), (64, 64), (97, 97)])
@pytest.mark.parametrize("k", [(0, 0, 0), K])
def test_columns(ctx, ncols, ld, k):
    for single in (False, True):
        _run(ctx, 3, 4, 2, k, ncols, ld, single, 3)


# cells with 5 and 9 atoms: the update's own loop and further projection passes
@pytest.mark.parametrize("atoms", [4, 5, 9])
@pytest.mark.parametrize("k", [(0, 0, 0), K])
def test_many_atoms_per_cell(ctx, atoms, k):
    for single in (False, True):
        _run(ctx, 2, 5, atoms, k, 18, 18, single, 4)


# a mesh of 7 cells per side: tiles of 4 cells, one of them beyond the mesh
def test_ragged_wide_tile(ctx):
    _run(ctx, 7, 3, 2, (0, 0, 0), 20, 20, False, 2)


# problems of unequal size in one batch: rounds of a ragged block, both
# parities of the degree, blocks in storage of their own (single precision)
# and in place, eager and as a captured graph on changing blocks; each problem
# as the single-problem filter does it
@pytest.mark.parametrize("k", [(0, 0, 0), K])
@pytest.mark.parametrize("single", [False, True])
@pytest.mark.parametrize("m", [1, 4, 5])
def test_batched_filter(ctx, k, single, m):
    p = 4
    sizes = [(2, 2, 9), (3, 0, 40), (5, 3, 33), (1, 0, 1), (4, 5, 17)]
    ops = [lib.Operator(ctx, workloads.small_system(nc, p, na, seed=nc, has_proj=na > 0, k=k)) for nc, na, _ in sizes]
    cplx = ops[0].is_complex
    prec = {(False, False): lib.F64, (False, True): lib.F32, (True, False): lib.C128, (True, True): lib.C64}[cplx, single]
    b = [40.0 + nc for nc, _, _ in sizes]
    a = [0.3 * x for x in b]
    aL = [-1.0] * len(ops)
    for graph in (False, True, True):
        Xs = [torch.from_numpy(workloads.start_block(op.M, c, seed=3 + c + graph, complex_=cplx)).cuda()
              for op, (_, _, c) in zip(ops, sizes)] if not graph or not hasattr(ctx, "_blocks") else ctx._blocks
        ctx._blocks = Xs
        want = [X.clone() for X in Xs]
        for op, W, bb, aa, al in zip(ops, want, b, a, aL):
            op.filter(W, m, aa, bb, al, prec=prec, block=16)
        ctx.filter_batched(ops, Xs, m, a, b, aL, prec, block=16, use_graph=graph)
        torch.cuda.synchronize()
        for X, W in zip(Xs, want):
            assert _relerr(X.cpu().numpy(), W.cpu().numpy()) < (1e-4 if single else 1e-11)
            X /= X.abs().max()
    del ctx._blocks


# Gram blocks of 64 columns and rotation slabs of 256 where they end, in place
# with a leading dimension of its own; tolerances of the orthonormalisation and
# Rayleigh-Ritz tests of smaller blocks (1e-11, 1e-9)
@pytest.mark.parametrize("N", [1, 15, 17, 48, 63, 65, 130, 257, 300])
@pytest.mark.parametrize("k", [(0, 0, 0), K])
def test_subspace_widths(ctx, N, k):
    s = workloads.small_system(3, 5, 2, seed=21, has_proj=True, k=k)
    op = lib.Operator(ctx, s)
    X = workloads.start_block(op.M, N, seed=N, complex_=op.is_complex)
    buf = torch.full((op.M, N + 3), 4.0, dtype=torch.from_numpy(X).dtype, device="cuda")
    buf[:, :N] = torch.from_numpy(X).cuda()
    Xo, Lref, _ = ochfsi.cholgs(X)
    L = np.zeros((N, N), dtype=X.dtype)
    ctx.check(ctx.lib.chfsi_orthonormalize(op.h, lib._tptr(buf), N, N + 3,
                                           L.ctypes.data_as(ctypes.POINTER(ctypes.c_double))))
    got = buf.cpu().numpy()
    assert _relerr(got[:, :N], Xo) < 1e-11
    assert _relerr(L, Lref) < 1e-11
    assert np.all(got[:, N:] == 4)
    H = fe.assemble(fe.build_operator(s))
    th_ref = ochfsi.rayleigh_ritz(lambda v: H @ v, Xo)[0]
    Xd = torch.from_numpy(Xo).cuda()
    th, r = op.rayleigh_ritz(Xd)
    assert np.max(np.abs(th - th_ref)) < 1e-10 * max(1.0, np.max(np.abs(th_ref)))
    Psi = Xd.cpu().numpy()
    assert np.max(np.abs(np.linalg.norm(H @ Psi - Psi * th, axis=0) - r)) < 1e-9


# one column (the narrow projection and the update in parts), real and complex:
# bounds of 1 and more steps against the same recurrence on the host
@pytest.mark.parametrize("steps", [1, 2, 9])
@pytest.mark.parametrize("k", [(0, 0, 0), K])
def test_bounds_recurrence(ctx, steps, k):
    s = workloads.small_system(3, 5, 3, seed=4, has_proj=True, k=k)
    op = lib.Operator(ctx, s)
    H = fe.assemble(fe.build_operator(s))
    v = workloads.lanczos_start(op.M, 9, op.is_complex)
    got = op.bounds(steps, torch.from_numpy(v).cuda())
    f, prev, beta, al, be = v, 0.0 * v, 0.0, [], []
    for i in range(steps):
        nrm = np.linalg.norm(f)
        if i:
            be.append(nrm)
        q = f / nrm
        f = H @ q - (nrm * prev if i else 0.0)
        al.append(np.vdot(q, f).real)
        f = f - al[-1] * q
        prev = q
    ev = np.linalg.eigvalsh(np.diag(al) + np.diag(be, 1) + np.diag(be, -1))
    # one product each step: 1e-12 of the norm, growing with the steps
    assert abs(got[0] - (ev[-1] + np.linalg.norm(f))) < 1e-10 * ev[-1]
    assert abs(got[1] - ev[0]) < 1e-10 * ev[-1]


def test_bounds_refuses_a_zero_start(ctx):
    op = lib.Operator(ctx, workloads.small_system(2, 3, 1, seed=4))
    with pytest.raises(lib.ChfsiError):
        op.bounds(4, torch.zeros(op.M, dtype=torch.float64, device="cuda"))


# widths around the narrow projection's 16 columns
@pytest.mark.parametrize("ncols", [2, 3, 9, 16, 17])
@pytest.mark.parametrize("k", [(0, 0, 0), K])
def test_narrow_projection(ctx, ncols, k):
    for single in (False, True):
        _run(ctx, 3, 5, 3, k, ncols, ncols + 1, single, 2)


# planes of 2 GB go to the dense kernel (32-bit offsets in a plane), smaller
# ones to the tensor-product kernel: 4^2 nodes x 2^24 doubles, and one less
@pytest.mark.parametrize("ld", [2 ** 24 - 1, 2 ** 24])
def test_plane_limit(ctx, ld):
    s = workloads.small_system(2, 2, 1, seed=2, has_proj=True)
    op = lib.Operator(ctx, s)
    H = fe.assemble(fe.build_operator(s))
    X = workloads.start_block(op.M, 3, seed=7)
    buf = torch.zeros(op.M, ld, dtype=torch.float64, device="cuda")
    out = torch.full_like(buf, 5.0)
    buf[:, :3] = torch.from_numpy(X).cuda()
    for call in (ctx.lib.chfsi_apply, ctx.lib.chfsi_apply_noalloc):
        ctx.check(call(op.h, lib._tptr(buf), lib._tptr(out), 3, ld, lib.F64))
        torch.cuda.synchronize()
        assert _relerr(out[:, :3].cpu().numpy(), H @ X) < 1e-12
        assert bool((out[:, 3:5] == 5).all()) and bool((out[:, -2:] == 5).all())
        out[:, :3] = 5.0
    b = float(abs(H).sum(axis=1).max())
    want = ochfsi.cheb_filter(lambda v: H @ v, X, 3, 0.3 * b, b, -1.0)
    ctx.check(ctx.lib.chfsi_filter(op.h, lib._tptr(buf), 3, ld, 3, 0.3 * b, b, -1.0, lib.F64, 0))
    torch.cuda.synchronize()
    assert _relerr(buf[:, :3].cpu().numpy(), want) < 1e-11
