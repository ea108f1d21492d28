"""H~X of a product on its own, on both sides of the line between the dense cell
kernel (small meshes of order 2 and 3 with projectors) and the tensor-product
kernel: against the oracle, in the default and in the deterministic mode, and
which of the two kernels ran.

The tensor-product kernel gives every node's sum in a fixed order and is taken
in the deterministic mode at every size here, so a default product that took it
has the same bits; the dense kernel forms other sums and differs in the last
ones.  Tolerances of the parity tests: 1e-12 of max|Y| in FP64, 2e-5 in FP32."""
import numpy as np
import pytest

import workloads
from oracle import fe

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2203_07820_amd as lib  # noqa: E402

K = (0.1, -0.2, 0.15)

CASES = [
    # (p, ncell, atoms, complex, single, columns, dense)
    (2, 2, 1, False, False, 33, True),
    (2, 4, 1, False, True, 128, True),
    (2, 4, 0, False, False, 33, False),       # no projectors
    (3, 2, 1, True, True, 17, True),
    (3, 3, 1, False, False, 1, True),
    (3, 3, 1, True, False, 128, True),
    (3, 5, 2, True, False, 128, True),        # 64,000
    (3, 5, 2, True, False, 129, False),
    (3, 6, 2, False, False, 138, True),       # 29,808
    (3, 6, 2, False, False, 139, False),      # 30,024
    (3, 6, 2, False, True, 33, True),
    (3, 7, 2, False, True, 33, False),
    (3, 8, 3, False, False, 58, True),        # 29,696
    (3, 8, 3, False, False, 59, False),
    (2, 9, 3, False, False, 5, False),
    (4, 2, 1, False, False, 33, False),
]


def _relerr(got, want):
    return float(np.max(np.abs(got - want)) / np.max(np.abs(want)))


@pytest.mark.parametrize("case", CASES)
def test_single_product(case):
    p, nc, atoms, cplx, single, ncols, dense = case
    s = workloads.small_system(nc, p, atoms, seed=31, has_proj=atoms > 0, k=K if cplx else (0, 0, 0))
    ctx = lib.Context(0)
    op = lib.Operator(ctx, s)
    X = workloads.start_block(op.M, ncols, seed=7, complex_=cplx)
    if single:
        X = X.astype(np.complex64 if cplx else np.float32)
    prec = {(False, False): lib.F64, (False, True): lib.F32, (True, False): lib.C128, (True, True): lib.C64}[cplx, single]
    want = fe.assemble(fe.build_operator(s)) @ X.astype(np.complex128 if cplx else np.float64)
    ld = ncols + 3
    buf = torch.full((op.M, ld), 3.0, dtype=torch.from_numpy(X).dtype, device="cuda")
    buf[:, :ncols] = torch.from_numpy(X).cuda()

    def run(call):
        out = torch.full_like(buf, 5.0)
        ctx.check(call(op.h, lib._tptr(buf), lib._tptr(out), ncols, ld, prec))
        torch.cuda.synchronize()
        Y = out.cpu().numpy()
        assert np.all(Y[:, ncols:] == 5)
        assert _relerr(Y[:, :ncols], want) < (2e-5 if single else 1e-12)
        return Y[:, :ncols]

    plain = [run(ctx.lib.chfsi_apply), run(ctx.lib.chfsi_apply_noalloc)]
    ctx.set_deterministic(True)
    fixed = [run(ctx.lib.chfsi_apply), run(ctx.lib.chfsi_apply_noalloc)]
    ctx.set_deterministic(False)
    assert np.array_equal(fixed[0], fixed[1])
    for Y in plain:
        assert np.array_equal(Y, fixed[0]) == (not dense)
    op.close()
    ctx.close()


# the callers of single products inside the library, on a mesh of either side:
# spectral bounds, Rayleigh-Ritz and the split step, against the other mode
# (1e-10 of the largest value: a few hundred roundings of sums of that size)
@pytest.mark.parametrize("p,nc,cplx", [(3, 3, False), (3, 4, True), (2, 9, False), (4, 3, True)])
def test_callers(p, nc, cplx):
    s = workloads.small_system(nc, p, 2, seed=33, has_proj=True, k=K if cplx else (0, 0, 0))
    ctx = lib.Context(0)
    op = lib.Operator(ctx, s)
    X = torch.from_numpy(workloads.start_block(op.M, 24, seed=8, complex_=cplx)).cuda()
    op.orthonormalize(X)
    v = X[:, 0].contiguous()

    def values():
        th, r = op.rayleigh_ritz(X.clone())
        F = torch.empty(op.M, 6, dtype=X.dtype, device="cuda")
        ths = op.rayleigh_ritz_split(X.clone(), 6, F)
        return np.concatenate([np.array(op.bounds(8, v)), th, r, ths])

    a = values()
    ctx.set_deterministic(True)
    b = values()
    assert np.max(np.abs(a - b)) < 1e-10 * np.max(np.abs(b))
    op.close()
    ctx.close()
