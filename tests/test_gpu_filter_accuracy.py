"""Error of the single-precision filter on the tensor-product path.

The tensor-product kernel and the nonlocal update behind it form other sums, with
other scalars, than the dense cell kernel.  Their error against the FP64 filter
may be no larger than the dense kernel's on the same blocks: a batch that holds
one quadrature-potential operator goes by the dense kernel as a whole, which
gives that error for the other operators in it.  A single case scatters by the
luck of its roundings (0.3 to 1.4 times), so the bound, 1, is on the geometric
mean over the cases; a factor of 2 on each."""
import numpy as np
import pytest

import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2203_07820_amd as lib  # noqa: E402

# (order, cells per side, box side): cells of 0.6 to 10 bohr, so that the kernel's
# scaling by the cell side is no power of two everywhere
BOXES = [(p, nc, L) for p, nc in [(3, 5), (4, 4), (5, 4), (6, 4), (7, 4)] for L in (3.0, 8.0, 40.0)]


@pytest.mark.parametrize("cplx", [False, True])
def test_single_precision_filter_is_no_less_accurate_than_dense(cplx):
    c = lib.Context(0)
    dt = torch.complex128 if cplx else torch.float64
    single = lib.C64 if cplx else lib.F32
    ratios = []
    for p, nc, L in BOXES:
        s = workloads.make_system(L, nc, p, 3, seed=3, d_min=0.5, has_proj=True)
        small = workloads.make_system(4.0, 2, p, 1, seed=4, d_min=0.5, has_proj=False)
        if cplx:
            s, small = s.with_k(workloads.kpoints_mp4(L)[1]), small.with_k(workloads.kpoints_mp4(4.0)[1])
        op, dense = lib.Operator(c, s), lib.Operator(c, small, potential="quadrature")
        g = torch.Generator(device="cuda").manual_seed(p)
        X = torch.randn(op.M, 24, dtype=dt, device="cuda", generator=g)
        b = 1.05 * float(op.bounds(20, X[:, 0].contiguous())[0])
        iv = (0.2 * b, b, -1.0)
        want, tens, den = X.clone(), X.clone(), X.clone()
        other = torch.randn(dense.M, 8, dtype=dt, device="cuda", generator=g)
        op.filter(want, 10, *iv)
        op.filter(tens, 10, *iv, prec=single)
        bd = 1.05 * float(dense.bounds(20, other[:, 0].contiguous())[0])
        c.filter_batched([op, dense], [den, other], 10, [iv[0], 0.2 * bd], [iv[1], bd], [iv[2], -1.0], single)
        torch.cuda.synchronize()
        e = [float((Y - want).norm() / want.norm()) for Y in (tens, den)]
        print(f"p{p} nc{nc} L{L}: {e[0]:.2e} {e[1]:.2e}")
        assert 0.0 < e[0] < 5e-6 and 0.0 < e[1] < 5e-6
        ratios.append(e[0] / e[1])
        op.close()
        dense.close()
    c.close()
    assert max(ratios) < 2.0
    assert np.exp(np.mean(np.log(ratios))) < 1.0
