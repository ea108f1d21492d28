"""Overlap of more columns than the Gram products' block rows fit into one
dimension of a launch: 23,168 columns are 65,703 blocks of 64 x 64, where a grid
holds 65,535.

Tolerance: an entry of Q^T Q sums M products of entries of orthonormal columns
made from a block of condition number below 10, so M eps = 6e-12; 1e-10."""
import pytest

import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2203_07820_amd as lib  # noqa: E402


def test_orthonormalize_23168_columns():
    N = 23168
    c = lib.Context(0)
    op = lib.Operator(c, workloads.small_system(5, 6, 1, seed=3, has_proj=False))
    assert op.M == 27000
    j = torch.arange(N, device="cuda")
    X = torch.zeros(op.M, N, dtype=torch.float64, device="cuda")
    X[j, j] = 1.0 + (j % 7).double() / 7.0
    X[N + j % (op.M - N), j] = 0.25
    X[(j + 61) % N, j] += 0.25
    first = X[:, 0].clone()
    op.orthonormalize(X)
    torch.cuda.synchronize()
    assert torch.allclose(X[:, 0], first / torch.linalg.norm(first), rtol=0, atol=1e-12)
    G = X.T @ X
    G.diagonal().sub_(1.0)
    assert float(G.abs().max()) < 1e-10
    del X, G
    op.close()
    c.close()
    torch.cuda.empty_cache()
