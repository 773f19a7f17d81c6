"""Reductions of the solvers at right-hand-side counts that change their split: one
column (sixteen threads share a block's entries), odd counts, counts above half a block,
and 16 columns with more than 16 basis vectors (four entries per finalizing block).

The solver stops on its own norms; the residual is formed here with the operator and
torch's FP64 sums.  tol = 1e-10 is met by every column with a factor two: norms that
missed or repeated an entry of n = 3072 would be off by far more than the 1e-13 the sums
round, while the Krylov residual and the true one differ by the rounding of the solution,
1e-15 times the condition number (below 1e3 here).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_common import to_gpu, from_gpu  # noqa: E402
from lattice_inputs import gauge_field, random_spinor  # noqa: E402


@pytest.mark.parametrize("nrhs", [1, 2, 7, 16, 100, 129, 256])
@pytest.mark.parametrize("kind", ["gmres", "mg"])
def test_solver_norms(nrhs, kind):
    import torch
    import paper_2509_11424_amd as m
    dims = (4, 4, 4, 4)
    U = gauge_field(dims, 0.4, 91)
    op = m.Operator(m.Context(0), U, 0.3, 1.0)
    h = m.Hierarchy(op, [(2, 2, 2, 2)], [8], seed=5, max_nrhs=nrhs, restart=24)
    b = to_gpu(random_spinor(dims, 92, batch=nrhs).reshape(nrhs, -1, 12))
    x = h.solve(0, b, m.solve_desc(tol=1e-10, kind=kind))
    x = x[0] if isinstance(x, tuple) else x
    r = b - op.apply(x)
    torch.cuda.synchronize()
    nr = from_gpu(r).reshape(nrhs, -1)
    nb = from_gpu(b).reshape(nrhs, -1)
    assert np.all(np.linalg.norm(nr, axis=1) <= 2e-10 * np.linalg.norm(nb, axis=1))


@pytest.mark.parametrize("nrhs", [1, 2, 3, 6, 8, 12])
def test_mixed_solver_column_counts(nrhs):
    """Scaled conversions and MR updates at 1, 2 and 4 columns per thread: the FP64 outer
    residual meets the tolerance whatever the inner precision, if no column is lost."""
    import torch
    import paper_2509_11424_amd as m
    dims = (8, 8, 8, 8)
    U = gauge_field(dims, 0.4, 93)
    op = m.Operator(m.Context(0), U, 0.3, 1.0)
    h = m.Hierarchy(op, [(2, 2, 2, 2)], [8], seed=5, max_nrhs=nrhs, restart=12, mixed=2)
    b = to_gpu(random_spinor(dims, 94, batch=nrhs).reshape(nrhs, -1, 12))
    x, st = h.solve(0, b, m.solve_desc(tol=1e-10, kind="mg_mixed", smooth=4))
    r = b - op.apply(x)
    torch.cuda.synchronize()
    nr = from_gpu(r).reshape(nrhs, -1)
    nb = from_gpu(b).reshape(nrhs, -1)
    assert st["fallbacks"] == 0
    assert np.all(np.linalg.norm(nr, axis=1) <= 2e-10 * np.linalg.norm(nb, axis=1))
