"""The solvers' reductions column by column: every column of a batch is a power of two times
one right-hand side, so that its solve is the single one scaled exactly, up to the order
of the sums.  A norm or dot that misses or repeats one of the n = 3072 entries changes the
Krylov coefficients by 1e-4, and the solutions, stopped at 1e-6, in the sixth digit; the
orders of the sums change them by 2^-53 times the number of steps and the condition number
(below 1e3): 1e-10.  Iteration counts are those of the single solve, and the residual that
the solver reports is the one formed from its solution in FP64 (1e-7: rounding 1e-15 of |b|
in a residual of 1e-6 is 1e-9)."""
import pytest

pytestmark = pytest.mark.gpu

from gpu_common import to_gpu  # noqa: E402
from lattice_inputs import gauge_field, random_spinor  # noqa: E402


@pytest.mark.parametrize("nrhs", [2, 7, 16, 20, 100, 129, 256])
@pytest.mark.parametrize("kind", ["gmres", "mg"])
def test_columns_of_a_batch(nrhs, kind):
    import torch
    import paper_2509_11424_amd as m
    dims = (4, 4, 4, 4)
    op = m.Operator(m.Context(0), gauge_field(dims, 0.4, 91), 0.3, 1.0)
    h = m.Hierarchy(op, [(2, 2, 2, 2)], [8], seed=5, max_nrhs=nrhs, restart=24)
    b1 = to_gpu(random_spinor(dims, 92, batch=1).reshape(1, -1, 12))
    scale = 2.0 ** (torch.arange(nrhs, device="cuda:0") % 7)
    b = (b1 * scale).contiguous()
    desc = m.solve_desc(tol=1e-6, kind=kind)
    x1, st1 = h.solve(0, b1, desc)
    x, st = h.solve(0, b, desc)
    torch.cuda.synchronize()
    assert st["iterations"] == st1["iterations"], (st, st1)
    off = (x - x1 * scale).abs().square().sum(dim=(0, 1)).sqrt() / (x1 * scale).abs().square().sum(dim=(0, 1)).sqrt()
    assert torch.all(off <= 1e-10), off.max()
    r = b - op.apply(x)
    torch.cuda.synchronize()
    rel = r.abs().square().sum(dim=(0, 1)).sqrt() / b.abs().square().sum(dim=(0, 1)).sqrt()
    assert abs(rel.max().item() - st["max_rel_residual"]) <= 1e-7 * rel.max().item()
