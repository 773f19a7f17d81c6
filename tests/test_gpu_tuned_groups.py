"""A tuned solve repeated with the autotuner off, and in another context from the saved
report: the same column groups of the FP16 smoother, seen in the bytes of a step's launch,
and the same launch variants, so the same bits.  8^4 at 16 right-hand sides, where untuned
solves form no groups."""
import pytest

pytestmark = pytest.mark.gpu

from gpu_common import to_gpu  # noqa: E402
from lattice_inputs import gauge_field, random_spinor  # noqa: E402


def _solve(h, ctx, b, desc):
    ctx.profile(True)
    ctx.profile_reset()
    try:
        x, _ = h.solve(0, b, desc)
        q = ctx.profile_query("dslash_step")
    finally:
        ctx.profile(False)
    assert q["launches"] > 0
    return x, q["bytes"] / q["launches"]


def test_tuned_solve_repeats():
    import torch
    import paper_2509_11424_amd as m
    dims, nrhs = (8, 8, 8, 8), 16
    U = gauge_field(dims, 0.4, 95)
    ctxs = [m.Context(0) for _ in range(3)]
    hs = [m.Hierarchy(m.Operator(c, U, 0.1, 1.0), [(2, 2, 2, 2)], [8], seed=5, max_nrhs=nrhs, restart=12, mixed=1)
          for c in ctxs]
    b = to_gpu(random_spinor(dims, 96, batch=nrhs).reshape(nrhs, -1, 12))
    desc = m.solve_desc(tol=1e-10, kind="mg_mixed", smooth=4)
    ctxs[0].autotune(True)
    hs[0].solve(0, b, desc)  # tunes
    x1, per1 = _solve(hs[0], ctxs[0], b, desc)
    ctxs[0].autotune(False)
    x2, per2 = _solve(hs[0], ctxs[0], b, desc)
    rep = ctxs[0].tune_report()
    assert "dslash_step/%d/%d/8" % (m.api.PREC["f16"], 4096) in rep
    for k, (v, _) in rep.items():
        ctxs[1].tune_set(k, v)
    x3, per3 = _solve(hs[1], ctxs[1], b, desc)
    _, untuned = _solve(hs[2], ctxs[2], b, desc)
    torch.cuda.synchronize()
    assert per1 < untuned
    assert per2 == per1 and per3 == per1
    assert torch.equal(x1, x2)
    assert torch.equal(x1, x3)
