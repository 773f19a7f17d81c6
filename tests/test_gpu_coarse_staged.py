"""Default forms of the coarse stencils at the edges of their tiles: dof counts
that fill no row tile or k chunk (d = 2 N_tv), right-hand sides around 16, 32
and 128.  Every form multiplies and adds in the same order, so the default
equals the one-wave-per-tile form (variant 0) bit for bit; that form against
the oracle is covered by the stencil tests.  Infinities in one right-hand
side stay in its column."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from lattice_inputs import gauge_field  # noqa: E402

TAG = {"f64": "coarse64", "f32": "coarse32", "bf16": "coarsebf16"}


@pytest.mark.parametrize("ntv", [1, 3, 8, 9, 13, 16, 20, 24, 29, 32, 33])
def test_default_equals_first_form(ntv):
    import torch
    import paper_2509_11424_amd as m
    ctxs = [m.Context(0), m.Context(0)]
    U = gauge_field((4, 4, 4, 6), 0.6, 73)
    hs = [m.Hierarchy(m.Operator(c, U, 0.05, 1.0), [(2, 2, 2, 2)], [ntv], seed=3, setup_steps=1, max_nrhs=2, restart=2,
                      mixed=2, max_nrhs_level=[2, 130]) for c in ctxs]
    V, d, _ = hs[0].level_info(1)
    g = torch.Generator(device="cuda:0").manual_seed(ntv)
    for nrhs in (1, 15, 16, 17, 33, 50, 130):
        for prec in ("f64", "f32", "bf16"):
            ctxs[0].tune_set("%s/%d/%d/%d" % (TAG[prec], V, d, nrhs), 0)
            dt = torch.float64 if prec == "f64" else torch.float32
            x = torch.view_as_complex(torch.randn((d, V, nrhs, 2), generator=g, device="cuda:0", dtype=dt))
            a, b = hs[0].apply_prec(1, x, prec), hs[1].apply_prec(1, x, prec)
            assert torch.equal(a, b), (nrhs, prec)
            assert bool(torch.isfinite(torch.view_as_real(b)).all())
            if nrhs > 1:
                x[:, :, nrhs - 1] = float("inf")
                c = hs[1].apply_prec(1, x, prec)
                assert torch.equal(c[:, :, :-1], b[:, :, :-1]), (nrhs, prec)
