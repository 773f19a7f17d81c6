"""Every launch form of the coarse stencils and the default against the one-wave-per-tile
form (variant 0), where the choice of the default changes: fewer sites than CUs and more,
one to four row tiles, one tile of 16 right-hand sides and more than four.  All forms multiply and add in
the same order, so they give the same bits; an infinity in one right-hand side stays in
its column."""
import pytest

pytestmark = pytest.mark.gpu

from lattice_inputs import gauge_field  # noqa: E402

TAG = {"f64": "coarse64", "f32": "coarse32", "bf16": "coarsebf16"}


@pytest.mark.parametrize("dims,ntvs", [((4, 4, 4, 4), (4, 11, 20, 28)), ((16, 16, 8, 16), (4, 12, 32))])
def test_every_form_and_default(dims, ntvs):
    import torch
    import paper_2509_11424_amd as m
    U = gauge_field(dims, 0.6, 77)
    for ntv in ntvs:
        pinned, free = m.Context(0), m.Context(0)
        hs = [m.Hierarchy(m.Operator(c, U, 0.05, 1.0), [(2, 2, 2, 2)], [ntv], seed=3, setup_steps=1, max_nrhs=2,
                          restart=2, mixed=2, max_nrhs_level=[2, 100]) for c in (pinned, free)]
        V, d, _ = hs[0].level_info(1)
        g = torch.Generator(device="cuda:0").manual_seed(ntv)
        for nrhs in (3, 16, 20, 70, 100):
            for prec in ("f64", "f32", "bf16"):
                key = "%s/%d/%d/%d" % (TAG[prec], V, d, nrhs)
                dt = torch.float64 if prec == "f64" else torch.float32
                x = torch.view_as_complex(torch.randn((d, V, nrhs, 2), generator=g, device="cuda:0", dtype=dt))
                pinned.tune_set(key, 0)
                y0 = hs[0].apply_prec(1, x, prec)
                assert torch.equal(hs[1].apply_prec(1, x, prec), y0), key
                free.autotune(True)
                hs[1].apply_prec(1, x, prec)
                free.autotune(False)
                forms = len(free.tune_report()[key][1])
                assert forms >= 2  # at least one staged form
                bad = x.clone()
                bad[:, :, nrhs // 2] = float("inf")
                for v in range(1, forms):
                    pinned.tune_set(key, v)
                    assert torch.equal(hs[0].apply_prec(1, x, prec), y0), (key, v)
                    z = hs[0].apply_prec(1, bad, prec)
                    assert torch.equal(z[:, :, :nrhs // 2], y0[:, :, :nrhs // 2]), (key, v)
                    assert torch.equal(z[:, :, nrhs // 2 + 1:], y0[:, :, nrhs // 2 + 1:]), (key, v)
