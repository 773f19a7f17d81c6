"""The dslash in boxes of sites, pinned so that a lattice without a box raises, against the
untiled form (pinned variant 0): blocks of 640 to 768 threads with more than 64 KiB of LDS,
boxes with odd extents, odd site counts in the halving sums of the dots (60, 36 and 30 sites),
blocks that are no whole waves (180, 210, 252 threads), boxes as long as the lattice.

Both forms add the same terms of a site in the same order, so y is the same bits.  The
dots are FP64 sums of n products in another order: 1e-13 of the norms (n < 2^20 terms
of rounding 2^-53, whose errors add up as sqrt(n))."""
import pytest

pytestmark = pytest.mark.gpu

from lattice_inputs import gauge_field  # noqa: E402

CASES = {
    (16, 16, 16, 32): [("f64", 20, "both"), ("f64", 3, "both"), ("f32", 8, "both")],
    (16, 16, 16, 16): [("f64", 12, "both"), ("f64", 1, "both"), ("f32", 3, "apply"), ("f32", 8, "both")],
    (15, 10, 12, 14): [("f64", 3, "apply"), ("f64", 7, "apply"), ("f64", 12, "both"), ("f64", 20, "both"),
                       ("f32", 14, "apply")],
    (12, 15, 10, 14): [("f64", 7, "apply"), ("f64", 12, "both"), ("f64", 20, "both"), ("f32", 14, "apply")],
    (12, 9, 10, 14): [("f64", 5, "apply"), ("f64", 20, "both")],
    (12, 10, 14, 18): [("f64", 8, "both"), ("f64", 12, "both"), ("f32", 8, "dot"), ("f32", 14, "apply")],
    (2, 2, 48, 64): [("f64", 16, "both")],
    (4, 2, 48, 64): [("f32", 32, "apply"), ("f64", 8, "both")],
}


@pytest.mark.parametrize("dims", sorted(CASES))
def test_boxes_match_the_untiled_form(dims):
    import torch
    import paper_2509_11424_amd as m
    U = gauge_field(dims, 0.6, 89)
    box, plain = (m.Operator(m.Context(0), U, 0.03, 1.0) for _ in range(2))
    for prec, nrhs, which in CASES[dims]:
        for kind in ("dslash", "dslash_dot"):
            if which == "both" or (which == "dot") == (kind == "dslash_dot"):
                box.ctx.tune_set("%s_form@%dx%dx%dx%d/%d/%d/%d" % ((kind,) + dims + (m.api.PREC[prec], box.V, nrhs)), 1)
            plain.ctx.tune_set("%s/%d/%d/%d" % (kind, m.api.PREC[prec], box.V, nrhs), 0)
        g = torch.Generator(device="cuda:0").manual_seed(nrhs)
        x = torch.view_as_complex(torch.randn((12, box.V, nrhs, 2), generator=g, device="cuda:0", dtype=torch.float64))
        if prec == "f32":
            x = x.to(torch.complex64)
        if which != "dot":
            assert torch.equal(box.apply(x, prec=prec), plain.apply(x, prec=prec)), (prec, nrhs)
        if which != "apply":
            (da, qra, qqa), (db, qrb, qqb) = box.apply_dot(x, prec=prec), plain.apply_dot(x, prec=prec)
            assert torch.equal(da, db), (prec, nrhs)
            n = qqb.sqrt() * x.to(torch.complex128).abs().square().sum(dim=(0, 1)).sqrt()
            assert torch.all((qra - qrb).abs() <= 1e-13 * n), (prec, nrhs)
            assert torch.all((qqa - qqb).abs() <= 1e-13 * qqb), (prec, nrhs)
