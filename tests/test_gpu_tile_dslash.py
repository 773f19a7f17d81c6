"""Tiled dslash against the untiled form (pinned variant 0): tiles that reach
over a whole extent (hops wrap inside the tile), boxes with odd extents, counts whose
blocks are not whole waves, the antiperiodic boundary on a tile's edge, the large
tiles of the FP64 dots.

Both forms add the same terms of a site in the same order, so y is the same bits.  The
dots are FP64 sums of n products in another order: 1e-13 of the norms (n < 2^20 terms
of rounding 2^-53, whose errors add up as sqrt(n)).
"""
import pytest

pytestmark = pytest.mark.gpu

from lattice_inputs import gauge_field  # noqa: E402


@pytest.mark.parametrize("dims,prec,nrhs", [
    ((8, 8, 8, 16), "f64", 4), ((8, 8, 8, 16), "f64", 12), ((16, 8, 6, 12), "f64", 8), ((16, 8, 6, 12), "f32", 6),
    ((9, 6, 15, 10), "f64", 7), ((9, 6, 15, 10), "f32", 14), ((12, 10, 14, 18), "f64", 8), ((16, 16, 16, 16), "f64", 1),
    ((16, 16, 16, 16), "f32", 3), ((2, 2, 48, 64), "f64", 16), ((4, 2, 48, 64), "f32", 32), ((8, 8, 8, 8), "f64", 32)])
def test_tiles_match_the_untiled_form(dims, prec, nrhs):
    import torch
    import paper_2509_11424_amd as m
    U = gauge_field(dims, 0.6, 81)
    tiled, plain = (m.Operator(m.Context(0), U, 0.03, 1.0) for _ in range(2))
    V = tiled.V
    for k in ("dslash/", "dslash_dot/"):
        plain.ctx.tune_set(k + "%d/%d/%d" % (m.api.PREC[prec], V, nrhs), 0)
    g = torch.Generator(device="cuda:0").manual_seed(nrhs)
    x = torch.view_as_complex(torch.randn((12, V, nrhs, 2), generator=g, device="cuda:0", dtype=torch.float64))
    if prec == "f32":
        x = x.to(torch.complex64)
    ya, yb = tiled.apply(x, prec=prec), plain.apply(x, prec=prec)
    (da, qra, qqa), (db, qrb, qqb) = tiled.apply_dot(x, prec=prec), plain.apply_dot(x, prec=prec)
    torch.cuda.synchronize()
    assert torch.equal(ya, yb) and torch.equal(da, db) and torch.equal(ya, da)
    n = qqb.sqrt() * x.to(torch.complex128).abs().square().sum(dim=(0, 1)).sqrt()
    assert torch.all((qra - qrb).abs() <= 1e-13 * n)
    assert torch.all((qqa - qqb).abs() <= 1e-13 * qqb)


@pytest.mark.parametrize("dims,prec,nrhs", [((16, 16, 16, 32), "f64", 12), ((32, 32, 8, 8), "f32", 12),
                                           ((16, 16, 32, 32), "f32", 12), ((16, 16, 32, 32), "f16", 24)])
def test_long_vectors_match_single_columns(dims, prec, nrhs):
    """Results stored past the caches (over 256 MB) and boxes walked in bands, against
    launches of one column, which take neither; the same sums, so the same bits in FP64 and
    FP32.  FP16 marching and site-parallel forms may sum in another order: one ulp."""
    import torch
    import paper_2509_11424_amd as m
    op = m.Operator(m.Context(0), gauge_field(dims, 0.6, 83), 0.03, 1.0)
    g = torch.Generator(device="cuda:0").manual_seed(nrhs)
    xr = torch.randn((12, op.V, nrhs, 2), generator=g, device="cuda:0", dtype=torch.float32)
    x = {"f64": lambda: torch.view_as_complex(xr.double()), "f32": lambda: torch.view_as_complex(xr),
         "f16": lambda: xr.to(torch.float16)}[prec]()
    y = op.apply(x, prec=prec)
    for r in (0, 1, nrhs - 1):
        y1 = op.apply(x[:, :, r:r + 1].contiguous(), prec=prec)
        torch.cuda.synchronize()
        a, b = y[:, :, r], y1[:, :, 0]
        if prec == "f16":
            a, b = a.double(), b.double()
            assert torch.all((a - b).abs() <= 2.0 ** -10 * b.abs() + 2.0 ** -14)
        else:
            assert torch.equal(a, b)
