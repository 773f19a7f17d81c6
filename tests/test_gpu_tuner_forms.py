"""The launch forms beside the listed variants (boxes of sites, the site-parallel smoother
step): the report holds the time of every variant it names, a report set again in another
context gives the same launches, a pinned variant goes before a measured form, and
every form is checked against the listed ones.

Boxes and the untiled form add the same terms in the same order (the same bits).  The step
forms with one and two right-hand sides per thread do so too, so that their dots, FP64 sums
over the sites in another order, agree to 1e-12; r' may round to FP16 in one step with its last
product or after it.  Against the marching form (pinned variant 0) the dots, FP32 sums
per site, agree to 1e-6.  r' and x' agree to one FP16 ulp (2^-10 relative, 2^-14 near zero)."""
import pytest

pytestmark = pytest.mark.gpu

from lattice_inputs import gauge_field  # noqa: E402


def _ops(dims, n):
    import paper_2509_11424_amd as m
    U = gauge_field(dims, 0.6, 87)
    return [m.Operator(m.Context(0), U, 0.03, 1.0) for _ in range(n)]


def _form_key(kind, op, prec, nrhs):
    import paper_2509_11424_amd as m
    return "%s_form@%dx%dx%dx%d/%d/%d/%d" % ((kind,) + op.dims + (m.api.PREC[prec], op.V, nrhs))


def _check_report(rep):
    for k, (v, ms) in rep.items():
        assert 0 <= v < len(ms) and all(t > 0 for t in ms), (k, v, ms)


@pytest.mark.parametrize("dims,prec,nrhs", [((16, 16, 16, 16), "f64", 4), ((16, 16, 16, 8), "f32", 12)])
def test_box_form_in_the_report(dims, prec, nrhs):
    import torch
    import paper_2509_11424_amd as m
    tuned, again, box, free = _ops(dims, 4)
    dt = torch.complex128 if prec == "f64" else torch.complex64
    g = torch.Generator(device="cuda:0").manual_seed(nrhs)
    x = torch.view_as_complex(torch.randn((12, tuned.V, nrhs, 2), generator=g, device="cuda:0",
                                          dtype=torch.float64)).to(dt)
    tuned.ctx.autotune(True)
    y = tuned.apply(x, prec=prec)
    tuned.ctx.autotune(False)
    rep = tuned.ctx.tune_report()
    _check_report(rep)
    key, fkey = "dslash/%d/%d/%d" % (m.api.PREC[prec], tuned.V, nrhs), _form_key("dslash", tuned, prec, nrhs)
    assert set(rep) == {key, fkey} and len(rep[fkey][1]) == 2
    assert rep[fkey][1][0] == rep[key][1][rep[key][0]]
    for k, (v, _) in rep.items():
        again.ctx.tune_set(k, v)
    box.ctx.tune_set(fkey, 1)
    box.ctx.tune_set(key, 0)  # the pinned form goes before it
    torch.cuda.synchronize()
    for op in (again, box, free):
        z = op.apply(x, prec=prec)
        torch.cuda.synchronize()
        d = (z - y).abs()
        assert torch.equal(z, y) if prec == "f64" else torch.all(d <= 1e-5 * y.abs() + 1e-6 * y.abs().max())
    box.ctx.tune_set(fkey, 2)
    with pytest.raises(m.MgmError):
        box.apply(x, prec=prec)


def test_box_form_refused_where_there_is_none():
    import torch
    import paper_2509_11424_amd as m
    op, = _ops((8, 8, 8, 8), 1)
    x = torch.ones((12, op.V, 1), dtype=torch.complex128, device="cuda:0")
    op.ctx.tune_set(_form_key("dslash", op, "f64", 1), 1)
    with pytest.raises(m.MgmError):
        op.apply(x)
    op.ctx.tune_set(_form_key("dslash", op, "f64", 1), 0)
    op.apply(x)
    torch.cuda.synchronize()


@pytest.mark.parametrize("dims", [(8, 8, 8, 3), (16, 8, 8, 5)])
@pytest.mark.parametrize("nrhs", [1, 2, 6, 8, 12, 50])
def test_step_forms(dims, nrhs):
    import torch
    import paper_2509_11424_amd as m
    march, one, two, tuned = _ops(dims, 4)
    if not march.step_fusable(nrhs):
        pytest.skip("no marching shape: the step is refused")
    key, fkey = "dslash_step/%d/%d/%d" % (m.api.PREC["f16"], march.V, nrhs), _form_key("dslash_step", march, "f16", nrhs)
    g = torch.Generator(device="cuda:0").manual_seed(nrhs)
    r, x0 = (torch.randn((12, march.V, nrhs, 2), generator=g, device="cuda:0").to(torch.float16) for _ in range(2))
    qq = torch.rand(nrhs, generator=g, device="cuda:0", dtype=torch.float64) + 0.5
    qr = torch.complex(0.1 * qq, 0.02 * torch.rand(nrhs, generator=g, device="cuda:0", dtype=torch.float64))
    qq[0] = 0.0

    def step(op):
        x = x0.clone()
        rn, yx, yy = op.smoother_step(r, x, qr, qq)
        torch.cuda.synchronize()
        return rn.double(), x.double(), yx, yy

    march.ctx.tune_set(key, 0)
    one.ctx.tune_set(fkey, 1)
    a, b = step(march), step(one)
    norm = a[3].sqrt() * r.double().square().sum(dim=(0, 1, 3)).sqrt()

    def close(a, b, dots):
        assert torch.all((a[0] - b[0]).abs() <= 2.0 ** -10 * a[0].abs() + 2.0 ** -14)
        assert torch.all((a[1] - b[1]).abs() <= 2.0 ** -10 * a[1].abs() + 2.0 ** -14)
        assert torch.all((a[2] - b[2]).abs() <= dots * norm)
        assert torch.all((a[3] - b[3]).abs() <= dots * a[3])

    close(a, b, 1e-6)
    two.ctx.tune_set(fkey, 2)
    if nrhs % 2:
        with pytest.raises(m.MgmError):
            step(two)
    else:
        close(b, step(two), 1e-12)
    tuned.ctx.autotune(True)
    step(tuned)
    tuned.ctx.autotune(False)
    rep = tuned.ctx.tune_report()
    _check_report(rep)
    assert len(rep[key][1]) % 2 == 0 and len(rep[fkey][1]) == (2 if nrhs % 2 else 3)
    tuned.ctx.tune_set(key, 0)  # goes before whatever form was measured
    d = step(tuned)
    assert all(torch.equal(p, q) for p, q in zip(a, d))
