"""The autotuner with two lattices of one volume in one context, whose lists of launch
variants differ (a box or marching shapes on one of them only): each call is tuned for
its own lattice, none is refused, and a pinned variant holds for both.

FP64 and FP32 forms add the same terms in the same order except the marching ones, so the
tuned y is within 1e-5 of the untuned one element by element (FP32; the same bits in FP64).
"""
import pytest

pytestmark = pytest.mark.gpu

from lattice_inputs import gauge_field  # noqa: E402

BOX, NONE = (16, 16, 11, 13), (11, 13, 16, 16)
MARCH, FEW = (8, 16, 8, 4), (4, 4, 4, 64)


@pytest.mark.parametrize("first,second,prec,nrhs", [
    (BOX, NONE, "f64", 4), (NONE, BOX, "f64", 4), (BOX, NONE, "f32", 8), (MARCH, FEW, "f32", 4), (MARCH, FEW, "f16", 4)])
def test_two_lattices_of_one_volume(first, second, prec, nrhs):
    import torch
    import paper_2509_11424_amd as m
    tuned, plain = m.Context(0), m.Context(0)
    fields = [gauge_field(d, 0.6, 85) for d in (first, second)]
    ops = [[m.Operator(c, U, 0.03, 1.0) for U in fields] for c in (tuned, plain)]
    V = ops[0][0].V
    g = torch.Generator(device="cuda:0").manual_seed(nrhs)
    xr = torch.randn((12, V, nrhs, 2), generator=g, device="cuda:0", dtype=torch.float64)
    x = {"f64": lambda: torch.view_as_complex(xr), "f32": lambda: torch.view_as_complex(xr.float()),
         "f16": lambda: xr.to(torch.float16)}[prec]()
    tuned.autotune(True)
    ys = [[op.apply(x, prec=prec), *op.apply_dot(x, prec=prec)] for op in ops[0]]
    tuned.autotune(False)
    again = [op.apply(x, prec=prec) for op in ops[0]]
    torch.cuda.synchronize()
    for k in range(2):
        want = [ops[1][k].apply(x, prec=prec), *ops[1][k].apply_dot(x, prec=prec)]
        torch.cuda.synchronize()
        assert torch.equal(ys[k][0], again[k])
        for got, ref in ((ys[k][0], want[0]), (ys[k][1], want[1])):
            if prec == "f64":
                assert torch.equal(got, ref)
            elif prec == "f32":
                assert torch.all((got - ref).abs() <= 1e-5 * ref.abs() + 1e-6 * ref.abs().max())
            else:  # one FP16 ulp
                a, b = got.double(), ref.double()
                assert torch.all((a - b).abs() <= 2.0 ** -10 * b.abs() + 2.0 ** -14)
        assert torch.all((ys[k][3] - want[3]).abs() <= 2e-3 * want[3])
    rep = tuned.tune_report()
    for kind in ("dslash", "dslash_dot"):
        rest = "/%d/%d/%d" % (m.api.PREC[prec], V, nrhs)
        assert kind + rest in rep
        assert "%s@%dx%dx%dx%d%s" % ((kind,) + second + (rest,)) in rep
    # a pin names the volume alone and holds for both lattices
    tuned.tune_set("dslash/%d/%d/%d" % (m.api.PREC[prec], V, nrhs), 99)
    for op in ops[0]:
        with pytest.raises(m.MgmError):
            op.apply(x, prec=prec)
