"""Links and clover in groups of 16 bytes: lattices whose volume no group size divides
(odd ones too), every storage format, one or two right-hand sides per thread.

A row of D sums terms whose magnitudes add up to at most 12 |x| (the mass and clover
term, eight hops), each of rounded factors, against |D x| of at least |x|: 12 units
of the format, 12 * 2^-24 in FP32 and 12 * 2^-11 in FP16, 1e-13 in FP64.
"""
import pytest

pytestmark = pytest.mark.gpu

from gpu_common import to_gpu, from_gpu, rel  # noqa: E402
from lattice_inputs import gauge_field, random_spinor  # noqa: E402


@pytest.mark.parametrize("dims", [(5, 3, 11, 7), (3, 3, 3, 3), (2, 3, 2, 3), (9, 2, 3, 7)])
@pytest.mark.parametrize("prec,nrhs,tol", [("f64", 1, 1e-13), ("f64", 5, 1e-13), ("f32", 1, 12 * 2.0 ** -24),
                                           ("f32", 4, 12 * 2.0 ** -24), ("f16", 1, 12 * 2.0 ** -11),
                                           ("f16", 6, 12 * 2.0 ** -11)])
def test_apply_on_undivided_volumes(dims, prec, nrhs, tol):
    import torch
    import paper_2509_11424_amd as m
    from oracle.dirac import WilsonClover
    U = gauge_field(dims, 0.6, 71)
    op = m.Operator(m.Context(0), U, 0.03, 1.0)
    xs = random_spinor(dims, 72, batch=nrhs)
    x = to_gpu(xs.reshape(nrhs, -1, 12))
    if prec == "f32":
        x = x.to(torch.complex64)
    if prec == "f16":
        x = torch.view_as_real(x).to(torch.float16)
    y = op.apply(x, prec=prec)
    yd, yx, yy = op.apply_dot(x, prec=prec)
    torch.cuda.synchronize()
    as64 = (lambda t: torch.view_as_complex(t.double())) if prec == "f16" else (lambda t: t.to(torch.complex128))
    want = WilsonClover(U, 0.03, 1.0).apply(xs).reshape(nrhs, -1)
    assert rel(from_gpu(as64(y)).reshape(nrhs, -1), want) < tol
    assert rel(from_gpu(as64(yd)).reshape(nrhs, -1), want) < tol
