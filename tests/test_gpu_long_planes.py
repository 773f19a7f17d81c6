"""Planes past 4 GiB, which take the kernels with 64-bit byte offsets, against launches of
one column, which take those with 32-bit ones: the dslash and its dots (32^3 x 64, 128
right-hand sides in FP64, 256 in FP32, 512 in FP16: planes of 2^32 bytes) and a network layer (256).
The same sums in the same order: the same bits in FP64 and FP32, one ulp in FP16 (the
default form of a single column may march); dots of n = 2.5e7 products in another order,
2^-53 sqrt(n) = 6e-13 of the norms: 2e-12.  Vectors are 51.5 GB each; the links are a small field
repeated."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from lattice_inputs import gauge_field  # noqa: E402


@pytest.fixture(scope="module")
def op():
    import torch
    import paper_2509_11424_amd as m
    yield m.Operator(m.Context(0), np.tile(gauge_field((8, 8, 8, 8), 0.6, 93), (8, 4, 4, 4, 1, 1, 1)), 0.03, 1.0)
    torch.cuda.empty_cache()


def _room(gb):
    import gc
    import torch
    gc.collect()
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gb * 1e9:
        pytest.skip("needs %d GB of free device memory" % gb)


@pytest.mark.parametrize("prec,nrhs", [("f64", 128), ("f32", 256), ("f16", 512)])
def test_dslash(op, prec, nrhs):
    import torch
    _room(115)
    g = torch.Generator(device="cuda:0").manual_seed(nrhs)
    dt = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}[prec]
    xr = torch.empty((12, op.V, nrhs, 2), dtype=dt, device="cuda:0")
    for k in range(12):
        xr[k].normal_(generator=g)
    x = xr if prec == "f16" else torch.view_as_complex(xr)
    y = torch.empty_like(x)
    op.apply(x, y, prec)
    kept = {r: y[:, :, r].clone() for r in (0, 1, nrhs - 1)}
    if prec != "f16":  # at most 256 right-hand sides
        _, yx, yy = op.apply_dot(x, y, prec)
    for r, col in kept.items():
        x1 = x[:, :, r:r + 1].contiguous()
        y1, yx1, yy1 = op.apply_dot(x1, prec=prec)
        one = op.apply(x1, prec=prec)[:, :, 0]
        torch.cuda.synchronize()
        if prec == "f16":
            a, b = col.double(), one.double()
            assert torch.all((a - b).abs() <= 2.0 ** -10 * b.abs() + 2.0 ** -14), r
            continue
        assert torch.equal(col, one) and torch.equal(y[:, :, r], y1[:, :, 0]), r
        n = yy1[0].sqrt() * x1.to(torch.complex128).abs().square().sum().sqrt()
        assert (yx[r] - yx1[0]).abs() <= 2e-12 * n and (yy[r] - yy1[0]).abs() <= 2e-12 * yy1[0], r


def test_network_layer(op):
    import torch
    import paper_2509_11424_amd as m
    _room(215)
    nrhs = 256
    net = m.Net(op, (4, 4), seed=1, max_nrhs=nrhs)
    g = torch.Generator(device="cuda:0").manual_seed(5)
    xr = torch.empty((12, op.V, nrhs, 2), dtype=torch.float32, device="cuda:0")
    for k in range(12):
        xr[k].normal_(generator=g)
    x = torch.view_as_complex(xr)
    y = net.apply(x, torch.empty_like(x))
    for r in (0, 100, nrhs - 1):
        x1 = x[:, :, r:r + 1].contiguous()
        y1 = net.apply(x1, torch.empty_like(x1))
        torch.cuda.synchronize()
        assert torch.equal(y[:, :, r], y1[:, :, 0]), r
