"""Transfers at the edges of their tiles: test-vector counts around 8, 16 and
32, right-hand sides around 8, 16 and 32, aggregates whose rows do not fill a
step, with one and with four waves per aggregate.  Against products with the
exported P in FP64: 1e-13 in norm for FP64 (sums of up to 324 products); the
mixed forms use P rounded to FP16 (relative 2^-11 an entry) with FP32 sums:
1e-3 in norm."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from lattice_inputs import gauge_field  # noqa: E402


@pytest.mark.parametrize("dims,block", [((4, 6, 4, 4), (2, 3, 1, 2)), ((6, 6, 6, 4), (3, 3, 3, 2))])
@pytest.mark.parametrize("ntv", [1, 7, 8, 9, 17, 24, 33])
def test_transfer_tiles(dims, block, ntv):
    import torch
    import paper_2509_11424_amd as m
    op = m.Operator(m.Context(0), gauge_field(dims, 0.6, 71), 0.05, 1.0)
    h = m.Hierarchy(op, [block], [ntv], seed=3, setup_steps=1, max_nrhs=33, restart=2, mixed=2)
    (vf, df, _), (vc, dc, _) = h.level_info(0), h.level_info(1)
    P = torch.from_numpy(h.export(0, "P")).cuda()
    rows = torch.from_numpy(h.export(0, "agg_map")).cuda()
    site, dof = rows // df, rows % df

    def restrict(x):
        w = x[dof, site]
        return (P.conj().unsqueeze(-1) * w.unsqueeze(3)).sum(2).reshape(vc, dc, -1).permute(1, 0, 2)

    def prolong(c):
        w = c.reshape(2, ntv, vc, -1).permute(2, 0, 1, 3)
        y = torch.empty((df, vf, c.shape[2]), dtype=c.dtype, device="cuda")
        y[dof, site] = (P.unsqueeze(-1) * w.unsqueeze(2)).sum(3)
        return y

    def off(a, b):
        return ((a.to(torch.complex128) - b).abs().square().sum() / b.abs().square().sum()).sqrt().item()

    g = torch.Generator(device="cuda:0").manual_seed(ntv)
    for nrhs in (1, 7, 8, 9, 17, 25, 33):
        x = torch.view_as_complex(torch.randn((df, vf, nrhs, 2), generator=g, device="cuda:0", dtype=torch.float64))
        c = torch.view_as_complex(torch.randn((dc, vc, nrhs, 2), generator=g, device="cuda:0", dtype=torch.float64))
        assert off(h.restrict(0, x), restrict(x)) < 1e-13, nrhs
        assert off(h.prolong(0, c), prolong(c)) < 1e-13, nrhs
        assert off(h.project_out(0, x), x - prolong(restrict(x))) < 1e-13, nrhs
        x32, c32 = x.to(torch.complex64), c.to(torch.complex64)
        x16 = torch.view_as_real(x32).to(torch.float16).contiguous()
        xe = torch.view_as_complex(x16.double())
        s = torch.rand(nrhs, generator=g, device="cuda:0", dtype=torch.float64) + 0.5
        assert off(h.restrict(0, x32, "f32"), restrict(x)) < 1e-3, nrhs
        assert off(h.prolong(0, c32, "f32"), prolong(c)) < 1e-3, nrhs
        assert off(h.restrict_f16(0, x16, s), restrict(xe * s)) < 1e-3, nrhs
        assert off(h.prolong_add_f16(0, c32, x16, s), xe * s + prolong(c)) < 1e-3, nrhs
