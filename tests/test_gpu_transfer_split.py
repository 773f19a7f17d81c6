"""Transfers where the split over workgroups changes: few aggregates (four waves on
aggregates of few rows, fewer tiles of right-hand sides per workgroup) and many (one wave), one
to nine tiles of 8 right-hand sides, test vectors over one to three tiles.  Every column
equals that of a launch of its own eight: the same products, summed in another order
where the rows are split over waves, 1e-14 in norm in FP64 and 1e-6 in FP32."""
import pytest

pytestmark = pytest.mark.gpu

from lattice_inputs import gauge_field  # noqa: E402


@pytest.mark.parametrize("dims,block,ntv", [((4, 4, 4, 4), (2, 2, 2, 2), 8), ((4, 4, 4, 8), (2, 2, 2, 4), 40),
                                            ((16, 16, 8, 16), (2, 2, 2, 2), 12), ((8, 8, 16, 32), (2, 2, 2, 2), 20),
                                            ((8, 8, 8, 8), (4, 4, 4, 4), 17)])
def test_columns_do_not_depend_on_the_split(dims, block, ntv):
    import torch
    import paper_2509_11424_amd as m
    op = m.Operator(m.Context(0), gauge_field(dims, 0.6, 75), 0.05, 1.0)
    h = m.Hierarchy(op, [block], [ntv], seed=3, setup_steps=1, max_nrhs=72, restart=2, mixed=2)
    (vf, df, _), (vc, dc, _) = h.level_info(0), h.level_info(1)
    g = torch.Generator(device="cuda:0").manual_seed(ntv)
    x = torch.view_as_complex(torch.randn((df, vf, 72, 2), generator=g, device="cuda:0", dtype=torch.float64))
    c = torch.view_as_complex(torch.randn((dc, vc, 72, 2), generator=g, device="cuda:0", dtype=torch.float64))
    s = torch.rand(72, generator=g, device="cuda:0", dtype=torch.float64) + 0.5

    def off(a, b):
        a, b = a.to(torch.complex128), b.to(torch.complex128)
        return ((a - b).abs().square().sum() / b.abs().square().sum()).sqrt().item()

    def calls(k):
        x1, c1 = x[:, :, k].contiguous(), c[:, :, k].contiguous()
        x32, c32 = x1.to(torch.complex64), c1.to(torch.complex64)
        x16 = torch.view_as_real(x32).half().contiguous()
        return [h.restrict(0, x1), h.prolong(0, c1), h.project_out(0, x1), h.restrict(0, x32, "f32"),
                h.prolong(0, c32, "f32"), h.restrict_f16(0, x16, s[k].contiguous()),
                h.prolong_add_f16(0, c32, x16, s[k].contiguous())]

    single = [torch.cat(p, dim=2) for p in zip(*(calls(slice(r, r + 8)) for r in range(0, 72, 8)))]
    for nrhs in (1, 9, 16, 17, 25, 33, 41, 50, 64, 72):
        for i, y in enumerate(calls(slice(0, nrhs))):
            assert off(y, single[i][:, :, :nrhs]) < (1e-14 if i < 3 else 1e-6), (nrhs, i)
