"""Mixed-precision transfers against 64-bit products with the P they use (rounded to
FP16), so that their own summation error shows: FP32 sums of n products of random sign
round to about 2^-24 sqrt(n / 6) in norm, 6e-7 at the 648 real products of the longest sum here;
1e-6.  FP16 inputs below the normal range (6.1e-5) count in full.  An infinity in one
right-hand side changes no bit of the others.  Row counts 72 and 324 (one wave and four
per aggregate), test vectors around 8, 16 and 32, one to five tiles of 8 right-hand sides."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from lattice_inputs import gauge_field  # noqa: E402


@pytest.mark.parametrize("dims,block", [((4, 6, 4, 4), (2, 3, 1, 2)), ((6, 6, 6, 4), (3, 3, 3, 2))])
@pytest.mark.parametrize("ntv", [1, 7, 9, 12, 24, 33])
def test_transfers_against_rounded_p(dims, block, ntv):
    import torch
    import paper_2509_11424_amd as m
    op = m.Operator(m.Context(0), gauge_field(dims, 0.6, 71), 0.05, 1.0)
    h = m.Hierarchy(op, [block], [ntv], seed=3, setup_steps=1, max_nrhs=50, restart=2, mixed=2)
    (vf, df, _), (vc, dc, _) = h.level_info(0), h.level_info(1)
    P64 = np.ascontiguousarray(h.export(0, "P")).view(np.float64)
    P = torch.from_numpy(P64.astype(np.float16).astype(np.float64).view(np.complex128)).cuda()
    rows = torch.from_numpy(h.export(0, "agg_map")).cuda()
    site, dof = rows // df, rows % df

    def restrict(x):
        return (P.conj().unsqueeze(-1) * x[dof, site].unsqueeze(3)).sum(2).reshape(vc, dc, -1).permute(1, 0, 2)

    def prolong(c):
        y = torch.empty((df, vf, c.shape[2]), dtype=c.dtype, device="cuda")
        y[dof, site] = (P.unsqueeze(-1) * c.reshape(2, ntv, vc, -1).permute(2, 0, 1, 3).unsqueeze(2)).sum(3)
        return y

    def off(a, b):
        return ((a.to(torch.complex128) - b).abs().square().sum() / b.abs().square().sum()).sqrt().item()

    g = torch.Generator(device="cuda:0").manual_seed(ntv)
    for nrhs in (1, 9, 16, 25, 33, 40, 50):
        x = torch.view_as_complex(torch.randn((df, vf, nrhs, 2), generator=g, device="cuda:0", dtype=torch.float32))
        c = torch.view_as_complex(torch.randn((dc, vc, nrhs, 2), generator=g, device="cuda:0", dtype=torch.float32))
        x64, c64 = x.to(torch.complex128), c.to(torch.complex128)
        yr, yp = h.restrict(0, x, "f32"), h.prolong(0, c, "f32")
        assert off(yr, restrict(x64)) < 1e-6, nrhs
        assert off(yp, prolong(c64)) < 1e-6, nrhs
        # FP16 vectors of unit size, and scaled down to where most entries are subnormal
        for scale in (1.0, 2.0 ** -17):
            x16 = (torch.view_as_real(x) * scale).half().contiguous()
            xe = torch.view_as_complex(x16.double())
            s = (torch.rand(nrhs, generator=g, device="cuda:0", dtype=torch.float64) + 0.5) / scale
            assert off(h.restrict_f16(0, x16, s), restrict(xe * s)) < 1e-6, (nrhs, scale)
            assert off(h.prolong_add_f16(0, c, x16, s), xe * s + prolong(c64)) < 1e-6, (nrhs, scale)
        if nrhs == 1:
            continue
        x16 = torch.view_as_real(x).half().contiguous()
        s = torch.ones(nrhs, device="cuda:0", dtype=torch.float64)
        calls = [(lambda: h.restrict(0, x, "f32")), (lambda: h.prolong(0, c, "f32")), (lambda: h.restrict(0, x64)),
                 (lambda: h.prolong(0, c64)), (lambda: h.restrict_f16(0, x16, s)),
                 (lambda: h.prolong_add_f16(0, c, x16, s)), (lambda: h.project_out(0, x64))]
        clean = [f() for f in calls]
        for t in (x, x64, c, c64, x16):
            t[:, :, nrhs // 2] = float("inf")
        for f, want in zip(calls, clean):
            got = f()
            for part in (slice(0, nrhs // 2), slice(nrhs // 2 + 1, nrhs)):
                assert torch.equal(got[:, :, part], want[:, :, part]), nrhs
