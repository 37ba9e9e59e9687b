"""Whole-solve CGNR launch at the sizes where its exchange changes form (tagged
sums up to 128 coarse sites, arrival counters above) and at row counts that
take one, two or four operator rows per thread, in each precision class,
against the chunks of launches: bit for bit in 32-bit arithmetic, to the
rounding of 10^-3 CG iterates (1e-11) in FP64, iteration counts equal."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,block,nv", [((4, 4, 4, 4), (2, 2, 2, 2), 3), ((8, 8, 8, 8), (2, 2, 2, 4), 5),
                                        ((8, 8, 6, 6), (2, 2, 2, 2), 8), ((8, 8, 8, 16), (2, 2, 2, 2), 12)])
def test_exchange_forms(cuda, L, block, nv):
    import paper_1005_3043_amd as mgwd
    U, starts = W.gauge_field(L, 0.3, 9), W.setup_starts(L, nv, 9)
    Lc = [a // b for a, b in zip(L, block)]
    vol = Lc[0] * Lc[1] * Lc[2] * Lc[3]
    for prec in ("f64", "f32", "f16"):
        ctx = mgwd.MG(torch.from_numpy(U).cuda(), 0.1, [block], [nv], [torch.from_numpy(starts).cuda()],
                      setup_rounds=1, precond_prec=prec)
        ctx.set_coarse_variant(0)
        g = torch.Generator().manual_seed(vol)
        b = torch.randn(1, Lc[3], Lc[2], Lc[1], Lc[0], 2 * nv, dtype=torch.complex128, generator=g).cuda()
        out = []
        for on in (True, False, True):
            ctx.set_cgnr_persistent(on)
            out.append(ctx.coarse_solve(b, prec))
        ctx.close()
        (x1, i1), (x0, i0), (x2, i2) = out
        assert i1 == i0 == i2 and i1[0] > 3, (prec, i1, i0, i2)
        assert torch.equal(x1, x2), prec
        if prec == "f64":
            assert (x1 - x0).norm() <= 1e-11 * x0.norm()
        else:
            assert torch.equal(x1, x0), prec
