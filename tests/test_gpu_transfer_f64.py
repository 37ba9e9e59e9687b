"""FP64 fine-level transfers on the matrix cores, on canonical arrays
(mg_restrict, mg_prolong) and, with several right-hand sides, inside the FP64
V-cycle: aggregates that are not whole 16-site chunks or whole tiles, Nv
that is not a multiple of the tile or k-step, and right-hand sides from one
to more than a workgroup takes; against the oracle's P."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import solvers as so
from oracle import transfer as tr

pytestmark = pytest.mark.gpu

CASES = [((4, 4, 4, 4), (2, 1, 1, 1), 1), ((6, 6, 4, 6), (3, 3, 2, 3), 17), ((6, 4, 2, 8), (3, 2, 1, 4), 5),
         ((8, 8, 4, 8), (4, 4, 4, 4), 32), ((8, 4, 4, 4), (4, 4, 4, 4), 9)]


@pytest.mark.parametrize("L,block,nv", CASES)
def test_canonical_transfers(cuda, L, block, nv):
    import paper_1005_3043_amd as mgwd
    U, starts = W.gauge_field(L, 0.3, 2), W.setup_starts(L, nv, 2)
    ctx = mgwd.MG(torch.from_numpy(U).cuda(), 0.1, [block], [nv], [torch.from_numpy(starts).cuda()], setup_rounds=1)
    geom = tr.BlockGeometry(L, block)
    P = ctx.export_P(0)  # [Vc, 2, rows, nv]
    for nrhs in (1, 2, 12, 16, 17, 33):
        psi = W.gaussian_spinor(L, nrhs, batch=(nrhs,))
        F = geom.blockify(tr.fine_to_generic(psi))  # [nrhs, Vc, 2, rows]
        cref = np.einsum("cxri,ncxr->ncxi", np.conj(P), F).reshape(nrhs, -1)
        c = ctx.restrict(0, torch.from_numpy(psi).cuda())
        got = c.cpu().numpy().reshape(nrhs, -1)
        assert np.linalg.norm(got - cref) <= 1e-13 * np.linalg.norm(cref), nrhs
        fref = geom.unblockify(np.einsum("cxri,ncxi->ncxr", P, got.reshape(nrhs, geom.Vc, 2, nv)))
        f = ctx.prolong(0, c).cpu().numpy().reshape(fref.shape)
        assert np.linalg.norm(f - fref) <= 1e-13 * np.linalg.norm(fref), nrhs


def test_vcycle_several_rhs(cuda):
    """The V-cycle's own transfers (internal layout, prolongation added into
    the smoothed vector) with 3 right-hand sides against the oracle."""
    import paper_1005_3043_amd as mgwd
    L, block, nv, m = (6, 4, 4, 6), (3, 2, 2, 3), 5, -0.1
    U, starts = W.gauge_field(L, 0.3, 2), W.setup_starts(L, nv, 2)
    ctx = mgwd.MG(torch.from_numpy(U).cuda(), m, [block], [nv], [torch.from_numpy(starts).cuda()], max_rhs=3)
    h = so.mg_setup(U, m, so.MGParams(blocks=[block], nv=[nv]), starts)
    r = W.gaussian_spinor(L, 5, batch=(3,))
    z, _ = ctx.vcycle(torch.from_numpy(r).cuda(), "f64")
    z = z.cpu().numpy()
    for k in range(3):
        ref = h.vcycle(r[k], 0)
        assert np.linalg.norm(z[k] - ref) <= 1e-10 * np.linalg.norm(ref)


@pytest.mark.parametrize("L,nv,nrhs", [
    ((8, 8, 16, 16), 9, (12, 13, 16, 17)),  # 64 aggregates: both lines (768 and 1024 aggregates times vectors)
    ((12, 12, 12, 12), 17, (1, 12, 13)),    # 81: restriction's, with two row tiles
    ((16, 16, 16, 16), 9, (1, 2, 5)),       # 256: prolongation of one vector too
    ((8, 8, 8, 20), 32, (26,)),             # 40, the largest Nv, two groups of 13 vectors
])
def test_lines_between_kernels(cuda, L, nv, nrhs):
    """4^4 aggregates, few and many of them: both sides of the lines between
    the matrix-core and the vector kernels."""
    import paper_1005_3043_amd as mgwd
    block = (4, 4, 4, 4)
    U, starts = W.gauge_field(L, 0.3, 2), W.setup_starts(L, nv, 2)
    ctx = mgwd.MG(torch.from_numpy(U).cuda(), 0.1, [block], [nv], [torch.from_numpy(starts).cuda()], setup_rounds=0)
    geom = tr.BlockGeometry(L, block)
    P = ctx.export_P(0)
    for k in nrhs:
        psi = W.gaussian_spinor(L, k, batch=(k,))
        F = geom.blockify(tr.fine_to_generic(psi))
        cref = np.einsum("cxri,ncxr->ncxi", np.conj(P), F, optimize=True).reshape(k, -1)
        c = ctx.restrict(0, torch.from_numpy(psi).cuda())
        got = c.cpu().numpy().reshape(k, -1)
        assert np.linalg.norm(got - cref) <= 1e-13 * np.linalg.norm(cref), k
        fref = geom.unblockify(np.einsum("cxri,ncxi->ncxr", P, got.reshape(k, geom.Vc, 2, nv), optimize=True))
        f = ctx.prolong(0, c).cpu().numpy().reshape(fref.shape)
        assert np.linalg.norm(f - fref) <= 1e-13 * np.linalg.norm(fref), k
    ctx.close()
