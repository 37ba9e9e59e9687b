"""Rounding of the FP64 matrix-core kernels: their sums are as short as those
of the vector kernels.  The reference is the same sum in extended precision
(numpy longdouble) of the same FP64 operands, so that only the kernel's own
rounding is left."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import transfer as tr

pytestmark = pytest.mark.gpu

LD = np.clongdouble


def _rel(a, b):
    return float(np.sqrt((np.abs(a.astype(LD) - b) ** 2).sum() / (np.abs(b) ** 2).sum()))


def _context(L, block, nv):
    import paper_1005_3043_amd as mgwd
    U, starts = W.gauge_field(L, 0.3, 2), W.setup_starts(L, nv, 2)
    return mgwd.MG(torch.from_numpy(U).cuda(), 0.1, [block], [nv], [torch.from_numpy(starts).cuda()], setup_rounds=1)


@pytest.mark.parametrize("L,block,nv", [((8, 8, 8, 8), (4, 4, 4, 4), 24), ((8, 8, 4, 8), (4, 4, 4, 4), 8),
                                        ((6, 6, 4, 6), (3, 3, 2, 3), 17), ((8, 12, 16, 16), (4, 4, 4, 4), 24),
                                        ((8, 12, 16, 16), (4, 4, 4, 4), 8)])
def test_restriction(cuda, L, block, nv):
    """P^dag f sums 6 |B| complex products.  A rounding is 0.47e-16 rms of the
    partial sum it is made on, and a partial sum of a random sum is on average
    half way there: a chain of d additions gives 0.47e-16 sqrt(d / 2), a tree
    0.47e-16 per level's square root.  12 products per thread and 8 levels make
    1.8e-16, the bound leaves a third; one chain of 1536 makes 13e-16."""
    ctx = _context(L, block, nv)
    geom = tr.BlockGeometry(L, block)
    P = ctx.export_P(0).astype(LD)  # [Vc, 2, rows, nv]
    for nrhs in (1, 2, 12):
        psi = W.gaussian_spinor(L, nrhs, batch=(nrhs,))
        F = geom.blockify(tr.fine_to_generic(psi)).astype(LD)
        ref = np.einsum("cxri,ncxr->ncxi", np.conj(P), F).reshape(nrhs, -1)
        got = ctx.restrict(0, torch.from_numpy(psi).cuda()).cpu().numpy().reshape(nrhs, -1)
        err = _rel(got, ref)
        print(f"restriction {L} nv {nv} x{nrhs}: {err:.2e}")
        assert err <= 2.5e-16, nrhs
    ctx.close()


@pytest.mark.parametrize("L,block,nv", [((8, 8, 8, 8), (4, 4, 4, 4), 8), ((16, 8, 8, 8), (4, 4, 4, 4), 24),
                                        ((8, 8, 4, 8), (4, 4, 4, 4), 32), ((8, 8, 8, 16), (4, 4, 4, 4), 10)])
def test_coarse_operator(cuda, L, block, nv):
    """Several right-hand sides of the coarse stencil round no more than one at
    a time, which the vector kernel sums (a tenth is left for the sample);
    160 of them, so that the matrix-core kernel
    takes them on these few sites too."""
    ctx = _context(L, block, nv)
    X, Y = (a.astype(LD) for a in ctx.export_coarse_op(1))
    rng = np.random.default_rng(nv)
    nrhs = 160
    v = rng.standard_normal((nrhs,) + X.shape[:-1]) + 1j * rng.standard_normal((nrhs,) + X.shape[:-1])
    ref = np.einsum("...ij,n...j->n...i", X, v.astype(LD))
    for d in range(8):
        mu, back = divmod(d, 2)
        nb = np.roll(v.astype(LD), 1 if back else -1, axis=(-2, -3, -4, -5)[mu])
        ref += np.einsum("...ij,n...j->n...i", Y[d], nb)
    dv = torch.from_numpy(v).cuda()
    one = np.concatenate([ctx.coarse_apply(1, dv[k:k + 1]).cpu().numpy().reshape(1, *v.shape[1:]) for k in range(12)])
    several = ctx.coarse_apply(1, dv).cpu().numpy().reshape(v.shape)
    ctx.close()
    e1, en = _rel(one, ref[:12]), _rel(several, ref)
    print(f"coarse operator n {2 * nv}: one at a time {e1:.2e}, several {en:.2e}")
    assert en <= 1.1 * e1
