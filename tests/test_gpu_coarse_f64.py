"""FP64 coarse stencil with several right-hand sides (FP64 matrix cores):
row counts that are not whole tiles or k-steps, right-hand sides at and over
what one workgroup takes, the operator and its adjoint, against the oracle
stencil on the exported operator."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import coarse as co

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,block,nv", [((4, 4, 4, 4), (2, 2, 2, 2), 1), ((6, 4, 2, 4), (3, 2, 1, 2), 5),
                                        ((8, 8, 4, 8), (4, 4, 4, 4), 9), ((8, 4, 4, 8), (4, 4, 4, 4), 32)])
def test_several_rhs(cuda, L, block, nv):
    import paper_1005_3043_amd as mgwd
    U, starts = W.gauge_field(L, 0.3, 4), W.setup_starts(L, nv, 4)
    ctx = mgwd.MG(torch.from_numpy(U).cuda(), 0.1, [block], [nv], [torch.from_numpy(starts).cuda()], setup_rounds=1)
    X, Y = ctx.export_coarse_op(1)
    rng = np.random.default_rng(nv)
    for nrhs in (2, 3, 12, 16, 17, 24):
        shp = (nrhs,) + X.shape[:-1]
        v = rng.standard_normal(shp) + 1j * rng.standard_normal(shp)
        d = torch.from_numpy(v).cuda()
        for dag, ref in ((False, co.coarse_apply), (True, co.coarse_apply_dag)):
            got = ctx.coarse_apply(1, d, dagger=dag).cpu().numpy()
            for k in range(nrhs):
                r = ref(X, Y, v[k])
                assert np.linalg.norm(got[k] - r) <= 1e-13 * np.linalg.norm(r), (nrhs, dag, k)


@pytest.mark.parametrize("L,block,nv,nrhs", [
    ((4, 4, 4, 4), (2, 2, 2, 2), 1, (64, 65)),     # 16 sites: both sides of the line, n = 2
    ((6, 4, 2, 4), (3, 2, 1, 2), 5, (65, 80)),     # n = 10, groups of 13 and of 16 right-hand sides
    ((8, 8, 4, 8), (4, 4, 4, 4), 9, (128, 129)),   # 8 sites: the line again, n = 18
    ((8, 4, 4, 8), (4, 4, 4, 4), 32, (128, 129)),  # 4 sites, not a multiple of 8: half as many
    ((4, 4, 4, 6), (2, 2, 2, 2), 10, (43,)),       # n = 20: the last batch of k-steps is half empty
    ((4, 4, 4, 6), (2, 2, 2, 2), 7, (1, 43)),      # n = 14
])
def test_matrix_cores_and_their_line(cuda, L, block, nv, nrhs):
    """Operator and adjoint on both sides of the line between one workgroup per
    site and one per site and right-hand side."""
    import paper_1005_3043_amd as mgwd
    U, starts = W.gauge_field(L, 0.3, 4), W.setup_starts(L, nv, 4)
    ctx = mgwd.MG(torch.from_numpy(U).cuda(), 0.1, [block], [nv], [torch.from_numpy(starts).cuda()], setup_rounds=1)
    X, Y = ctx.export_coarse_op(1)
    rng = np.random.default_rng(nv)
    for k in nrhs:
        shp = (k,) + X.shape[:-1]
        v = rng.standard_normal(shp) + 1j * rng.standard_normal(shp)
        d = torch.from_numpy(v).cuda()
        for dag, ref in ((False, co.coarse_apply), (True, co.coarse_apply_dag)):
            got = ctx.coarse_apply(1, d, dagger=dag).cpu().numpy()
            r = np.stack([ref(X, Y, u) for u in v])
            err = np.sqrt((np.abs(got.reshape(r.shape) - r) ** 2).reshape(k, -1).sum(1) /
                          (np.abs(r) ** 2).reshape(k, -1).sum(1))
            assert err.max() <= 1e-13, (k, dag)
    ctx.close()
