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
