"""Fine stencil in its two forms, the hops of a tile on eight wavefronts (few
tiles) and a site per thread with the workgroup's own sites in LDS: volumes of
whole tiles and blocks, with a remainder, and of whole aggregates, with
right-hand sides that make full and ragged groups of two and of three, in each
precision class, against the oracle.  Bounds: rounding of about 1500 operations per site in
FP64 and FP32, half a binary16 unit (4.9e-4) in links and spinors otherwise."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import wilson as wi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,block", [((4, 4, 4, 4), (2, 2, 2, 2)), ((6, 4, 2, 6), (3, 2, 1, 2)),
                                     ((8, 4, 4, 8), (4, 4, 4, 4)), ((5, 4, 8, 4), (5, 4, 4, 2)),
                                     ((8, 8, 8, 16), (4, 4, 4, 4)), ((11, 13, 16, 15), (11, 1, 2, 3)),
                                     ((16, 16, 16, 9), (4, 4, 4, 3))])
def test_groups(cuda, L, block):
    import paper_1005_3043_amd as mgwd
    U, starts = W.gauge_field(L, 0.4, 6), W.setup_starts(L, 2, 6)
    m = 0.15
    rng = np.random.default_rng(L[0])
    shp = (7, L[3], L[2], L[1], L[0], 4, 3)
    v = rng.standard_normal(shp) + 1j * rng.standard_normal(shp)
    ref = np.stack([wi.apply_D(U, v[k], m) for k in range(7)])
    ctx = mgwd.MG(torch.from_numpy(U).cuda(), m, [block], [2], [torch.from_numpy(starts).cuda()], setup_rounds=0)
    for prec, tol in (("f64", 1e-13), ("f32", 1e-5), ("f16", 2e-3)):
        for nrhs in (1, 2, 3, 4, 5, 7):
            got = ctx.apply_op(0, torch.from_numpy(v[:nrhs]).cuda(), prec).cpu().numpy()
            for k in range(nrhs):
                assert np.linalg.norm(got[k] - ref[k]) <= tol * np.linalg.norm(ref[k]), (prec, nrhs, k)
    ctx.close()
