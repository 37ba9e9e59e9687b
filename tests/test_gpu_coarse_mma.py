"""FP32 matrix-core coarse stencil (every variant, FP32 and binary16 storage)
at the largest row counts, where a workgroup's LDS passes 64 KB (n = 64 with
twelve right-hand sides: 60 KB of staged vectors or 64 KB of sums, and 6 KB
beside them), and at counts that are not whole row tiles, against the oracle
stencil on the exported operator.  Bounds: 9 n products of FP32 rounding, 6e-8
sqrt(9 n) with the operator's own 6e-8, and binary16's 4.9e-4 in its storage."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import coarse as co

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nv,nrhs", [(32, 12), (32, 1), (27, 12), (25, 14), (25, 5), (9, 16)])
@pytest.mark.parametrize("L,block", [((8, 8, 8, 8), (4, 4, 4, 4)), ((8, 4, 12, 4), (4, 2, 4, 4))])
def test_variants(cuda, L, block, nv, nrhs):
    import paper_1005_3043_amd as mgwd
    U, starts = W.gauge_field(L, 0.3, 4), W.setup_starts(L, nv, 4)
    ctx = mgwd.MG(torch.from_numpy(U).cuda(), 0.1, [block], [nv], [torch.from_numpy(starts).cuda()], setup_rounds=1,
                  max_rhs=16)
    X, Y = ctx.export_coarse_op(1)
    rng = np.random.default_rng(nv)
    v = rng.standard_normal((nrhs,) + X.shape[:-1]) + 1j * rng.standard_normal((nrhs,) + X.shape[:-1])
    ref = np.stack([co.coarse_apply(X, Y, u) for u in v])
    d = torch.from_numpy(v).cuda()
    for variant in (0, 1, 2, 4, 9, 10, 12):
        ctx.set_coarse_variant(variant)
        for prec, tol in (("f32", 3e-6), ("f16", 1e-3)):
            got = ctx.apply_op(1, d, prec).cpu().numpy().reshape(ref.shape)
            for k in range(nrhs):
                e = np.linalg.norm(got[k] - ref[k]) / np.linalg.norm(ref[k])
                assert e <= tol, (variant, prec, k, e)
    ctx.close()
