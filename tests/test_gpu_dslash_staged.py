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


def test_modes_with_a_remainder(cuda):
    """Every mode of the stencil (MR partial sums in FP64, the q recursion in
    the FP32 classes, residuals) and one right-hand side's FP64 transfers on a
    volume that is neither whole tiles nor whole 256-site blocks and too large
    for the latency form (34 320 sites, aggregates of 66), through the V-cycle
    against the oracle's.  One, three (a ragged group of two, a whole one of
    three) and four right-hand sides (groups of two).  Bounds: those of the
    V-cycle's parity on small lattices, 1e-10 in FP64, rounding of some 50
    vector operations of 6e-8 and of stored binary16 otherwise."""
    import paper_1005_3043_amd as mgwd
    from oracle import solvers as so
    L, block, nv, m = (11, 13, 16, 15), (11, 1, 2, 3), 2, 0.15
    U, starts = W.gauge_field(L, 0.4, 6), W.setup_starts(L, nv, 6)
    h = so.mg_setup(U, m, so.MGParams(blocks=[block], nv=[nv], setup_rounds=1), starts)
    r = W.gaussian_spinor(L, 5, batch=(4,))
    ref = []
    for k in range(4):
        ref.append(h.vcycle(r[k], 0))
        print(f"oracle cycle {k}", flush=True)
    ctx = mgwd.MG(torch.from_numpy(U).cuda(), m, [block], [nv], [torch.from_numpy(starts).cuda()], setup_rounds=1,
                  max_rhs=4)
    for prec, tol in (("f64", 1e-10), ("f32", 1e-4), ("f16", 2e-3)):
        for nrhs in (1, 3, 4):
            z, _ = ctx.vcycle(torch.from_numpy(r[:nrhs]).cuda(), prec)
            z = z.cpu().numpy().reshape((nrhs,) + ref[0].shape)
            for k in range(nrhs):
                e = np.linalg.norm(z[k] - ref[k]) / np.linalg.norm(ref[k])
                print(f"{prec} x{nrhs} rhs {k}: {e:.2e}")
                assert e <= tol, (prec, nrhs, k)
    ctx.close()


@pytest.mark.timeout(240)
def test_groups_chunk_by_chunk(cuda):
    """Twelve right-hand sides on 16^3 x 64: two chunks of 512 blocks in the
    order of the right-hand-side groups (two or three per thread).  The
    operator in each class on 2048 sampled sites against the oracle, bounds as
    above; and the V-cycle, which in the binary16 class keeps its residuals in
    binary16 with a scale per site, against one FP64 right-hand side at a time
    (another kernel and no chunks).  There eight smoothing steps round links,
    operator and residual by 4.9e-4 of the site's scale each: 1e-2 in the
    norm, and no entry further off than a quarter of the rms entry, where a
    block out of place would be off by the entry itself."""
    import paper_1005_3043_amd as mgwd
    L, block, nv, m = (16, 16, 16, 64), (4, 4, 4, 4), 2, 0.15
    U, starts = W.gauge_field(L, 0.3, 6), W.setup_starts(L, nv, 6)
    rng = np.random.default_rng(7)
    sites = np.stack([rng.integers(0, L[mu], 2048) for mu in range(4)], 1)
    sites[:4] = [(0, 0, 0, 0), (15, 15, 15, 63), (0, 15, 0, 31), (15, 0, 15, 32)]
    v = W.gaussian_spinor(L, 8, batch=(12,))
    ref = wi.apply_D_sites(U, v, m, sites)
    ctx = mgwd.MG(torch.from_numpy(U).cuda(), m, [block], [nv], [torch.from_numpy(starts).cuda()], setup_rounds=1,
                  max_rhs=12, coarse_tol=1e-6)
    d = torch.from_numpy(v).cuda()
    for prec, tol in (("f64", 1e-13), ("f32", 1e-5), ("f16", 2e-3)):
        got = ctx.apply_op(0, d, prec).cpu().numpy()[:, sites[:, 3], sites[:, 2], sites[:, 1], sites[:, 0]]
        for k in range(12):
            assert np.linalg.norm(got[k] - ref[k]) <= tol * np.linalg.norm(ref[k]), (prec, k)
            assert np.abs(got[k] - ref[k]).max() <= 20 * tol, (prec, k)
    z64 = torch.stack([ctx.vcycle(d[k], "f64")[0].reshape(v.shape[1:]) for k in range(12)])
    print("FP64 cycles done", flush=True)
    for prec, tol in (("f64", 1e-10), ("f32", 1e-4), ("f16", 1e-2)):
        z, _ = ctx.vcycle(d, prec)
        for k in range(12):
            e = float((z[k] - z64[k]).norm() / z64[k].norm())
            worst = float((z[k] - z64[k]).abs().max() / (z64[k].norm() / z64[k].numel() ** 0.5))
            if k == 0:
                print(f"{prec}: {e:.2e}, largest entry {worst:.2e} rms", flush=True)
            assert e <= tol and worst <= 0.25, (prec, k, e, worst)
    ctx.close()
