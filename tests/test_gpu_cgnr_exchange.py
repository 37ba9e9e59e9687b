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


@pytest.mark.parametrize("maxiter", [2**31 - 1, 2**31 - 2, 2**30])
def test_iteration_caps_near_the_largest(cuda, maxiter):
    """Coarse solves that follow one of a single iteration, with an iteration
    cap of "no limit": a launch must not take the words that the one before it
    left for its own (their tags repeated when they went up by twice the cap,
    modulo 2^32).  Against the same solves under a cap of 100, bit for bit, on 16
    coarse sites (tagged words)."""
    import paper_1005_3043_amd as mgwd
    L, block, nv = (8, 8, 8, 8), (4, 4, 4, 4), 8
    U, starts = W.gauge_field(L, 0.3, 9), W.setup_starts(L, nv, 9)
    g = torch.Generator().manual_seed(1)
    b = torch.randn(3, 1, 2, 2, 2, 2, 2 * nv, dtype=torch.complex128, generator=g).cuda()
    for prec in ("f64", "f32", "f16"):
        out = []
        for cap in (100, maxiter):
            ctx = mgwd.MG(torch.from_numpy(U).cuda(), 0.1, [block], [nv], [torch.from_numpy(starts).cuda()],
                          setup_rounds=1, coarse_tol=0.95, coarse_maxiter=cap)
            ctx.set_coarse_variant(0)
            out.append([ctx.coarse_solve(b[k], prec) for k in (0, 1, 2, 0, 1)])
            ctx.close()
        assert all(it == [1] for _, it in out[0]), [it for _, it in out[0]]
        for (x0, i0), (x1, i1) in zip(*out):
            assert i0 == i1 and torch.equal(x0, x1), prec


@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
def test_chunks_under_the_largest_cap(cuda, prec):
    """The number of chunks under a cap of 2^31 - 1 (it overflowed, no chunk
    ran and the solution was zero), one and three right-hand sides."""
    import paper_1005_3043_amd as mgwd
    L, block, nv = (8, 8, 8, 8), (4, 4, 4, 4), 8
    U, starts = W.gauge_field(L, 0.3, 9), W.setup_starts(L, nv, 9)
    g = torch.Generator().manual_seed(2)
    b = torch.randn(3, 2, 2, 2, 2, 2 * nv, dtype=torch.complex128, generator=g).cuda()
    out = []
    for cap in (100, 2**31 - 1):
        ctx = mgwd.MG(torch.from_numpy(U).cuda(), 0.1, [block], [nv], [torch.from_numpy(starts).cuda()],
                      setup_rounds=1, coarse_maxiter=cap, max_rhs=3)
        ctx.set_coarse_variant(0)
        ctx.set_cgnr_persistent(False)
        out.append([ctx.coarse_solve(b[:k], prec) for k in (1, 3)])
        ctx.close()
    for (x0, i0), (x1, i1) in zip(*out):
        assert i0 == i1 and min(i0) > 2 and torch.equal(x0, x1)


@pytest.mark.parametrize("L,block,nv", [((4, 4, 4, 4), (2, 2, 2, 2), 3), ((8, 8, 8, 8), (2, 2, 2, 4), 5),
                                        ((8, 8, 6, 6), (2, 2, 2, 2), 5), ((8, 8, 8, 16), (2, 2, 2, 2), 4)])
def test_whole_solve_runs_and_equals_the_chunks(cuda, L, block, nv):
    """In every precision class, FP64 too, the whole-solve launch ran (one timed
    launch per coarsest solve and no fallback; chunks take two per iteration)
    and its iterates are those of the chunks, bit for bit; 16, 128, 144 and 512
    coarse sites."""
    import paper_1005_3043_amd as mgwd
    U, starts = W.gauge_field(L, 0.3, 9), W.setup_starts(L, nv, 9)
    ctx = mgwd.MG(torch.from_numpy(U).cuda(), 0.1, [block], [nv], [torch.from_numpy(starts).cuda()], setup_rounds=1)
    ctx.set_coarse_variant(0)
    ctx.set_timing(True)
    g = torch.Generator().manual_seed(3)
    b = torch.randn(1, *(L[3 - k] // block[3 - k] for k in range(4)), 2 * nv, dtype=torch.complex128, generator=g)
    b = b.cuda()
    f = torch.randn(L[3], L[2], L[1], L[0], 4, 3, dtype=torch.complex128, generator=g).cuda()
    for prec, name in (("f64", "coarse_f64"), ("f32", "cgnr_f32"), ("f16", "cgnr_f16")):
        ctx.set_precond_prec(prec)
        out = {}
        for on in (True, False):
            ctx.set_cgnr_persistent(on)
            x, it = ctx.coarse_solve(b, prec)
            _, info, _ = ctx.solve(f, 1e-8)
            assert info["n_cgnr_fallbacks"] == 0
            launches = info["kernels"][name]["launches"]
            if on:
                assert launches == info["n_vcycles"], (prec, launches)
            elif prec == "f64":
                assert launches >= 2 * info["n_cgnr_iters"], launches
            else:
                assert launches == 0
            out[on] = (x, it, info["iters"][0], info["n_cgnr_iters"])
        assert out[True][1:] == out[False][1:] and out[True][1][0] > 3, prec
        assert torch.equal(out[True][0], out[False][0]), prec
    ctx.close()


def test_refused_shape_takes_the_chunks(cuda):
    """n = 40 in FP64 needs 30 operator entries per thread, more than the launch
    keeps in registers: chunks, without a fallback being counted; the FP32
    classes run the launch on the same 64 coarse sites."""
    import paper_1005_3043_amd as mgwd
    L, block, nv = (8, 8, 8, 8), (2, 2, 4, 4), 20
    U, starts = W.gauge_field(L, 0.3, 9), W.setup_starts(L, nv, 9)
    ctx = mgwd.MG(torch.from_numpy(U).cuda(), 0.1, [block], [nv], [torch.from_numpy(starts).cuda()], setup_rounds=1)
    ctx.set_coarse_variant(0)
    ctx.set_timing(True)
    f = torch.from_numpy(W.gaussian_spinor(L, 1)).cuda()
    for prec, name in (("f64", "coarse_f64"), ("f32", "cgnr_f32"), ("f16", "cgnr_f16")):
        ctx.set_precond_prec(prec)
        _, info, rc = ctx.solve(f, 1e-8)
        assert rc == 0 and info["n_cgnr_fallbacks"] == 0
        launches = info["kernels"][name]["launches"]
        if prec == "f64":
            assert launches >= 2 * info["n_cgnr_iters"], launches
        else:
            assert launches == info["n_vcycles"], (prec, launches)
    ctx.close()


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_tagged_words_give_up_cleanly(cuda, prec):
    """A wait limited to two polls on 128 coarse sites, where the words are
    tagged: the launch gives up (every wait is bounded, so all workgroups leave),
    the chunks solve again from the right-hand side, and later launches, whose
    words start cleared, are right again."""
    import paper_1005_3043_amd as mgwd
    L, block, nv = (8, 8, 8, 8), (2, 2, 2, 4), 5
    U, starts = W.gauge_field(L, 0.3, 9), W.setup_starts(L, nv, 9)
    ctx = mgwd.MG(torch.from_numpy(U).cuda(), 0.1, [block], [nv], [torch.from_numpy(starts).cuda()], setup_rounds=1,
                  precond_prec=prec)
    ctx.set_coarse_variant(0)
    f = torch.from_numpy(W.gaussian_spinor(L, 1)).cuda()
    out = []
    for on, polls in ((True, 2), (False, None), (True, None)):
        ctx.set_cgnr_persistent(on, polls=polls)
        x, info, rc = ctx.solve(f, 1e-10)
        out.append((x.clone(), info["iters"], info["n_cgnr_iters"], info["n_cgnr_fallbacks"], rc))
    ctx.close()
    print(f"{prec}: fallbacks {[o[3] for o in out]}")
    assert out[0][3] >= 1 and out[1][3] == out[2][3] == 0
    for o in out:
        assert o[4] == 0 and o[1:3] == out[1][1:3] and torch.equal(o[0], out[1][0])
