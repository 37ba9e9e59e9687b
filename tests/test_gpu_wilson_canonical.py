"""wilson_apply on the canonical arrays: every form of its kernel (the
latency form for few tiles; one, two, three and four right-hand sides per
workgroup in the streaming form) at ragged tiles and lattice edges, in every
precision, and an output that shares memory with the input."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import cref, wilson as wi

from test_gpu_wilson import _h16_round

pytestmark = pytest.mark.gpu

# 512 tiles x right-hand sides is the last call of the latency form
CASES = [((1, 1, 1, 1), 2), ((3, 1, 7, 3), 1), ((2, 4, 2, 4), 3),  # below, at and above one 64-site tile
         ((8, 8, 8, 32), 2), ((8, 8, 8, 32), 3),                   # both sides of the forms' border
         ((9, 7, 5, 113), 1),                                      # streaming, one RHS, ragged last tile and blocks
         ((9, 7, 5, 29), 5), ((9, 7, 5, 29), 6), ((5, 11, 9, 21), 7), ((16, 6, 10, 12), 4), ((16, 6, 10, 12), 10)]


@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
@pytest.mark.parametrize("L,nrhs", CASES)
def test_forms_against_oracle(cuda, L, nrhs, prec):
    import paper_1005_3043_amd as mgwd
    U, psi = W.gauge_field(L, 0.3, 3), W.gaussian_spinor(L, 4, batch=(nrhs,))
    got = mgwd.wilson_apply(torch.from_numpy(U).cuda(), torch.from_numpy(psi).cuda(), -0.25, prec=prec).cpu().numpy()
    # the class's rounding of the inputs is part of its definition; what is
    # left is the arithmetic's: about ten roundings per entry of 8 hops and
    # the diagonal in FP64 / FP32, one binary16 unit of the site's scale
    if prec == "f16":
        U = U.real.astype(np.float16).astype(np.float64) + 1j * U.imag.astype(np.float16).astype(np.float64)
        psi, _ = _h16_round(psi)
    tol = {"f64": 1e-14, "f32": 1e-6, "f16": 2.0 ** -11 + 2e-6}[prec]
    for k in range(nrhs):
        ref = wi.apply_D(U, psi[k], -0.25)
        assert np.linalg.norm(got[k] - ref) <= tol * np.linalg.norm(ref), k
        if prec == "f16":
            ref_r, m = _h16_round(ref)
            assert np.max(np.abs(got[k] - ref_r) / np.maximum(m, 1e-300)[..., None, None]) <= 2.0 ** -10 * 1.01


def test_link_rounding_to_binary16_is_single(cuda):
    """Links whose FP32 rounding falls on a binary16 midpoint, and subnormal
    ones, round as numpy's double -> binary16 does (nearest even, once)."""
    import paper_1005_3043_amd as mgwd
    L = (2, 2, 2, 2)
    mid = 0.5 + 2.0 ** -12  # halfway between two binary16 neighbours
    vals = [mid, mid + 2.0 ** -40, mid - 2.0 ** -40, -mid - 2.0 ** -40, 3e-6, 2.0 ** -25 * 1.5, -1e-5, 0.0, 1.0 / 3]
    U = np.zeros((4, 2, 2, 2, 2, 3, 3), dtype=np.complex128)
    U[0] = np.array(vals).reshape(3, 3)
    psi = np.zeros((2, 2, 2, 2, 4, 3), dtype=np.complex128)
    psi[..., 0, 0] = 1.0  # picks column 0 forwards; backwards row 0
    got = mgwd.wilson_apply(torch.from_numpy(U).cuda(), torch.from_numpy(psi).cuda(), 0.0, prec="f16").cpu().numpy()
    ref, _ = _h16_round(wi.apply_D(U.real.astype(np.float16).astype(np.complex128), psi, 0.0))
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("nrhs", [2, 3])
def test_output_sharing_memory_with_the_input(cuda, nrhs):
    import paper_1005_3043_amd as mgwd
    L = (6, 4, 2, 10)
    U, psi = W.gauge_field(L, 0.3, 5), W.gaussian_spinor(L, 6, batch=(nrhs,))
    dU = torch.from_numpy(U).cuda()
    buf = torch.zeros((nrhs + 1,) + psi.shape[1:], dtype=torch.complex128, device="cuda")
    for apply in (mgwd.wilson_apply, lambda u, p, m, out: mgwd.wilson_apply_noalloc(u, p, m, out)):
        buf[:nrhs] = torch.from_numpy(psi).cuda()
        out = apply(dU, buf[:nrhs], -0.2, out=buf[1:])
        ref = np.stack([cref.apply_D(U, p, -0.2) for p in psi])
        assert np.linalg.norm(out.cpu().numpy() - ref) < 1e-12 * np.linalg.norm(ref)
