"""GPU parity of the parallel-transport network (learned null-vector
proposal) against the oracle: forward pass, subspace-fit loss, weight
gradients of both layers, and the Adam step; plus argument errors."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import ptc as op
from oracle import transfer as tr

pytestmark = pytest.mark.gpu

CASES = {
    # name: (L, block, n_hidden, n_out, n_targets, eps, seed)
    "8x4x4x8 b4^4 8->6": ((8, 4, 4, 8), (4, 4, 4, 4), 8, 6, 5, 0.3, 0),
    "4^4 b2^4 3->4": ((4, 4, 4, 4), (2, 2, 2, 2), 3, 4, 3, 0.4, 1),
}


def _rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - np.asarray(b)) / max(np.linalg.norm(np.asarray(b)), 1e-300))


@pytest.fixture(scope="module", params=list(CASES))
def case(request, cuda):
    import paper_1005_3043_amd as mgwd
    L, blk, nh, no, nt, eps, seed = CASES[request.param]
    U = W.gauge_field(L, eps, seed)
    W1, W2 = W.ptc_init_weights(nh, no, seed)
    eta = W.noise_spinor(L, seed)
    V = W.gaussian_spinor(L, seed + 7, batch=(nt,))
    net = mgwd.PTC(L, blk, nh, no)
    net.set_links(torch.from_numpy(U).cuda())
    net.set_targets(torch.from_numpy(V).cuda())
    dev = dict(W1=torch.from_numpy(W1.astype(np.complex64)).cuda(),
               W2=torch.from_numpy(W2.astype(np.complex64)).cuda(),
               eta=torch.from_numpy(eta).cuda())
    return request.param, net, U, W1, W2, eta, V, tr.BlockGeometry(L, blk), dev


def test_forward(case):
    name, net, U, W1, W2, eta, V, geom, d = case
    Y = net.forward(d["W1"], d["W2"], d["eta"]).cpu().numpy()
    # the oracle runs on the same FP32-rounded weights
    _, Yref = op.forward(W1.astype(np.complex64).astype(np.complex128),
                         W2.astype(np.complex64).astype(np.complex128), U, eta)
    e = _rel(Y, Yref)
    print(f"{name}: forward rel err {e:.2e}")
    assert e < 2e-6


def test_loss_and_gradients(case):
    name, net, U, W1, W2, eta, V, geom, d = case
    loss, g1, g2 = net.loss_grad(d["W1"], d["W2"], d["eta"])
    W1r = W1.astype(np.complex64).astype(np.complex128)
    W2r = W2.astype(np.complex64).astype(np.complex128)
    lref, g1r, g2r = op.loss_and_grad(W1r, W2r, U, eta, V, geom)
    el, e1, e2 = abs(loss - lref) / lref, _rel(g1.cpu().numpy(), g1r), _rel(g2.cpu().numpy(), g2r)
    print(f"{name}: loss {loss:.6f} (oracle {lref:.6f}, rel {el:.1e}), gW1 rel err {e1:.2e}, gW2 rel err {e2:.2e}")
    assert el < 1e-5 and e1 < 1e-4 and e2 < 1e-4


def test_adam_matches_oracle(cuda):
    import paper_1005_3043_amd as mgwd
    rng = np.random.default_rng(3)
    p = (rng.standard_normal(50) + 1j * rng.standard_normal(50)).astype(np.complex64)
    Wd = torch.from_numpy(p.copy()).cuda()
    m = torch.zeros_like(Wd)
    v = torch.zeros(100, dtype=torch.float32, device="cuda")
    opt = op.Adam(lr=1e-2)
    pr = p.astype(np.complex128)
    for step in range(1, 4):
        g = (rng.standard_normal(50) + 1j * rng.standard_normal(50)).astype(np.complex64)
        mgwd.ptc_adam(Wd, torch.from_numpy(g).cuda(), m, v, step, lr=1e-2)
        (pr,) = opt.step([pr], [g.astype(np.complex128)])
    assert _rel(Wd.cpu().numpy(), pr) < 1e-6


def test_errors(cuda):
    import paper_1005_3043_amd as mgwd
    with pytest.raises(mgwd.MGError) as e:
        mgwd.PTC((8, 8, 8, 8), (3, 4, 4, 4), 8, 6)
    assert e.value.rc == -2
    with pytest.raises(mgwd.MGError) as e:
        mgwd.PTC((8, 8, 8, 8), (4, 4, 4, 4), 8, 40)
    assert e.value.rc == -1


@pytest.mark.parametrize("L,block,nh,no,nt", [
    ((4, 4, 4, 4), (2, 2, 2, 2), 1, 1, 9),      # one channel, more targets than a tile's fill
    ((6, 2, 4, 6), (3, 1, 2, 3), 2, 17, 17),    # 18-site blocks (not whole groups of four), one past a row tile
    ((2, 2, 3, 4), (2, 1, 3, 2), 5, 7, 40),     # volume below one 64-site tile, three target tiles
    ((8, 4, 4, 4), (4, 4, 4, 4), 8, 32, 32),    # the largest output count
])
def test_matrix_core_edges(cuda, L, block, nh, no, nt):
    """Forward pass, loss and both weight gradients where rows, columns, hops
    and sites are not whole matrix-core tiles (bounds as above)."""
    import paper_1005_3043_amd as mgwd
    U, eta, V = W.gauge_field(L, 0.3, 11), W.noise_spinor(L, 11), W.gaussian_spinor(L, 12, batch=(nt,))
    W1, W2 = (w.astype(np.complex64) for w in W.ptc_init_weights(nh, no, 11))
    net = mgwd.PTC(L, block, nh, no)
    net.set_links(torch.from_numpy(U).cuda())
    net.set_targets(torch.from_numpy(V).cuda())
    d1, d2, de = torch.from_numpy(W1).cuda(), torch.from_numpy(W2).cuda(), torch.from_numpy(eta).cuda()
    W1r, W2r = W1.astype(np.complex128), W2.astype(np.complex128)
    _, Yref = op.forward(W1r, W2r, U, eta)
    assert _rel(net.forward(d1, d2, de).cpu().numpy(), Yref) < 2e-6
    loss, g1, g2 = net.loss_grad(d1, d2, de)
    lref, g1r, g2r = op.loss_and_grad(W1r, W2r, U, eta, V, tr.BlockGeometry(L, block))
    assert abs(loss - lref) / lref < 1e-5
    # the fit's conditioning multiplies the FP32 rounding of Y (2e-7) once more
    cond = max(np.linalg.cond(b) for b in
               tr.BlockGeometry(L, block).blockify(tr.fine_to_generic(Yref)).transpose(1, 2, 3, 0).reshape(-1, int(np.prod(block)) * 6, no))
    tol = max(1e-4, 1e-6 * cond)
    assert _rel(g1.cpu().numpy(), g1r) < tol and _rel(g2.cpu().numpy(), g2r) < tol


def test_weight_gradient_rounding(cuda):
    """Layer 2's weight gradient on 16^3 x 64 with 64 hidden channels, where
    the site sum is dealt to the fewest wavefronts.  Unit links, hidden channel b
    a pure hop of FP32 noise and one output equal to it keep the transported
    fields exact, so that what is left is the rounding of the fit's residual and
    gradient (four roundings per site, 0.7e-7) and of the sum: FP32 chains of 32
    products, then FP64, 1.4e-7 (a rounding is 0.34e-7 rms, a chain of d products
    0.34e-7 sqrt(d / 2)); 1.6e-7 together, the bound is twice that.  One FP32 sum
    over a wavefront's 558 blocks of 16 sites would make 6e-7."""
    import paper_1005_3043_amd as mgwd
    L, nh = (16, 16, 16, 64), 64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)

    def noise(*lead):
        return torch.randn(*lead, L[3], L[2], L[1], L[0], 4, 3, dtype=torch.complex64, device="cuda",
                           generator=gen).to(torch.complex128)

    def hop(f, k):  # T_k with unit links, periodic
        return f if k == 0 else torch.roll(f, 1 if (k - 1) % 2 else -1, (-3, -4, -5, -6)[(k - 1) // 2])

    one = torch.eye(4, dtype=torch.complex64, device="cuda")
    W1 = torch.zeros(nh, 1, 9, 4, 4, dtype=torch.complex64, device="cuda")
    for b in range(nh):
        W1[b, 0, b % 9] = one
    W2 = torch.zeros(1, nh, 9, 4, 4, dtype=torch.complex64, device="cuda")
    W2[0, 0, 0] = one
    eta, V = noise(), noise(1)
    U = torch.zeros(4, L[3], L[2], L[1], L[0], 3, 3, dtype=torch.complex128, device="cuda")
    U[...] = torch.eye(3, device="cuda")
    net = mgwd.PTC(L, (4, 4, 4, 4), nh, 1, t_antiperiodic=False)
    net.set_links(U)
    net.set_targets(V)
    _, _, g2 = net.loss_grad(W1, W2, eta)

    def blocks(f):  # [aggregate, site and component of a chirality] per chirality
        f = f.reshape(L[3] // 4, 4, L[2] // 4, 4, L[1] // 4, 4, L[0] // 4, 4, 2, 6)
        return f.permute(0, 2, 4, 6, 8, 1, 3, 5, 7, 9).reshape(-1, 256 * 6)

    Y, T = blocks(eta), blocks(V[0])
    C = (Y.conj() * T).sum(1) / (Y.conj() * Y).sum(1)
    G = -2.0 / (T.abs() ** 2).sum() * (T - C[:, None] * Y) * C[:, None].conj()
    G = G.reshape(L[3] // 4, L[2] // 4, L[1] // 4, L[0] // 4, 2, 4, 4, 4, 4, 6).permute(0, 5, 1, 6, 2, 7, 3, 8, 4, 9)
    G = G.reshape(eta.shape).permute(4, 0, 1, 2, 3, 5).reshape(4, -1)
    ref = torch.stack([torch.stack([
        torch.matmul(G, hop(hop(eta, b), k).permute(4, 0, 1, 2, 3, 5).reshape(4, -1).conj().t().contiguous())
        for k in range(9)]) for b in range(9)])
    for b0 in range(0, 63, 9):
        err = float((g2[0, b0:b0 + 9].to(torch.complex128) - ref).norm() / ref.norm())
        print(f"weight gradient, channels {b0}..{b0 + 8}: {err:.2e}")
        assert err <= 3.2e-7


@pytest.mark.parametrize("nh,no,nt", [(4, 12, 4), (2, 24, 24), (13, 13, 1)])
def test_row_tile_groups(cuda, nh, no, nt):
    """Three, six and four row tiles in one group of the mixing, one to three
    column tiles of the Gram matrices (the other counts are above)."""
    test_matrix_core_edges(cuda, (4, 4, 4, 4), (2, 2, 2, 2), nh, no, nt)
