"""Meshes at which a rule hands a launch back to the kernel with a thread per
node, each against a reference that does not depend on the choice."""

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dgm():
    from paper_2006_15698_amd import dg
    return dg


@pytest.mark.parametrize("p,n", [(2, (9, 46, 46)), (2, (6, 50, 50)), (3, (16, 23, 23)), (3, (15, 24, 25)),
                                 (7, (5, 16, 16))])
def test_stage_node_kernels_bitwise(dgm, p, n):
    """The rate and two steps of the default exchange against the trace
    exchange, bit for bit."""
    import torch
    print(f"[node stage p={p} n={n}]", flush=True)
    Q0 = torch.from_numpy(W.random_smooth(n, p, seed=20 + p, noise=0.02)).cuda()
    outs = []
    for exchange in (dgm.DG_EXCHANGE_TRACES, dgm.DG_EXCHANGE_NEIGHBOUR):
        s = dgm.Solver(n, p)
        s.set_option(dgm.DG_OPT_EXCHANGE, exchange)
        dt = 0.2 * s.dt_cfl(Q0, 1.0)
        Q, res = Q0.clone(), torch.ones_like(Q0)
        R = s.rhs(Q)
        s.step(Q, res, dt, nsteps=2)
        torch.cuda.synchronize()
        outs.append((R, Q, res))
    assert bool(torch.isfinite(outs[0][1]).all())
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("p,n", [(1, (1, 49, 49)), (2, (1, 23, 23)), (3, (2, 20, 20)), (4, (3, 15, 17)),
                                 (4, (5, 13, 21))])
def test_split_node_kernels_vs_oracle(dgm, p, n):
    """The split form on short rows (the last mesh: lines, with a short last
    block): seeded elements against the oracle on the
    3x3x3 periodic patch around each, summand-scaled 1e-12; and one step
    against the rates of its stages."""
    import numpy as np
    import torch
    from oracle import lserk
    from oracle.splitform import SplitFormDG
    from tests.parity import TOL, patch_rhs, split_summand_scale
    L = (1.0, 0.8, 1.3)
    print(f"[node split p={p} n={n}]", flush=True)
    Q = W.random_smooth(n, p, seed=30 + p, L=L, noise=0.02)
    s = dgm.Solver(n, p, L=L, volume_form=dgm.DG_VOLUME_KEP)
    Qd = torch.from_numpy(Q).cuda()
    R = s.rhs(Qd).cpu().numpy()
    nx, ny, nz = n
    rng = np.random.default_rng(p)
    elems = {(0, 0, 0), (nx - 1, ny - 1, nz - 1), (nx - 1, 0, 1)}
    elems |= {tuple(int(rng.integers(0, m)) for m in n) for _ in range(4)}
    ref = patch_rhs(n, p, L, Q, sorted(elems), make=SplitFormDG)
    small = SplitFormDG((3, 3, 3), p, L=tuple(3 * np.array(L) / np.array(n)))
    for (ex, ey, ez), Ro in ref.items():
        patch = np.ascontiguousarray(Q[:, [(ez + o) % nz for o in (-1, 0, 1)]][:, :, [(ey + o) % ny for o in (-1, 0, 1)]]
                                     [:, :, :, [(ex + o) % nx for o in (-1, 0, 1)]])
        scale = split_summand_scale(small, patch) + np.abs(Ro).reshape(5, -1).max(axis=1)
        err = np.abs(R[:, ez, ey, ex] - Ro).reshape(5, -1).max(axis=1) / scale
        assert np.all(err <= TOL), ((ex, ey, ez), err)
    Qs, res, Qr, rr = Qd.clone(), torch.zeros_like(Qd), Qd.clone(), torch.zeros_like(Qd)
    s.step(Qs, res, 1e-4)
    for a, b in zip(lserk.A, lserk.B):
        rr = a * rr + 1e-4 * s.rhs(Qr)
        Qr = Qr + b * rr
    torch.cuda.synchronize()
    assert float((Qs - Qr).abs().max()) <= 1e-13 * float(Qr.abs().max())


@pytest.mark.parametrize("p,n", [(1, (1, 30, 30)), (2, (2, 20, 20)), (3, (17, 12, 13)), (4, (19, 9, 8)),
                                 (5, (8, 27, 27)), (7, (5, 24, 24))])
def test_viscous_kernels_vs_oracle(dgm, p, n):
    """The viscous form on short rows (nodes) and, with short last blocks,
    just above the lines' smallest launches: elements at the row ends against
    the oracle on the 5x5x5 periodic patch around each, summand-scaled 1e-12;
    and bitwise the same with the inviscid rate from a launch of its own."""
    import numpy as np
    import torch
    from oracle.viscous import NavierStokesDG
    from tests.parity import TOL, patch_rhs_viscous, summand_scale, visc_summand_scale
    L, mu, pr = (1.0, 0.8, 1.3), 0.01, 0.71
    print(f"[viscous routes p={p} n={n}]", flush=True)
    Q = W.random_smooth(n, p, seed=10 + p, L=L, noise=0.01)
    Qd = torch.from_numpy(Q).cuda()
    outs = []
    for fused in (1, 0):
        s = dgm.Solver(n, p, L=L, mu=mu, prandtl=pr)
        s.set_option(dgm.DG_OPT_VISC_FUSED, fused)
        Qs, res = Qd.clone(), torch.ones_like(Qd)
        R = s.rhs(Qd)
        s.step(Qs, res, 1e-6, nsteps=2)
        torch.cuda.synchronize()
        outs.append((R, Qs, res))
    for a, b in zip(*outs):
        assert torch.equal(a, b)
    R = outs[0][0].cpu().numpy()
    nx, ny, nz = n
    elems = [(0, 0, 0), (nx - 1, ny - 1, nz - 1), (nx // 2, 0, nz - 2)]
    ref = patch_rhs_viscous(n, p, L, Q, elems, mu, pr)
    small = NavierStokesDG((5, 5, 5), p, L=tuple(5 * np.array(L) / np.array(n)), mu=mu, prandtl=pr)
    for (ex, ey, ez), Ro in ref.items():
        xs, ys, zs = ([(e + o) % m for o in range(-2, 3)] for e, m in zip((ex, ey, ez), n))
        patch = np.ascontiguousarray(Q[:, zs][:, :, ys][:, :, :, xs])
        scale = summand_scale(small, patch) + visc_summand_scale(small, patch) + np.abs(Ro).reshape(5, -1).max(axis=1)
        err = np.abs(R[:, ez, ey, ex] - Ro).reshape(5, -1).max(axis=1) / scale
        assert np.all(err <= TOL), ((ex, ey, ez), err)


@pytest.mark.parametrize("p", [1, 3, 4, 5])
def test_batch_lines_and_nodes_bitwise(dgm, p):
    """A batch of one small mesh (a thread per node) and of forty copies of it
    (a thread per line): the rate and two steps of every copy are the one's
    bit for bit, as they are with every tile built for the degree."""
    import torch
    n = (7, 5, 3)
    print(f"[batch routes p={p}]", flush=True)
    q = torch.from_numpy(W.random_smooth(n, p, seed=70 + p, noise=0.02)).cuda()
    outs = []
    for count in (1, 40):
        for tile in dgm.dg_batch_tile_options(p):
            b = dgm.Batch([n] * count, [p] * count, [(1.0, 1.0, 1.0)] * count, tiles={p: tile})
            Q = b.empty()
            for i in range(count):
                b.view(Q, i).copy_(q)
            b.set_dt([1e-3] * count)
            R, res = b.rhs(Q), torch.zeros_like(Q)
            b.step(Q, res, nsteps=2)
            torch.cuda.synchronize()
            for i in (0, count // 2, count - 1):
                outs.append([b.view(x, i).clone() for x in (R, Q, res)])
    for o in outs[1:]:
        for a, c in zip(outs[0], o):
            assert torch.equal(a, c)


def test_variable_degree_node_round_bitwise(dgm):
    """1800 waves of p = 3 (a thread per node) against the same mesh tiled to
    3600 (a thread per line), bit for bit."""
    import numpy as np
    import torch
    n, p = (20, 20, 18), 3
    print("[varp node round]", flush=True)
    q = torch.from_numpy(np.ascontiguousarray(
        W.random_smooth(n, p, seed=3, L=(20.0, 20.0, 18.0), noise=0.02).reshape(5, n[2], n[1] * n[0] * (p + 1) ** 3))).cuda()
    outs = []
    for t in (1, 2):
        m = (n[0], n[1], t * n[2])
        v = dgm.VariableDegree(m, np.full(m[0] * m[1] * m[2], p), L=tuple(float(x) for x in m))
        Q = q.repeat(1, t, 1).reshape(-1).contiguous()
        res = torch.zeros_like(Q)
        R = v.rhs(Q).clone()
        v.step(Q, res, 1e-3, nsteps=2)
        torch.cuda.synchronize()
        outs.append([x.view(5, t, -1) for x in (R, Q, res)])
    assert bool(torch.isfinite(outs[0][1]).all())
    for a, b in zip(*outs):
        assert torch.equal(a[:, 0], b[:, 0]) and torch.equal(a[:, 0], b[:, 1])


def test_adjoint_of_small_and_larger_meshes_p7(dgm):
    """p = 7 at 128 elements (a thread per node) and at twice and 1.5 times as
    many (lines): products and reverse stages of the default exchange against
    the trace exchange, bit for bit."""
    import torch
    p = 7
    for n in ((4, 4, 8), (3, 8, 8), (4, 8, 8)):
        print(f"[adjoint routes n={n}]", flush=True)
        Q = torch.from_numpy(W.random_smooth(n, p, seed=5, noise=0.02)).cuda()
        gen = torch.Generator().manual_seed(7)
        g0, r0 = (torch.randn(Q.shape, dtype=torch.float64, generator=gen).cuda() for _ in range(2))
        outs = []
        for exchange in (dgm.DG_EXCHANGE_NEIGHBOUR, dgm.DG_EXCHANGE_TRACES):
            s = dgm.Solver(n, p)
            s.set_option(dgm.DG_OPT_EXCHANGE, exchange)
            gQ, gres = g0.clone(), r0.clone()
            dgm.dg_rk_stage_vjp(s.ctx, 2, Q, gQ, gres, 1e-3)
            outs.append((s.rhs_vjp(Q, g0), gQ, gres))
            torch.cuda.synchronize()
        for a, b in zip(*outs):
            assert torch.equal(a, b)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_batch_deal_of_items_bitwise(dgm, prec):
    """Windows of items, the plain spread and contiguous parts give the same
    bits (5000 items of p = 3, 1024 to a window)."""
    import torch
    n, p, count = (9, 8, 7), 3, 30
    print(f"[batch deal {prec}]", flush=True)
    b = dgm.Batch([n] * count, [p] * count, [(1.0, 1.0, 1.0)] * count,
                  precision=dgm.DG_FP64 if prec == "fp64" else dgm.DG_FP32_MFMA)
    assert b.options()["xcd_remap"] == 0 and b.options()["xcd_window"] == 1
    q = torch.from_numpy(W.random_smooth(n, p, seed=9, noise=0.02)).cuda()
    Q0 = b.empty()
    for i in range(count):
        b.view(Q0, i).copy_(q * (1.0 + 0.001 * i))
    b.set_dt([1e-3] * count)
    outs = []
    for xcd, window in ((0, 1), (0, 0), (1, 0), (1, 1)):
        b.set_option(dgm.DG_OPT_XCD_REMAP, xcd)
        b.set_option(dgm.DG_OPT_XCD_WINDOW, window)
        assert b.options()["xcd_remap"] == xcd and b.options()["xcd_window"] == window
        Q, res = Q0.clone(), torch.zeros_like(Q0)
        b.step(Q, res, nsteps=2)
        torch.cuda.synchronize()
        outs.append((Q, res))
    assert bool(torch.isfinite(outs[0][0]).all())
    for o in outs[1:]:
        assert torch.equal(o[0], outs[0][0]) and torch.equal(o[1], outs[0][1])


@pytest.mark.parametrize("form", ["euler", "fp32", "kep"])
def test_stage_to_is_one_launch(dgm, form):
    """The out-of-place stage leaves the workspace, the second state buffer
    included, as it was."""
    import torch
    n, p = (5, 4, 6), 3
    print(f"[stage to {form}]", flush=True)
    s = dgm.Solver(n, p, precision=dgm.DG_FP32_MFMA if form == "fp32" else dgm.DG_FP64,
                   volume_form=dgm.DG_VOLUME_KEP if form == "kep" else dgm.DG_VOLUME_STANDARD)
    Q = torch.from_numpy(W.random_smooth(n, p, seed=6, noise=0.02)).cuda()
    Q0, res, nxt = Q.clone(), torch.zeros_like(Q), torch.empty_like(Q)
    s.rhs(Q)   # (the call below uses the context's stream)
    s.workspace.fill_(0xa5)
    dgm.dg_rk_stage_to(s.ctx, 0, Q, nxt, res, 1e-4)
    torch.cuda.synchronize()
    assert torch.equal(Q, Q0) and not torch.equal(nxt, Q0)
    assert bool((s.workspace == 0xa5).all())
