"""The one-thread-per-line stage kernel against the trace-buffer kernel,
which holds a node per thread and shares only the arithmetic: both round the
same operations in the same order, so rates and steps are equal bit for bit.
Meshes large enough for the line kernel (more than 512 waves), with rows that
leave short blocks, one-element rows (an element its own x-neighbour), whole
and left-over parts of the XCD-shared slabs, and arrays that start at an odd
multiple of 8 bytes."""

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dgm():
    from paper_2006_15698_amd import dg
    return dg


def _odd(t):
    """A copy of t that starts 8 bytes past a 16-byte boundary."""
    import torch
    flat = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    v = flat[1:].view(t.shape)
    v.copy_(t)
    assert v.data_ptr() % 16 == 8
    return v


@pytest.mark.parametrize("p,n", [(1, (17, 13, 21)), (1, (32, 16, 17)), (2, (5, 9, 21)), (2, (6, 3, 2)), (3, (5, 13, 21)),
                                 (3, (4, 24, 25)), (4, (3, 13, 21)), (4, (1, 24, 24)), (4, (4, 18, 16)),
                                 (5, (3, 13, 21)), (6, (2, 13, 21)), (7, (1, 25, 21))])
def test_line_kernel_bitwise_equals_node_kernel(dgm, p, n):
    import torch
    print(f"[line kernel p={p} n={n}]", flush=True)
    Q0 = torch.from_numpy(W.random_smooth(n, p, seed=60 + p, noise=0.02)).cuda()
    outs = []
    for exchange, pencil_z, place in ((dgm.DG_EXCHANGE_TRACES, 1, lambda t: t.clone()),
                                      (dgm.DG_EXCHANGE_NEIGHBOUR, 1, lambda t: t.clone()),
                                      (dgm.DG_EXCHANGE_NEIGHBOUR, 3, _odd)):
        s = dgm.Solver(n, p)
        s.set_option(dgm.DG_OPT_EXCHANGE, exchange)
        s.set_option(dgm.DG_OPT_PENCIL_Z, pencil_z)
        dt = 0.2 * s.dt_cfl(Q0, 1.0)
        Q, res = place(Q0), place(torch.ones_like(Q0))
        R = s.rhs(Q, out=place(torch.empty_like(Q0)))
        s.step(Q, res, dt, nsteps=2)
        torch.cuda.synchronize()
        outs.append((R, Q, res))
    assert bool(torch.isfinite(outs[0][1]).all())
    for o in outs[1:]:
        for a, b in zip(outs[0], o):
            assert torch.equal(a, b)


@pytest.mark.parametrize("p,n", [(1, (33, 5, 4)), (2, (7, 5, 4)), (3, (5, 13, 21)), (4, (3, 13, 21)), (5, (3, 13, 21)),
                                 (6, (1, 25, 21)), (7, (2, 13, 21))])
def test_split_line_kernel_vs_oracle(dgm, p, n):
    """The split form's line kernel (meshes of more than 384 waves) on
    elements at the row ends and corners and seeded ones, each against the
    oracle on the 3x3x3 periodic patch around it, summand-scaled 1e-12."""
    import numpy as np
    import torch
    from oracle.splitform import SplitFormDG
    from tests.parity import TOL, patch_rhs, split_summand_scale
    L = (1.0, 0.8, 1.3)
    print(f"[split line kernel p={p} n={n}]", flush=True)
    Q = W.random_smooth(n, p, seed=70 + p, L=L, noise=0.02)
    s = dgm.Solver(n, p, L=L, volume_form=dgm.DG_VOLUME_KEP)
    R = s.rhs(torch.from_numpy(Q).cuda()).cpu().numpy()
    nx, ny, nz = n
    rng = np.random.default_rng(p)
    elems = {(0, 0, 0), (nx - 1, ny - 1, nz - 1), (nx - 1, 0, 1), (0, ny - 1, nz - 2)}
    elems |= {tuple(int(rng.integers(0, m)) for m in n) for _ in range(4)}
    ref = patch_rhs(n, p, L, Q, sorted(elems), make=SplitFormDG)
    small = SplitFormDG((3, 3, 3), p, L=tuple(3 * np.array(L) / np.array(n)))
    for (ex, ey, ez), Ro in ref.items():
        patch = np.ascontiguousarray(Q[:, [(ez + o) % nz for o in (-1, 0, 1)]][:, :, [(ey + o) % ny for o in (-1, 0, 1)]]
                                     [:, :, :, [(ex + o) % nx for o in (-1, 0, 1)]])
        scale = split_summand_scale(small, patch) + np.abs(Ro).reshape(5, -1).max(axis=1)
        err = np.abs(R[:, ez, ey, ex] - Ro).reshape(5, -1).max(axis=1) / scale
        assert np.all(err <= TOL), ((ex, ey, ez), err)


@pytest.mark.parametrize("p,n", [(1, (33, 5, 4)), (2, (7, 5, 4)), (3, (5, 13, 21)), (4, (3, 13, 21)), (5, (6, 28, 25)),
                                 (6, (2, 13, 21)), (7, (5, 21, 20))])
def test_viscous_line_kernels(dgm, p, n):
    """The viscous line kernels (meshes above their smallest size) on elements
    at the row ends and corners, each against the oracle on the 5x5x5 periodic
    patch around it, summand-scaled 1e-12; and bitwise the same with the
    inviscid rate from a launch of its own."""
    import numpy as np
    import torch
    from oracle.viscous import NavierStokesDG
    from tests.parity import TOL, patch_rhs_viscous, summand_scale, visc_summand_scale
    L, mu, pr = (1.0, 0.8, 1.3), 0.01, 0.71
    print(f"[viscous line kernels p={p} n={n}]", flush=True)
    Q = W.random_smooth(n, p, seed=80 + p, L=L, noise=0.01)
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


@pytest.mark.parametrize("p,n", [(1, (5, 3, 4)), (2, (7, 2, 3)), (3, (5, 3, 4)), (4, (3, 5, 2)), (5, (3, 2, 4)),
                                 (6, (3, 2, 4)), (6, (1, 1, 1)), (7, (2, 3, 3))])
def test_reverse_stage_bitwise(dgm, p, n):
    """The reverse stage folded into the adjoint launch (neighbour reads; the
    line kernel at p = 6, 7) against the trace-buffer sequence of separate
    launches, for every stage; and the product alone."""
    import torch
    print(f"[reverse stage p={p} n={n}]", flush=True)
    Q = torch.from_numpy(W.random_smooth(n, p, seed=90 + p, noise=0.02)).cuda()
    gen = torch.Generator().manual_seed(p)
    g0, r0 = (torch.randn(Q.shape, dtype=torch.float64, generator=gen).cuda() for _ in range(2))
    outs = []
    for exchange in (dgm.DG_EXCHANGE_NEIGHBOUR, dgm.DG_EXCHANGE_TRACES):
        s = dgm.Solver(n, p)
        s.set_option(dgm.DG_OPT_EXCHANGE, exchange)
        got = [s.rhs_vjp(Q, g0)]
        for k in range(5):
            gQ, gres = g0.clone(), r0.clone()
            dgm.dg_rk_stage_vjp(s.ctx, k, Q, gQ, gres, 1e-3)
            got += [gQ, gres]
        torch.cuda.synchronize()
        outs.append(got)
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("form", ["euler", "fp32", "kep", "viscous"])
@pytest.mark.parametrize("p,n", [(1, (5, 3, 4)), (4, (3, 13, 21))])
def test_odd_stage_counts_and_stage_to(dgm, form, p, n):
    """Calls of one, two, three and five steps (the odd ones end by way of the
    third state buffer), graph replay of each, and the out-of-place stage: all
    bitwise those of the stages one by one in place."""
    import torch
    print(f"[odd stage counts {form} p={p} n={n}]", flush=True)
    s = dgm.Solver(n, p, precision=dgm.DG_FP32_MFMA if form == "fp32" else dgm.DG_FP64,
                   mu=0.01 if form == "viscous" else 0.0,
                   volume_form=dgm.DG_VOLUME_KEP if form == "kep" else dgm.DG_VOLUME_STANDARD)
    Q0 = torch.from_numpy(W.random_smooth(n, p, seed=95, noise=0.01)).cuda()
    dt = 0.1 * s.dt_cfl(Q0, 1.0)
    for nsteps in (1, 2, 3, 5):
        Q, res, Qt, rest = Q0.clone(), torch.zeros_like(Q0), Q0.clone(), torch.zeros_like(Q0)
        for _ in range(nsteps):
            for k in range(5):
                s.rk_stage(k, Q, res, dt)
                nxt = torch.full_like(Q0, float("nan"))
                dgm.dg_rk_stage_to(s.ctx, k, Qt, nxt, rest, dt)
                Qt = nxt
        ends = [(Qt, rest)]
        for graph in (False, True, True):
            Qg, resg = Q0.clone(), torch.zeros_like(Q0)
            s.step(Qg, resg, dt, nsteps, graph=graph)
            ends.append((Qg, resg))
        torch.cuda.synchronize()
        for a, b in ends:
            assert torch.equal(a, Q) and torch.equal(b, res), nsteps
    with pytest.raises(dgm.DGError):
        dgm.dg_rk_stage_to(s.ctx, 0, Q0, Q0, torch.zeros_like(Q0), dt)


@pytest.mark.parametrize("p,other,refined", [(3, 2, True), (4, 5, True), (4, 4, True), (5, 0, False), (5, 6, True),
                                             (6, 7, True)])
def test_variable_degree_groups_bitwise(dgm, p, other, refined):
    """A mesh of two degrees, some cells refined, against the same mesh tiled
    periodically: the elements of the small one run with a thread per node,
    the tiled one's groups of degree p are large enough for a thread per line.
    The rate and two steps (with the face traces handed on between stages)
    agree bit for bit in every copy."""
    import torch
    print(f"[varp lines p={p} other={other} refined={refined}]", flush=True)
    tile, n = (4, 4, 2), (5, 4, 5)
    rng = np.random.default_rng(820 + p)
    ref = (rng.random((n[2], n[1], n[0])) < 0.15).astype(int) * int(refined)
    count = np.where(ref == 1, 8, 1)
    deg = [np.where(rng.random(c) < 0.85, p, other) for c in count.reshape(-1)]
    q = [np.stack([1.0 + 0.1 * rng.random((d + 1) ** 3), *(0.2 * rng.random((3, (d + 1) ** 3))),
                   2.5 + 0.1 * rng.random((d + 1) ** 3)]) for cell in deg for d in cell]
    first = np.concatenate([[0], np.cumsum(count.reshape(-1))])

    def mesh(t):
        m = tuple(a * b for a, b in zip(n, t))
        cells = [(cz % n[2] * n[1] + cy % n[1]) * n[0] + cx % n[0]
                 for cz in range(m[2]) for cy in range(m[1]) for cx in range(m[0])]
        elems = np.concatenate([np.arange(first[c], first[c + 1]) for c in cells])
        r = np.tile(ref, t[::-1])
        v = dgm.VariableDegree(m, np.concatenate([deg[c] for c in cells]), L=tuple(float(x) for x in t),
                               refine=r if refined else None)
        Q = torch.from_numpy(np.concatenate([q[e] for e in elems], axis=1).reshape(-1)).cuda()
        res = torch.zeros_like(Q)
        out = [v.rhs(Q).clone()]
        v.step(Q, res, 2e-4, nsteps=2)
        torch.cuda.synchronize()
        return elems, [x.cpu().numpy().reshape(5, -1) for x in out + [Q, res]], v.offsets

    _, small, off = mesh((1, 1, 1))
    elems, tiled, _ = mesh(tile)
    at = np.concatenate([np.arange(off[e], off[e + 1]) for e in elems])
    for a, b in zip(small, tiled):
        assert np.isfinite(a).all() and np.array_equal(b, a[:, at])
