"""Steps on meshes whose arrays exceed the last-level cache: slabs shared by
the XCDs and new states stored as not reused, against kernels or meshes that
know neither, bit for bit."""

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dgm():
    from paper_2006_15698_amd import dg
    return dg


@pytest.mark.parametrize("p,n", [(2, (56, 55, 50)), (3, (41, 39, 40)), (3, (36, 35, 36)), (4, (4, 8, 1100)),
                                 (6, (24, 24, 25)), (7, (17, 17, 17))])
def test_steps_beyond_the_cache_equal_the_trace_exchange(dgm, p, n):
    """Neighbour reads against the trace-buffer kernel (a node per thread,
    index order, plain stores)."""
    import torch
    print(f"[stream p={p} n={n}]", flush=True)
    Q0 = torch.from_numpy(W.random_smooth(n, p, seed=40 + p, noise=0.02)).cuda()
    outs = []
    for exchange in (dgm.DG_EXCHANGE_TRACES, dgm.DG_EXCHANGE_NEIGHBOUR):
        s = dgm.Solver(n, p)
        s.set_option(dgm.DG_OPT_EXCHANGE, exchange)
        dt = 0.2 * s.dt_cfl(Q0, 1.0)
        Q, res = Q0.clone(), torch.zeros_like(Q0)
        s.step(Q, res, dt, nsteps=3)
        torch.cuda.synchronize()
        outs.append((Q, res))
    assert bool(torch.isfinite(outs[0][0]).all())
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("p,m", [(2, 28), (3, 20), (6, 12)])
def test_split_steps_beyond_the_cache_equal_a_periodic_tile(dgm, p, m):
    """The split form on eight periodic copies of a mesh that fits the cache
    against that mesh."""
    import torch
    print(f"[stream split p={p} m={m}]", flush=True)
    q = torch.from_numpy(W.random_smooth((m, m, m), p, seed=50 + p, noise=0.02)).cuda()
    outs = []
    for t in (1, 2):
        s = dgm.Solver((t * m,) * 3, p, L=(float(t),) * 3, volume_form=dgm.DG_VOLUME_KEP)
        Q = q.repeat(1, t, t, t, 1, 1, 1).contiguous()
        res = torch.zeros_like(Q)
        s.step(Q, res, 1e-4, nsteps=3)
        torch.cuda.synchronize()
        outs.append((Q, res))
    assert bool(torch.isfinite(outs[0][0]).all())
    for a, b in zip(*outs):
        for z in (0, m):
            for y in (0, m):
                for x in (0, m):
                    assert torch.equal(a, b[:, z:z + m, y:y + m, x:x + m])
