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
