"""The one-thread-per-line stage kernel against the trace-buffer kernel,
which holds a node per thread and shares only the arithmetic: both round the
same operations in the same order, so rates and steps are equal bit for bit.
Meshes large enough for the line kernel (more than 512 waves), with rows that
leave short blocks, one-element rows (an element its own x-neighbour), whole
and left-over parts of the XCD-shared slabs, and arrays that start at an odd
multiple of 8 bytes."""

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
