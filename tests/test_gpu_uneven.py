"""Ensembles of one large instance and many small ones: the calls that visit the
whole state give each instance what its own run holds, and are paced by the
cells and not by the number of instances."""
import numpy as np
import pytest

from paper_2411_15001_amd import binding as B
from paper_2411_15001_amd import cases

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch

    assert torch.cuda.is_available()
    B.lib()
    return torch


def timed(f, torch):
    best = 1e9
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


@pytest.mark.parametrize("large,small", [((1024, 1024), (64, 64)), ((1030, 701), (33, 40)), ((64, 3), (512, 70))])
@pytest.mark.parametrize("prec", [0, 1])
def test_uneven_instances_hold_their_own_states(large, small, prec, gpu):
    from paper_2411_15001_amd.solver import BatchSolver, Solver

    print("uneven", large, small, prec, flush=True)
    torch = gpu
    sides = [small] * 3 + [large] + [small] * 40
    u0s = [np.ascontiguousarray(cases.riemann4(max(nx, ny, 4), seed=i)[:, :ny, :nx]) for i, (nx, ny) in enumerate(sides)]
    kw = dict(limiters=9, bc_x=1, bc_y=1, precision=prec)
    b = BatchSolver(u0s, **kw)
    b.step(2)
    state = b.get_state()
    b.set_state(state)
    assert torch.equal(b.get_state(), state)
    for i in (0, 3, 4, len(sides) - 1):
        s = Solver(u0s[i], **kw)
        d0 = s.diagnostics()
        s.step(2)
        assert torch.equal(b.moments(i, check=False)[0], s.moments())
        d, ref = b.diagnostics(i), s.diagnostics()
        assert d["lam"] == ref["lam"] and d0["lam"] > 0.0
        s.close()
    b.close()


def test_a_large_instance_keeps_its_blocks(gpu):
    """Loading one instance of 4096^2 and 255 of 64^2 takes less than 2.5 times
    the load of the large one alone (6% more cells; with the same few blocks for
    every instance it took 4.9 times)."""
    from paper_2411_15001_amd.solver import BatchSolver, Solver

    torch = gpu

    def uniform(n):
        u = torch.zeros((4, n, n), dtype=torch.float64, device="cuda")
        u[0], u[3] = 1.0, 2.5
        return u

    s = Solver(uniform(4096), limiters=9)
    state = s.get_state()
    alone = timed(lambda: s.set_state(state), torch)
    s.close()
    del s, state
    b = BatchSolver([uniform(4096)] + [uniform(64)] * 255, limiters=9)
    state = b.get_state()
    together = timed(lambda: b.set_state(state), torch)
    b.close()
    print("  load %.0f / %.0f us" % (alone * 1e3, together * 1e3))
    assert together < 2.5 * alone
