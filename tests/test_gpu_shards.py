"""The step kernels spread their wavespeed maxima and event counts over several
records per instance, which are folded into the instance's own before the host
reads it: whatever mix of eager steps, caller-recorded graphs, loads and reads
comes between, the counters, lambda and t are those of one plain run."""
import numpy as np
import pytest

from paper_2411_15001_amd import binding as B
from paper_2411_15001_amd import cases

pytestmark = pytest.mark.gpu

KEYS = ("lam", "t", "n_limited", "n_guard", "n_lmp", "n_bad", "min_rho", "min_rhoe")
KW = dict(limiters=1 | 2 | 8, a_beta=1.1, bc_x=1, bc_y=1)


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch

    assert torch.cuda.is_available()
    B.lib()
    return torch


def plain(u0, kw, steps):
    from paper_2411_15001_amd.solver import Solver

    s = Solver(u0, **kw)
    s.step(steps)
    d, x = s.diagnostics(), s.get_state()
    s.close()
    return d, x


def same(d, ref):
    for k in KEYS:
        assert d[k] == ref[k], (k, d[k], ref[k])


@pytest.mark.parametrize("n", [96, 128, 330])  # planar and blocked layouts, one and many strips per record
def test_replays_of_a_callers_graph_are_counted(n, gpu):
    from paper_2411_15001_amd.solver import Solver

    print("replay", n, flush=True)
    torch = gpu
    u0 = cases.riemann4(n, seed=2)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        s = Solver(u0, **KW)
        s.step(6)
        same(s.diagnostics(), plain(u0, KW, 6)[0])  # folds the eager steps
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            s.step(6)
        for k in range(3):
            g.replay()
            side.synchronize()
            d = s.diagnostics()
            same(d, plain(u0, KW, 6 * (k + 2))[0])
        s.step(5)
        same(s.diagnostics(), plain(u0, KW, 29)[0])
        del g
        s.close()


def test_load_recorded_into_a_graph_keeps_the_counts(gpu):
    from paper_2411_15001_amd.solver import Solver

    torch = gpu
    u0 = cases.riemann4(192, seed=5)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        s = Solver(u0, **KW)
        start = s.get_state()
        s.step(6)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            s.set_state(start)
        d, ref = s.diagnostics(), plain(u0, KW, 6)[0]
        same(d, ref)
        g.replay()
        s.step(6)
        d = s.diagnostics()
        assert d["n_limited"] == 2 * ref["n_limited"] and d["lam"] == ref["lam"]
        del g
        s.close()


def test_counts_of_an_ensemble_and_their_reset(gpu):
    from paper_2411_15001_amd.solver import BatchSolver

    sides = [64, 320, 128, 256]
    u0s = [cases.riemann4(n, seed=10 + i) for i, n in enumerate(sides)]
    b = BatchSolver(u0s, **KW)
    b.step(7)
    for i, u0 in enumerate(u0s):
        ref, x = plain(u0, KW, 7)
        same(b.diagnostics(i), ref)
        assert np.array_equal(b.moments(i, check=False)[0].cpu().numpy(), x[:4].cpu().numpy())
        if i == 0:  # the first read clears every counter
            b.step(0)
            assert all(b.diagnostics(k)["n_limited"] == 0 for k in range(len(sides)))
            break
    b.step(4)
    for i, u0 in enumerate(u0s):
        r7, r11 = plain(u0, KW, 7)[0], plain(u0, KW, 11)[0]
        assert b.diagnostics(i)["n_limited"] == r11["n_limited"] - r7["n_limited"]
    b.close()


def test_what_counts_after_a_read_cleared_the_counters_is_reported(gpu):
    """lbm_moments skips its read where nothing can have counted since it
    cleared the counters: steps, loads and the adjoint's reduction end that."""
    from paper_2411_15001_amd.solver import Solver

    torch = gpu
    n = 96
    u0 = cases.riemann4(n, seed=6)
    s = Solver(u0, **KW)
    start = s.get_state()
    bad = start.clone()
    bad[0, 5, 7] = -1.0
    for _ in range(2):
        s.step(3)
        assert s.diagnostics()["n_limited"] > 0
        for _ in range(3):
            m, st = s.moments(check=False)
            assert st == B.LBM_OK and s.diagnostics()["n_limited"] == 0
        assert torch.equal(m, s.get_state()[:4])
    s.set_state(bad)
    assert s.moments(check=False)[1] == B.LBM_EPOSITIVITY
    assert s.moments(check=False)[1] == B.LBM_OK
    s.set_state(start)
    tx, ty = s.step_theta()
    s.moments()
    out = torch.empty_like(start)
    B.lbm_step_adjoint_theta(s.ctx, bad, tx, ty, start, out)
    assert s.moments(check=False)[1] == B.LBM_EPOSITIVITY
    s.set_state(start)
    s.step(1)
    d, ref = s.diagnostics(), plain(u0, KW, 1)[0]
    assert d["n_limited"] == ref["n_limited"] and d["lam"] == ref["lam"] and d["min_rho"] == ref["min_rho"]
    s.close()
