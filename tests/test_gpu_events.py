"""The events that lbm_moments reports: whatever raised them (eager work, or
loads and adjoint steps that the caller recorded into a graph and replays), the
next call returns them and the one after it starts from zero."""
import pytest

from paper_2411_15001_amd import binding as B
from paper_2411_15001_amd import cases

pytestmark = pytest.mark.gpu

KW = dict(limiters=1 | 2 | 8, a_beta=1.1, bc_x=1, bc_y=1)


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch

    assert torch.cuda.is_available()
    B.lib()
    return torch


def record(kind, s, state, torch):
    """A graph of one call that counts the non-admissible cells of `state`."""
    bar, out = torch.ones_like(state), torch.empty_like(state)
    tx = torch.ones((s.ny, s.nx + 1), dtype=torch.float64, device="cuda")
    ty = torch.ones((s.ny + 1, s.nx), dtype=torch.float64, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.current_stream()):
        if kind == "load":
            s.set_state(state)
        elif kind == "adjoint":
            B.lbm_step_adjoint(s.ctx, state, bar, out)
        else:
            B.lbm_step_adjoint_theta(s.ctx, state, tx, ty, bar, out)
    return g, (bar, out, tx, ty)


@pytest.mark.parametrize("kind", ["load", "adjoint", "adjoint_theta"])
@pytest.mark.parametrize("n", [64, 100])  # blocked and planar layouts
def test_replays_of_recorded_work_that_counts_are_reported(kind, n, gpu):
    from paper_2411_15001_amd.solver import Solver

    print("events", kind, n, flush=True)
    torch = gpu
    with torch.cuda.stream(torch.cuda.Stream()):
        s = Solver(cases.riemann4(n, seed=5), **KW)
        s.step(6)
        good = s.get_state()
        state = good.clone()
        g, keep = record(kind, s, state, torch)
        for value, want in ((None, B.LBM_OK), (-1.0, B.LBM_EPOSITIVITY), (float("nan"), B.LBM_ENONFINITE),
                            (None, B.LBM_OK), (-1.0, B.LBM_EPOSITIVITY)):
            s.moments(check=False)  # clears the counters
            assert s.moments(check=False)[1] == B.LBM_OK
            state.copy_(good)
            if value is not None:
                state[0, 5, 7] = value
            g.replay()
            assert s.moments(check=False)[1] == want, value
        del g, keep
        s.close()


def test_replays_of_a_recorded_load_of_an_ensemble_are_reported(gpu):
    from paper_2411_15001_amd.solver import BatchSolver

    torch = gpu
    with torch.cuda.stream(torch.cuda.Stream()):
        b = BatchSolver([cases.riemann4(n, seed=n) for n in (40, 64, 33)], **KW)
        good = b.get_state()
        state = good.clone()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=torch.cuda.current_stream()):
            b.set_state(state)
        for bad in (False, True, False, True):
            b.moments(0, check=False)
            assert b.moments(0, check=False)[1] == B.LBM_OK
            state.copy_(good)
            if bad:
                state.view(torch.float64)[40 * 40 + 17] = -1.0  # rho of a cell of the second instance
            g.replay()
            assert b.moments(0, check=False)[1] == (B.LBM_EPOSITIVITY if bad else B.LBM_OK)
        del g
        b.close()


def test_nothing_is_pending_when_moments_returns(gpu):
    """The call synchronises with everything it enqueues, the clearing of the
    counters included."""
    from paper_2411_15001_amd.solver import Solver

    torch = gpu
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        s = Solver(cases.riemann4(96, seed=6), **KW)
        out = torch.empty((4, 96, 96), dtype=torch.float64, device="cuda")
        for _ in range(40):
            s.step(2)
            B.lbm_moments(s.ctx, 0, out)
            assert stream.query()
        s.step(2)
        assert s.diagnostics()["n_limited"] > 0  # so every call above had counts to clear
        s.close()


@pytest.mark.parametrize("n", [24, 64, 100, 150, 200, 330, 512])  # 1 to 32 records an instance
def test_load_after_steps_folds_every_record(n, gpu):
    """A load folds the records that the steps before it raised: the counters
    stay the sum of all of them and lambda becomes the loaded state's."""
    from paper_2411_15001_amd.solver import BatchSolver, Solver

    u0 = cases.riemann4(n, seed=3)
    s = Solver(u0, **KW)
    s.step(5)
    ref = s.diagnostics()
    assert ref["n_limited"] > 0
    s.set_state(s.get_state())
    got = s.diagnostics()
    assert all(got[k] == ref[k] for k in ("lam", "t", "n_limited", "n_guard", "n_lmp", "n_bad"))
    s.close()
    b = BatchSolver([u0, cases.riemann4(40, seed=4)], **KW)
    b.step(5)
    b.set_state(b.get_state())
    got = b.diagnostics(0)
    assert all(got[k] == ref[k] for k in ("lam", "n_limited", "n_guard", "n_lmp", "n_bad"))
    b.close()


def test_counts_of_every_instance_of_an_ensemble(gpu):
    """Before any read clears them, each instance's counters, lambda and minima
    are those of its own run; after the first lbm_moments all start from zero."""
    from paper_2411_15001_amd.solver import BatchSolver, Solver

    sides = [64, 320, 128, 256, 33]
    u0s = [cases.riemann4(n, seed=10 + i) for i, n in enumerate(sides)]
    keys = ("lam", "t", "n_limited", "n_guard", "n_lmp", "n_bad", "min_rho", "min_rhoe")
    b = BatchSolver(u0s, **KW)
    runs = [Solver(u0, **KW) for u0 in u0s]
    for part in (7, 4):
        b.step(part)
        for s in runs:
            s.step(part)
        for i, s in enumerate(runs):
            got, ref = b.diagnostics(i), s.diagnostics()
            assert ref["n_limited"] > 0 and all(got[k] == ref[k] for k in keys), i
        for i, s in enumerate(runs):
            assert gpu.equal(b.moments(i), s.moments())
            assert b.diagnostics(i)["n_limited"] == 0
    for s in runs:
        s.close()
    b.close()
