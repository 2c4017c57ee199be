"""The strip tables of a context: what rebuilds them, and that work recorded
before keeps its own."""
import time

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


def field(nx, ny, seed):
    return np.ascontiguousarray(cases.riemann4(max(nx, ny), seed=seed)[:, :ny, :nx])


def uniform(nx, ny, torch):
    u = torch.zeros((4, ny, nx), dtype=torch.float64, device="cuda")
    u[0], u[3] = 1.0, 2.5
    return u


def test_update_of_a_description_does_not_rebuild_the_tables(gpu):
    """Updating one side's cells of one instance costs what that side's cells
    cost, however many strips the ensemble has: 16 instances of one column and
    131072 rows (524288 groups of four strip rows) against 16 of one column and
    four rows.  (A rebuild walks and uploads all of them: 228 us against 34.)"""
    from paper_2411_15001_amd.solver import BatchSolver

    torch = gpu
    best = []
    for ny in (4, 131072):
        b = BatchSolver([uniform(1, ny, torch) for _ in range(16)], limiters=9, bc_x=1, bc_y=1)
        kind = torch.ones(1, dtype=torch.uint8, device="cuda")
        b.set_boundary(0, 2, kind)
        times = []
        for k in range(20):
            torch.cuda.synchronize()
            t = time.perf_counter()
            b.set_boundary(k % 16, 2 + k % 2, kind)
            times.append(time.perf_counter() - t)
        best.append(min(times))
        b.step(2)
        m = b.moments(3)
        assert torch.equal(m, uniform(1, ny, torch))
        b.close()
    print("  set_boundary %.1f / %.1f us" % (best[0] * 1e6, best[1] * 1e6))
    assert best[1] < 4.0 * best[0]


SMALL = [(40, 41), (64, 3), (129, 70), (200, 33)]  # the row kernel
LARGE = [(700, 690), (650, 701), (690, 700), (701, 640)]  # float64 under density bounds: the marches
SHAPE = {
    "grid": lambda b: B.lbm_set_grid(b.ctx, 2),
    "waves": lambda b: B.lbm_set_launch(b.ctx, 0, 2),
    "rows": lambda b: B.lbm_set_launch(b.ctx, 8, 0),
    "mode": lambda b: B.lbm_set_strip_mode(b.ctx, 1),
}


@pytest.mark.parametrize("sides", [SMALL, LARGE])
@pytest.mark.parametrize("shape", list(SHAPE))
def test_recorded_steps_outlive_a_first_launch_shape(sides, shape, gpu):
    """Steps of an ensemble that a caller recorded while nobody had set a launch
    shape read the strip table they were recorded with after one is set."""
    from paper_2411_15001_amd.solver import BatchSolver

    print("tables", sides[0], shape, flush=True)
    torch = gpu
    u0s = [field(nx, ny, 20 + i) for i, (nx, ny) in enumerate(sides)]
    kw = dict(limiters=11, a_beta=1.1, bc_x=1, bc_y=1)
    with torch.cuda.stream(torch.cuda.Stream()):
        ref = BatchSolver(u0s, **kw)
        b = BatchSolver(u0s, **kw)
        b.step(6)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=torch.cuda.current_stream()):
            b.step(6)
        ref.step(6)
        SHAPE[shape](b)
        for _ in range(2):
            g.replay()
            ref.step(6)
            assert torch.equal(b.get_state(), ref.get_state())
        b.step(3)  # in the new shape
        ref.step(3)
        assert torch.equal(b.get_state(), ref.get_state())
        for i in range(len(sides)):
            x, y = b.diagnostics(i), ref.diagnostics(i)
            assert all(x[k] == y[k] for k in ("lam", "t", "n_limited", "n_lmp", "n_bad"))
        del g
        b.close()
        ref.close()


def test_recorded_steps_outlive_the_last_description(gpu):
    """Described boundaries bring their own launch: steps recorded with them
    still find its table when the last description has gone."""
    from paper_2411_15001_amd.solver import BatchSolver

    torch = gpu
    u0s = [field(nx, ny, 50 + i) for i, (nx, ny) in enumerate(LARGE)]
    kw = dict(limiters=11, a_beta=1.1, bc_x=1, bc_y=1)
    kind = torch.ones(LARGE[1][0], dtype=torch.uint8, device="cuda")
    with torch.cuda.stream(torch.cuda.Stream()):
        runs = []
        for recorded in (True, False):
            b = BatchSolver(u0s, **kw)
            b.set_boundary(1, 2, kind)
            b.step(6)
            if recorded:
                g = torch.cuda.CUDAGraph()
                with torch.cuda.graph(g, stream=torch.cuda.current_stream()):
                    b.step(6)
            b.set_boundary(1, 2, None)
            for _ in range(2):
                g.replay() if recorded else b.step(6)
            b.step(3)
            runs.append((b.get_state(), [b.diagnostics(i)["n_limited"] for i in range(len(LARGE))]))
            b.close()
        del g
    assert torch.equal(runs[0][0], runs[1][0]) and runs[0][1] == runs[1][1]
