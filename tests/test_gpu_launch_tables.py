"""The strip tables of a context: what rebuilds them, and that work recorded
before keeps its own."""
import time

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
