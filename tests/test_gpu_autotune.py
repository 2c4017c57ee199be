"""The tuner weighs the launch that runs while nobody sets a shape, and reads its
own file back."""
import json

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


def test_the_untuned_launch_is_a_candidate(gpu, tmp_path):
    """1536^2 in float64: the strips of 12 rows that run untuned take 161 us a
    step, the best of the tuner's own heights 172 and more, so it must keep the
    former."""
    from paper_2411_15001_amd.solver import Solver

    path = str(tmp_path / "tune.json")
    s = Solver(cases.blast(1536), limiters=9)
    untuned = B.lbm_get_grid(s.ctx)[1]
    s.autotune(path)
    (entry,) = json.load(open(path)).values()
    assert entry == [0, 0, 0, 0]
    assert B.lbm_get_grid(s.ctx)[1] == untuned
    s.close()


def test_entries_of_the_file(gpu, tmp_path):
    """[0, 0, ...] is the library's own choice; zero rows with a number of waves
    keep the current height, as in lbm_set_launch."""
    from paper_2411_15001_amd.solver import Solver

    u0 = cases.riemann4(96, seed=1)
    path = str(tmp_path / "tune.json")
    s = Solver(u0, limiters=9)
    untuned, shape = B.lbm_get_grid(s.ctx)[1], B.lbm_get_launch(s.ctx)
    s.autotune(path)
    s.close()
    (key,) = json.load(open(path))
    for entry, launch, groups in (([0, 0, 0, 0], shape, untuned), ([0, 2, 0, 0], (shape[0], 2), None),
                                  ([8, 2, 0, 0], (8, 2), None)):
        with open(path, "w") as f:
            json.dump({key: entry}, f)
        s = Solver(u0, limiters=9)
        s.autotune(path)
        assert B.lbm_get_launch(s.ctx) == launch, entry
        if groups is not None:
            assert B.lbm_get_grid(s.ctx)[1] == groups
        else:
            strips = 2 * -(-96 // launch[0])
            assert B.lbm_get_grid(s.ctx)[1] == -(-(-(-strips // launch[1])) // 8) * 8
        s.close()
