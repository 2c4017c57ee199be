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
