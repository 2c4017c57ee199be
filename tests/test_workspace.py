"""Workspace sizes, which the library computes without a GPU."""
import pytest

from paper_2411_15001_amd import binding as B


@pytest.mark.parametrize("n", [4, 8, 16, 33])
@pytest.mark.parametrize("lims", [9, 11])
@pytest.mark.parametrize("bc", [0, 1])
def test_small_instances_need_little_beside_their_states(n, lims, bc):
    """Beside the two states of 20 values a cell, an instance of an ensemble
    takes less than 1 KB for its record, its place in the strip tables and its
    boundary description (further records only where its waves would queue at
    one: 4 KB each with all of them)."""
    k = 1000
    p = B.make_params(n, n, precision=B.LBM_FP32_STATE, limiters=lims, bc_x=bc, bc_y=bc)
    states = 2 * 20 * 4 * n * n * k
    beside = B.lbm_batch_workspace_bytes(p, [n] * k, [n] * k) - states
    assert 0 < beside < 1024 * k + (1 << 17)


def test_records_of_large_instances_are_reserved():
    p = B.make_params(4096, 4096, limiters=9)
    assert B.lbm_workspace_bytes(p) - 2 * 20 * 8 * 4096 * 4096 > 33 * 128
