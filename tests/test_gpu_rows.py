"""The row kernel (one row of a 64-column strip per wave; grids whose launch
shape nobody set, up to the sizes its rule names) against the marches (a
launch shape set by the caller): states, face factors, lambda, t and every
counter are the same bit for bit, on widths and heights around the strip's 64
columns, the workgroup's four rows and the two halo layers, in both storage
types, for every limiter set, with sponges, described boundaries and in
ensembles."""
import numpy as np
import pytest

from paper_2411_15001_amd import binding as B
from paper_2411_15001_amd import cases

pytestmark = pytest.mark.gpu

KEYS = ("lam", "t", "n_limited", "n_guard", "n_lmp", "n_bad", "n_nonfinite", "n_rho", "n_rhoe", "bouchut")
SIZES = [(1, 1), (2, 3), (63, 4), (64, 5), (65, 2), (128, 9), (130, 6), (192, 64), (200, 33)]


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch

    assert torch.cuda.is_available()
    B.lib()
    return torch


def field(nx, ny, seed):
    return np.ascontiguousarray(cases.riemann4(max(nx, ny, 4), seed=seed)[:, :ny, :nx])


def run(u0, kw, launch, steps=7, bnd=None):
    from paper_2411_15001_amd.solver import Solver

    s = Solver(u0, **kw)
    for side, (k, st) in (bnd or {}).items():
        s.set_boundary(side, k, st)
    if launch:
        s.set_launch(*launch)
    s.step(steps - 1)
    tx, ty = s.step_theta()
    out = (s.get_state(), tx, ty, s.diagnostics())
    s.close()
    return out


def check(a, b, torch):
    for x, y in zip(a[:3], b[:3]):
        assert torch.equal(x, y)
    for k in KEYS:
        assert a[3][k] == b[3][k] or (a[3][k] != a[3][k] and b[3][k] != b[3][k]), k


@pytest.mark.parametrize("nx,ny", SIZES)
@pytest.mark.parametrize("lims", [0, 1, 8, 9, 11, 13, 2, 15])
@pytest.mark.parametrize("prec", [0, 1])
def test_rows_equal_marches(nx, ny, lims, prec, gpu):
    print("rows", nx, ny, lims, prec, flush=True)
    for k, (bx, by, sponge) in enumerate([(0, 0, 0), (1, 1, 0), (1, 0, 2)]):
        kw = dict(limiters=lims, a_beta=1.1, bc_x=bx, bc_y=by, sponge=sponge, precision=prec)
        u0 = field(nx, ny, 3 + k)
        check(run(u0, kw, None), run(u0, kw, (8, 2)), gpu)


@pytest.mark.parametrize("nx,ny", [(1, 1030), (64, 1030), (200, 1029), (1030, 66)])
@pytest.mark.parametrize("lims", [2, 11, 13, 15])
def test_rows_under_bounds_beyond_one_group_per_cu(nx, ny, lims, gpu):
    """float64 under density bounds with more than 256 workgroups: the form of
    the row kernel that loads each face's values in turn."""
    for k, (bx, by, sponge) in enumerate([(0, 0, 0), (1, 1, 0), (1, 0, 2), (0, 1, 3)]):
        kw = dict(limiters=lims, a_beta=1.1, bc_x=bx, bc_y=by, sponge=sponge)
        u0 = field(nx, ny, 30 + k)
        check(run(u0, kw, None, steps=4), run(u0, kw, (8, 2), steps=4), gpu)


@pytest.mark.parametrize("nx,ny", [(2, 2), (65, 5), (130, 40), (64, 64)])
@pytest.mark.parametrize("lims", [9, 13])
@pytest.mark.parametrize("prec", [0, 1])
def test_rows_equal_marches_with_described_boundaries(nx, ny, lims, prec, gpu):
    print("bnd rows", nx, ny, lims, prec, flush=True)
    u0 = field(nx, ny, 8)
    rng = np.random.default_rng(1)
    bnd = {}
    for side in range(4):
        n = ny if side < 2 else nx
        st = cases.prim_to_cons(rng.uniform(0.5, 1.5, n), rng.uniform(-1, 1, n), rng.uniform(-1, 1, n),
                                rng.uniform(0.5, 1.5, n), 1.4)
        bnd[side] = (rng.integers(0, 3, n).astype(np.uint8), st)
    for by in (1, 0):
        kw = dict(limiters=lims, a_beta=1.1, bc_x=1, bc_y=by, precision=prec)
        sides = {k: v for k, v in bnd.items() if by or k < 2}
        check(run(u0, kw, None, bnd=sides), run(u0, kw, (4, 1), bnd=sides), gpu)


@pytest.mark.parametrize("nx,ny", [(3, 2), (130, 6), (257, 30)])
@pytest.mark.parametrize("lims,sponge", [(11, 0), (9, 2), (11, 2), (13, 2), (15, 0), (2, 0)])
@pytest.mark.parametrize("prec", [0, 1])
def test_described_boundaries_with_the_limiter_set_fixed_or_read(nx, ny, lims, sponge, prec, gpu):
    """The sets with PP and pressure are fixed at compile time unless a sponge
    or another set asks for the general form."""
    print("bnd limiters", nx, ny, lims, sponge, prec, flush=True)
    rng = np.random.default_rng(5)
    bnd = {}
    for side in range(4):
        n = ny if side < 2 else nx
        st = cases.prim_to_cons(rng.uniform(0.5, 1.5, n), rng.uniform(-1, 1, n), rng.uniform(-1, 1, n),
                                rng.uniform(0.5, 1.5, n), 1.4)
        bnd[side] = (rng.integers(0, 3, n).astype(np.uint8), st)
    kw = dict(limiters=lims, a_beta=1.1, bc_x=1, bc_y=1, sponge=sponge, precision=prec)
    u0 = field(nx, ny, 12)
    check(run(u0, kw, None, bnd=bnd), run(u0, kw, (4, 1), bnd=bnd), gpu)


@pytest.mark.parametrize("sides", [[(40, 41), (64, 3), (129, 70), (1, 1)], [(64, 64), (128, 5), (192, 130)]])
@pytest.mark.parametrize("lims", [9, 11])
def test_rows_of_an_ensemble_equal_marches(sides, lims, gpu):
    from paper_2411_15001_amd.solver import BatchSolver

    u0s = [field(nx, ny, 20 + i) for i, (nx, ny) in enumerate(sides)]
    kw = dict(limiters=lims, a_beta=1.1, bc_x=1, bc_y=1)
    got = []
    for launch in (None, (4, 3)):
        b = BatchSolver(u0s, **kw)
        if launch:
            b.set_launch(*launch)
        b.step_graph(6)
        b.step(3)
        got.append((b.get_state(), [b.diagnostics(i) for i in range(len(sides))]))
        b.close()
    assert gpu.equal(got[0][0], got[1][0])
    for x, y in zip(got[0][1], got[1][1]):
        assert all(x[k] == y[k] for k in KEYS)


@pytest.mark.parametrize("nx,ny,rows", [(896, 896, True), (960, 960, False)])
def test_both_sides_of_the_size_rule(nx, ny, rows, gpu):
    """The largest grids the rule gives the row kernel, and the next ones: the
    workgroups of a launch tell which kernel runs."""
    from paper_2411_15001_amd.solver import Solver

    kw = dict(limiters=9)
    u0 = cases.blast(nx)
    s = Solver(u0, **kw)
    groups = B.lbm_get_grid(s.ctx)[1]
    assert (groups == (nx // 64) * ((ny + 3) // 4)) == rows
    s.close()
    a, b = run(u0, kw, None, steps=3), run(u0, kw, (8, 2), steps=3)
    check(a, b, gpu)


@pytest.mark.parametrize("nx,ny,lims,prec,rows", [(900, 900, 11, 0, True), (960, 920, 11, 0, False),
                                                  (1024, 1025, 9, 1, True), (1024, 1026, 9, 1, False),
                                                  (896, 900, 13, 1, True), (896, 901, 13, 1, False)])
def test_size_rule_by_type_and_bounds(nx, ny, lims, prec, rows, gpu):
    from paper_2411_15001_amd.solver import Solver

    kw = dict(limiters=lims, precision=prec, bc_x=1, bc_y=1)
    u0 = np.ascontiguousarray(cases.double_rarefaction(max(nx, ny))[:, :ny, :nx])
    s = Solver(u0, **kw)
    groups = -(-((nx + 63) // 64 * ((ny + 3) // 4)) // 8) * 8  # a multiple of the XCDs
    assert (B.lbm_get_grid(s.ctx)[1] == groups) == rows
    s.close()
    check(run(u0, kw, None, steps=3), run(u0, kw, (20, 3), steps=3), gpu)


@pytest.mark.parametrize("nx,ny", [(1100, 1030), (1024, 2048)])
@pytest.mark.parametrize("lims,prec", [(9, 0), (11, 0), (9, 1), (13, 1)])
def test_chosen_strip_height_keeps_the_results(nx, ny, lims, prec, gpu):
    """Grids beyond the row kernel: the strip height that the library picks
    while nobody sets one, ragged and full strips, against a given one."""
    u0 = np.ascontiguousarray(cases.double_rarefaction(max(nx, ny))[:, :ny, :nx])
    kw = dict(limiters=lims, bc_x=1, bc_y=1, precision=prec)
    check(run(u0, kw, None, steps=3), run(u0, kw, (20, 3), steps=3), gpu)


def test_autotuned_choice_keeps_the_results(gpu, tmp_path):
    """The tuner weighs the row kernel too; its recorded choice is taken back
    from the file, and an explicit shape afterwards replaces it."""
    from paper_2411_15001_amd.solver import Solver

    u0 = field(100, 90, 4)
    kw = dict(limiters=11, a_beta=1.1, bc_x=1, bc_y=1)
    ref = run(u0, kw, (8, 2))
    path = str(tmp_path / "tune.json")
    for _ in range(2):
        s = Solver(u0, **kw)
        s.autotune(path)
        rows, waves = B.lbm_get_launch(s.ctx)
        assert rows >= 4 and 1 <= waves <= 4
        s.step(6)
        tx, ty = s.step_theta()
        check((s.get_state(), tx, ty, s.diagnostics()), ref, gpu)
        s.close()


@pytest.mark.parametrize("nx,ny,prec", [(320, 320, 0), (336, 320, 0), (321, 320, 0), (448, 448, 1), (464, 464, 1),
                                        (447, 448, 1), (1280, 1280, 1), (1344, 1280, 1), (1281, 1320, 1)])
@pytest.mark.parametrize("lims", [9, 11])
def test_both_sides_of_the_store_rule(nx, ny, prec, lims, gpu):
    """The state is stored past the caches or through L2 by its size and by how
    its rows are aligned: around the limits, in both kernels."""
    print("store", nx, ny, prec, lims, flush=True)
    kw = dict(limiters=lims, a_beta=1.1, bc_x=1, bc_y=1, precision=prec)
    u0 = np.ascontiguousarray(cases.double_rarefaction(max(nx, ny))[:, :ny, :nx])
    check(run(u0, kw, None, steps=3), run(u0, kw, (20, 3), steps=3), gpu)


@pytest.mark.parametrize("sides", [[(48, 5), (80, 6)], [(48, 5), (81, 6), (16, 16)], [(32, 3), (16, 1), (96, 70)]])
@pytest.mark.parametrize("lims", [9, 11, 13])
def test_float32_rows_that_start_on_64_bytes_and_elsewhere(sides, lims, gpu):
    """Instances whose rows start on 64 bytes and others, in one buffer: each, in
    both kernels, against its own run."""
    from paper_2411_15001_amd.solver import BatchSolver

    u0s = [field(nx, ny, 40 + i) for i, (nx, ny) in enumerate(sides)]
    kw = dict(limiters=lims, a_beta=1.1, bc_x=1, bc_y=0, precision=1)
    single = [run(u, kw, None, steps=6) for u in u0s]
    for launch in (None, (4, 3)):
        b = BatchSolver(u0s, **kw)
        if launch:
            b.set_launch(*launch)
        b.step(6)
        for i, one in enumerate(single):
            assert gpu.equal(b.moments(i), one[0][:4].double())
        b.close()
