"""Which way the collided solve takes for a mesh, its directions and materials:
that each way gives the oracle's values (FP64: 1e-10 relative in the L2 and max
norms, the bound of every parity test) and is not one that a mesh should avoid."""
import numpy as np
import pytest

from gpu_util import log
from plan_util import sweep_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available()
    from paper_2511_16821_amd import slh
    slh.lib()
    return slh


def _problem(nx, ny, n_mat, **kw):
    """n_mat materials at random, or (0) one per cell; cells that are not square."""
    from paper_2511_16821_amd import workloads as W
    rng = np.random.default_rng(nx * 10007 + ny)
    p = W.homogeneous_box(n=max(nx, ny), L=2.0, n_s=0, n_particles=3000, **kw)
    h = 2.0 / max(nx, ny)
    p.update(nx=nx, ny=ny, x_hi=h * nx, y_hi=1.3 * h * ny)
    pick = rng.integers(0, max(1, n_mat), size=(ny, nx))
    for f in ("sigma_s", "sigma_a"):
        p[f] = rng.uniform(0.05, 3.0, size=(ny, nx)) if n_mat == 0 \
            else rng.uniform(0.05, 3.0, size=n_mat)[pick]
    p["q"] = np.zeros((ny, nx))
    p["q"][ny // 3:ny // 2 + 1, nx // 4:nx // 2 + 1] = 1.0
    return p


def _solve_ms(solver):
    """The shortest collided solve of five steps."""
    ms = []
    for _ in range(5):
        solver.advance(1)
        solver.synchronize(allow_not_converged=True)
        ms.append(solver.get_stats()["ms_dg"])
    return min(ms)


def test_material_per_cell_on_long_rows(S):
    """Twelve iterations with a material per cell take little more than with a
    table of five (by 1.07 measured; 1.7 where the lanes of a wave read sigma_e
    from 64 cache lines at each step)."""
    ms = []
    for n_mat in (5, 0):
        s = S.Solver(_problem(3800, 250, n_mat, dt=1e-4, sn_order=2, si_tol=1e-300,
                              si_max_iter=12))
        s.set_timing(True)
        s.set_si_batch(12)
        ms.append(_solve_ms(s))
        s.destroy()
    log("3800 x 250, S_2: table %.2f ms, material per cell %.2f ms" % tuple(ms))
    assert ms[1] < 1.4 * ms[0], ms


def test_many_materials_and_directions(S):
    """50 x 50 cells, S_32: a material per cell takes about as long as five (by
    1.0 measured; 2.0 where a table of 2500 materials kept other directions'
    workgroups off the compute unit)."""
    ms = []
    for n_mat in (5, 0):
        s = S.Solver(_problem(50, 50, n_mat, dt=1e-2, sn_order=32, si_tol=1e-300, si_max_iter=12))
        s.set_timing(True)
        s.set_si_batch(12)
        ms.append(_solve_ms(s))
        s.destroy()
    log("50 x 50, S_32: five materials %.2f ms, one per cell %.2f ms" % tuple(ms))
    assert ms[1] < 1.5 * ms[0], ms


def _check(S, oracle, p, steps=1):
    from gpu_util import compare_step
    log("sweep", p["nx"], p["ny"], "S_%d" % p["sn_order"], "boundary", p.get("boundary", 0))
    o = oracle.HybridOracle(p)
    s = S.Solver(p)
    for _ in range(steps):
        r = o.step()
        s.advance(1)
        compare_step(S, s, r)
        assert s.get_stats()["si_iterations"] == r["si_iters"]
    s.destroy()


def test_few_strips_along_the_long_side(S):
    """1000 x 65: sixteen directions take about as long as four (by 1.05
    measured; 2.4 where they walked the 65 rows' way, sixteen strips one after
    the other with four directions per wave)."""
    ms = []
    for sn in (2, 4):
        s = S.Solver(_problem(1000, 65, 5, dt=1e-3, sn_order=sn, si_tol=1e-300, si_max_iter=12))
        s.set_timing(True)
        s.set_si_batch(12)
        ms.append(_solve_ms(s))
        s.destroy()
    log("1000 x 65: S_2 %.2f ms, S_4 %.2f ms" % tuple(ms))
    assert ms[1] < 1.6 * ms[0], ms


def test_four_directions_where_one_side_is_long(S):
    """3000 x 1000 cells, S_16, need the planes of 2000 x 1500 (four times as
    many where the long side's traces kept the directions one by one)."""
    b = [S.slh_footprint_bytes(_problem(nx, ny, 5, dt=1e-3, sn_order=16))
         for nx, ny in ((3000, 1000), (2000, 1500))]
    assert b[0] < 1.1 * b[1], b


@pytest.mark.parametrize("nx,ny,sn,boundary,n_mat,per,nu", [
    (700, 65, 4, 15, 5, 1, 700),  # two strips along the long side, the second of one row
    (65, 700, 2, 6, 0, 1, 700),
    (129, 500, 4, 9, 0, 1, 500),  # three strips
    (200, 66, 8, 3, 5, 1, 200),
    (144, 65, 32, 0, 5, 4, 144)])  # four directions along the side of more wave-steps
def test_strips_along_either_side(S, oracle, nx, ny, sn, boundary, n_mat, per, nu):
    plan = sweep_plan(S, nx, ny, sn, n_mat or nx * ny, boundary != 0)
    assert (plan.per, plan.nu) == (per, nu)
    _check(S, oracle, _problem(nx, ny, n_mat, dt=1e-3, sn_order=sn, boundary=boundary, si_tol=1e-4))


def test_cells_of_extreme_width(S, oracle):
    """Cells 1e-155 wide, four directions per wave: 1/|z|^2 of the element's
    modes is no number there, the inverses themselves are."""
    p = _problem(256, 250, 5, sn_order=16)
    assert sweep_plan(S, 256, 250, 16, 5).per == 4
    p.update(x_hi=256e-155, steady=True, horizon=30e-155, q=1e250 * p["q"])
    _check(S, oracle, p)


@pytest.mark.parametrize("n_mat", [4600, 4900, 5119, 5200])
def test_as_many_materials_as_a_table_holds(S, oracle, n_mat):
    """130 x 129 cells whose materials fill the table's LDS, or are one more
    than it could hold, or more than are counted."""
    p = _problem(130, 129, n_mat, dt=0.1, sn_order=2, boundary=9)
    assert sweep_plan(S, 130, 129, 2, n_mat, True).table == (n_mat <= 4900)
    for k, f in enumerate(("sigma_s", "sigma_a")):  # every material in some cell
        v = np.random.default_rng(7 + k).uniform(0.05, 3.0, size=n_mat)
        p[f] = v[np.random.default_rng(3).permutation(130 * 129) % n_mat].reshape(129, 130)
    _check(S, oracle, p, steps=2)
