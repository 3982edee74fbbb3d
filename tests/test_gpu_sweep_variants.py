"""Every instantiation of the DG sweep against the CPU oracle (FP64: 1e-10
relative in the L2 and max norms, the bound of every parity test), with the
plan that makes it run asserted, so that a change of the plan's estimate shows
here instead of leaving a variant without a test."""
import numpy as np
import pytest

from gpu_util import compare_step, log
from plan_util import sweep_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available()
    from paper_2511_16821_amd import slh
    slh.lib()
    return slh


def _check(S, oracle, nx, ny, sn, boundary, n_mat, sweeps, plan):
    from paper_2511_16821_amd import workloads as W
    rng = np.random.default_rng(nx * 10007 + ny)
    p = W.homogeneous_box(n=max(nx, ny), L=2.0, n_s=0, n_particles=3000, dt=1e-3, sn_order=sn,
                          boundary=boundary, si_tol=1e-6, si_max_iter=sweeps)
    h = 2.0 / max(nx, ny)
    p.update(nx=nx, ny=ny, x_hi=h * nx, y_hi=1.3 * h * ny)
    pick = rng.integers(0, max(1, n_mat), size=(ny, nx))
    for f in ("sigma_s", "sigma_a"):
        p[f] = rng.uniform(0.05, 3.0, size=(ny, nx)) if n_mat == 0 \
            else rng.uniform(0.05, 3.0, size=n_mat)[pick]
    p["q"] = np.zeros((ny, nx))
    p["q"][ny // 3:ny // 2 + 1, nx // 4:nx // 2 + 1] = 1.0
    got = sweep_plan(S, nx, ny, sn, len(np.unique(p["sigma_a"] + p["sigma_s"])), boundary != 0)
    assert {k: getattr(got, k) for k in plan} == plan
    log("sweep", nx, ny, "S_%d" % sn, "boundary", boundary, "materials", n_mat, plan)
    o = oracle.HybridOracle(p)
    r = o.step()
    s = S.Solver(p)
    s.advance(1)
    compare_step(S, s, r)
    assert s.get_stats()["si_iterations"] == r["si_iters"]
    s.destroy()


@pytest.mark.parametrize("nx,ny,boundary,n_mat,swap,strips", [
    (600, 560, 15, 5, 0, 9),     # up to sixteen waves with reflective sides
    (560, 600, 6, 0, 1, 9),
    (590, 530, 0, 0, 0, 9),
    (1040, 1100, 0, 0, 0, 18),   # more strips than waves without the table
    (1090, 1030, 9, 0, 1, 18),
    (1030, 1090, 15, 7, 0, 18)])
def test_one_direction_many_strips(S, oracle, nx, ny, boundary, n_mat, swap, strips):
    _check(S, oracle, nx, ny, 2, boundary, n_mat, 2,
           dict(per=1, swap=swap, n_strips=strips, n_waves=min(strips, 16), n_blk=1,
                table=n_mat > 0))


@pytest.mark.parametrize("nx,ny,sn,boundary,n_mat,sweeps,swap,groups,blocks", [
    (300, 290, 16, 0, 300, 1, 1, 16, 2),  # the table beyond a handful of entries, groups in pairs
    (290, 300, 14, 0, 400, 1, 0, 13, 2),  # an odd count of groups, the last of one direction
    (930, 900, 4, 0, 300, 2, 1, 1, 4),    # one group, four workgroups of four strips
    (900, 950, 4, 13, 0, 2, 0, 1, 4),     # with reflective sides, a material per cell
    (300, 260, 16, 6, 0, 1, 1, 16, 2),    # the same, the lanes along x
    (330, 300, 14, 9, 40, 1, 0, 13, 2)])
def test_four_directions(S, oracle, nx, ny, sn, boundary, n_mat, sweeps, swap, groups, blocks):
    """(One sweep of many directions, two of few: the oracle takes seconds.)"""
    _check(S, oracle, nx, ny, sn, boundary, n_mat, sweeps,
           dict(per=4, swap=swap, n_grp=groups, n_blk=blocks, table=n_mat > 0))
