"""The DG sweep at the edges of its strips of 64 rows, blocks of eight columns,
sixteen strips per workgroup and four directions per wave, against the CPU
oracle (FP64: 1e-10 relative in the L2 and max norms, the bound of every parity
test), with few materials (the table) and a material per cell."""
import numpy as np
import pytest

from gpu_util import compare_step, log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available()
    from paper_2511_16821_amd import slh
    slh.lib()
    return slh


def _problem(nx, ny, per_cell, **kw):
    from paper_2511_16821_amd import workloads as W
    rng = np.random.default_rng(nx * 10007 + ny)
    p = W.homogeneous_box(n=max(nx, ny), L=2.0, n_s=0, n_particles=3000, **kw)
    h = 2.0 / max(nx, ny)
    p.update(nx=nx, ny=ny, x_hi=h * nx, y_hi=1.3 * h * ny)
    mats = rng.uniform(0.05, 3.0, size=(2, 5))
    pick = rng.integers(0, 5, size=(ny, nx))
    for k, f in enumerate(("sigma_s", "sigma_a")):
        p[f] = rng.uniform(0.05, 3.0, size=(ny, nx)) if per_cell else mats[k][pick]
    p["q"] = np.zeros((ny, nx))
    p["q"][ny // 3:ny // 2 + 1, nx // 4:nx // 2 + 1] = 1.0
    return p


def _check(S, oracle, p, steps):
    log("sweep", p["nx"], p["ny"], "S_%d" % p["sn_order"], "boundary", p.get("boundary", 0))
    o = oracle.HybridOracle(p)
    s = S.Solver(p)
    for _ in range(steps):
        r = o.step()
        s.advance(1)
        compare_step(S, s, r)
        assert s.get_stats()["si_iterations"] == r["si_iters"]
    s.destroy()


@pytest.mark.parametrize("per_cell", [False, True])
@pytest.mark.parametrize("nx,ny,boundary", [
    (1, 1, 0), (1, 70, 15), (70, 1, 13), (3, 8, 1), (8, 3, 4), (63, 64, 2), (64, 65, 8),
    (65, 129, 0), (129, 65, 15), (200, 7, 10), (7, 200, 5), (130, 130, 0)])
def test_strip_edges(S, oracle, nx, ny, boundary, per_cell):
    _check(S, oracle, _problem(nx, ny, per_cell, dt=0.1, sn_order=4, boundary=boundary), 2)


def test_more_strips_than_waves(S, oracle):
    """1040 x 1030 cells: seventeen strips, so that a wave takes two."""
    _check(S, oracle, _problem(1040, 1030, False, dt=1e-3, sn_order=2, si_tol=1e-4), 1)


@pytest.mark.parametrize("nx,ny,sn,boundary,per_cell", [
    (560, 330, 14, 15, False),  # 49 directions per quadrant: thirteen groups, the last of one
    (330, 560, 14, 0, True),    # the lanes along x
    (520, 300, 16, 6, True)])
def test_four_directions_per_wave(S, oracle, nx, ny, sn, boundary, per_cell):
    """Several workgroups per group of directions (five and six strips); a
    short step and a loose tolerance leave the oracle two or three sweeps."""
    _check(S, oracle, _problem(nx, ny, per_cell, dt=1e-3, sn_order=sn, boundary=boundary,
                               si_tol=1e-4), 1)


@pytest.mark.parametrize("per_cell", [False, True])
@pytest.mark.parametrize("n,boundary", [
    (2, 15), (64, 0), (65, 13), (128, 7), (1024, 0), (1025, 15), (2500, 14)])
@pytest.mark.parametrize("along_x", [True, False])
def test_one_row(S, oracle, n, boundary, along_x, per_cell):
    """One row or one column of cells: a wave's, a workgroup's, and more cells
    than a workgroup has threads (two and three for a thread)."""
    nx, ny = (n, 1) if along_x else (1, n)
    _check(S, oracle, _problem(nx, ny, per_cell, dt=0.1, sn_order=4, boundary=boundary), 2)


@pytest.mark.parametrize("nx,ny,sn,kw", [
    (16, 1, 2, dict(boundary=5)),
    (1, 33, 4, dict(boundary=15)),
    (113, 1, 4, dict(boundary=10)),
    (100, 1, 4, dict(si_batch=3)),              # batches that end before the iteration does
    (32, 1, 4, dict(boundary=4, si_norm=1)),    # the whole flux as the reference
    (96, 1, 8, dict(boundary=13)),              # more directions than one workgroup takes
    (128, 1, 10, dict(boundary=12, si_accel=1)),  # with the diffusion correction
])
def test_short_row(S, oracle, nx, ny, sn, kw):
    """Short rows, whose iterations run in one workgroup, and their limits."""
    kw = dict(kw)
    batch = kw.pop("si_batch", 0)
    p = _problem(nx, ny, True, dt=0.1, sn_order=sn, **kw)
    log("short row", nx, ny, sn, kw, batch)
    o = oracle.HybridOracle(p)
    s = S.Solver(p)
    if batch:
        s.set_si_batch(batch)
    for _ in range(2):
        r = o.step()
        s.advance(1)
        compare_step(S, s, r)
        assert s.get_stats()["si_iterations"] == r["si_iters"]
    s.destroy()


@pytest.mark.parametrize("nx,ny,sn,boundary,per_cell", [
    (256, 250, 16, 9, False),  # four strips: one workgroup per group, no hand-over
    (770, 768, 4, 0, True)])   # one group of four directions per quadrant
def test_four_directions_one_block_or_group(S, oracle, nx, ny, sn, boundary, per_cell):
    _check(S, oracle, _problem(nx, ny, per_cell, dt=1e-3, sn_order=sn, boundary=boundary,
                               si_tol=1e-4), 1)
