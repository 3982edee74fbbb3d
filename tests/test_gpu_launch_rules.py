"""Where a launch changes its shape with the size of its work: the conjugate
gradients' grids, the tiles of the census decisions and the runs of the
emission, against the CPU oracle (FP64: 1e-10 relative in the L2 and max norms,
counts equal, the bound of every parity test)."""
import numpy as np
import pytest

from gpu_util import compare_balance, compare_step, log, rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available()
    from paper_2511_16821_amd import slh
    slh.lib()
    return slh


@pytest.mark.parametrize("nx,ny", [
    (80, 70),     # 22 blocks, not a multiple of eight
    (96, 64),     # 24 blocks, in runs
    (400, 327),   # 511 blocks: one counter
    (512, 256),   # 512 blocks: eight counters, in runs
    (400, 330)])  # 516 blocks: groups of 65 and 64
def test_conjugate_gradient_grids(S, oracle, nx, ny):
    from paper_2511_16821_amd import workloads as W
    rng = np.random.default_rng(nx + ny)
    p = W.homogeneous_box(n=nx, L=2.0, n_s=1, n_particles=2000, dt=0.05)
    p.update(nx=nx, ny=ny, x_hi=4.0, y_hi=4.0 * ny / nx, closure=1)
    for f in ("sigma_s", "sigma_a"):
        p[f] = rng.uniform(0.05, 3.0, size=(ny, nx))
    p["q"] = np.ones((ny, nx))
    log("cg", nx, ny)
    o = oracle.HybridOracle(p)
    s = S.Solver(p)
    for _ in range(2):
        r = o.step()
        s.advance(1)
        compare_step(S, s, r)
        assert s.get_stats()["si_iterations"] == r["si_iters"]
    s.destroy()


@pytest.mark.parametrize("n_particles,cap", [
    (122000, 132383),  # 2^18 candidates: tiles of 512
    (122000, 132384),  # one more: tiles of 4096, the last of one candidate
    (122000, 4001),    # a small kept fraction
    (270000, 300000),  # emission in runs, nothing thinned in the first step
    (65, 64)])
def test_census_tiles_and_emission_runs(S, oracle, n_particles, cap):
    """A 12 x 10 mesh over two steps, most histories reaching the census: the
    second step's candidates exceed the cap."""
    from paper_2511_16821_amd import workloads as W
    p = W.homogeneous_box(n=12, L=2.0, n_s=1, n_particles=n_particles, dt=0.02, sn_order=4)
    p.update(ny=10, census_cap=cap)
    for f in ("sigma_s", "sigma_a", "q"):
        p[f] = np.asarray(p[f])[:10]
    log("census", n_particles, cap)
    o = oracle.HybridOracle(p)
    s = S.Solver(p)
    for _ in range(2):
        r = o.step()
        s.advance(1)
        compare_step(S, s, r)
        compare_balance(s, r)
        st = s.get_stats()
        assert st["census_alive"] == r["census_alive"]
        assert st["census_kept"] == r["census_kept"]
        assert st["segments_total"] == r["segments"]
        c, b = s.get_census(), o.bank
        assert np.array_equal(c["hid"], b.hid) and np.array_equal(c["cell"], b.cell)
        for f in ("x", "y", "ox", "oy", "w"):
            assert rel_l2(c[f], getattr(b, f)) <= 1e-12, f
    s.destroy()


@pytest.mark.parametrize("nx,ny", [(1, 1), (1, 70), (1024, 1), (41, 25), (63, 65), (64, 64)])
@pytest.mark.parametrize("kw", [dict(closure=1), dict(si_accel=1)])
def test_conjugate_gradients_in_one_workgroup(S, oracle, nx, ny, kw):
    """Up to 4096 cells, one to four per thread: the closing stage and the
    corrections of the source iteration."""
    from paper_2511_16821_amd import workloads as W
    rng = np.random.default_rng(nx * 31 + ny)
    p = W.homogeneous_box(n=max(nx, ny), L=2.0, n_s=1, n_particles=2000, dt=0.1, sn_order=4, **kw)
    p.update(nx=nx, ny=ny, x_hi=0.2 * nx, y_hi=0.25 * ny, boundary=6)
    for f in ("sigma_s", "sigma_a"):
        p[f] = rng.uniform(0.05, 3.0, size=(ny, nx))
    p["q"] = np.ones((ny, nx))
    log("one workgroup", nx, ny, kw)
    o = oracle.HybridOracle(p)
    s = S.Solver(p)
    for _ in range(2):
        r = o.step()
        s.advance(1)
        compare_step(S, s, r)
        assert s.get_stats()["si_iterations"] == r["si_iters"]
    s.destroy()
