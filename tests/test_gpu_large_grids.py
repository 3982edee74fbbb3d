"""More work than a grid has threads: the conjugate gradients with several
cells per thread and the emission in runs of several particles per thread,
against the CPU oracle (FP64: 1e-10 relative in the L2 and max norms, counts
equal, the bound of every parity test)."""
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
    (700, 521),     # 364700 cells on 262144 threads: some threads have a second cell
    (1033, 1031)])  # 1065023: a fifth, past the four that a thread loads at once
def test_conjugate_gradients_with_several_cells_per_thread(S, oracle, nx, ny):
    from paper_2511_16821_amd import workloads as W
    rng = np.random.default_rng(nx + ny)
    p = W.homogeneous_box(n=max(nx, ny), L=2.0, n_s=1, n_particles=2000, dt=0.02, closure=1,
                          si_tol=1e-9)
    p.update(nx=nx, ny=ny, x_hi=4.0, y_hi=4.0 * ny / nx)
    for f in ("sigma_s", "sigma_a"):
        p[f] = rng.uniform(0.05, 3.0, size=(ny, nx))
    p["q"] = np.ones((ny, nx))
    log("cg", nx, ny)
    r = oracle.HybridOracle(p).step()
    assert r["si_iters"] < 200
    s = S.Solver(p)
    s.advance(1)
    compare_step(S, s, r)
    assert s.get_stats()["si_iterations"] == r["si_iters"]
    s.destroy()


@pytest.mark.parametrize("n_particles,run", [
    (530001, 2),    # a thread takes two, the last one not both
    (2200003, 8)])  # the longest run, the last one partial
def test_emission_runs(S, oracle, n_particles, run):
    """A source in every cell of 41 x 29, so that runs span emitters; the
    first step's census shows every particle."""
    from paper_2511_16821_amd import workloads as W
    rng = np.random.default_rng(n_particles)
    p = W.homogeneous_box(n=41, L=2.0, n_s=1, n_particles=n_particles, dt=0.005, sn_order=2)
    p.update(ny=29, census_cap=2 * n_particles)
    for f in ("sigma_s", "sigma_a"):
        p[f] = np.asarray(p[f])[:29]
    p["q"] = rng.uniform(0.1, 2.0, size=(29, 41))
    log("emission", n_particles, "runs of", run)
    assert 1024 * 256 * run <= n_particles < 2048 * 256 * 8
    o = oracle.HybridOracle(p)
    r = o.step()
    s = S.Solver(p)
    s.advance(1)
    compare_step(S, s, r)
    compare_balance(s, r)
    assert s.get_stats()["census_alive"] == r["census_alive"]
    c, b = s.get_census(), o.bank
    assert np.array_equal(c["hid"], b.hid) and np.array_equal(c["cell"], b.cell)
    for f in ("x", "y", "ox", "oy", "w"):
        assert rel_l2(c[f], getattr(b, f)) <= 1e-12, f
    s.destroy()
