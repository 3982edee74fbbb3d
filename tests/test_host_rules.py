"""Host-only checks of the launch rules inside the library (no device work):
what a launch refuses and which sweep a mesh gets, through internal symbols."""
import ctypes as C
import os

import pytest

from plan_util import sweep_plan

HIP_INVALID_VALUE = 1


@pytest.fixture(scope="module")
def S():
    from paper_2511_16821_amd import slh
    if not os.path.exists(slh.LIB_PATH):
        from paper_2511_16821_amd import build
        build.build()
    slh.lib()
    return slh


@pytest.mark.parametrize("nx,ny", [(4097, 1), (65, 64), (64, 65), (1024, 1024), (65536, 65536),
                                   (0, 5), (-3, 7)])
def test_one_workgroup_cg_refuses_other_meshes(S, nx, ny):
    """The one-workgroup solve holds 4096 cells in registers and LDS; a launch
    for more would leave cells unsolved and read past the LDS row.  Refused on
    the host, before any launch (65536 x 65536: the count is not 32-bit)."""
    f = S.lib()._ZN3slh25launch_cg_solve_one_blockERKNS_6CgArgsEdiP12ihipStream_t
    f.argtypes = [C.c_void_p, C.c_double, C.c_int, C.c_void_p]
    f.restype = C.c_int
    args = (C.c_int32 * 64)(nx, ny)  # CgArgs: the mesh, then pointers
    assert f(args, 1e-2, 32, None) == HIP_INVALID_VALUE


@pytest.mark.parametrize("nx,ny,sn,n_mat,plan", [
    # one row or column: the scan of its cells, whatever the order
    (80, 1, 4, 5, dict(per=1, nu=80, nv=1)),
    (1, 16, 64, 5, dict(per=1, nu=16, nv=1)),
    (1, 4095, 64, 0, dict(per=1, nu=4095, nv=1)),
    # few strips along the long side
    (1000, 65, 4, 5, dict(per=1, nu=1000)),
    (65, 2300, 8, 0, dict(per=1, nu=2300)),
    # squares: one direction while the planes are small, then four
    (256, 256, 8, 5, dict(per=1)),
    (1024, 1024, 16, 1024, dict(per=4, n_blk=4, table=True)),
    # four directions along the side whose traces fit the LDS
    (3000, 1000, 16, 5, dict(per=4, nu=1000)),
    (1000, 3000, 16, 5, dict(per=4, nu=1000)),
    # the table: where it costs no turns, where it is a number
    (50, 50, 16, 2000, dict(per=1, table=True)),
    (50, 50, 32, 2500, dict(per=1, table=False))])
def test_plan_of_a_sweep(S, nx, ny, sn, n_mat, plan):
    p = sweep_plan(S, nx, ny, sn, n_mat)
    assert {k: getattr(p, k) for k in plan} == plan


def test_plan_without_squares(S):
    """Extreme cells: no table of 1/|z|^2 with four directions per wave; with one
    the table holds the inverses themselves."""
    assert sweep_plan(S, 1024, 1024, 16, 8).table
    assert not sweep_plan(S, 1024, 1024, 16, 8, squares=False).table
    assert sweep_plan(S, 256, 256, 8, 8, squares=False).table


@pytest.mark.parametrize("nx", [1, 2, 63, 64, 65, 700, 1500, 2425, 3000, 4000])
@pytest.mark.parametrize("sn", [2, 4, 14, 64])
def test_plans_are_consistent(S, nx, sn):
    """Every plan covers its mesh and directions, fits the LDS and never takes
    more planes than there are directions."""
    for ny in (1, 2, 64, 65, 129, 1000, 1500, 2425):
        if nx + ny > 4096:
            continue
        for n_mat in (0, 1, 300, 5121):
            for refl in (False, True):
                p = sweep_plan(S, nx, ny, sn, n_mat, refl)
                assert (p.nu, p.nv) == ((ny, nx) if p.swap else (nx, ny))
                assert p.n_strips == (p.nv + 63) // 64 and p.per in (1, 4)
                assert 4 * p.n_grp <= max(sn * sn, 4) and p.n_grp * p.per >= sn * sn // 4
                assert 1 <= p.n_waves <= (4 if p.per == 4 else 16)
                assert p.n_blk * p.n_waves >= p.n_strips if p.per == 4 else p.n_blk == 1
                rows = n_mat + 1 if p.table else 0
                lds = 16 * p.per * (p.nu + 135)
                if refl:
                    lds += 16 * p.per * (64 * p.n_waves if p.per == 4 else p.nv)
                lds += rows * (72 if p.per == 4 else 32)
                lds += 4 * (p.n_waves if p.per == 4 else p.n_strips)
                assert lds <= 160 * 1024, (nx, ny, sn, n_mat, refl)


def _plane_bytes(p, cells):
    return 4 * p.n_grp * cells * 32 + 4 * p.n_grp * (p.n_blk - 1) * p.nu * 4 * p.per * 8


@pytest.mark.parametrize("sn", [2, 4, 8, 16, 24, 64])
def test_plan_of_unknown_materials_bounds_all(S, sn):
    """Without fields the footprint is a bound: the planes of no number of
    materials need more."""
    for nx in (4, 33, 65, 100, 144, 274, 316, 512, 667, 1000, 2047, 2251, 3000):
        for ny in (3, 12, 36, 65, 73, 113, 129, 325, 432, 1000, 2047):
            if nx + ny > 4096:
                continue
            for refl in (False, True):
                bound = _plane_bytes(sweep_plan(S, nx, ny, sn, -1, refl), nx * ny)
                for n_mat in (0, 1, 50, 500, 1000, 2000, 4000, 5121):
                    for squares in (True, False):
                        p = sweep_plan(S, nx, ny, sn, n_mat, refl, squares)
                        assert _plane_bytes(p, nx * ny) <= bound, (nx, ny, sn, n_mat, refl, squares)


def test_footprint_without_fields_bounds_the_one_with(S):
    import numpy as np
    from paper_2511_16821_amd import workloads as W
    rng = np.random.default_rng(4)
    for nx, ny, sn in ((20, 20, 8), (65, 300, 16), (300, 65, 8), (120, 130, 24), (1000, 65, 4)):
        for n_mat in (1, 300, 2000):
            p = W.homogeneous_box(n=max(nx, ny), n_particles=1000, sn_order=sn)
            v = rng.uniform(0.1, 2.0, size=n_mat)
            f = v[rng.integers(0, n_mat, size=(ny, nx))]
            p.update(nx=nx, ny=ny, sigma_s=f, sigma_a=f, q=f)
            st, keep = S.make_problem(p)
            exact = S.lib().slh_footprint_bytes(C.byref(st))
            st.sigma_s = st.sigma_a = None
            assert 0 < exact <= S.lib().slh_footprint_bytes(C.byref(st)), (nx, ny, sn, n_mat)
