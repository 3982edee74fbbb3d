"""The sweep plan that the library chooses for a mesh, asked on the host through
its internal symbol."""
import ctypes as C

LDS = 160 * 1024  # bytes per workgroup on MI355X


class Plan(C.Structure):
    _fields_ = [(k, C.c_int) for k in ("swap", "nu", "nv", "n_strips", "n_waves", "n_blk", "per",
                                       "n_grp")] + [("table", C.c_bool)]


def sweep_plan(S, nx, ny, sn_order, n_mat, reflective=False, squares=True):
    """n_mat: distinct sigma_e.  per: directions per wave; swap: lanes along x;
    n_blk: workgroups per group of directions."""
    f = S.lib()._ZN3slh7dg_planEiiixbbm
    f.argtypes = [C.c_int, C.c_int, C.c_int, C.c_longlong, C.c_bool, C.c_bool, C.c_size_t]
    f.restype = Plan
    return f(nx, ny, sn_order ** 2, n_mat, squares, reflective, LDS)
