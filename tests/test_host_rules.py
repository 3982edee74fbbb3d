"""Host-only checks of the launch rules inside the library (no device work):
what a launch refuses, through its internal symbols."""
import ctypes as C
import os

import pytest

HIP_INVALID_VALUE = 1


@pytest.fixture(scope="module")
def L():
    from paper_2511_16821_amd import slh
    if not os.path.exists(slh.LIB_PATH):
        from paper_2511_16821_amd import build
        build.build()
    return slh.lib()


@pytest.mark.parametrize("nx,ny", [(4097, 1), (65, 64), (64, 65), (1024, 1024), (65536, 65536),
                                   (0, 5), (-3, 7)])
def test_one_workgroup_cg_refuses_other_meshes(L, nx, ny):
    """The one-workgroup solve holds 4096 cells in registers and LDS; a launch
    for more would leave cells unsolved and read past the LDS row.  Refused on
    the host, before any launch (65536 x 65536: the count is not 32-bit)."""
    f = L._ZN3slh25launch_cg_solve_one_blockERKNS_6CgArgsEdiP12ihipStream_t
    f.argtypes = [C.c_void_p, C.c_double, C.c_int, C.c_void_p]
    f.restype = C.c_int
    args = (C.c_int32 * 64)(nx, ny)  # CgArgs: the mesh, then pointers
    assert f(args, 1e-2, 32, None) == HIP_INVALID_VALUE
