"""Functions inside the library that a test calls by their C++ names: the two rules that need no GPU, and the launch of the
direct GEMM kernel with a row-block count of the test's own."""
import ctypes as C

import paper_2512_10236_amd as ficco
from paper_2512_10236_amd.binding import _ptr

CUS = 256
TILES = {1: (256, 256), 2: (128, 128), 3: (256, 128), 4: (128, 256), 5: (64, 256), 6: (32, 256), 7: (128, 128), 8: (128, 192), 9: (256, 192), 10: (64, 128), 11: (64, 64), 12: (32, 64)}


def choose_tile(plan, whole_rows=False):
    """(tile rows, tile columns), estimated microseconds: the tile rule's answer for a plan on a whole MI355X."""
    f = ficco.load()._ZN5ficco11choose_tileEPK12ficco_plan_sibPd
    f.argtypes, f.restype = [C.c_void_p, C.c_int, C.c_bool, C.POINTER(C.c_double)], C.c_int
    us = C.c_double()
    return TILES[f(plan, CUS, whole_rows, C.byref(us))], us.value


def direct_row_blocks(M, K, N):
    """How ficco_gemm_static goes about a product: row blocks of the direct kernel, or 0 where it packs the weight."""
    f = ficco.load()._ZN5ficco17direct_row_blocksElllid
    f.argtypes, f.restype = [C.c_int64, C.c_int64, C.c_int64, C.c_int, C.c_double], C.c_int
    plan = ficco.ficco_plan(M, K, N, 1, 1, ficco.FICCO_FINE_PERSISTENT)
    try:
        ficco.ficco_plan_set(plan, ficco.FICCO_OPT_MODE, ficco.FICCO_MODE_GEMM_ONLY)
        return f(M, K, N, CUS, choose_tile(plan)[1])
    finally:
        ficco.ficco_destroy(plan)


class _DirectLaunch(C.Structure):
    _fields_ = [("A", C.c_void_p), ("W", C.c_void_p), ("C", C.c_void_p), ("M", C.c_int32), ("N", C.c_int32), ("K", C.c_int32),
                ("tiles_m", C.c_int32), ("tiles_n", C.c_int32)]


def launch_direct(row_blocks, A, W, out, stream):
    (M, K), N = A.shape, W.shape[1]
    assert W.shape[0] == K and out.shape[0] >= M and out.shape[1] == N and all(t.is_contiguous() and t.element_size() == 2 for t in (A, W, out))
    f = ficco.load()._ZN5ficco13launch_directEiRKNS_12DirectLaunchEP12ihipStream_t
    f.argtypes, f.restype = [C.c_int, C.POINTER(_DirectLaunch), C.c_void_p], C.c_int
    rc = f(row_blocks, C.byref(_DirectLaunch(_ptr(A), _ptr(W), _ptr(out), M, N, K, 0, 0)), _ptr(stream))
    assert rc == 0, rc
