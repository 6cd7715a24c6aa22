"""The library's own choice between single steps and passes of several steps, asked on
the host: lbm_init calls these functions of csrc/lbm_multi.h (no part of the C ABI, hence
the C++ names)."""
import ctypes as C

from paper_1510_07328_amd import lbm

CUS = 256


class MultiPlan(C.Structure):
    _fields_ = [("best", C.c_int), ("time", C.c_double), ("ly", C.c_int * 8), ("next", C.c_byte * 2 * 25)]


class TilePlan(C.Structure):
    _fields_ = [("sx", C.c_int), ("sy", C.c_int), ("h", C.c_int), ("time", C.c_double), ("one", C.c_bool)]


def tile(shape, fp64=False, walls=False, porous=False):
    """d2v9 in LDS: the tile, its steps per launch, and whether a launch of one step pays."""
    f = lbm.load()._ZN3lbm9tile_planEiibbbii
    f.restype, f.argtypes = TilePlan, [C.c_int] * 2 + [C.c_bool] * 3 + [C.c_int] * 2
    return f(shape[0], shape[1], walls, walls, porous, int(fp64), CUS)


def planes_per_segment(shape, bc=(0, 0, 0), fp64=False):
    """d3v19: planes per segment of a pass of two steps, 0 for single steps."""
    f = lbm.load()._ZN3lbm11multi3_planEiiiiii
    f.restype, f.argtypes = C.c_int, [C.c_int] * 6
    walls = 3 if bc[0] else 2 if bc[1] else 1 if bc[2] else 0
    return f(*shape, int(fp64), walls, CUS)


def depths(shape, n, fp64=False, links=False, push=False):
    """d2v9 in registers: the launches of a call of n steps (1: a single step)."""
    lib = lbm.load()
    plan, depth = lib._ZN3lbm10multi_planEiiibbi, lib._ZN3lbm11multi_depthERKNS_9MultiPlanEli
    plan.restype, plan.argtypes = MultiPlan, [C.c_int] * 3 + [C.c_bool] * 2 + [C.c_int]
    depth.restype, depth.argtypes = C.c_int, [C.POINTER(MultiPlan), C.c_int64, C.c_int]
    p = plan(shape[0], shape[1], int(fp64), links, push, CUS)
    out, odd = [], n & 1 if push else 0
    while n > 0:
        h = depth(C.byref(p), n, odd) or 1
        out.append(h)
        n, odd = n - h, odd ^ 1
    return out
