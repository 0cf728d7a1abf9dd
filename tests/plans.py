"""The library's host-side choices of kernel and tile (molt::gemm_plan, molt::moe_plan), through their
C++ symbols, so that a test can assert which path its case takes."""
import ctypes

import paper_2607_21653_amd as molt
from paper_2607_21653_amd import _lib

F32, BF16, FP8 = 0, 1, 2


class GemmPlan(ctypes.Structure):
    _fields_ = [("bm", ctypes.c_int), ("splits", ctypes.c_int), ("ab", ctypes.c_int)]


class MoePlan(ctypes.Structure):
    _fields_ = [("tile_m", ctypes.c_int), ("big", ctypes.c_bool)]


def _fn(name, res, args):
    molt.load()
    f = getattr(ctypes.CDLL(_lib.LIB_PATH), name)
    f.restype, f.argtypes = res, args
    return f


def gemm_plan(M, N, K, part_elems=1 << 62, rope=False):
    i = ctypes.c_int
    return _fn("_ZN4molt9gemm_planEiiilb", GemmPlan, [i, i, i, ctypes.c_long, ctypes.c_bool])(M, N, K, part_elems, rope)


def moe_plan(dtype, T, K, E, d, F):
    return _fn("_ZN4molt8moe_planE10molt_dtypeiiiii", MoePlan, [ctypes.c_int] * 6)(dtype, T, K, E, d, F)
