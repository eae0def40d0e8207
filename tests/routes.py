"""The library's own rules for which kernel takes a projection, so that a test can say that it reaches the one it is for."""
import ctypes as C

from paper_2303_06865_amd import binding as B


def _rule(name, *args):
    f = getattr(B.lib(), name)
    f.restype, f.argtypes = C.c_bool, [C.c_int64 if isinstance(a, int) else type(a) for a in args]
    return bool(f(*args))


def few_rows(dtype, n, k, m):
    """fg::gemm_fewrows_takes (csrc/fg_gemm_fewrows.hip); asked before any other kernel"""
    return _rule("_ZN2fg18gemm_fewrows_takesEilll", C.c_int(dtype), n, k, m)


def f16_tiles(n, k, m, residual=True):
    """fg::gemm_f16_tiles_takes (csrc/fg_gemm_f16_tiles.hip)"""
    return _rule("_ZN2fg20gemm_f16_tiles_takesEilllb", C.c_int(B.FG_F16), n, k, m, C.c_bool(residual))
