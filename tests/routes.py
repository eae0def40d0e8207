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


class _Pick(C.Structure):
    _fields_ = [("mt", C.c_int), ("nt", C.c_int), ("splits", C.c_int), ("items", C.c_int64), ("us", C.c_float)]


def f16_tile(n, k, m):
    """(rows / 32, columns / 32) of the tiles and ranges of the contraction, fg::gemm_f16_tiles_pick with the scratch that
    fg::linear_workspace_bytes asks for"""
    need = B.lib()._ZN2fg22linear_workspace_bytesEilll
    need.restype, need.argtypes = C.c_size_t, [C.c_int] + 3 * [C.c_int64]
    pick = B.lib()._ZN2fg19gemm_f16_tiles_pickElllm
    pick.restype, pick.argtypes = _Pick, 3 * [C.c_int64] + [C.c_size_t]
    p = pick(n, k, m, need(B.FG_F16, n, k, m))
    return p.mt, p.nt, p.splits
