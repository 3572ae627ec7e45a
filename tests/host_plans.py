"""The library's launch plans, asked on the host (no GPU): the planners are C++ functions of libfocus.so, called by
their linker names."""
import ctypes

from paper_2608_01847_amd import focus

i32, i64 = ctypes.c_int, ctypes.c_int64


class FwdPlan(ctypes.Structure):
    _fields_ = [("path", i32), ("tile_m", i64), ("mtiles", i64), ("ws_bytes", ctypes.c_size_t)]


class BwdPlan(ctypes.Structure):
    _fields_ = [("path", i32), ("tile", i32), ("splits", i64), ("chunk", i64), ("ws_bytes", ctypes.c_size_t)]


class DxPlan(ctypes.Structure):
    _fields_ = [("path", i32), ("splits", i64), ("chunk", i64), ("ws_bytes", ctypes.c_size_t)]


def _planner(symbol, result, arguments):
    f = getattr(focus.lib(), symbol)
    f.restype, f.argtypes = result, arguments
    return f


def plan_fwd(op_dt, M, N, K):
    return _planner("_ZN5focus8plan_fwdEilll", FwdPlan, [i32, i64, i64, i64])(op_dt, M, N, K)


def fwd_tile_rows(M, N, mx):
    return _planner("_ZN5focus13fwd_tile_rowsEllb", i64, [i64, i64, ctypes.c_bool])(M, N, mx)


def fwd_finish_in_one(mtiles, N):
    return _planner("_ZN5focus17fwd_finish_in_oneEll", ctypes.c_bool, [i64, i64])(mtiles, N)


def plan_bwd(op_dt, fmt, sb, M, N, K, want_G=False):
    return _planner("_ZN5focus8plan_bwdEiiilllb", BwdPlan, [i32, i32, i32, i64, i64, i64, ctypes.c_bool])(
        op_dt, fmt, sb, M, N, K, want_G)


def plan_dx(op_dt, M, N, K):
    return _planner("_ZN5focus7plan_dxEilll", DxPlan, [i32, i64, i64, i64])(op_dt, M, N, K)
