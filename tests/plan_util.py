"""The library's GEMM launch planner, called on the host through its C++
symbols (no GPU), and the sizes a plan needs."""
import ctypes

import paper_2606_20543_amd as ssd

ROWS_MAX = 128  # most rows of the few-row kernel


class GemmPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("MT", "NT", "KCB", "WV", "S", "n_fb", "kchunks", "bn", "xcd", "tile",
                                            "m_tiles", "depth", "tail_fb", "tail_S", "tail_nt")]


def _planner(symbol):
    f = getattr(ssd.lib(), symbol)
    f.argtypes, f.restype = [ctypes.c_int] * 4, GemmPlan
    return f


def plan(M, N, K, xcd=8):
    return _planner("_ZN3ssd14gemm_plan_bf16Eiiii")(M, N, K, xcd)


def plan_guided(M, N, K, xcd=8):
    """The plan of a guided session's block."""
    return _planner("_ZN3ssd16gemm_plan_guidedEiiii")(M, N, K, xcd)


def partials(p, M):
    """Floats of split-K partial sums a plan needs."""
    f = getattr(ssd.lib(), "_ZN3ssd20gemm_partials_floatsERKNS_8GemmPlanEi")
    f.argtypes, f.restype = [ctypes.POINTER(GemmPlan), ctypes.c_int], ctypes.c_size_t
    return f(ctypes.byref(p), M)


def counters(p):
    """Arrival counters a plan uses: one per output tile of a split launch."""
    if p.tile and p.tail_fb:
        return 0 if p.tail_nt else (p.n_fb - p.tail_fb) * p.m_tiles
    return p.n_fb * (p.m_tiles if p.tile else 1) if p.S > 1 else 0


def row_classes():
    """The row counts workspaces are sized over: the few-row kernel's classes (up to 16, 32, 48, 64, 96 and 128
    rows), then each count of 128-row tiles to 256."""
    return [1, 16, 17, 32, 33, 48, 49, 64, 65, 96, 97, 128] + [128 * t for t in range(2, 257)]
