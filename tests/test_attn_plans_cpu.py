"""Session workspaces are sized from attn_plan_bound: for every block length and
context a session can meet, attn_plan must need no more chunk partials or
arrival counters (host code inside libssd.so, called through its C++ symbols)."""
import ctypes

import pytest

import paper_2606_20543_amd as ssd
import synth


class Dims(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("L", "d", "Hq", "Hkv", "D", "dff", "V", "img_lo", "img_hi", "Vimg")] + [
        ("bf16", ctypes.c_bool), ("eps", ctypes.c_float), ("theta", ctypes.c_float)]


class AttnPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("chunk", "nchunk", "qpw", "qs", "nqg", "rows", "xcd")]


@pytest.fixture(scope="module")
def planner():
    L = ssd.lib()
    plan = getattr(L, "_ZN3ssd9attn_planERKNS_4DimsEiiiii")
    plan.argtypes, plan.restype = [ctypes.POINTER(Dims)] + [ctypes.c_int] * 5, AttnPlan
    bound = getattr(L, "_ZN3ssd15attn_plan_boundERKNS_4DimsEiii")
    bound.argtypes, bound.restype = [ctypes.POINTER(Dims)] + [ctypes.c_int] * 3, AttnPlan
    return plan, bound


@pytest.mark.parametrize("Hq,Hkv,D", [(16, 16, 128), (32, 32, 128), (32, 8, 128), (32, 8, 64), (8, 1, 64), (64, 1, 128)])
@pytest.mark.parametrize("B", [1, 2, 3, 8, 33])
def test_bound_covers_every_context(planner, Hq, Hkv, D, B):
    plan, bound = planner
    dm = Dims(1, Hq * D, Hq, Hkv, D, 512, 64, 0, 64, 64, True, 1e-5, 1e4)
    for max_ctx in (64, 640, 4352, 20032):
        for K in (1, 2, 5, 15, 16, 17, 31, 32, 33, 48, 64, 96, 127, 128, 256, 300):
            b = bound(dm, B, K, max_ctx)
            for ctx in {1, 63, 64, 65, 127, 128, 129, *range(1, max_ctx + 1, 61 if max_ctx < 5000 else 509), max_ctx}:
                if ctx > max_ctx:
                    continue
                for xcd in (0, 8):
                    p = plan(dm, B, K, ctx, xcd, 0)
                    where = f"B={B} K={K} ctx={ctx} of {max_ctx}"
                    assert (p.qpw, p.qs, p.nqg, p.rows) == (b.qpw, b.qs, b.nqg, b.rows), where
                    assert 1 <= p.nchunk <= b.nchunk, where
