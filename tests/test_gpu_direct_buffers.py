"""Callers' arrays in device memory are read and written in place; arrays in
host memory, and device arrays not aligned for vector accesses, go through the
session's own.  All of them must give the same bits: verify rounds of every
rule, plain and guided, commits with and without logits, strict rounds, and
draft head runs.  Device arrays that end before the call's last element are
refused, and calls on device arrays can be captured into a graph."""
import ctypes

import numpy as np
import pytest

import paper_2606_20543_amd as ssd
import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

BF16 = synth.ModelShape(2, 512, 8, 2, 64, 768, 640, 512, "bf16")
F32 = synth.ModelShape(2, 64, 4, 2, 16, 100, 90, 70, "f32")  # rows of 70 codes: no 16-byte rows


class Dev:
    """A device copy of an array, `skew` bytes past an aligned address."""

    def __init__(self, a, skew):
        raw = np.zeros(a.nbytes + skew, np.uint8)
        raw[skew:] = np.ascontiguousarray(a).view(np.uint8).reshape(-1)
        self.a, self.skew, self.mem = a, skew, G.DeviceArray(raw)
        self.ptr = self.mem.ptr + skew

    def numpy(self):
        out = self.mem.numpy()[self.skew:].copy().view(self.a.dtype).reshape(self.a.shape)
        self.mem.free()
        return out


def _step(sess, K, tokens, prm, V, d, where, ref=None, logits=True):
    n = tokens.shape[0]
    host = [tokens.copy(), ref, np.zeros((n, K), np.uint8), np.zeros(n, np.int32), np.zeros(n, np.int32),
            np.zeros((n, K, V), np.float32) if logits else None, np.zeros((n, K, d), np.float32)]
    if where == "host":
        t, r, a, c, f, l, h = host
        ssd.ssd_verify_step(sess, K, t, prm, ref_logits=r, accept_mask=a, accept_count=c, frontier=f, logits_out=l,
                            h_pre_out=h)
        return [t, a, c, f, l, h]
    dev = [None if x is None else Dev(x, 4 if where == "skewed" else 0) for x in host]
    t, r, a, c, f, l, h = [None if x is None else x.ptr for x in dev]
    ssd.ssd_verify_step(sess, K, t, prm, ref_logits=r, accept_mask=a, accept_count=c, frontier=f, logits_out=l,
                        h_pre_out=h)
    return [None if x is None else x.numpy() for i, x in enumerate(dev) if i != 1]


def _script(shape, model, where, guided):
    """A sequence of calls on one session; every output of each."""
    B, P, K = (4, 19, 9)
    n = B // 2 if guided else B
    prefix = synth.prompt(shape, B, P).astype(np.int32)
    blk = (synth.random_codes(shape, (n, K)) + shape.img_lo).astype(np.int32)
    ref = np.random.default_rng(3).standard_normal((n, K, shape.v_img)).astype(np.float32)
    sess = ssd.ssd_prefill(model, B, P, prefix, P + 4 * K, K)
    out = []
    try:
        if guided:
            ssd.ssd_session_set_cfg(sess, 4.0)
        args = (shape.v_img, shape.d_model, where)
        out.append(_step(sess, K, blk, G.vparams(0, rnd=0), *args))
        out.append(_step(sess, K, blk, G.vparams(1, top_k=20, rnd=1, n_fixed=1), *args))
        out.append(_step(sess, K, blk, G.vparams(2, top_k=30, rnd=2), *args, ref=ref))
        out.append(_step(sess, K, blk, G.vparams(2, rnd=3), *args, logits=False))
        if not guided:
            out.append(_step(sess, K, blk, G.vparams(0, rnd=4, truncate=1, n_fixed=1), *args))
        out.append(_step(sess, K, blk, G.vparams(commit=1), *args)[3:])
        out.append(_step(sess, K, blk, G.vparams(0, rnd=5), *args))
        out.append(_step(sess, K, blk, G.vparams(commit=1), *args, logits=False)[3:4])
        carry = np.zeros((n, shape.v_img), np.float32)
        ssd.ssd_get_carry(sess, carry)
        out.append([carry])
    finally:
        ssd.ssd_free_session(sess)
    return out


def _equal(a, b):
    return all(x is None if y is None else np.array_equal(x, y) for p, q in zip(a, b) for x, y in zip(p, q))


@pytest.mark.parametrize("shape", [BF16, F32], ids=["bf16", "f32"])
@pytest.mark.parametrize("guided", [False, True])
def test_verify_steps(shape, guided):
    pair = G.Pair(shape, gain_std=0.1, oracle=False)
    try:
        host = _script(shape, pair.model, "host", guided)
        for where in ("device", "skewed"):
            assert _equal(_script(shape, pair.model, where, guided), host), where
    finally:
        pair.close()


@pytest.mark.parametrize("shape,R", [(BF16, 5), (BF16, 64), (BF16, 70), (F32, 9)])
def test_draft_head_runs(shape, R):
    pair = G.Pair(shape, gain_std=0.1, oracle=False)
    try:
        head = ssd.ssd_draft_head_init(pair.model, 512, synth.draft_head_weights(shape.d_model, 512, gain_std=0.1,
                                                                                 dtype=shape.dtype), R)
        h = synth.hidden_states(R, shape.d_model)
        tok = (synth.random_codes(shape, (R,)) + shape.img_lo).astype(np.int32)
        want = (np.zeros(R, np.int32), np.zeros((R, shape.v_img), np.float32))
        ssd.ssd_draft_head_run(head, R, h, tok, *want)
        for run in (ssd.ssd_draft_head_run, ssd.ssd_draft_head_run_noalloc):
            for skew in (0, 4):
                a = [Dev(x, skew) for x in (h, tok, np.zeros(R, np.int32), np.zeros((R, shape.v_img), np.float32))]
                run(head, R, *[x.ptr for x in a])
                got = [x.numpy() for x in a]
                assert np.array_equal(got[2], want[0]) and np.array_equal(got[3], want[1]), (run.__name__, skew)
        ssd.ssd_free_draft_head(head)
    finally:
        pair.close()


def _short(a):
    """A device array one element short of `a`; what is missing lies in the page that the rest ends in."""
    e = a.dtype.itemsize
    assert (a.nbytes - 1) // 4096 == (a.nbytes - e - 1) // 4096
    return G.DeviceArray(np.ascontiguousarray(a).reshape(-1)[:-1])


@pytest.mark.parametrize("guided", [False, True])
@pytest.mark.parametrize("which", range(6), ids=["tokens", "ref", "mask", "count", "logits", "h_pre"])
def test_short_device_arrays_are_refused(which, guided):
    pair = G.Pair(F32, gain_std=0.1, oracle=False)
    B, P, K = 4, 6, 5
    n = B // 2 if guided else B
    sess = ssd.ssd_prefill(pair.model, B, P, synth.prompt(F32, B, P).astype(np.int32), P + K, K)
    try:
        if guided:
            ssd.ssd_session_set_cfg(sess, 4.0)
        host = [(synth.random_codes(F32, (n, K)) + F32.img_lo).astype(np.int32), np.zeros((n, K, F32.v_img), np.float32),
                np.zeros((n, K), np.uint8), np.zeros(n, np.int32), np.zeros((n, K, F32.v_img), np.float32),
                np.zeros((n, K, F32.d_model), np.float32)]
        dev = [_short(x) if i == which else G.DeviceArray(x) for i, x in enumerate(host)]
        t, r, a, c, lg, h = [x.ptr for x in dev]
        with pytest.raises(ssd.SSDError):
            ssd.ssd_verify_step(sess, K, t, G.vparams(2), ref_logits=r, accept_mask=a, accept_count=c, logits_out=lg,
                                h_pre_out=h)
        for x in dev:
            x.free()
    finally:
        ssd.ssd_free_session(sess)
        pair.close()


@pytest.mark.parametrize("which", range(4), ids=["h", "tokens", "drafts", "logits"])
@pytest.mark.parametrize("run", [ssd.ssd_draft_head_run, ssd.ssd_draft_head_run_noalloc])
def test_short_device_arrays_are_refused_by_heads(which, run):
    pair, R = G.Pair(BF16, gain_std=0.1, oracle=False), 9
    w = synth.draft_head_weights(BF16.d_model, 512, gain_std=0.1)
    head = ssd.ssd_draft_head_init(pair.model, 512, w, R)
    try:
        host = [synth.hidden_states(R, BF16.d_model), (synth.random_codes(BF16, (R,)) + BF16.img_lo).astype(np.int32),
                np.zeros(R, np.int32), np.zeros((R, BF16.v_img), np.float32)]
        dev = [_short(x) if i == which else G.DeviceArray(x) for i, x in enumerate(host)]
        with pytest.raises(ssd.SSDError):
            run(head, R, *[x.ptr for x in dev])
        for x in dev:
            x.free()
    finally:
        ssd.ssd_free_draft_head(head)
        pair.close()


def test_captured_calls_replay():
    """A verify round and an allocation-free head run on device arrays, captured once and replayed on new inputs
    (the graph's kernels read and write the arrays themselves)."""
    hip = G.DeviceArray.hip()
    vp = ctypes.c_void_p
    stream, graph, exe = vp(), vp(), vp()
    assert hip.hipStreamCreate(ctypes.byref(stream)) == 0
    shape, B, P, K, R = BF16, 3, 19, 8, 20
    model = ssd.ssd_init_model(G.cfg_of(shape), synth.weights(shape, gain_std=0.1), stream.value)
    head = ssd.ssd_draft_head_init(model, 512, synth.draft_head_weights(shape.d_model, 512, gain_std=0.1), R)
    sess = ssd.ssd_prefill(model, B, P, synth.prompt(shape, B, P).astype(np.int32), P + K, K, stream.value)
    V, d = shape.v_img, shape.d_model

    def inputs(i):
        return ((synth.random_codes(shape, (B, K), seed=i) + shape.img_lo).astype(np.int32),
                synth.hidden_states(R, d, stream=i), (synth.random_codes(shape, (R,), seed=i + 9) + shape.img_lo).astype(np.int32))

    blk, h, tok = inputs(0)
    dev = [G.DeviceArray(x) for x in (blk, np.zeros((B, K), np.uint8), np.zeros(B, np.int32), np.zeros((B, K, V), np.float32),
                                      np.zeros((B, K, d), np.float32), h, tok, np.zeros(R, np.int32),
                                      np.zeros((R, V), np.float32))]

    def load(i):
        for a, x in zip((dev[0], dev[5], dev[6]), inputs(i)):
            assert hip.hipMemcpy(a.ptr, np.ascontiguousarray(x).ctypes.data, a.nbytes, 1) == 0

    def calls():
        ssd.ssd_verify_step(sess, K, dev[0].ptr, G.vparams(1, top_k=40), accept_mask=dev[1].ptr, accept_count=dev[2].ptr,
                            logits_out=dev[3].ptr, h_pre_out=dev[4].ptr)
        ssd.ssd_draft_head_run_noalloc(head, R, *[x.ptr for x in dev[5:9]])

    try:
        want = []
        for i in range(3):
            load(i)
            calls()
            want.append([x.numpy() for x in dev])
        assert hip.hipStreamBeginCapture(stream, 0) == 0
        calls()
        assert hip.hipStreamEndCapture(stream, ctypes.byref(graph)) == 0
        assert hip.hipGraphInstantiate(ctypes.byref(exe), graph, None, None, ctypes.c_size_t(0)) == 0
        for i in (2, 0, 1):
            load(i)
            assert hip.hipGraphLaunch(exe, stream) == 0
            got = [x.numpy() for x in dev]
            assert all(np.array_equal(a, b) for a, b in zip(got, want[i])), i
            load((i + 1) % 3)  # the calls themselves between replays
            calls()
            assert all(np.array_equal(x.numpy(), b) for x, b in zip(dev, want[(i + 1) % 3])), i
    finally:
        if exe:
            hip.hipGraphExecDestroy(exe)
        if graph:
            hip.hipGraphDestroy(graph)
        for x in dev:
            x.free()
        ssd.ssd_free_session(sess)
        ssd.ssd_free_draft_head(head)
        ssd.ssd_free_model(model)
        hip.hipStreamDestroy(stream)
