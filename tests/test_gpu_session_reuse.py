"""Sessions that take over a freed session's workspace: the same bits as on a
model that never had another session, whatever the earlier session left in it
(larger and smaller shapes, other requests, NaN in every cached key and value),
several live sessions at once never share one, threads may create and free them,
and a session may be freed after its model."""
import ctypes
import threading

import numpy as np
import pytest

import paper_2606_20543_amd as ssd
import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

SHAPE = synth.ModelShape(2, 512, 8, 2, 64, 768, 640, 512, "bf16")


def _use(model, B, P, K, seed, stream=None):
    prefix = synth.prompt(SHAPE, B, P, seed=seed).astype(np.int32)
    block = (synth.random_codes(SHAPE, (B, K), seed=seed) + SHAPE.img_lo).astype(np.int32)
    sess = ssd.ssd_prefill(model, B, P, prefix, P + 4 * K, K, stream)
    carry = np.zeros((B, SHAPE.v_img), np.float32)
    ssd.ssd_get_carry(sess, carry)
    outs = [carry]
    for rnd in range(2):
        outs.append(G.gpu_verify(sess, SHAPE, block, G.vparams(2, top_k=50, rnd=rnd), want_h=True))
    outs.append(G.gpu_verify(sess, SHAPE, block, G.vparams(commit=1)))
    return sess, outs


def _same(a, b):
    if isinstance(a, dict):
        return all(_same(a[k], b[k]) for k in a)
    return (a is None and b is None) or np.array_equal(a, b)


def test_reused_workspace_gives_the_same_bits():
    uses = [(2, 70, 16, 1), (2, 64, 16, 2), (1, 70, 9, 3), (4, 130, 33, 4), (2, 70, 16, 1), (3, 90, 24, 5), (4, 130, 33, 4)]
    fresh = {}
    for u in set(uses):
        pair = G.Pair(SHAPE, gain_std=0.1, oracle=False)
        sess, fresh[u] = _use(pair.model, *u)
        ssd.ssd_free_session(sess)
        pair.close()
    pair = G.Pair(SHAPE, gain_std=0.1, oracle=False)
    try:
        for u in uses:  # one after the other: each may take the last one's block
            sess, got = _use(pair.model, *u)
            ssd.ssd_free_session(sess)
            assert all(_same(a, b) for a, b in zip(got, fresh[u])), u
        live = [(_use(pair.model, *u), u) for u in uses[:3]]  # together: none shares
        for (sess, got), u in live:
            assert all(_same(a, b) for a, b in zip(got, fresh[u])), u
            prm = G.vparams(commit=1)
            tok = np.full((u[0], u[2]), SHAPE.img_lo, np.int32)
            G.gpu_verify(sess, SHAPE, tok, prm)
        for (sess, _), _u in live:
            ssd.ssd_free_session(sess)
    finally:
        pair.close()


@pytest.mark.parametrize("shape", [
    SHAPE,
    synth.ModelShape(2, 512, 4, 1, 128, 768, 640, 512, "bf16"),  # head dim 128: blocks of many query rows (below)
    synth.ModelShape(2, 64, 4, 2, 16, 100, 90, 70, "f32"),
    synth.ModelShape(2, 24, 4, 2, 6, 36, 40, 30, "f32"),  # head dim that 16-byte loads cannot take
], ids=["bf16-64", "bf16-128", "f32-16", "f32-6"])
@pytest.mark.parametrize("K", [3, 40])
def test_keys_of_an_earlier_session_are_never_seen(shape, K):
    """Token 0's embedding is NaN, so a prompt that begins with it leaves NaN keys and values in the whole workspace;
    the next session's keys are not cleared, and must be masked without entering any sum."""
    w = synth.weights(shape, gain_std=0.1)
    w[:shape.d_model] = 0x7FC0 if shape.dtype == "bf16" else np.nan
    B, P = 2, 130
    rng = np.random.default_rng(7)
    clean = rng.integers(1, shape.vocab, (B, P)).astype(np.int32)
    nan = clean.copy()
    nan[:, 0] = 0
    blk = rng.integers(max(shape.img_lo, 1), shape.img_hi, (B, K)).astype(np.int32)

    def use(model, prefix):
        sess = ssd.ssd_prefill(model, B, P, prefix, P + 2 * K, K)
        outs = [G.gpu_verify(sess, shape, blk, G.vparams(), want_h=True), G.gpu_verify(sess, shape, blk, G.vparams(commit=1))]
        outs.append(G.gpu_verify(sess, shape, blk, G.vparams(1, top_k=9, rnd=1), want_h=True))
        ssd.ssd_free_session(sess)
        return outs

    models = [ssd.ssd_init_model(G.cfg_of(shape), w) for _ in range(2)]
    want = use(models[0], clean)
    left = use(models[1], nan)
    assert np.isnan(left[0]["logits"]).all() and np.isfinite(want[0]["logits"]).all()
    got = use(models[1], clean)
    assert all(_same(a, b) for a, b in zip(got, want))
    for m in models:
        ssd.ssd_free_model(m)


def test_a_session_outlives_its_model():
    pair = G.Pair(SHAPE, gain_std=0.1, oracle=False)
    first, _ = _use(pair.model, 2, 70, 16, 1)
    second, _ = _use(pair.model, 1, 70, 9, 3)
    ssd.ssd_free_session(first)  # its workspace is kept, and freed with the model
    pair.close()
    ssd.ssd_free_session(second)


def test_threads_with_streams_of_their_own():
    """Sessions of one model created, used and freed by three threads, each on its own stream: whichever takes the
    kept workspace gets the bits of a session that shares with nobody."""
    hip = G.DeviceArray.hip()
    uses = [(2, 70, 16, 1), (1, 70, 9, 3), (3, 90, 24, 5)]
    pair = G.Pair(SHAPE, gain_std=0.1, oracle=False)
    want, wrong, streams = [], [], []
    try:
        for u in uses:
            sess, outs = _use(pair.model, *u)
            ssd.ssd_free_session(sess)
            want.append(outs)
        for _ in uses:
            s = ctypes.c_void_p()
            assert hip.hipStreamCreate(ctypes.byref(s)) == 0
            streams.append(s)

        def work(i):
            try:
                for _ in range(8):
                    sess, outs = _use(pair.model, *uses[i], stream=streams[i].value)
                    ssd.ssd_free_session(sess)
                    if not all(_same(a, b) for a, b in zip(outs, want[i])):
                        wrong.append(uses[i])
            except Exception as e:  # noqa: BLE001 (reported by the assertion below)
                wrong.append(e)

        threads = [threading.Thread(target=work, args=(i,)) for i in range(len(uses))]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not wrong
    finally:
        pair.close()
        for s in streams:
            hip.hipStreamDestroy(s)
