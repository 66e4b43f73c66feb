"""Sessions that take over a freed session's workspace: the same bits as on a
model that never had another session, whatever the earlier session left in it
(larger and smaller shapes, another stream of requests, a poisoned-looking
fill), and several live sessions at once never share one."""
import numpy as np
import pytest

import paper_2606_20543_amd as ssd
import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

SHAPE = synth.ModelShape(2, 512, 8, 2, 64, 768, 640, 512, "bf16")


def _use(model, B, P, K, seed):
    prefix = synth.prompt(SHAPE, B, P, seed=seed).astype(np.int32)
    block = (synth.random_codes(SHAPE, (B, K), seed=seed) + SHAPE.img_lo).astype(np.int32)
    sess = ssd.ssd_prefill(model, B, P, prefix, P + 4 * K, K)
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
