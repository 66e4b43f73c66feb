"""Rules (B) and (C) at the edges of the sampling kernel: rows that 16-byte
loads can and cannot take, one partial 256-code group up to many, kept sets
that are listed in LDS (up to 4096 codes), too large for it, or the whole row,
boundary ties that cross waves, references with ties and masked (-inf) codes,
and a reference equal to the scoring logits.  Decisions are those of the
oracle's rule on the GPU's own logits; float64 on both sides, so they agree
unless a uniform falls within rounding of a boundary (24-bit uniforms against
sums of 1e4 terms: about 1e-9 per decision)."""
import numpy as np
import pytest

import paper_2606_20543_amd as ssd
import synth
from oracle import select as R
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def _model(v_img, ties):
    shape = synth.ModelShape(1, 32, 4, 2, 8, 48, v_img + 6, v_img, "f32")
    w = synth.weights(shape, gain_std=0.1)
    if ties > 1:  # equal output rows: equal logits
        lm = w[-shape.vocab * shape.d_model:].reshape(shape.vocab, shape.d_model)
        lm[:] = lm[np.arange(shape.vocab) // ties * ties]
    return shape, ssd.ssd_init_model(G.cfg_of(shape), w)


@pytest.mark.parametrize("v_img,ties,top_k", [
    (70, 1, 0), (70, 7, 33), (250, 3, 249), (1026, 1, 1), (4096, 64, 1000), (10002, 1, 4096), (10002, 5, 4097),
    (16384, 16, 2000), (16384, 4096, 5000), (32768, 1, 0), (32768, 32768, 100),
])
def test_sampling_matches_oracle_rule(v_img, ties, top_k):
    shape, model = _model(v_img, ties)
    B, P, K = 2, 9, 6
    try:
        sess = ssd.ssd_prefill(model, B, P, synth.prompt(shape, B, P).astype(np.int32), P + K, K)
        carry = np.zeros((B, v_img), np.float32)
        ssd.ssd_get_carry(sess, carry)
        block = synth.random_codes(shape, (B, K))
        rng = np.random.default_rng(5)
        try:
            for rnd, (rule, T) in enumerate([(R.RULE_SAMPLE, 1.0), (R.RULE_SAMPLE, 0.7), (R.RULE_ACCEPT_REJECT, 1.0),
                                             (R.RULE_ACCEPT_REJECT, 1.3), (R.RULE_ACCEPT_REJECT, 1.0)]):
                ref = None
                if rule == R.RULE_ACCEPT_REJECT:
                    ref = np.round(rng.standard_normal((B, K, v_img)) * 4).astype(np.float32) / 8 + 0.0  # many ties, no -0
                    ref[:, 1, : v_img // 3] = -np.inf
                    if rnd == 4:  # the scoring logits themselves: nothing is rejected
                        ref[:, 0], ref[:, 1:] = carry, out["logits"][:, :-1]
                prm = G.vparams(rule, top_k=top_k, T=T, rnd=rnd)
                f = np.full(B, P)
                out = G.gpu_verify(sess, shape, block + shape.img_lo, prm, ref=ref)
                refs = None if ref is None else [[ref[b, k].astype(np.float64) for k in range(K)] for b in range(B)]
                new, acc, cnt, _ = G.oracle_rule_on(out["logits"], carry, block, 0, rule, rnd, 3, f, T, top_k, refs)
                assert np.array_equal(out["tokens"] - shape.img_lo, new), (rule, T)
                assert np.array_equal(out["accept"], acc)
                assert np.array_equal(out["count"], cnt)
                if rnd == 3:
                    block = new  # same block again below, so that its logits are known beforehand
                    out = G.gpu_verify(sess, shape, block + shape.img_lo, G.vparams(R.RULE_GREEDY, rnd=9))
                elif rnd == 4:
                    assert acc.all()
        finally:
            ssd.ssd_free_session(sess)
    finally:
        ssd.ssd_free_model(model)
