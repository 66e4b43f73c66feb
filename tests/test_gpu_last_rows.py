"""Passes whose caller reads each sequence's last row alone (prefills, commits
without logits): the last layer's projections behind the attention run on those
rows only.  Carries against the oracle where the row counts cross the classes of
the projections (one to several 16-row tiles before and after the gather, more
than 64 last rows, more rows than a tiled GEMM's block), and a commit with and
without the pass's logits."""
import numpy as np
import pytest

import paper_2606_20543_amd as ssd
import synth
from oracle import model as M
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

SHAPE = synth.ModelShape(2, 512, 8, 2, 64, 768, 640, 512, "bf16")


@pytest.fixture(scope="module")
def pair():
    p = G.Pair(SHAPE, gain_std=0.1)
    yield p
    p.close()


@pytest.mark.parametrize("B,P", [(1, 16), (1, 17), (8, 2), (9, 3), (17, 2), (5, 27), (2, 64), (65, 2), (100, 3), (1, 200)])
def test_prefill_carry(pair, B, P):
    prefix = synth.prompt(SHAPE, B, P).astype(np.int32)
    sess = ssd.ssd_prefill(pair.model, B, P, prefix, P + 1, 1)
    carry = np.zeros((B, SHAPE.v_img), np.float32)
    try:
        ssd.ssd_get_carry(sess, carry)
    finally:
        ssd.ssd_free_session(sess)
    assert np.abs(carry - M.forward_nocache(pair.om, prefix)[0][:, -1]).max() < G.TOL["bf16"]


@pytest.mark.parametrize("B,K", [(1, 24), (3, 11), (6, 32)])
def test_commit_with_and_without_logits(pair, B, K):
    P = 19
    prefix = synth.prompt(SHAPE, B, P).astype(np.int32)
    block = (synth.random_codes(SHAPE, (B, K)) + SHAPE.img_lo).astype(np.int32)
    want = M.forward_nocache(pair.om, np.concatenate([prefix, block], 1))[0]
    prm = ssd.ssd_verify_params()
    prm.rule, prm.temperature, prm.commit = ssd.SSD_GREEDY, 1.0, 1
    for logits in (None, np.zeros((B, K, SHAPE.v_img), np.float32)):
        sess = ssd.ssd_prefill(pair.model, B, P, prefix, P + 2 * K, K)
        try:
            ssd.ssd_verify_step(sess, K, block.copy(), prm, logits_out=logits)
            carry = np.zeros((B, SHAPE.v_img), np.float32)
            ssd.ssd_get_carry(sess, carry)
            # the committed keys and values serve the next block
            again = np.zeros((B, 1, SHAPE.v_img), np.float32)
            nxt = ssd.ssd_verify_params()
            nxt.rule, nxt.temperature = ssd.SSD_GREEDY, 1.0
            ssd.ssd_verify_step(sess, 1, block[:, :1].copy(), nxt, logits_out=again)
        finally:
            ssd.ssd_free_session(sess)
        assert np.abs(carry - want[:, -1]).max() < G.TOL["bf16"]
        whole = np.concatenate([prefix, block, block[:, :1]], 1)
        assert np.abs(again[:, 0] - M.forward_nocache(pair.om, whole)[0][:, -1]).max() < G.TOL["bf16"]
