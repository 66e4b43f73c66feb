"""bf16 passes around the edges of the few-row projections: one row, whole and
partial 16-row tiles, the last row count they take and the first of the tiled
kernels (65 rows, whose output layer over 65 16-feature tiles stays on the
few-row kernel in chunks), feature tiles that the workgroups' blocks do not
divide, K ranges that the waves share unevenly and that are split across
workgroups, and reductions fenced across XCDs.  Logits and states of a verify
round against the oracle, and the carry a prefill of the same rows leaves."""
import os

import numpy as np
import pytest

import paper_2606_20543_amd as ssd
import synth
from oracle import model as M
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

# layers, d, heads, kv heads, head dim, mlp, vocab, image codes
SHAPES = {
    "d768": synth.ModelShape(2, 768, 6, 2, 128, 1280, 1100, 1040, "bf16"),
    "d1024-k3328": synth.ModelShape(1, 1024, 16, 16, 64, 3328, 600, 528, "bf16"),  # 104 k-blocks in the down projection
    "d256": synth.ModelShape(2, 256, 4, 1, 64, 256, 300, 272, "bf16"),  # one k-block a wave
}


@pytest.fixture(scope="module", params=[(n, x) for n in SHAPES for x in ("local", "fenced")], ids="-".join)
def pair(request):
    name, xcd = request.param
    old = os.environ.get("SSD_NO_XCD_LOCAL")
    os.environ["SSD_NO_XCD_LOCAL"] = "1" if xcd == "fenced" else "0"
    try:
        p = G.Pair(SHAPES[name], gain_std=0.1)
    finally:
        if old is None:
            os.environ.pop("SSD_NO_XCD_LOCAL", None)
        else:
            os.environ["SSD_NO_XCD_LOCAL"] = old
    yield p
    p.close()


@pytest.mark.parametrize("B,K", [(1, 1), (1, 5), (1, 16), (1, 17), (2, 16), (1, 33), (3, 16), (7, 7), (1, 63), (2, 32),
                                 (5, 13), (3, 43)])
def test_verify_round_and_prefill(pair, B, K):
    shape, P = pair.shape, 21
    prefix = synth.prompt(shape, B, P).astype(np.int32)
    block = (synth.random_codes(shape, (B, K)) + shape.img_lo).astype(np.int32)
    whole = np.concatenate([prefix, block], 1)
    want, want_h = M.forward_nocache(pair.om, whole)
    sess = ssd.ssd_prefill(pair.model, B, P, prefix, P + K, K)
    try:
        out = G.gpu_verify(sess, shape, block, G.vparams(), want_h=True)
    finally:
        ssd.ssd_free_session(sess)
    assert np.abs(out["logits"] - want[:, P:]).max() < G.TOL["bf16"]
    h = want_h[:, P:]
    rms = np.sqrt((h * h).mean(-1, keepdims=True))
    assert (np.abs(out["h_pre"] - h) / rms).max() < G.H_RTOL["bf16"]
    # a prefill of K rows per sequence computes the output layer of each sequence's last row only
    pre = block if K > 1 else prefix[:, :1]
    sess = ssd.ssd_prefill(pair.model, B, K, np.ascontiguousarray(pre), K + 1, 1)
    carry = np.zeros((B, shape.v_img), np.float32)
    try:
        ssd.ssd_get_carry(sess, carry)
    finally:
        ssd.ssd_free_session(sess)
    assert np.abs(carry - M.forward_nocache(pair.om, pre)[0][:, -1]).max() < G.TOL["bf16"]
