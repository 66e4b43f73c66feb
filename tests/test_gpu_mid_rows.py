"""Passes of 65 to 128 rows: two row groups of 48 or 64 rows on the few-row
projections, their layouts (operand tiles or rows, as each reader takes them)
where a projection of the pass runs on the wide tiles instead, and the row
counts around the groups' edges.  Logits and states of a verify round and the
carry of a prefill against the oracle.  The wide shapes are there for their
plans, which the tests look up."""
import os

import numpy as np
import pytest

import paper_2606_20543_amd as ssd
import synth
from oracle import model as M
from tests import gpu_util as G
from tests.plan_util import plan

# layers, d, heads, kv heads, head dim, mlp, vocab, image codes: feature tiles that blocks do not divide and K
# ranges shared unevenly; projections on wide tiles beside few-row ones
SHAPES = {
    "d768": synth.ModelShape(2, 768, 6, 2, 128, 1280, 1100, 1040, "bf16"),
    "d2048-wide": synth.ModelShape(2, 2048, 16, 4, 128, 24576, 32768, 32768, "bf16"),
    "d4096-gate-up": synth.ModelShape(1, 4096, 16, 2, 128, 14336, 1024, 1024, "bf16"),
    "d4096-output": synth.ModelShape(1, 4096, 16, 2, 128, 1024, 32768, 32768, "bf16"),
}


def _plans(m, M):
    """(tile, feature tiles, K splits) of QKV, O, gate/up, down and the output layer of M rows."""
    d = m.d_model
    nk = [((m.n_heads + 2 * m.n_kv_heads) * m.head_dim, d), (d, m.n_heads * m.head_dim), (2 * m.d_ff, d), (d, m.d_ff),
          (m.v_img, d)]
    return [(p.tile, p.NT, p.S) for p in (plan(M, N, K) for N, K in nk)]


def test_shapes_take_the_plans_they_are_here_for():
    for M in (65, 96, 97, 128):
        assert all(p[0] == 0 for p in _plans(SHAPES["d768"], M))
        qkv, o, gu, down, lm = _plans(SHAPES["d2048-wide"], M)
        # 128 x 192 tiles above 96 rows, between few-row projections
        assert gu[:2] == ((3, 3) if M > 96 else (0, 6)) and (o[0], down[0], lm[0]) == (0, 0, 0)
        qkv, o, gu, down, lm = _plans(SHAPES["d4096-gate-up"], M)
        assert gu == (3, 4, 2) and (o[0], down[0], lm[0]) == (0, 0, 0)  # one row tile of 128 x 256, K split
        qkv, o, gu, down, lm = _plans(SHAPES["d4096-output"], M)
        assert lm == ((3, 4, 2) if M > 96 else (0, 4, 1))  # a few-row down projection writes rows for it
        assert (gu[0], down[0]) == (0, 0)


@pytest.fixture(scope="module", params=[("d768", "local"), ("d768", "fenced"), ("d2048-wide", "local"),
                                        ("d4096-gate-up", "local"), ("d4096-output", "local")], ids="-".join)
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


@pytest.mark.gpu
@pytest.mark.parametrize("B,K", [(1, 65), (5, 16), (2, 48), (1, 97), (7, 16), (1, 127), (2, 64), (3, 43)])
def test_verify_round_and_prefill(pair, B, K):
    shape, P = pair.shape, 5
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
    sess = ssd.ssd_prefill(pair.model, B, K, block, K + 1, 1)
    carry = np.zeros((B, shape.v_img), np.float32)
    try:
        ssd.ssd_get_carry(sess, carry)
    finally:
        ssd.ssd_free_session(sess)
    assert np.abs(carry - M.forward_nocache(pair.om, block)[0][:, -1]).max() < G.TOL["bf16"]
