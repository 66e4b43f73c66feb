"""fp32 models at the edges of the matrix-core GEMM tiles (16 features x 16 or
64 tokens, 16-input chunks over four waves), of the attention's 64-key rounds
and four-query workgroups, and of the rule that keeps widths 16-byte loads
cannot take on the scalar kernels: verify rounds against the oracle, and the
same block token by token, whose bits must not depend on the block."""
import numpy as np
import pytest

import paper_2606_20543_amd as ssd
import synth
from oracle import model as M
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

SHAPES = {
    # layers, d, heads, kv heads, head dim, mlp, vocab, image codes
    "d32": synth.ModelShape(2, 32, 4, 2, 8, 48, 40, 32, "f32"),
    "d100-gqa5": synth.ModelShape(2, 100, 5, 1, 20, 52, 96, 70, "f32"),  # partial chunks and feature blocks
    "d30-scalar": synth.ModelShape(2, 30, 3, 1, 10, 37, 40, 34, "f32"),  # rows of two floats past 16 bytes
    "d256-16h": synth.ModelShape(1, 256, 16, 4, 64, 100, 128, 128, "f32"),
}


@pytest.mark.parametrize("name,B,P,K", [
    ("d32", 1, 1, 1), ("d32", 3, 61, 5), ("d100-gqa5", 2, 64, 17), ("d100-gqa5", 5, 3, 13), ("d30-scalar", 2, 70, 9),
    ("d256-16h", 8, 20, 33),  # 4224 queries: four a workgroup, the last one of a block alone
    ("d256-16h", 8, 120, 31),  # 3968: one a workgroup
])
def test_verify_round_matches_oracle(name, B, P, K):
    shape = SHAPES[name]
    pair = G.Pair(shape, gain_std=0.1)
    try:
        prefix = synth.prompt(shape, B, P).astype(np.int32)
        block = (synth.random_codes(shape, (B, K)) + shape.img_lo).astype(np.int32)
        sess = ssd.ssd_prefill(pair.model, B, P, prefix, P + K, K)
        try:
            out = G.gpu_verify(sess, shape, block, G.vparams(), want_h=True)
            # token by token (commits of one position each)
            one = np.zeros((B, K, shape.v_img), np.float32)
            for k in range(K):
                lg = np.zeros((B, 1, shape.v_img), np.float32)
                ssd.ssd_verify_step(sess, 1, np.ascontiguousarray(block[:, k:k + 1]), G.vparams(commit=1),
                                    logits_out=lg)
                one[:, k] = lg[:, 0]
        finally:
            ssd.ssd_free_session(sess)
        want = M.forward_nocache(pair.om, np.concatenate([prefix, block], 1))[0][:, P:]
        assert np.abs(out["logits"] - want).max() < G.TOL["f32"]
        assert np.array_equal(out["logits"], one)
    finally:
        pair.close()
