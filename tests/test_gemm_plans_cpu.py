"""Host-side invariants of the bf16 GEMM launch plans (no GPU: the planner is
host code inside libssd.so, called here through its C++ symbols).

Every plan, of common passes and of guided blocks, must tile its problem
exactly (feature blocks x block width cover N, splits x chunks x chunk width =
K), give the tiled kernel's pipeline a stage count it runs (a multiple of the
depth for depths 2 and 4, at least two stages for depth 3) and the few-row
kernel's eight waves a k-block each, and fit the workspaces that sessions
and draft heads size once, at creation, by planning a fixed set of row
counts: a plan for any row count must need no more split-K partials,
arrival counters or per-row x^2 parts than the largest of that set, or a
launch would write past its buffer.  Shapes: the projections of the 1B, 7B
and 8B backbones and of a draft head (m = 2d), row counts 1..4352.
"""
import pytest

import synth
from tests.plan_util import ROWS_MAX, counters, partials, plan, plan_guided, row_classes

TILE_ROWS, TILE_KT = 128, 64
PLANNERS = pytest.mark.parametrize("planner", [plan, plan_guided])


def shapes(m):
    d, D = m.d_model, m.head_dim
    mi = 2 * d
    return [((m.n_heads + 2 * m.n_kv_heads) * D, d), (d, m.n_heads * D), (2 * m.d_ff, d), (d, m.d_ff),
            (m.v_img, d), (d, 2 * d), (2 * mi, d), (d, mi)]


ROWS = sorted(set(list(range(1, 300)) + list(range(300, 4353, 37)) + [512, 1024, 2048, 4224, 4288, 4352]))


@pytest.mark.parametrize("model", [synth.M1B, synth.M7B, synth.M8B], ids=["1b", "7b", "8b"])
@PLANNERS
def test_plans_tile_their_problem(planner, model):
    for N, K in shapes(model):
        for M in ROWS:
            p = planner(M, N, K)
            where = f"M={M} N={N} K={K}"
            assert p.S >= 1 and p.n_fb >= 1, where
            if p.tile == 3:
                # 128 x 256 (or 128 x 192) tiles of eight waves: K split within 256 workgroups, >= 32 stages each
                assert M > 64, where
                assert p.NT in (3, 4) and p.bn == 64 * p.NT and p.n_fb * p.bn == N and p.WV == 8, where
                assert p.m_tiles == (M + TILE_ROWS - 1) // TILE_ROWS, where
                assert p.kchunks * p.S * TILE_KT == K and p.kchunks >= 32, where
                assert p.S == 1 or p.n_fb * p.m_tiles * p.S <= 256, where
                if p.NT == 3:
                    # only where the 256-feature grid would leave CUs idle, and never on a residual projection
                    assert N > K and p.n_fb * p.m_tiles * p.S <= 256 and not p.tail_fb, where
                    assert (N // 256) * p.m_tiles * p.S < p.n_fb * p.m_tiles * p.S, where
                if p.tail_fb:
                    # whole rounds of 256 tiles, then the remaining feature blocks K-split within one more,
                    # or as 128 x 192 tiles in one more
                    assert p.S == 1 and p.NT == 4 and 0 < p.tail_fb < p.n_fb, where
                    assert (p.tail_fb * p.m_tiles) % 256 == 0, where
                    r = (p.n_fb - p.tail_fb) * p.m_tiles
                    assert 0 < r < 256, where
                    if p.tail_nt:
                        fr = (p.n_fb - p.tail_fb) * 256
                        assert p.tail_nt == 3 and p.tail_S == 1 and N > K and fr % 192 == 0, where
                        assert r < (fr // 192) * p.m_tiles <= 256, where
                    else:
                        assert r * p.tail_S <= 256 and p.tail_S > 1, where
                        assert (K // TILE_KT) % p.tail_S == 0 and K // TILE_KT // p.tail_S >= 16, where
                else:
                    assert p.tail_S == 1 and p.tail_nt == 0, where
            elif p.tile:
                assert M > 64, where
                assert p.NT in (2, 4) and p.bn == 32 * p.NT and p.n_fb * p.bn == N, where
                assert p.m_tiles == (M + TILE_ROWS - 1) // TILE_ROWS, where
                assert p.kchunks * p.S * TILE_KT == K, where
                # depth 3 (128-feature tiles): any count of at least two stages;
                # depths 2 and 4 run whole groups of stages per trip
                if p.depth == 3:
                    assert p.NT == 4 and p.kchunks >= 2, where
                else:
                    assert p.depth in (2, 4) and p.kchunks % p.depth == 0, where
                if p.S > 1:
                    assert p.n_fb * p.m_tiles * p.S < 512, where  # splits stop once the grid fills the CUs
            else:
                # few-row kernel: eight waves share each split's k-blocks; 16 MT rows a launch
                assert p.MT in (1, 2, 3, 4, 6, 8) and 16 * p.MT >= min(M, ROWS_MAX) > 16 * (p.MT - 2), where
                assert p.NT in (1, 2, 3, 4, 6) and p.bn == 16 * p.NT, where
                assert p.n_fb * p.bn >= N > (p.n_fb - 1) * p.bn, where
                assert p.KCB * p.S * 32 == K and p.kchunks == 1 and (p.S == 1 or p.KCB >= 8), where
            if N == model.d_model:
                # the x^2 sums of a residual projection: one per row and feature block, buffers for N / 16
                assert p.n_fb <= N // 16, where


@pytest.mark.parametrize("model", [synth.M1B, synth.M7B, synth.M8B], ids=["1b", "7b", "8b"])
@PLANNERS
def test_workspace_classes_bound_every_row_count(planner, model):
    for N, K in shapes(model):
        cap_part = max(partials(planner(Mc, N, K, 0), Mc) for Mc in row_classes())
        cap_cnt = max(counters(planner(Mc, N, K, 0)) for Mc in row_classes())
        for M in ROWS:
            for xcd in (0, 8):
                p = planner(M, N, K, xcd)
                assert partials(p, M) <= cap_part, f"M={M} N={N} K={K}: split-K partials beyond the workspace"
                assert counters(p) <= cap_cnt, f"M={M} N={N} K={K}: arrival counters beyond the workspace"


def test_tiled_plan_choices():
    """The measured choices: 128 x 256 eight-wave tiles where each workgroup
    keeps at least 32 stages after the K split (at most 256 workgroups), else
    128-feature tiles (three weight stages) where they make at least 160
    workgroups, 64-feature tiles with four pipeline stages otherwise, K split
    until the grid reaches 256 workgroups; 128 x 192 eight-wave tiles where
    the 256-feature grid leaves CUs idle; the few-row
    kernel up to 64 rows, and up to 128 where the wide tiles' modelled time is not
    less; guided blocks of 65 to 128 rows keep the tiles."""
    m = synth.M8B
    gu = plan(512, 2 * m.d_ff, m.d_model)  # 112 x 4 = 448 tiles of 128 x 256: 256, then 192 as 256 of 128 x 192
    assert (gu.tile, gu.bn, gu.S, gu.tail_fb, gu.tail_nt, gu.tail_S) == (3, 256, 1, 64, 3, 1)
    lm = plan(512, m.v_img, m.d_model)  # 128 x 4 = 512
    assert (lm.tile, lm.S) == (3, 1)
    dn = plan(512, m.d_model, m.d_ff)  # 16 x 4 tiles, 224 stages in 4 splits of 56
    assert (dn.tile, dn.S, dn.kchunks) == (3, 4, 56)
    nq = (m.n_heads + 2 * m.n_kv_heads) * m.head_dim
    qkv = plan(512, nq, m.d_model)  # 32 x 4 tiles of 128 x 192 in 2 splits of 32 stages (24 x 4 x 2 of 256: 192 CUs)
    assert (qkv.tile, qkv.NT, qkv.bn, qkv.S, qkv.kchunks) == (3, 3, 192, 2, 32)
    qkv1k = plan(1024, nq, m.d_model)  # 32 x 8 tiles of 128 x 192, no split
    assert (qkv1k.tile, qkv1k.NT, qkv1k.S) == (3, 3, 1)
    o = plan(512, m.d_model, m.n_heads * m.head_dim)  # 16 x 4 x 4 splits would leave 16 stages: 128 x 128
    assert (o.tile, o.NT, o.S, o.depth) == (1, 2, 1, 4)
    gu1k = plan(1024, 2 * m.d_ff, m.d_model)  # 896 tiles: 768 in three full rounds, 128 in two splits of 32
    assert (gu1k.tile, gu1k.S, gu1k.tail_fb, gu1k.tail_S, gu1k.tail_nt) == (3, 1, 96, 2, 0)
    assert lm.tail_fb == 0 and (lm.NT, dn.NT) == (4, 4)  # two whole rounds; a residual projection
    o1 = plan(256, synth.M1B.d_model, synth.M1B.d_model)  # 32 x 2 tiles of 64 features: 4 splits
    assert (o1.tile, o1.NT, o1.S) == (1, 2, 4)
    for M in (1, 24, 48, 64):
        assert plan(M, 2 * synth.M1B.d_ff, synth.M1B.d_model).tile == 0
    for M in (96, 128):  # 8B: gate/up on the wide tiles, the output layer too beyond 96 rows
        assert plan(M, 2 * m.d_ff, m.d_model).tile == 3
        assert plan(M, m.v_img, m.d_model).tile == (3 if M > 96 else 0)
        assert plan(M, m.d_model, m.d_ff).tile == 0
        assert plan(M, 2 * synth.M1B.d_ff, synth.M1B.d_model).tile == 0
        assert plan_guided(M, 2 * synth.M1B.d_ff, synth.M1B.d_model).tile == 1
