"""The bf16 attention backward of up to 224 tokens with more pairs than the chip holds at once, so that workgroups take a second
and third one, at token counts on and beside the edges of its 32-token tiles."""
import numpy as np
import pytest

import d2ft_inputs as di
from helpers import TOL, gpu_block, oracle_block, rel_inf
from test_gpu_attn_stream import channel, crafted
from test_gpu_block import draw_block, run_case
from test_gpu_microbatch import run_mb

pytestmark = pytest.mark.gpu

FULL, FWD, SKIP = di.OP_FULL, di.OP_FWD, di.OP_SKIP


@pytest.mark.parametrize("batch,tokens,ops", [(1040, 17, [FULL, FULL, FULL]), (600, 33, [FULL, FULL, FULL]), (280, 64, [FULL, SKIP, FULL, FULL, FULL]),
                                              (130, 129, [FULL, FWD, FULL, FULL]), (90, 193, [FULL, FULL, FULL]), (170, 224, [FWD, FULL, FULL, FULL])])
def test_more_pairs_than_workgroups(batch, tokens, ops):
    import paper_2504_12471_amd as P
    w = di.Workload("attn_bwd_pairs", batch, tokens, 64, len(ops), 64, 64, 1, "bf16")
    P.d2ft_timing_enable(True)
    try:
        run_case(w, ops, seed=tokens)
        names = {r["name"] for r in P.d2ft_timing_read()}
    finally:
        P.d2ft_timing_enable(False)
    assert "attn_bwd_mfma" in names, names


def test_micro_batches_whose_slots_have_no_pair():
    """Slots are as many as the busiest micro-batch has p_f heads: workgroups skip the other images' empty ones."""
    w = di.Workload("attn_bwd_slots", 150, 193, 64, 3, 64, 64, 1, "bf16")
    run_mb(w, [[FULL, FULL, FULL], [SKIP, FWD, FULL], [FWD, SKIP, FWD]], [40, 60, 50], seed=5)


def codes(heads, full):
    """Micro-batch i: full[i] p_f heads from head i on, the others forward-only and skipped in turn."""
    return [[FULL if (h - i) % heads < n else (FWD, SKIP)[h % 2] for h in range(heads)] for i, n in enumerate(full)]


# pairs and zero blocks: uneven counts; eight positions, which divide the workgroups; more zero blocks than workgroups and a few
# pairs; workgroups that only write zeros; a last micro-batch without a pair
@pytest.mark.parametrize("tokens,heads,full,images", [(177, 12, (9, 7, 7, 7, 6), (13, 13, 13, 13, 12)), (200, 8, (8, 3, 3, 3, 0), (9, 20, 13, 13, 12)),
                                                      (33, 12, (1, 0, 0, 0, 12), (60, 64, 50, 3, 2)), (70, 5, (1, 4, 2), (3, 1, 5)),
                                                      (20, 3, (0, 3, 0), (200, 1, 180))])
def test_micro_batches_with_uneven_pairs(tokens, heads, full, images):
    w = di.Workload("attn_bwd_uneven", sum(images), tokens, 64, heads, 64, 64, 1, "bf16")
    run_mb(w, codes(heads, full), list(images), seed=tokens)


# lengths on both sides of the 32, 96 and 128 tokens, few pairs and more than two rounds of the chip
@pytest.mark.parametrize("tokens", [17, 40, 65, 128, 197])
@pytest.mark.parametrize("images", [2, 140])
def test_key_bias_gradient_shows_what_is_not_finite(tokens, images):
    w = di.Workload("nan_token", images, tokens, 128, 2, 64, 64, 1, "bf16")
    x, wt, dy = draw_block(w, 89)
    assert np.all(gpu_block(w, wt, [FULL, FULL], x, dy, ("b_qkv",))[2]["b_qkv"][1] == 0)   # a common shift of the keys changes nothing
    x[1, 3, 5] = np.nan
    assert np.isnan(gpu_block(w, wt, [FULL, FULL], x, dy, ("b_qkv",))[2]["b_qkv"]).all()


@pytest.mark.parametrize("tokens,images", [(24, 3), (64, 3), (100, 150), (197, 150)])
def test_only_the_channel_that_overflows_shows_it(tokens, images):
    """Queries of 2^127 in a channel whose keys are zero leave the scores alone, and dK = sum_q dS Q overflows in that channel."""
    w = di.Workload("overflow", images, tokens, 128, 2, 64, 64, 1, "bf16")
    x, wt, dy = draw_block(w, 90)
    for plane, bias in ((0, 2.0 ** 127), (1, 0.0)):
        wt["w_qkv"][plane, 1, 7], wt["b_qkv"][plane, 1, 7] = 0.0, bias
    b = gpu_block(w, wt, [FULL, FULL], x, dy * 2.0 ** 12, ("b_qkv",))[2]["b_qkv"]
    assert not np.isfinite(b[1, 1, 7])
    b[1, 1, 7] = 0.0
    assert np.isfinite(b).all()


def images_of(n, w, x):
    return di.Workload(w.name, n, w.tokens, 64, 1, 64, 64, 1, w.dtype, ln_eps=w.ln_eps), np.repeat(x, n, 0)


@pytest.mark.parametrize("tokens,images", [(16, 2), (32, 2), (64, 2), (64, 600), (128, 2), (128, 300)])
def test_value_bias_gradient_adds_unrounded_dv(tokens, images):
    """dV = 1 + 2^-8 in one half of the images, which bf16 rounds to 1, and -1 in the others: every step is exact in fp32."""
    w, wt, x = crafted(np.ones(tokens), "bf16", (0, 0), (0, 0), (0, 1.0), 1.0)
    w, x = images_of(images, w, x)
    dy = np.full(x.shape, -1.0, np.float32)
    dy[::2] = np.where(np.arange(tokens) % 2 == 0, 1.0, 1.0 + 2.0 ** -7)[None, :, None]
    b = gpu_block(w, wt, [FULL], x, dy, ("b_qkv",))[2]["b_qkv"]
    assert np.all(b[2] == images / 2 * tokens * 2.0 ** -8)


@pytest.mark.parametrize("tokens,images", [(24, 1), (100, 1), (100, 300), (197, 1), (197, 300)])
def test_value_bias_gradient_of_an_infinite_dv_is_infinite(tokens, images):
    """Places of keys beyond the last token have probability zero: zero times infinity is not part of the sum."""
    w, wt, x = crafted(np.ones(tokens), "bf16", (0, 0), (0, 0), (0, 0), 1.0)
    w, x = images_of(images, w, x)
    wt["w_o"][:, 7] = 2.0 ** 127   # dO of the first token overflows in one channel
    dy = np.zeros_like(x)
    dy[:, 0] = 1.0
    b = gpu_block(w, wt, [FULL], x, dy, ("b_qkv",))[2]["b_qkv"][2, 0]
    assert b[7] == np.inf and np.isfinite(np.delete(b, 7)).all()


@pytest.mark.parametrize("tokens,images", [(16, 1), (64, 1), (64, 600), (128, 300)])
def test_query_bias_gradient_of_infinite_score_gradients_is_infinite(tokens, images):
    """dP of +-2^130 overflows, O and delta are zero, and every dS * K is +infinity in one channel."""
    s = np.where(np.arange(tokens) % 2 == 0, 1.0, -1.0)
    w, wt, x = crafted(s, "bf16", (0, 0), (0, channel(1, 1.0)), (0, channel(0, 2.0 ** 100)), 1.0)
    w, x = images_of(images, w, x)
    b = gpu_block(w, wt, [FULL], x, np.full_like(x, 2.0 ** 30), ("b_qkv",))[2]["b_qkv"][0, 0]
    assert b[1] == np.inf


@pytest.mark.parametrize("tokens,images", [(17, 1), (33, 1), (33, 200), (100, 1), (100, 200), (193, 1), (197, 150)])
def test_keys_that_are_not_finite_reach_no_query_past_the_last(tokens, images):
    """A key of minus infinity under positive queries has probability zero, and its dV is zero, not NaN from places of the last tile
    that hold no query."""
    s = np.where(np.arange(tokens) == 5, -1.0, 1.0)
    w, wt, x = crafted(s, "bf16", (channel(0, 1.0), 0), (0, 0), (0.5, 1.0), 4.0, ln_eps=1e-12)
    w, x = images_of(images, w, x)
    top = float(di.round_to_bf16(np.full(1, 3.3e38, np.float32))[0])   # k of token 5: -(top + top), of the others: top - top
    wt["w_qkv"][1, 0, 0, 0] = top
    wt["b_qkv"][1, 0, 0] = -top
    dy = np.ones(x.shape, np.float32)
    y, _, g = gpu_block(w, wt, [FULL], x, dy, ("w_qkv", "b_qkv"))
    # the same without that key: its probability is zero either way
    wt["w_qkv"][1, 0, 0, 0], wt["b_qkv"][1, 0, 0] = 2.0 ** 20, -(2.0 ** 20)
    ry, _, rg, _ = oracle_block(w, wt, [FULL], x, dy)
    assert rel_inf(y, ry) < TOL["bf16"] and rel_inf(g["w_qkv"][2], rg["w_qkv"][2]) < TOL["bf16"] and rel_inf(g["b_qkv"][2], rg["b_qkv"][2]) < TOL["bf16"]
