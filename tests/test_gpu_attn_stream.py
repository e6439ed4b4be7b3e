"""GPU parity of the streaming attention kernels (kernels_attn_stream.hip) through one block forward + backward: token
counts at and beside the edges of tiles, stages and workgroups, the smallest and the largest."""
import numpy as np
import pytest

import d2ft_inputs as di
from helpers import TOL, gpu_block, oracle_block, rel_inf
from test_gpu_block import draw_block, run_case
from test_gpu_ln_product import kernels_of

pytestmark = pytest.mark.gpu

FULL, FWD, SKIP = di.OP_FULL, di.OP_FWD, di.OP_SKIP


@pytest.mark.parametrize("tokens", [1, 31, 32, 33, 64, 127, 128, 129, 257])
def test_fp32_token_edges(tokens):
    run_case(di.Workload("stream_f32", 2, tokens, 128, 3, 64, 64, 1, "f32"), [FULL, FWD, FULL], seed=81)


@pytest.mark.parametrize("tokens", [17, 32, 33, 96, 97])   # with 130 pairs: the fp32 instruction up to 64 tokens, parts beyond
def test_fp32_many_pairs(tokens):
    names = kernels_of(lambda: run_case(di.Workload("stream_f32_many", 65, tokens, 128, 2, 64, 64, 1, "f32"), [FULL, FULL], seed=86))
    assert names >= fp32_kernels(tokens > 64), names


def fp32_kernels(parts):
    return {"attn_fwd_stream_kernel<float%s>" % (", Parts" if parts else ""), "attn_bwd_stream_kernel<float, 1%s>" % (", Parts" if parts else "")}


@pytest.mark.parametrize("tokens,images,parts", [(32, 1, False), (33, 64, True), (33, 65, False), (64, 65, False), (65, 384, True),
                                                 (65, 385, False), (96, 385, False), (97, 768, True), (97, 769, False),
                                                 (128, 769, False), (129, 769, True)])
def test_which_products_fp32_attention_takes(tokens, images, parts):
    """Two p_f heads and one p_o head per image; forward and backward take the same."""
    w = di.Workload("which_f32", images, tokens, 64, 3, 64, 64, 1, "f32")
    names = kernels_of(lambda: run_case(w, [FULL, FWD, FULL], seed=96))
    assert names >= fp32_kernels(parts) and not names & fp32_kernels(not parts), names


@pytest.mark.parametrize("tokens", [33, 64, 65])
def test_fp32_forward_alone(tokens):
    """Without p_f heads, 576 pairs: the fp32 instruction up to 64 tokens."""
    names = kernels_of(lambda: run_case(di.Workload("stream_f32_forward", 144, tokens, 64, 4, 64, 64, 1, "f32"), [FWD] * 4, seed=95))
    assert "attn_fwd_stream_kernel<float%s>" % (", Parts" if tokens == 65 else "") in names, names


@pytest.mark.parametrize("tokens", [225, 256, 257, 289, 320, 577])
def test_bf16_token_edges(tokens):
    run_case(di.Workload("stream_bf16", 2, tokens, 128, 3, 64, 64, 1, "bf16"), [FWD, FULL, FULL], seed=82)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_most_tokens(dtype):
    run_case(di.Workload("stream_max", 1, 1024, 64, 2, 64, 64, 1, dtype), [FULL, FWD], seed=83)


@pytest.mark.parametrize("tokens", [17, 64, 65, 128, 129, 197, 224])
def test_bf16_few_pairs_below_225_tokens(tokens):
    run_case(di.Workload("stream_few", 3, tokens, 128, 3, 64, 64, 1, "bf16"), [FULL, FWD, FULL], seed=84)


# ---------------------------------------------------------------------------
# crafted scores: one head, tokens x = s * e with e = (+1, -1, ..) and s = +-1, so that LayerNorm gives exactly x
# ---------------------------------------------------------------------------
E = np.where(np.arange(64) % 2 == 0, 1.0, -1.0).astype(np.float32)


def crafted(s, dtype, q, k, v, w_o, ln_eps=1e-6):
    """Workload, weights and x of one image of len(s) tokens.  q, k, v: (constant, coefficient of s) per channel [64]."""
    T = len(s)
    w = di.Workload("crafted", 1, T, 64, 1, 64, 64, 1, dtype, ln_eps=ln_eps)
    z = lambda *sh: np.zeros(sh, np.float32)
    w_qkv, b_qkv = z(3, 1, 64, 64), z(3, 1, 64)
    for p, (const, coef) in enumerate((q, k, v)):
        b_qkv[p, 0] = const
        w_qkv[p, 0] = (np.broadcast_to(np.asarray(coef, np.float32), 64) / 64)[:, None] * E[None, :]
    wt = {"ln1_g": z(64) + 1, "ln1_b": z(64), "w_qkv": w_qkv, "b_qkv": b_qkv, "w_o": np.eye(64, dtype=np.float32) * np.float32(w_o),
          "b_o": z(64), "ln2_g": z(64) + 1, "ln2_b": z(64), "w1": z(64, 64), "b1": z(64), "w2": z(64, 64), "b2": z(64)}
    x = (np.asarray(s, np.float32)[:, None] * E[None, :])[None]
    return w, wt, x


def channel(c, value):
    a = np.zeros(64, np.float32)
    a[c] = value
    return a


@pytest.mark.parametrize("tokens", [258, 288, 578])
def test_bf16_probabilities_keep_their_bits(tokens):
    """Two kinds of keys whose probabilities differ by 2^-10 of themselves, less than bf16 resolves, and values that
    cancel: O and dV are that difference alone."""
    s = np.where(np.arange(tokens) % 2 == 0, 1.0, -1.0)
    a = channel(0, 2.0 ** -4)
    w, wt, x = crafted(s, "bf16", (0, a), (0, a), (0, 1.0), 2.0 ** 14)
    dy = (s[:, None] * np.full((1, 64), 2.0 ** -14))[None].astype(np.float32)
    y, _, g = gpu_block(w, wt, [FULL], x, dy, ("w_qkv",))
    ry, _, rg, _ = oracle_block(w, wt, [FULL], x, dy)
    # O and dV are rounded to bf16 once (2^-9), the weight gradient again
    assert rel_inf(y, ry) < 1e-2 and rel_inf(g["w_qkv"][2], rg["w_qkv"][2]) < 1e-2


def test_bf16_score_gradients_keep_their_bits():
    """Equal probabilities and score gradients of two sizes whose sum is zero, multiplied with 128 +- 1: rounded to bf16
    they leave a rest of 2.5 % of the result."""
    s = np.where(np.arange(288) % 6 == 0, 1.0, -1.0)
    w, wt, x = crafted(s, "bf16", (channel(0, 128), channel(0, 1)), (channel(1, 128), channel(1, 1)), (2.0, 3.0), 1.0)
    dy = ((2 + 3 * s)[:, None] * np.ones((1, 64)))[None].astype(np.float32)
    _, _, g = gpu_block(w, wt, [FULL], x, dy, ("w_qkv",))
    rg = oracle_block(w, wt, [FULL], x, dy)[2]
    for p in (0, 1):
        assert rel_inf(g["w_qkv"][p], rg["w_qkv"][p]) < 1e-2


def test_fp32_probability_of_a_single_key_is_one():
    """Scores of some 1e5: in one multiply-add with a rounded log-sum-exp the exponent would be off by 1e-2."""
    rng = np.random.default_rng(85)
    w = di.Workload("one_key", 8, 1, 64, 1, 64, 64, 1, "f32")
    _, wt, _ = crafted([1.0], "f32", (rng.standard_normal(64) * 600, 1.0), (rng.standard_normal(64) * 600, 1.0), (0, 1.0), 1.0)
    x = rng.standard_normal((8, 1, 64)).astype(np.float32)
    dy = rng.standard_normal((8, 1, 64)).astype(np.float32)
    _, _, g = gpu_block(w, wt, [FULL], x, dy, ("w_qkv",))
    rg = oracle_block(w, wt, [FULL], x, dy)[2]
    assert rel_inf(g["w_qkv"][2], rg["w_qkv"][2]) < 1e-5   # sums of eight fp32 products


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("slope", [0.4, -0.4])
@pytest.mark.parametrize("tokens", [100, 577])
def test_maximum_in_every_stage(dtype, slope, tokens):
    """Scores that rise (or fall) by slope / 8 per token: the running maximum moves in every stage, or never."""
    rng = np.random.default_rng(86)
    n = np.arange(tokens)
    bits = np.where((n[:, None] >> np.arange(10)) & 1, 1.0, -1.0)
    x = np.concatenate([bits, -bits, np.broadcast_to(E[:44], (tokens, 44))], 1).astype(np.float32)[None]   # LayerNorm gives x
    w, wt, _ = crafted([1.0] * tokens, dtype, (0, 0), (0, 0), (0, 0), 4.0)
    half = 2.0 ** np.arange(10) / 2                       # key channel b: bit b of the position, times 2^b
    wt["b_qkv"][0, 0, :10] = di.round_to_bf16(np.full(1, slope, np.float32)) if dtype == "bf16" else slope
    wt["b_qkv"][1, 0, :10] = half
    wt["w_qkv"][1, 0, np.arange(10), np.arange(10)] = half
    wt["w_qkv"][2, 0] = np.sign(rng.standard_normal((64, 64))) / 8
    dy = np.sign(rng.standard_normal(x.shape)).astype(np.float32)
    fields = ("w_qkv", "w_o")
    y, dx, g = gpu_block(w, wt, [FULL], x, dy, fields)
    ry, rdx, rg, _ = oracle_block(w, wt, [FULL], x, dy)
    errs = {"y": rel_inf(y, ry), "dx": rel_inf(dx, rdx), "w_o": rel_inf(g["w_o"], rg["w_o"])}
    # With bf16 storage the sum of a query's score gradients is not zero but the rounding of its O, up to 2^-9, and keys of up
    # to 512 multiply it: dW_q may be off by 2^-9 * 512 of a score gradient whatever the kernel.  The other planes are not.
    for p in (0, 1, 2) if dtype == "f32" else (1, 2):
        errs[p] = rel_inf(g["w_qkv"][p], rg["w_qkv"][p])
    assert max(errs.values()) <= TOL[dtype], errs


@pytest.mark.parametrize("dtype,tokens", [("f32", 33), ("f32", 100), ("f32", 193), ("bf16", 300)])
def test_scores_that_overflow_to_minus_infinity(dtype, tokens):
    """Keys whose scores are below fp32's range have no part in the softmax, wherever they stand: here one query's first
    and last keys, whole tiles and stages of them."""
    n = np.arange(tokens)
    s = np.where((n < min(70, tokens // 2)) | (n > tokens - 4), -1.0, 1.0)
    big = 2.0 ** 66
    # q = 2^66, k = 0 or -2^66 in the same channel; LayerNorm's epsilon is small enough for k to be exactly 0
    w, wt, x = crafted(s, dtype, (channel(0, big), 0), (channel(0, -big / 2), channel(0, big / 2)), (0.5, 1.0), 4.0, ln_eps=1e-12)
    dy = ((2 + s)[:, None] * np.ones((1, 64)))[None].astype(np.float32)
    y, _, g = gpu_block(w, wt, [FULL], x, dy, ("w_qkv",))
    ry, _, rg, _ = oracle_block(w, wt, [FULL], x, dy)
    assert rel_inf(y, ry) < TOL[dtype] and rel_inf(g["w_qkv"][2], rg["w_qkv"][2]) < TOL[dtype]


@pytest.mark.parametrize("dtype,tokens", [("f32", 33), ("f32", 197), ("bf16", 300)])
def test_keys_that_are_not_finite_reach_no_query_past_the_last(dtype, tokens):
    """A key of minus infinity under positive queries has probability zero, and its dV is zero, not NaN from 0 * infinity
    with the empty rows of the last tile."""
    s = np.where(np.arange(tokens) == 5, -1.0, 1.0)
    w, wt, x = crafted(s, dtype, (channel(0, 1.0), 0), (0, 0), (0.5, 1.0), 4.0, ln_eps=1e-12)
    # k of token 5: -(max + max), of the others: max - max
    top = float(np.float32(3.4e38) if dtype == "f32" else di.round_to_bf16(np.full(1, 3.3e38, np.float32))[0])
    wt["w_qkv"][1, 0, 0, 0] = top
    wt["b_qkv"][1, 0, 0] = -top
    dy = np.ones(x.shape, np.float32)
    y, _, g = gpu_block(w, wt, [FULL], x, dy, ("w_qkv",))
    # the same without that key: its probability is zero either way
    wt["w_qkv"][1, 0, 0, 0], wt["b_qkv"][1, 0, 0] = 2.0 ** 20, -(2.0 ** 20)
    ry, _, rg, _ = oracle_block(w, wt, [FULL], x, dy)
    assert rel_inf(y, ry) < TOL[dtype] and rel_inf(g["w_qkv"][2], rg["w_qkv"][2]) < TOL[dtype]


@pytest.mark.parametrize("dtype,tokens", [("f32", 65), ("f32", 197), ("bf16", 300)])
def test_key_bias_gradient_shows_what_is_not_finite(dtype, tokens):
    w = di.Workload("nan_token", 2, tokens, 128, 2, 64, 64, 1, dtype)
    x, wt, dy = draw_block(w, 87)
    clean = gpu_block(w, wt, [FULL, FULL], x, dy, ("b_qkv",))[2]["b_qkv"]
    assert np.all(clean[1] == 0)   # a common shift of the keys changes nothing
    x[1, 3, 5] = np.nan
    b = gpu_block(w, wt, [FULL, FULL], x, dy, ("b_qkv",))[2]["b_qkv"]
    assert np.isnan(b).all()


@pytest.mark.parametrize("tokens,images,stream", [(129, 1, True), (129, 24, True), (129, 25, False), (129, 33, False), (224, 24, True),
                                                  (224, 25, False), (128, 1, False), (128, 33, False), (96, 40, False), (64, 64, False),
                                                  (49, 129, False), (33, 3, False)])
def test_which_kernel_runs_the_bf16_backward(tokens, images, stream):
    """Four heads per image, on both sides of the 128 tokens and 96 pairs up to which the streamed kernel is the faster one: the times
    of both kernels at these sizes are beside attn_bwd_stream_faster."""
    import paper_2504_12471_amd as P
    w = di.Workload("which", images, tokens, 64, 4, 64, 64, 1, "bf16")
    P.d2ft_timing_enable(True)
    try:
        run_case(w, [FULL] * 4, seed=88)
        names = {r["name"] for r in P.d2ft_timing_read()}
    finally:
        P.d2ft_timing_enable(False)
    assert ("attn_bwd_stream" in names) == stream and ("attn_bwd_mfma" in names) == (not stream), names


@pytest.mark.parametrize("tokens", [65, 197])
def test_fp32_values_without_bf16_parts(tokens):
    """A value channel of 2^105 has no bf16 parts: its workgroups form their rows again with the fp32 instruction, and
    everything else comes out as it does without it.  The channel's rows of W_o bring it back to ordinary size."""
    w = di.Workload("no_parts", 2, tokens, 128, 2, 64, 64, 1, "f32")
    x, wt, dy = draw_block(w, 92)
    wt["b_qkv"][2, 1, 7] = np.float32(2.0 ** 105)
    wt["w_o"][:, 64 + 7] *= np.float32(2.0 ** -105)
    fields = ("w_qkv", "b_qkv", "w_o")
    out = []
    names = kernels_of(lambda: out.extend(gpu_block(w, wt, [FULL, FULL], x, dy, fields)))
    assert names >= fp32_kernels(parts=True), names
    y, dx, g = out
    ry, rdx, rg, _ = oracle_block(w, wt, [FULL, FULL], x, dy)
    assert rel_inf(y, ry) < TOL["f32"] and rel_inf(dx, rdx) < TOL["f32"]
    for k in ("w_qkv", "b_qkv"):
        for p in range(3):
            # the key bias gradient is what rounding leaves of zero
            assert rel_inf(g[k][p], rg[k][p]) < TOL["f32"] or (k, p) == ("b_qkv", 1), (k, p)
    keep = [c for c in range(128) if c != 64 + 7]
    assert rel_inf(g["w_o"][:, keep], rg["w_o"][:, keep]) < TOL["f32"]
    assert rel_inf(g["w_o"][:, 64 + 7], rg["w_o"][:, 64 + 7]) < TOL["f32"]


# ---------------------------------------------------------------------------
# fp32 by bf16 parts: scores whose sums in parts leave fp32's range, and scores that forward and backward must round alike
# ---------------------------------------------------------------------------
def positions(tokens):
    """x of one image whose first ten channels are the bits of the position (+-1), which LayerNorm returns as they are."""
    n = np.arange(tokens)
    bits = np.where((n[:, None] >> np.arange(10)) & 1, 1.0, -1.0)
    return np.concatenate([bits, -bits, np.broadcast_to(E[:44], (tokens, 44))], 1).astype(np.float32)[None]


def check_values(w, wt, x, dy):
    """y and what reaches the values; the other gradients are what rounding leaves of zero, times the scores' size."""
    out = []
    names = kernels_of(lambda: out.extend(gpu_block(w, wt, [FULL], x, dy, ("w_qkv", "b_qkv", "w_o"))))
    assert names >= fp32_kernels(parts=True), names
    y, _, g = out
    ry, _, rg, _ = oracle_block(w, wt, [FULL], x, dy)
    errs = {"y": rel_inf(y, ry), "w_o": rel_inf(g["w_o"], rg["w_o"])}
    errs.update({k: rel_inf(g[k][2], rg[k][2]) for k in ("w_qkv", "b_qkv")})
    print(errs, flush=True)
    assert max(errs.values()) < TOL["f32"], errs


@pytest.mark.parametrize("tokens", [33, 65, 197])
@pytest.mark.parametrize("first,unit,q", [
    (1, -2.0 ** 90, 2.0 ** 45),         # every score of every query below -2^80, the largest at the first key
    (1024, 2.0 ** 90, 2.0 ** 45),       # .. at the last
    (383, 2.0 ** 72 * 1.00167, 2.0 ** 36 * 1.0011),   # of 197 keys the first 128 below -2^80, the largest above it, at the last
])
def test_fp32_scores_below_the_range_of_parts(tokens, first, unit, q):
    """Score n is -first * |unit| + n * unit: the softmax is one key's, whose values get the whole gradient."""
    rng = np.random.default_rng(93)
    w, wt, _ = crafted([1.0] * tokens, "f32", (0, 0), (0, 0), (0, 0), 1.0, ln_eps=1e-30)
    x = positions(tokens)
    q = np.float32(q)
    k = np.float32(abs(unit) / float(q))
    wt["b_qkv"][0, 0, :11] = q
    half = np.float32(np.sign(unit)) * k * (2.0 ** np.arange(10) / 2).astype(np.float32)   # key channel b: bit b, times 2^b
    wt["b_qkv"][1, 0, :10] = half
    wt["w_qkv"][1, 0, np.arange(10), np.arange(10)] = half
    wt["b_qkv"][1, 0, 10] = -first * k
    wt["w_qkv"][2, 0] = np.sign(rng.standard_normal((64, 64))) / 8
    check_values(w, wt, x, np.sign(rng.standard_normal(x.shape)).astype(np.float32))


@pytest.mark.parametrize("tokens", [33, 65, 197])
def test_fp32_partial_sums_below_the_range_of_parts(tokens):
    """Scores of zero as -3 * 2^79 over the first 16 channels and 2^79 in each of three later ones, beside keys of -1.  (1 + eps
    is 1 for the oracle too, or its scores would be what rounding leaves of 2^79.)"""
    s = np.where(np.arange(tokens) % 3 == 0, 1.0, -1.0)
    big = np.zeros(64)
    big[:16] = -3 * 2.0 ** 36
    big[[16, 32, 48]] = 2.0 ** 40
    w, wt, x = crafted(s, "f32", (np.where(big != 0, 2.0 ** 39, 0) + channel(63, 1.0), 0),
                       (big / 2 - channel(63, 4.0), big / 2 + channel(63, 4.0)), (0.5, 1.0), 4.0, ln_eps=1e-30)
    check_values(w, wt, x, ((2 + s)[:, None] * np.ones((1, 64)))[None].astype(np.float32))


@pytest.mark.parametrize("heads,tokens,size,seed", [   # 64 pairs per head; sizes of 10 and 110: scores of some 800 and 1e5
    (1, 33, 10.0, 94), (1, 130, 10.0, 94), (8, 33, 10.0, 94), (8, 33, 110.0, 94), (8, 64, 10.0, 94), (8, 65, 10.0, 94), (8, 130, 110.0, 94),
    (13, 96, 10.0, 94), (13, 97, 110.0, 94),
    (8, 97, 10.0, 3), (8, 97, 10.0, 25),   # one of the 512 scores has other bits if the products of parts are added in another order
])
def test_fp32_probability_of_one_key_among_many_is_one(heads, tokens, size, seed):
    """Each query has a single key, whose probability is one if the backward forms its score with the forward's bits: a unit
    in the last place of a score of 800 is 6e-5 of it.  Image c has its gradient in channel c of each head."""
    rng = np.random.default_rng(seed)
    D = 64 * heads
    w = di.Workload("one_of_many", 64, tokens, D, heads, 64, 64, 1, "f32", ln_eps=1e-30)
    z = lambda *sh: np.zeros(sh, np.float32)
    wt = {"ln1_g": z(D) + 1, "ln1_b": z(D), "w_qkv": z(3, heads, 64, D), "b_qkv": z(3, heads, 64), "w_o": np.eye(D, dtype=np.float32),
          "b_o": z(D), "ln2_g": z(D) + 1, "ln2_b": z(D), "w1": z(64, D), "b1": z(64), "w2": z(D, 64), "b2": z(D)}
    code = np.where(rng.random((64, D // 2)) < 0.5, -1.0, 1.0)
    code = np.concatenate([code, -code], 1)                     # mean 0, variance 1: LayerNorm gives x itself
    x = np.repeat(-code[:, None, :], tokens, 1)
    x[:, tokens // 2] = code                                    # one key unlike the others
    x = x.astype(np.float32)
    for h in range(heads):
        wt["b_qkv"][0, h] = rng.uniform(0.5, 1.0, 64) * size
        # key channels: a part that all images share in sign, through a channel of x that is +1 in token `tokens // 2`
        wt["w_qkv"][1, h] = rng.standard_normal((64, D)) * (0.05 * size / np.sqrt(D))
    x[:, :, 0], x[:, :, D // 2] = -1.0, 1.0
    x[:, tokens // 2, 0], x[:, tokens // 2, D // 2] = 1.0, -1.0
    wt["w_qkv"][1, :, :, 0] += rng.uniform(0.8, 1.6, (heads, 64)).astype(np.float32) * np.float32(size)
    dy = z(64, tokens, D)
    for h in range(heads):
        dy[np.arange(64), :, 64 * h + np.arange(64)] = 1.0
    g = gpu_block(w, wt, [FULL] * heads, x, dy, ("w_qkv",))[2]["w_qkv"][2]     # [heads][channel = image][D]
    err = np.abs(g / (tokens * x[:, tokens // 2][None]) - 1).max(-1)
    print("off by more than 1e-5:", int((err > 1e-5).sum()), "of", err.size, "largest", err.max(), flush=True)
    assert err.max() < 1e-5   # sums of up to 130 fp32 products that are all one
