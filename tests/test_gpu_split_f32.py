"""GPU parity of the fp32 products by bf16 parts (kernels_gemm_split.hip) where its tiling can go wrong, their error
against fp64, and operands that have no parts: infinities, NaN and values that round up to infinity."""
import contextlib

import numpy as np
import pytest

import d2ft_inputs as di
from helpers import FLAG_GATE_FFN, TOL, gpu_block, oracle_block, rel_inf
from test_gpu_block import draw_block, run_case
from test_gpu_ffn_gate import run_gated

pytestmark = pytest.mark.gpu

FULL, FWD, SKIP = di.OP_FULL, di.OP_FWD, di.OP_SKIP

# the kernel's three forms: both operands with K contiguous, B with K strided, the grouped weight gradients
ROWS, B_COL, GROUPED = "<false, false, d2ft::GemmArgs>", "<false, true, d2ft::GemmArgs>", "<true, true, d2ft::Tile64Grouped>"


@contextlib.contextmanager
def runs(*forms):
    """the calls inside launch these forms of the split kernel: which kernel runs is a matter of a fitted cost"""
    import paper_2504_12471_amd as P
    P.d2ft_timing_enable(True)
    try:
        yield
        records = P.d2ft_timing_read()
    finally:
        P.d2ft_timing_enable(False)
    names = {r["name"] for r in records}
    print([(r["name"], r["launches"], r["flops"]) for r in records if "gemm" in r["name"]], flush=True)
    assert {"gemm_split_kernel" + f for f in forms} <= names, names


@pytest.mark.parametrize("batch,tokens,width,heads,mlp", [
    (16, 193, 328, 5, 1288),   # rows, columns and K beside the edges of 128, 64 and 32; column sums of a short band
    (30, 128, 384, 6, 1536),   # whole tiles; weight gradients in several splits of K
])
def test_block_at_tile_edges(batch, tokens, width, heads, mlp):
    w = di.Workload("split_f32", batch, tokens, width, heads, 64, mlp, 1, "f32")
    with runs(ROWS, B_COL, GROUPED):
        run_case(w, [FULL, FWD, FULL, SKIP, FULL, FULL][-heads:], seed=81)


def test_gated_slices_through_the_remaps():
    w = di.Workload("split_gate_f32", 20, 197, 384, 6, 64, 1536, 1, "f32")
    with runs(ROWS, B_COL, GROUPED):
        run_gated(w, [FULL, SKIP, FWD, FULL, FULL, SKIP], seed=82)


def test_operands_without_parts_through_remaps_and_splits():
    """Operands of 2^105 have no parts: what meets them is formed again with the fp32 instruction, in every form of the
    kernel.  Their partners are zero, or their results are left out below, so that everything compared is of ordinary size."""
    big = np.float32(2.0 ** 105)
    w = di.Workload("redo", 40, 197, 384, 6, 64, 1536, 1, "f32")
    ops = [FULL, SKIP, FWD, FULL, FULL, FULL]
    x, wt, dy = draw_block(w, 85)
    # columns 37 and 301 of w_qkv (read through a remap of its rows forward, of its K backward) times u = 0, and du times 0
    wt["ln1_g"][[37, 301]] = wt["ln1_b"][[37, 301]] = 0
    wt["w_qkv"][..., [37, 301]] = big
    # column 70 of w1 likewise: FC1 and dv
    wt["ln2_g"][70] = wt["ln2_b"][70] = 0
    wt["w1"][:, 70] = big
    # row 90 of w2 times dy = 0 in dz; FC2's column 90 is of its size
    wt["w2"][90, :] = big
    dy[:, :, 90] = 0
    # one element of dy, column 200: weight gradients' row 200, dx's element; its products with w2 and w_o are 0
    wt["w2"][200, :] = 0
    wt["w_o"][200, :] = 0
    dy[7, 11, 200] = big
    fields = ("w_qkv", "b_qkv", "w_o", "w1", "b1", "w2")
    with runs(ROWS, B_COL, GROUPED):
        y, dx, g = gpu_block(w, wt, ops, x, dy, fields, FLAG_GATE_FFN)
    ry, rdx, rg, _ = oracle_block(w, wt, ops, x, dy, gate_ffn=True)
    assert rel_inf(y[..., 90], ry[..., 90]) < TOL["f32"]
    for a in (y, ry): a[..., 90] = 0
    for a in (dx, rdx): a[7, 11, 200] = 0
    for k in ("w2", "w_o"):
        assert rel_inf(g[k][200], rg[k][200]) < TOL["f32"], k
        for a in (g[k], rg[k]): a[200] = 0
    errs = {"y": rel_inf(y, ry), "dx": rel_inf(dx, rdx), **{k: rel_inf(g[k], rg[k]) for k in fields}}
    print(errs, flush=True)
    assert max(errs.values()) < TOL["f32"], errs


def patch_embed(images, w_pe):
    """tokens of images through d2ft_patch_embed_fwd with zero bias, class token and positions"""
    import torch
    import paper_2504_12471_amd as P
    B, C, H, _ = images.shape
    D, np_ = w_pe.shape[0], (H // 16) ** 2
    d = P.EmbedDesc(B, C, H, H, 16, D, P.F32, 0)
    t = lambda a: torch.from_numpy(a).cuda()
    z = lambda *s: torch.zeros(s, device="cuda")
    tokens = z(B, np_ + 1, D)
    saved = torch.empty(P.d2ft_embed_saved_bytes(d), dtype=torch.uint8, device="cuda")
    scratch = torch.empty(P.d2ft_embed_scratch_bytes(d), dtype=torch.uint8, device="cuda")
    P.d2ft_patch_embed_fwd(d, t(images), t(w_pe), z(D), z(D), z(np_ + 1, D), tokens, saved, scratch)
    return tokens[:, 1:].cpu().numpy().reshape(B * np_, D)


def patches(images):
    B, C, H, _ = images.shape
    g = H // 16
    return images.reshape(B, C, g, 16, g, 16).transpose(0, 2, 4, 1, 3, 5).reshape(B * g * g, C * 256)


def test_error_against_fp64_and_operands_without_parts():
    rng = np.random.default_rng(83)
    images = rng.standard_normal((32, 3, 224, 224)).astype(np.float32)
    w = rng.standard_normal((384, 768)).astype(np.float32)
    images[3, 0, 40, 50] = np.inf            # one infinity in a row: the sign of the weight decides
    images[5, 1, 0, 0] = np.inf              # two in a row: NaN where their signs differ
    images[5, 2, 0, 0] = np.inf
    images[7, 2, 100, 100] = np.nan
    images[9, 0, 16, 16] = 3.4e38            # its first part rounds up to infinity
    w[11, 0] = 1e-3
    p = patches(images)
    row = 9 * 196 + 15                       # patch (1, 1): pixel (16, 16) is its first
    assert p[row, 0] == np.float32(3.4e38)
    with runs(ROWS):
        got = patch_embed(images, w)
    with np.errstate(invalid="ignore", over="ignore"):
        ref64 = p.astype(np.float64) @ w.astype(np.float64).T
        ref = ref64.astype(np.float32)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    odd = np.isinf(ref)
    assert odd.any() and np.array_equal(got[odd], ref[odd])
    ok = np.isfinite(ref)
    assert np.isfinite(got[ok]).all()
    big = np.zeros_like(ok)
    big[row] = True
    # fp32 products and sums in any order: 2-norm below sqrt(768) roundings of 2^-24 each (1.7e-6); measured 2e-7
    for part in (ok & ~big, ok & big):
        err = np.linalg.norm((got[part] - ref64[part]) / np.abs(ref64[part]).max()) / np.linalg.norm(ref64[part] / np.abs(ref64[part]).max())
        assert err < 1e-6, err


@pytest.mark.parametrize("up", [-126, -120, -108, 110])
def test_error_of_small_and_large_operands(up):
    """Operands far from 1, subnormal ones among them: their parts hold every bit, or the fp32 instruction takes over."""
    rng = np.random.default_rng(84)
    images = np.ldexp(rng.standard_normal((32, 3, 224, 224)).astype(np.float32), up)
    w = np.ldexp(rng.standard_normal((384, 768)).astype(np.float32), -up if abs(up) < 110 else (100 if up < 0 else -100))
    ref = patches(images).astype(np.float64) @ w.astype(np.float64).T
    with runs(ROWS):
        got = patch_embed(images, w)
    err = np.linalg.norm((got - ref) / np.abs(ref).max()) / np.linalg.norm(ref / np.abs(ref).max())
    assert err < 1e-6, err   # as above
