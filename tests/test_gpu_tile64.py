"""GPU parity of the small-tile GEMM (kernels_gemm_tile64.hip) through one block forward + backward, at the sizes
where its tiling can go wrong: rows and widths at and beside the tile edges, one and several K groups per workgroup,
K shorter than a slab, weight gradients with K split over several partial tiles and with every remap."""
import pytest

import d2ft_inputs as di
from test_gpu_block import run_case
from test_gpu_ffn_gate import run_gated

pytestmark = pytest.mark.gpu

FULL, FWD, SKIP = di.OP_FULL, di.OP_FWD, di.OP_SKIP


@pytest.mark.parametrize("batch,tokens,width,heads,mlp", [
    (1, 3, 8, 1, 8),          # K below one slab everywhere
    (1, 64, 64, 1, 64),       # one exact tile
    (5, 13, 56, 2, 72),       # one row and one piece of columns beside the tile edge
    (1, 63, 136, 2, 264),
    (8, 197, 192, 3, 768),    # weight gradients in several splits of K, K not a multiple of the slab
    (40, 50, 320, 5, 1280),
])
def test_fp32_tile_edges(batch, tokens, width, heads, mlp):
    w = di.Workload("tile64_f32", batch, tokens, width, heads, 64, mlp, 1, "f32")
    ops = [FULL, FWD, SKIP, FULL, FULL][-heads:]
    run_case(w, ops, seed=71)


def test_fp32_gated_slices_through_the_remaps():
    w = di.Workload("tile64_gate_f32", 6, 197, 256, 4, 64, 1024, 1, "f32")
    run_gated(w, [FULL, SKIP, FWD, FULL], seed=72)


@pytest.mark.parametrize("batch,tokens,width,heads,mlp", [
    (1, 3, 64, 1, 64),        # one tile, K of one slab
    (1, 33, 136, 2, 264),     # one row and one piece of columns beside the edge of a 32x32 tile, K not a multiple of 64
    (1, 197, 768, 12, 3072),  # 32x32 and 64x32 tiles, two and four K groups
    (1, 33, 64, 1, 4096),     # 32x32 tiles over a long K: a wavefront exchanges 16 slabs between its lanes
    (5, 65, 384, 6, 1536),    # 64x32 tiles with a row beside the edge, column sums on 64x64 tiles
    (5, 197, 320, 5, 1280),   # 64x64 tiles
    (8, 197, 192, 3, 768),    # weight gradients in several splits of K, the call's tail riding along
])
def test_bf16_tile_edges(batch, tokens, width, heads, mlp):
    w = di.Workload("tile64_bf16", batch, tokens, width, heads, 64, mlp, 1, "bf16")
    ops = ([FULL, FWD, SKIP, FULL, FULL] * 3)[-heads:]
    run_case(w, ops, seed=73)


@pytest.mark.parametrize("batch,tokens,width,heads,mlp", [
    (1, 33, 64, 1, 2568),     # 41 slabs, the last of 8: uneven over the groups
    (1, 65, 136, 2, 4096),    # one row and one piece of columns beside the tile
    (1, 197, 768, 12, 3072),
])
def test_bf16_eight_k_groups(batch, tokens, width, heads, mlp):
    import paper_2504_12471_amd as P
    w = di.Workload("tile64_wk8", batch, tokens, width, heads, 64, mlp, 1, "bf16")
    P.d2ft_timing_enable(True)
    try:
        run_case(w, ([FULL, FWD, SKIP] * 4)[:heads], seed=76)
        names = {r["name"] for r in P.d2ft_timing_read()}
    finally:
        P.d2ft_timing_enable(False)
    assert "gemm_tile64_kernel<__bf16, 32, 32, false, false, 8, d2ft::GemmArgs>" in names, names


def test_bf16_gated_slices_through_the_remaps():
    w = di.Workload("tile64_gate_bf16", 1, 197, 256, 4, 64, 1024, 1, "bf16")
    run_gated(w, [FULL, SKIP, FWD, FULL], seed=74)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("lora", [0, 4])
def test_vector_alu_kernels_on_request(dtype, lora):
    """D2FT_FLAG_NO_MFMA: the other kernel family, in either type."""
    import paper_2504_12471_amd as P
    w = di.Workload("vector", 2, 65, 128, 3, 64, 264, 1, dtype, lora_rank=lora, lora_b_zero=False)
    P.d2ft_timing_enable(True)
    try:
        run_case(w, [FULL, FWD, FULL], seed=75, flags=P.FLAG_NO_MFMA)
        names = {r["name"] for r in P.d2ft_timing_read()}
    finally:
        P.d2ft_timing_enable(False)
    assert {"gemm_simple_kernel", "attn_fwd_simple", "attn_bwd_simple"} <= names
    assert not [n for n in names if "mfma" in n or "tile64" in n or "split" in n or "stream" in n], names


@pytest.mark.parametrize("images,width,small", [(8, 768, False), (1, 768, True)])
def test_small_tiles_leave_long_products_to_the_large_ones(images, width, small):
    """The feed-forward products of eight images have K or N of 3072 and enough rows for the 128x128 tile; of one image not."""
    import paper_2504_12471_amd as P
    w = di.Workload("long", images, 197, width, 2, 64, 4 * width, 1, "bf16")
    P.d2ft_timing_enable(True)
    try:
        run_case(w, [SKIP, SKIP], seed=76)
        names = {r["name"] for r in P.d2ft_timing_read()}
    finally:
        P.d2ft_timing_enable(False)
    assert any("gemm_tile64" in n and "GemmArgs" in n for n in names) == small, names


@pytest.mark.parametrize("rows,width,heads,mlp,lora,small", [
    (4096, 128, 2, 512, 0, True), (4480, 384, 6, 1536, 0, False), (4480, 128, 2, 512, 0, True), (2048, 64, 1, 64, 8, True)])
def test_which_tiles_the_weight_gradients_take(rows, width, heads, mlp, lora, small):
    """bf16: on either side of the lines by multiply-adds and rows."""
    import paper_2504_12471_amd as P
    w = di.Workload("wgrad", rows // 64, 64, width, heads, 64, mlp, 1, "bf16", lora_rank=lora, lora_b_zero=False)
    P.d2ft_timing_enable(True)
    try:
        run_case(w, [FULL] * heads, seed=77, grad_fields=[k for k in di.WEIGHT_FIELDS if k.startswith("lora") == (lora > 0)])
        names = {r["name"] for r in P.d2ft_timing_read()}
    finally:
        P.d2ft_timing_enable(False)
    assert any("Tile64Grouped" in n for n in names) == small, names
