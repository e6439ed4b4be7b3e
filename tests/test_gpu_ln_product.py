"""GPU parity of LayerNorm fused into the product behind it (kernels_gemm_ln.hip) through one block forward + backward, at
the sizes where it can go wrong: rows and columns at and beside the edges of its 32x64 and 32x96 tiles, rows of x that end
inside and at the ends of the four lengths it is built for, both types, the remaps and merged weights."""
import pytest

import d2ft_inputs as di
from test_gpu_block import run_case
from test_gpu_ffn_gate import run_gated

pytestmark = pytest.mark.gpu

FULL, FWD, SKIP = di.OP_FULL, di.OP_FWD, di.OP_SKIP


def records_of(run):
    import paper_2504_12471_amd as P
    P.d2ft_timing_enable(True)
    try:
        run()
        return P.d2ft_timing_read()
    finally:
        P.d2ft_timing_enable(False)


def kernels_of(run):
    return {r["name"] for r in records_of(run)}


@pytest.mark.parametrize("dtype,batch,tokens,width,heads,mlp,form", [
    ("bf16", 1, 3, 64, 1, 64, "1, 64"),          # one slab of K: three of the four K groups have none
    ("bf16", 1, 33, 256, 2, 264, "1, 64"),       # one row and one piece of columns beside the tile; rows of 512 bytes
    ("bf16", 1, 31, 320, 3, 1280, "2, 64"),
    ("bf16", 2, 16, 512, 2, 520, "2, 64"),       # rows of 1024 bytes, one exact tile of rows
    ("bf16", 1, 65, 576, 2, 1032, "3, 64"),
    ("bf16", 1, 197, 768, 4, 1536, "3, 64"),     # rows of 1536 bytes
    ("bf16", 1, 33, 832, 1, 832, "4, 64"),
    ("bf16", 1, 65, 1024, 2, 1032, "4, 64"),     # the longest rows
    ("f32", 1, 3, 32, 1, 64, "1, 64"),
    ("f32", 1, 33, 128, 2, 264, "1, 64"),
    ("f32", 4, 65, 192, 3, 768, "2, 64"),
    ("f32", 4, 65, 288, 3, 1032, "3, 64"),
    ("f32", 2, 197, 384, 3, 1032, "3, 64"),
    ("f32", 1, 197, 512, 4, 2048, "4, 64"),
    ("bf16", 4, 197, 192, 2, 776, "1, 96"),   # a last tile of 8 columns, a last wavefront without any
    ("bf16", 2, 197, 384, 3, 1600, "2, 96"),
    ("bf16", 1, 225, 768, 3, 2648, "3, 96"),   # one row beside the tile
    ("bf16", 1, 129, 1024, 2, 4096, "4, 96"),
    ("f32", 5, 197, 192, 2, 768, "2, 96"),
    ("f32", 2, 197, 384, 3, 1600, "3, 96"),
    ("f32", 1, 257, 512, 2, 2048, "4, 96"),
])
def test_tile_and_row_edges(dtype, batch, tokens, width, heads, mlp, form):
    w = di.Workload("ln_product", batch, tokens, width, heads, 64, mlp, 1, dtype)
    names = kernels_of(lambda: run_case(w, [FULL, FWD, FULL, SKIP][:heads], seed=81))
    assert "gemm_ln_kernel<%s, %s>" % ("__bf16" if dtype == "bf16" else "float", form) in names, names


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("images,columns", [(2, 64), (12, 96)])   # tiles of 96 begin inside the remap's blocks
def test_gated_slices_through_the_remap(dtype, images, columns):
    w = di.Workload("ln_product_gate", images, 65, 256, 4, 64, 1024, 1, dtype)
    names = kernels_of(lambda: run_gated(w, [FULL, SKIP, FWD, FULL], seed=82))
    assert [n for n in names if n.startswith("gemm_ln_kernel") and n.endswith(", %d>" % columns)], names


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_merged_adapter_weights(dtype):
    w = di.Workload("ln_product_lora", 2, 65, 256, 4, 64, 512, 1, dtype, lora_rank=4, lora_b_zero=False)
    names = kernels_of(lambda: run_case(w, [FULL, SKIP, FWD, FULL], seed=83))
    assert [n for n in names if n.startswith("gemm_ln_kernel")], names


def test_timing_records_hold_the_norm_and_the_product():
    w = di.Workload("ln_product_records", 1, 33, 256, 2, 64, 264, 1, "f32")
    rec = [r for r in records_of(lambda: run_case(w, [FULL, FWD], seed=85)) if r["name"].startswith("gemm_ln_kernel")]
    assert sum(r["launches"] for r in rec) == 2   # before the QKV product and the first of the feed-forward network
    assert sum(r["bytes"] for r in rec) == 2 * (2 * 33 * 256 * 4 + 8 * 33)
    assert sum(r["flops"] for r in rec) == 2.0 * 33 * 256 * (2 * 192 + 264)


@pytest.mark.parametrize("tokens,fused", [(224, True), (353, False)])
def test_line_between_one_launch_and_two(tokens, fused):
    """Width 768 in bf16: a workgroup per CU at most."""
    w = di.Workload("ln_product_line", 1, tokens, 768, 12, 64, 768, 1, "bf16")
    names = kernels_of(lambda: run_case(w, [FULL] * 12, seed=84))
    assert ("launch_ln_fwd" in names) == (not fused), names
