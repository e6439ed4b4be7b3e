"""The weight gradients of a backward call in one launch of 256x256 tiles (gemm_wgrad_kernel), and their reduction."""
import numpy as np
import pytest

import d2ft_inputs as di
from helpers import TOL, gpu_block, oracle_block, rel_inf
from test_gpu_block import draw_block, run_case

pytestmark = pytest.mark.gpu

FULL, FWD, SKIP = di.OP_FULL, di.OP_FWD, di.OP_SKIP


# rows a multiple of the 32 of a slab, or 5 or 24 more; tiles with remainders both ways; rows and columns through the remaps;
# added to what is there; the adapters' product, whose sums stay fp32; one tile in eight runs of K
@pytest.mark.parametrize("B,T,D,heads,Dm,lora,accumulate", [
    (70, 64, 384, [FULL, SKIP, FULL, FWD, FULL, FULL], 1536, 0, False),
    (69, 65, 384, [FULL, FULL, SKIP, FULL, FULL, FULL], 1544, 0, True),
    (79, 104, 72, [FULL], 264, 0, False),
    (79, 104, 64, [FULL, SKIP, FULL, FULL], 64, 8, False)])
def test_weight_gradients(B, T, D, heads, Dm, lora, accumulate):
    import paper_2504_12471_amd as P
    w = di.Workload("wgrad", B, T, D, len(heads), 64, Dm, 1, "bf16", lora_rank=lora, lora_b_zero=False)
    fields = [k for k in di.WEIGHT_FIELDS if k.startswith("lora") == (lora > 0)]
    P.d2ft_timing_enable(True)
    try:
        if accumulate:
            x, wt, dy = draw_block(w, B + D)
            ref = oracle_block(w, wt, heads, x, dy)[2]
            init = {k: di.round_to_bf16(np.roll(ref[k].ravel(), 1).reshape(ref[k].shape)) for k in ("w1", "w2", "w_qkv", "w_o")}
            got = gpu_block(w, wt, heads, x, dy, list(init), 1, init)[2]
            for k, v in init.items():
                assert rel_inf(got[k], ref[k] + v) < TOL["bf16"], k
        else:
            run_case(w, heads, seed=B + D, grad_fields=fields)
        names = {r["name"] for r in P.d2ft_timing_read()}
    finally:
        P.d2ft_timing_enable(False)
    assert ("gemm_wgrad_kernel<%s>" % ("true" if B * T % 32 else "false")) in names, names


def test_infinity_stays_in_its_row_and_column():
    """An infinite dy of one token and channel: dw2's row of that channel and what dv carries on, nothing beyond."""
    import torch
    import paper_2504_12471_amd as P
    B, T, D, H, Dm = 70, 64, 384, 6, 1536
    gen = torch.Generator(device="cuda").manual_seed(3)
    mk = lambda *s, std=0.02: (torch.randn(s, generator=gen, device="cuda") * std).to(torch.bfloat16)
    wt = {"ln1_g": 1 + mk(D), "ln1_b": mk(D), "w_qkv": mk(3, H, 64, D), "b_qkv": mk(3, H, 64), "w_o": mk(D, 64 * H), "b_o": mk(D),
          "ln2_g": 1 + mk(D), "ln2_b": mk(D), "w1": mk(Dm, D), "b1": mk(Dm), "w2": mk(D, Dm), "b2": mk(D)}
    x, dy = mk(B, T, D, std=1.0), mk(B, T, D, std=1.0)
    ops = np.full((1, H), FULL, dtype=np.uint8)
    st = P.BlockStack(P.make_desc(B, T, D, H, Dm, "bf16"), [wt], "bf16", [])
    st.grads = [{n: (torch.zeros_like(wt[n]) if n in ("w1", "w2") else None) for n in P.WEIGHT_FIELDS}]
    st.step(x, dy, ops)
    clean = st.grads[0]["w2"].clone()
    dy[69, 63, 130] = float("inf")
    st.step(x, dy, ops)
    got = st.grads[0]["w2"]
    rest = torch.arange(D, device="cuda") != 130
    assert torch.equal(got[rest], clean[rest]) and not torch.isfinite(got[130]).any()


def units_of(records):
    """(256x256 tile, run of K) units of the one weight-gradient launch in the timing records: its reduction reads each once."""
    reads = [r for r in records if r["name"].startswith("launch_reduce_grouped")]
    assert len(reads) == 1 and reads[0]["launches"] == 1, records
    return round(reads[0]["bytes"] / (4 * 65536))


def weight_gradients_of(B, T, D, H, Dm, full, flags=0):
    """One backward call on random operands: its weights' gradients, the block's operands, the timing records."""
    import torch
    import paper_2504_12471_amd as P
    gen = torch.Generator(device="cuda").manual_seed(B * T + D)
    mk = lambda *s, std=0.02: (torch.randn(s, generator=gen, device="cuda") * std).to(torch.bfloat16)
    wt = {"ln1_g": 1 + mk(D), "ln1_b": mk(D), "w_qkv": mk(3, H, 64, D), "b_qkv": mk(3, H, 64), "w_o": mk(D, 64 * H), "b_o": mk(D),
          "ln2_g": 1 + mk(D), "ln2_b": mk(D), "w1": mk(Dm, D), "b1": mk(Dm), "w2": mk(D, Dm), "b2": mk(D)}
    x, dy = mk(B, T, D, std=1.0), mk(B, T, D, std=1.0)
    ops = np.array([[FULL] * full + [SKIP] * (H - full)], np.uint8)
    st = P.BlockStack(P.make_desc(B, T, D, H, Dm, "bf16", flags=flags), [wt], "bf16", [])
    st.grads = [{n: (torch.zeros_like(wt[n]) if n in ("w_qkv", "w_o", "w1", "w2") else None) for n in P.WEIGHT_FIELDS}]
    st.forward(x, ops)
    P.d2ft_timing_enable(True)
    try:
        st.backward(dy, ops)
        records = P.d2ft_timing_read()
    finally:
        P.d2ft_timing_enable(False)
    return st.grads[0], wt, x, dy, ops, records


# 93 tiles in one launch: two runs of K take 152.5 us with their reduction, five 167.6; 33 tiles: seven runs 63, eight 91
@pytest.mark.parametrize("H,Dm,full,tiles,runs", [(12, 3072, 6, 93, 2), (12, 3072, 4, 84, 3), (4, 1024, 2, 33, 7)])
def test_runs_per_tile(H, Dm, full, tiles, runs):
    assert units_of(weight_gradients_of(64, 197, 768, H, Dm, full)[5]) == tiles * runs


# rows, hidden units, tiles, 32-deep slabs of K: more tiles than the chip has CUs, so that a workgroup takes up to ten units, each
# with its first slabs requested ahead of the stores of the one before; runs of 2 to 10 slabs, i.e. fewer than, as many as and more than
# the five that are in LDS; rows that are no multiple of the 32 of a slab
@pytest.mark.parametrize("rows,Dm,tiles,slabs", [(303, 8192, 512, 10), (192, 13056, 816, 6), (160, 16384, 1024, 5), (97, 25600, 1600, 4), (64, 40960, 2560, 2)])
def test_more_units_than_workgroups_and_short_runs(rows, Dm, tiles, slabs):
    import torch
    D = 2048
    grads, wt, x, dy, _, records = weight_gradients_of(1, rows, D, 1, Dm, 0)
    assert ("gemm_wgrad_kernel<%s>" % ("true" if rows % 32 else "false")) in {r["name"] for r in records}
    assert units_of(records) == tiles and -(-rows // 32) == slabs   # one run of all slabs per tile

    r16 = lambda t: t.to(torch.bfloat16).float()
    f = {k: t.float() for k, t in wt.items()}
    x, dy = x[0].float(), dy[0].float()   # no head is live: the residual stream is x
    v = r16(torch.nn.functional.layer_norm(x, (D,), f["ln2_g"], f["ln2_b"], 1e-6))
    z = v @ f["w1"].T + f["b1"]
    phi = 0.5 * (1 + torch.erf(z * 0.5 ** 0.5))
    slope = r16(phi + z * torch.exp(-0.5 * z * z) * 0.3989422804014327)
    dz = r16((dy @ f["w2"]) * slope)
    # operands and results are rounded to bf16: 2^-9 each, up to four of them, adding in quadrature, is below 4e-3 in the norm
    # of any part; a slab left out is off by a third or more, a tile in another's place by more than one
    for name, ref in (("w2", dy.T @ r16(z * phi)), ("w1", dz.T @ v)):
        err = (grads[name].float() - ref).reshape(ref.shape[0] // 64, 64, ref.shape[1] // 64, 64).pow(2).sum((1, 3)).sqrt()
        size = ref.reshape(ref.shape[0] // 64, 64, ref.shape[1] // 64, 64).pow(2).sum((1, 3)).sqrt()
        assert (err / size).max() < 1e-2, (name, float((err / size).max()))
