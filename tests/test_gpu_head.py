"""GPU parity for the two subnets outside the blocks (Sec. IV-A): d2ft_patch_embed_fwd / _bwd and
d2ft_classifier_fwd_bwd against the oracle.  Tolerances as for the blocks (1e-4 fp32, 2e-2 bf16 per
tensor, infinity-norm relative); the loss is fp32 arithmetic on exact inputs: 1e-5."""
import numpy as np
import pytest

import d2ft_inputs as di
from helpers import TOL, rel_inf

pytestmark = pytest.mark.gpu


def grid(a, dtype):
    a = np.asarray(a, np.float32)
    return di.round_to_bf16(a) if dtype == "bf16" else a


def run_embed(dtype, B, C, H, W, P, D, seed, accumulate=False):
    import torch
    import paper_2504_12471_amd as Pk
    from oracle import d2ft_oracle as orc
    rng = np.random.default_rng(seed)
    T = 1 + (H // P) * (W // P)
    K = C * P * P
    h = dict(images=grid(rng.standard_normal((B, C, H, W)), dtype), w_pe=grid(rng.standard_normal((D, K)) * 0.05, dtype),
             b_pe=grid(rng.standard_normal(D) * 0.1, dtype), cls=grid(rng.standard_normal(D), dtype),
             pos=grid(rng.standard_normal((T, D)) * 0.5, dtype))
    dtok = grid(rng.standard_normal((B, T, D)), dtype)
    desc = Pk.EmbedDesc(B, C, H, W, P, D, Pk.BF16 if dtype == "bf16" else Pk.F32, 1 if accumulate else 0)
    dev = {k: Pk.to_device(v, dtype) for k, v in h.items()}
    tokens = torch.empty((B, T, D), dtype=Pk.torch_dtype(dtype), device="cuda")
    saved = torch.empty(Pk.d2ft_embed_saved_bytes(desc), dtype=torch.uint8, device="cuda")
    scratch = torch.empty(Pk.d2ft_embed_scratch_bytes(desc), dtype=torch.uint8, device="cuda")
    Pk.d2ft_patch_embed_fwd(desc, dev["images"], dev["w_pe"], dev["b_pe"], dev["cls"], dev["pos"], tokens, saved, scratch)
    init = {k: grid(rng.standard_normal(h[k].shape) * 0.1, dtype) for k in ("w_pe", "b_pe", "cls", "pos")}
    g = {k: (Pk.to_device(init[k], dtype) if accumulate else torch.full_like(dev[k], float("nan"))) for k in init}
    Pk.d2ft_patch_embed_bwd(desc, Pk.to_device(dtok, dtype), g["w_pe"], g["b_pe"], g["cls"], g["pos"], saved, scratch)
    torch.cuda.synchronize()
    rtok, cache = orc.patch_embed_fwd(h["images"], h["w_pe"], h["b_pe"], h["cls"], h["pos"], P)
    rg = orc.patch_embed_bwd(cache, dtok)
    tol = TOL[dtype]
    errs = {"tokens": rel_inf(tokens.float().cpu().numpy(), rtok)}
    for k in init:
        ref = rg[k] + (init[k] if accumulate else 0.0)
        errs["d" + k] = rel_inf(g[k].float().cpu().numpy(), ref)
    print(f"[embed {dtype} B={B} {C}x{H}x{W} P={P} D={D}] " + " ".join(f"{k}={v:.1e}" for k, v in errs.items()), flush=True)
    assert all(v <= tol for v in errs.values()), errs


def test_embed_fp32_small():
    run_embed("f32", 3, 3, 32, 24, 8, 40, 111)


def test_embed_fp32_accumulate():
    run_embed("f32", 2, 1, 16, 16, 8, 16, 112, accumulate=True)


def test_embed_bf16_vit_shape():
    """The ViT-B/16 embedding at a small batch: 224 x 224 x 3 images, 16 x 16 patches, 197 tokens, D = 768."""
    run_embed("bf16", 4, 3, 224, 224, 16, 768, 113)


def run_head(dtype, B, T, D, n, seed, frozen_ln=False):
    import torch
    import paper_2504_12471_amd as Pk
    from oracle import d2ft_oracle as orc
    rng = np.random.default_rng(seed)
    h = dict(tokens=grid(rng.standard_normal((B, T, D)), dtype), ln_g=grid(1 + 0.2 * rng.standard_normal(D), dtype),
             ln_b=grid(0.1 * rng.standard_normal(D), dtype), w_c=grid(rng.standard_normal((n, D)) * 0.2, dtype),
             b_c=grid(rng.standard_normal(n) * 0.1, dtype))
    labels = rng.integers(0, n, size=B)
    desc = Pk.HeadDesc(B, T, D, n, 1e-6, Pk.BF16 if dtype == "bf16" else Pk.F32, 0)
    dev = {k: Pk.to_device(v, dtype) for k, v in h.items()}
    dtok = torch.full_like(dev["tokens"], float("nan"))
    g = {k: torch.full_like(dev[k], float("nan")) for k in ("ln_g", "ln_b", "w_c", "b_c")}
    if frozen_ln:
        g["ln_g"] = g["ln_b"] = None
    scratch = torch.empty(Pk.d2ft_head_scratch_bytes(desc), dtype=torch.uint8, device="cuda")
    loss = Pk.d2ft_classifier_fwd_bwd(desc, dev["tokens"], dev["ln_g"], dev["ln_b"], dev["w_c"], dev["b_c"], labels, dtok,
                                      g["ln_g"], g["ln_b"], g["w_c"], g["b_c"], scratch)
    rloss, _, cache = orc.classifier_fwd(h["tokens"], h["ln_g"], h["ln_b"], h["w_c"], h["b_c"], labels)
    rdtok, rg = orc.classifier_bwd(cache)
    tol = TOL[dtype]
    assert abs(loss - rloss) <= 1e-5 * max(1.0, abs(rloss)), (loss, rloss)
    got = dtok.float().cpu().numpy()
    assert np.all(got[:, 1:] == 0.0) and not np.any(np.signbit(got[:, 1:]))
    errs = {"dtokens": rel_inf(got, rdtok)}
    for k, t in g.items():
        if t is not None:
            errs["d" + k] = rel_inf(t.float().cpu().numpy(), rg[k])
    print(f"[head {dtype} B={B} T={T} D={D} n={n}] loss={loss:.6f} ref={rloss:.6f} " +
          " ".join(f"{k}={v:.1e}" for k, v in errs.items()), flush=True)
    assert all(v <= tol for v in errs.values()), errs


def test_head_fp32_small():
    run_head("f32", 5, 4, 24, 7, 121)


def test_head_bf16_vit_shape_100_classes():
    run_head("bf16", 64, 197, 768, 100, 122)


def test_head_frozen_norm_and_single_class_count_edge():
    run_head("f32", 2, 1, 8, 1, 123, frozen_ln=True)        # one class: loss 0, zero gradients
    run_head("f32", 3, 2, 16, 300, 124, frozen_ln=True)     # more classes than threads in a workgroup


@pytest.mark.parametrize("dtype,B,T,D,n", [("f32", 257, 2, 264, 33), ("bf16", 3, 40, 520, 9), ("bf16", 2, 65, 1032, 1000),
                                           ("f32", 1, 1, 512, 8)])
def test_head_at_the_edges_of_its_pieces(dtype, B, T, D, n):
    """Images are staged by 256, channels taken by 512 and 256, classes by 8 and 32, cleared rows by 32 KiB."""
    run_head(dtype, B, T, D, n, 125)


@pytest.mark.parametrize("B", [7, 8, 9, 41])
def test_embed_images_over_the_lanes(B):
    run_embed("f32", B, 1, 16, 24, 8, 40, 126)              # 7 tokens x 5 pieces: the second workgroup is part empty


@pytest.mark.parametrize("dtype,B,accumulate", [("f32", 4, True), ("f32", 5, False), ("bf16", 16, True), ("f32", 17, False)])
def test_embed_lanes_by_images_and_pieces(dtype, B, accumulate):
    """4097 tokens x 13 pieces: one, two and eight lanes of images."""
    run_embed(dtype, B, 1, 512, 512, 8, 104, 128, accumulate)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_head_takes_pointers_of_element_alignment(dtype):
    """Every tensor one element past a 16-byte boundary: the same bits as from aligned ones."""
    import torch
    import paper_2504_12471_amd as Pk
    rng = np.random.default_rng(127)
    B, T, D, n = 3, 5, 72, 11
    labels = rng.integers(0, n, size=B)
    desc = Pk.HeadDesc(B, T, D, n, 1e-6, Pk.BF16 if dtype == "bf16" else Pk.F32, 0)
    h = {k: Pk.to_device(rng.standard_normal(s).astype(np.float32), dtype)
         for k, s in dict(tokens=(B, T, D), ln_g=D, ln_b=D, w_c=(n, D), b_c=n).items()}

    def shifted(t, by):
        return torch.empty(t.numel() + 8, dtype=t.dtype, device=t.device)[by:by + t.numel()].view(t.shape).copy_(t)

    def run(by):
        i = {k: shifted(t, by) for k, t in h.items()}
        o = {k: shifted(torch.full_like(t, float("nan")), by) for k, t in h.items()}
        scratch = torch.empty(Pk.d2ft_head_scratch_bytes(desc), dtype=torch.uint8, device="cuda")
        loss = Pk.d2ft_classifier_fwd_bwd(desc, i["tokens"], i["ln_g"], i["ln_b"], i["w_c"], i["b_c"], labels, o["tokens"],
                                          o["ln_g"], o["ln_b"], o["w_c"], o["b_c"], scratch)
        return loss, o

    (l0, o0), (l1, o1) = run(0), run(1)
    assert l0 == l1 and all(torch.equal(o0[k], o1[k]) for k in o0)


def test_bad_labels_and_shapes_are_rejected():
    import torch
    import paper_2504_12471_amd as Pk
    desc = Pk.HeadDesc(2, 3, 8, 4, 1e-6, Pk.F32, 0)
    z = lambda *s: torch.zeros(s, dtype=torch.float32, device="cuda")
    scratch = torch.empty(Pk.d2ft_head_scratch_bytes(desc), dtype=torch.uint8, device="cuda")
    with pytest.raises(Pk.D2ftError):
        Pk.d2ft_classifier_fwd_bwd(desc, z(2, 3, 8), z(8), z(8), z(4, 8), z(4), [0, 4], z(2, 3, 8), None, None, None, None, scratch)
    assert Pk.d2ft_embed_scratch_bytes(Pk.EmbedDesc(1, 3, 20, 16, 8, 16, Pk.F32, 0)) == 0     # 20 is not a multiple of 8
    assert Pk.d2ft_embed_scratch_bytes(Pk.EmbedDesc(1, 3, 16, 16, 4, 16, Pk.F32, 0)) == 0     # patch below 8
