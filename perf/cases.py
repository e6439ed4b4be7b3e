"""The work that a user of this package has it do, as a list of cases that can be timed and compared.

A case is a dict of plain values.  Its "kind" says which of the public entry points a pass goes through:

  step      one fine-tune pass over a stack of blocks: forward, then backward with the weight gradients
  forward   the forward half alone, as for evaluation: no head needs a backward pass
  finetune  a whole training step on images: patch embedding, blocks, classifier with its loss, the backward
            passes of all three, and the optimizer step with fp32 master weights
  select    the choice of operation codes: contribution scores of every block, then the bi-level knapsack

Sizes are those of a block as one device holds it: `heads` and `mlp` may be a share of the model's.  The op codes
are drawn from the seed with the exact counts that `full` and `fwd` (fractions of all subnets, the rest is
skipped) give, one per head and block, or one per head, block and micro-batch when `micro` > 1.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2504_12471_amd as P

FULL, FWD, SKIP = P.OP_FULL, P.OP_FWD, P.OP_SKIP
MATRICES = ("w_qkv", "w_o", "w1", "w2")


def _stack_case(name, kind, batch, tokens, width, heads, mlp, blocks, dtype, full, fwd, lora=0, gate=False, micro=1):
    c = {"kind": kind, "batch": batch, "tokens": tokens, "width": width, "heads": heads, "mlp": mlp, "blocks": blocks,
         "dtype": dtype, "full": full, "fwd": fwd, "lora": lora, "gate": gate, "micro": micro}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a single fp32 block of the tiny model with one head of each code: the smallest training call, all latency
        _stack_case("tiny_f32_block", "step", 4, 65, 192, 3, 768, 1, "f32", 1 / 3, 1 / 3),
        # the small model in fp32, 80 images as five micro-batches of 16 with codes of their own
        _stack_case("small_f32_micro5", "step", 80, 197, 384, 6, 1536, 12, "f32", 0.6, 0.2, micro=5),
        # an ordinary small batch in bf16, with tile remainders everywhere
        _stack_case("small_bf16_batch5", "step", 5, 197, 384, 6, 1536, 12, "bf16", 0.6, 0.2),
        # the base model, 64 images: the benchmark's own workload
        _stack_case("base_step", "step", 64, 197, 768, 12, 3072, 12, "bf16", 0.6, 0.2),
        # whole subnets gated (a head with its slice of the feed-forward network), five micro-batches
        _stack_case("base_gated_micro5", "step", 64, 197, 768, 12, 3072, 12, "bf16", 0.6, 0.2, gate=True, micro=5),
        # adapters on a frozen base: only the adapters' gradients
        _stack_case("base_lora", "step", 64, 197, 768, 12, 3072, 12, "bf16", 0.6, 0.0, lora=8),
        # one device's share of the base model: a third of the heads and of the feed-forward network
        _stack_case("base_share4", "step", 64, 197, 768, 4, 1024, 12, "bf16", 0.6, 0.05),
        # the large model: the largest training step
        _stack_case("large_step", "step", 32, 197, 1024, 16, 4096, 24, "bf16", 0.4, 0.2),
        # the base model on 384-pixel images: 24 x 24 patches and the class token
        _stack_case("base_384px", "step", 16, 577, 768, 12, 3072, 12, "bf16", 0.6, 0.2),
        # evaluation of one image: forward only, the latency of a prediction
        _stack_case("base_predict_one", "forward", 1, 197, 768, 12, 3072, 12, "bf16", 0.0, 1.0),
        # a whole training step of the small model from images to updated weights
        dict(_stack_case("small_finetune", "finetune", 80, 197, 384, 6, 1536, 12, "bf16", 0.6, 0.2, gate=True),
             pixels=224, patch=16, classes=100),
        # choosing the codes of the base model from one gradient set
        {"name": "base_select", "kind": "select", "width": 768, "heads": 12, "mlp": 3072, "blocks": 12, "dtype": "bf16",
         "gate": True, "devices": 1, "capacity": 0.6},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: models of 3 to 16 heads or a share of one, 1 to 24 blocks, 1 to 96 images,
    17 to 1024 tokens, either data type."""
    most = {}   # no drawn case does more arithmetic than the listed ones of its sort
    for c in listed():
        if c["kind"] != "select":
            sort = _sort(c)
            most[sort] = max(most.get(sort, 0.0), work(c)["flops"])
    while True:
        kind = rng.choices(("step", "forward", "finetune", "select"), (13, 3, 2, 2))[0]
        model = rng.randint(3, 16)
        width, blocks = 64 * model, _log_int(rng, 1, 24)
        dtype = rng.choices(("bf16", "f32"), (4, 1))[0]
        gate = rng.random() < 0.35
        if kind == "select":
            devices = rng.choice([d for d in range(1, model + 1) if model % d == 0])
            return {"kind": "select", "width": width, "heads": model, "mlp": 4 * width, "blocks": blocks, "dtype": dtype,
                    "gate": gate, "devices": devices, "capacity": round(rng.uniform(0.3, 0.9), 2)}
        heads = model
        if kind == "step" and rng.random() < 0.15:
            heads = rng.randint(1, max(1, model // 2))
        batch = _log_int(rng, 1, 96)
        full = rng.choice((0.4, 0.5, 0.6, 0.8, 1.0))
        fwd = round(rng.uniform(0.0, 1.0 - full), 2)
        if kind == "finetune":
            patch = rng.choice((8, 16, 32))
            side = rng.randint(4, 24)
            c = dict(_stack_case(None, "finetune", batch, 1 + side * side, width, heads, 4 * width, blocks, dtype, full, fwd,
                                 gate=gate), pixels=patch * side, patch=patch, classes=_log_int(rng, 10, 1000))
        else:
            tokens = _log_int(rng, 225, 1024) if rng.random() < 0.3 else _log_int(rng, 17, 224)
            if kind == "forward":
                full, fwd = 0.0, rng.choice((1.0, 0.8))
            lora = rng.choice((4, 8, 16)) if kind == "step" and not gate and rng.random() < 0.15 else 0
            micro = rng.randint(2, 8) if kind == "step" and batch >= 16 and rng.random() < 0.3 else 1
            c = _stack_case(None, kind, batch, tokens, width, heads, 256 * heads, blocks, dtype, full, fwd, lora, gate, micro)
        if work(c)["flops"] <= most[_sort(c)] and batch * c["tokens"] >= 32:
            return c


def _sort(c):
    if c["dtype"] == "f32":
        return "f32"
    return "long" if c["tokens"] > 224 else "bf16"


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _torch_dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _normal(gen, shape, dtype, mean=0.0, std=1.0):
    return (torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32) * std + mean).to(dtype)


def _weight_shapes(case):
    D, H, Dm, r = case["width"], case["heads"], case["mlp"], case.get("lora", 0)
    s = {"ln1_g": (D,), "ln1_b": (D,), "w_qkv": (3, H, 64, D), "b_qkv": (3, H, 64), "w_o": (D, 64 * H), "b_o": (D,),
         "ln2_g": (D,), "ln2_b": (D,), "w1": (Dm, D), "b1": (Dm,), "w2": (D, Dm), "b2": (D,)}
    if r:
        s.update({"lora_a_q": (H, r, D), "lora_a_v": (H, r, D), "lora_b_q": (H, 64, r), "lora_b_v": (H, 64, r)})
    return s


def _trained(case):
    """The tensors that get a gradient: normalisation layers are frozen, and under LoRA the whole base is."""
    names = list(_weight_shapes(case))
    return [n for n in names if n.startswith("lora")] if case.get("lora", 0) else [n for n in names if not n.startswith("ln")]


def _block_weights(gen, case):
    """Every tensor of the stack in one allocation, [blocks, ...], and the blocks' views of them."""
    L, dt = case["blocks"], _torch_dtype(case)
    stacked = {n: _normal(gen, (L,) + s, dt, 1.0 if n in ("ln1_g", "ln2_g") else 0.0, 0.02)
               for n, s in _weight_shapes(case).items()}
    return stacked, [{n: t[l] for n, t in stacked.items()} for l in range(L)]


def _micro_images(case):
    base, extra = divmod(case["batch"], case["micro"])
    return [base + (1 if i < extra else 0) for i in range(case["micro"])]


def _op_codes(case, seed):
    """Codes with exact counts over all subnets (and micro-batches), placed by a seeded shuffle."""
    shape = (case["blocks"], case["micro"], case["heads"])
    total = shape[0] * shape[1] * shape[2]
    n_full = int(round(case["full"] * total))
    n_fwd = min(total - n_full, int(round(case["fwd"] * total)))
    codes = np.array([FULL] * n_full + [FWD] * n_fwd + [SKIP] * (total - n_full - n_fwd), dtype=np.uint8)
    codes = np.random.default_rng([seed, 17]).permutation(codes).reshape(shape)
    return codes if case["micro"] > 1 else codes[:, 0]


def _make_stack(case, gen):
    stacked, weights = _block_weights(gen, case)
    desc = P.make_desc(case["batch"], case["tokens"], case["width"], case["heads"], case["mlp"], case["dtype"],
                       case["lora"], flags=P.FLAG_GATE_FFN if case["gate"] else 0)
    stack = P.BlockStack(desc, weights, case["dtype"], [], _micro_images(case) if case["micro"] > 1 else None)
    grads = {n: torch.zeros_like(stacked[n]) for n in _trained(case)} if case["kind"] != "forward" else {}
    stack.grads = [{n: (grads[n][l] if n in grads else None) for n in P.WEIGHT_FIELDS} for l in range(case["blocks"])]
    return stack, stacked, grads


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = _torch_dtype(case)
    if case["kind"] == "select":
        return _prepare_select(case, seed, gen)
    stack, stacked, grads = _make_stack(case, gen)
    shape = (case["batch"], case["tokens"], case["width"])
    s = {"kind": case["kind"], "stack": stack, "grads": grads, "ops": _op_codes(case, seed)}
    if case["kind"] != "finetune":
        s["x"] = _normal(gen, shape, dt)
        if case["kind"] == "step":
            s["dy"] = _normal(gen, shape, dt)
        return s

    B, D, px, patch, n = case["batch"], case["width"], case["pixels"], case["patch"], case["classes"]
    K = 3 * patch * patch
    code = P.F32 if case["dtype"] == "f32" else P.BF16
    s["embed_desc"] = P.EmbedDesc(B, 3, px, px, patch, D, code, 0)
    s["head_desc"] = P.HeadDesc(B, case["tokens"], D, n, 1e-6, code, 0)
    s["images"] = _normal(gen, (B, 3, px, px), dt)
    s["labels"] = np.random.default_rng([seed, 18]).integers(0, n, size=B).astype(np.int32)
    s["embed"] = {"w_pe": _normal(gen, (D, K), dt, std=0.02), "b_pe": _normal(gen, (D,), dt, std=0.02),
                  "cls": _normal(gen, (D,), dt, std=0.02), "pos": _normal(gen, (case["tokens"], D), dt, std=0.02)}
    s["head"] = {"ln_g": _normal(gen, (D,), dt, 1.0, 0.02), "ln_b": _normal(gen, (D,), dt, std=0.02),
                 "w_c": _normal(gen, (n, D), dt, std=0.02), "b_c": _normal(gen, (n,), dt, std=0.02)}
    s["embed_grads"] = {k: torch.empty_like(v) for k, v in s["embed"].items()}
    s["head_grads"] = {k: torch.empty_like(v) for k, v in s["head"].items()}
    s["tokens"] = torch.empty(shape, dtype=dt, device="cuda")
    s["dy"] = torch.empty(shape, dtype=dt, device="cuda")
    s["embed_saved"] = torch.empty(P.d2ft_embed_saved_bytes(s["embed_desc"]), dtype=torch.uint8, device="cuda")
    s["embed_scratch"] = torch.empty(P.d2ft_embed_scratch_bytes(s["embed_desc"]), dtype=torch.uint8, device="cuda")
    s["head_scratch"] = torch.empty(P.d2ft_head_scratch_bytes(s["head_desc"]), dtype=torch.uint8, device="cuda")
    # the optimizer's state: fp32 momentum and fp32 master copies of the trained block weights
    s["weights"] = {k: stacked[k] for k in grads}
    s["momentum"] = {k: torch.zeros(t.shape, dtype=torch.float32, device="cuda") for k, t in grads.items()}
    s["master"] = {k: stacked[k].float() for k in grads}
    L = case["blocks"]
    s["views"] = [tuple({k: t[l] for k, t in group.items()}
                        for group in (s["weights"], grads, s["momentum"], s["master"])) for l in range(L)]
    return s


def _prepare_select(case, seed, gen):
    _, weights = _block_weights(gen, case)
    dt = _torch_dtype(case)
    # gradients of one sample differ in size from block to block and head to head
    grads = []
    for _ in range(case["blocks"]):
        g = {n: _normal(gen, sh, dt, std=1e-3) for n, sh in _weight_shapes(case).items()}
        per_head = torch.rand(case["heads"], generator=gen, device="cuda") + 0.5
        g["w_qkv"] = (g["w_qkv"].float() * per_head[None, :, None, None]).to(dt)
        grads.append(g)
    desc = P.make_desc(1, 197, case["width"], case["heads"], case["mlp"], case["dtype"],
                       flags=P.FLAG_GATE_FFN if case["gate"] else 0)
    items = case["blocks"] * case["heads"] // case["devices"]
    budget = int(case["capacity"] * 3 * items + 1e-9)
    K = case["devices"]
    costs = [np.full(K, v, np.int32) for v in (1, 2, budget, budget % 3)]
    need = P.d2ft_knapsack_workspace_bytes(K, items, costs[2], costs[3])
    return {"kind": "select", "desc": desc, "weights": weights, "grads": grads, "costs": costs, "devices": K,
            "knapsack_space": torch.empty(need, dtype=torch.uint8, device="cuda")}


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    if s["kind"] == "step":
        y, dx = s["stack"].step(s["x"], s["dy"], s["ops"])
        return {"y": y, "dx": dx, "grads": s["grads"]}
    if s["kind"] == "forward":
        return s["stack"].forward(s["x"], s["ops"])
    if s["kind"] == "finetune":
        return _run_finetune(s)
    return _run_select(s)


def _run_finetune(s):
    e, h, eg, hg, stack = s["embed"], s["head"], s["embed_grads"], s["head_grads"], s["stack"]
    P.d2ft_patch_embed_fwd(s["embed_desc"], s["images"], e["w_pe"], e["b_pe"], e["cls"], e["pos"], s["tokens"],
                           s["embed_saved"], s["embed_scratch"])
    y = stack.forward(s["tokens"], s["ops"])
    loss = P.d2ft_classifier_fwd_bwd(s["head_desc"], y, h["ln_g"], h["ln_b"], h["w_c"], h["b_c"], s["labels"], s["dy"],
                                     hg["ln_g"], hg["ln_b"], hg["w_c"], hg["b_c"], s["head_scratch"])
    dtokens = stack.backward(s["dy"], s["ops"])
    P.d2ft_patch_embed_bwd(s["embed_desc"], dtokens, eg["w_pe"], eg["b_pe"], eg["cls"], eg["pos"], s["embed_saved"],
                           s["embed_scratch"])
    for l, (w, g, v, m) in enumerate(s["views"]):
        P.d2ft_sgd_step(stack.desc, w, g, v, m, s["ops"][l], 1e-3, 0.9, 1e-4)
    return {"loss": loss, "y": y, "dtokens": dtokens, "embed_grads": eg, "head_grads": hg, "grads": s["grads"],
            "weights": s["weights"], "momentum": s["momentum"], "master": s["master"]}


def _run_select(s):
    rows = []
    for g, w in zip(s["grads"], s["weights"]):
        rows.append((P.d2ft_subnet_scores(s["desc"], g, P.SCORE_FISHER),
                     P.d2ft_subnet_scores(s["desc"], w, P.SCORE_MAGNITUDE)))
    # device k holds the k-th group of every block's heads
    full, fwd = (np.stack([r[i] for r in rows]).reshape(len(rows), s["devices"], -1).transpose(1, 0, 2).reshape(s["devices"], -1)
                 for i in range(2))
    codes = P.d2ft_select_knapsack(full, fwd, *s["costs"], workspace=s["knapsack_space"])
    return {"codes": codes, "full": full, "fwd": fwd}


# ---------------------------------------------------------------------------
# what a pass cannot do without, and how far two correct ones may be apart
# ---------------------------------------------------------------------------
def work(case):
    es = 4 if case["dtype"] == "f32" else 2
    sizes = {n: math.prod(s) for n, s in _weight_shapes(case).items()}
    L = case["blocks"]
    if case["kind"] == "select":
        own = sum(v for n, v in sizes.items() if n in ("w_qkv", "b_qkv", "w_o") or (case["gate"] and n in ("w1", "b1", "w2")))
        return {"bytes": 2 * L * own * es, "flops": 3 * L * own}
    D, H, T, Dm, r = case["width"], case["heads"], case["tokens"], case["mlp"], case["lora"]
    M = case["batch"] * T
    n_full, n_live = L * H * case["full"], L * H * min(1.0, case["full"] + case["fwd"])
    head = 4.0 * M * 64 * (2 * D + T)             # Q, K, V, output projection and attention of one head, forward
    ffn = 4.0 * M * D * (Dm / H)                  # a head's share of the feed-forward network, forward
    flops = n_live * head
    back = 0.0 if case["kind"] == "forward" else 1.0
    if r:                                         # adapters only: no weight gradients of the base
        flops += n_live * 4.0 * M * r * (D + 64) + 2 * back * n_full * 4.0 * M * r * (D + 64)
        flops += back * n_full * head + (1 + back) * L * H * ffn
    else:
        flops += 2 * back * n_full * head
        flops += (n_live + 2 * back * n_full) * ffn if case["gate"] else (1 + 2 * back) * L * H * ffn
    weights = L * sum(sizes.values())
    grads = L * sum(sizes[n] for n in _trained(case)) if back else 0
    traffic = es * (weights + grads + (2 + 2 * back) * M * D)
    if case["kind"] == "finetune":
        K, px = 3 * case["patch"] ** 2, case["pixels"]
        flops += 4.0 * case["batch"] * (T - 1) * K * D + 6.0 * case["batch"] * case["classes"] * D
        traffic += es * (case["batch"] * 3 * px * px + 2 * D * K + 2 * case["classes"] * D)
        traffic += L * sum(sizes[n] for n in _trained(case)) * (2 * es + 16)   # weights out, gradients in, fp32 state in and out
    return {"bytes": traffic, "flops": flops}


def tolerance(case):
    if case["kind"] == "select":
        return {"rel": 1e-12}      # fp64 sums of exact terms: only their order is free
    if case["dtype"] == "f32":
        # against the same stack in fp64: up to 1e-6 (norm) and 2e-5 (largest)
        return {"rel": 4e-6, "max": 1e-4}
    # two kernel families of the same precision, 12 to 24 blocks: 7e-3 to 1.4e-2 (norm), 0.05 to 0.5 (largest)
    return {"rel": 2.8e-2, "max": 0.9}
