"""The forward's products on 128x256 tiles with two workgroups to a CU, where launch_gemm_mfma picks them."""
import numpy as np
import pytest
import torch

import paper_2504_12471_amd as P

pytestmark = pytest.mark.gpu


# (images, tokens, width, heads, hidden units, gated, some heads skipped): remainders of the 128 rows, of the 256 columns (and
# of a wavefront's 64), one slab of K and several, the workgroups' second to fourth tile, live heads that are no prefix of
# the weights
@pytest.mark.parametrize("B,T,D,H,Dm,gate,skip,kinds", [(64, 197, 768, 12, 3072, False, True, "1"), (83, 190, 384, 6, 1536, False, True, "1"),
                                                        (96, 181, 448, 7, 1792, True, True, "1"), (96, 193, 64, 1, 2568, False, False, "1"),
                                                        (91, 181, 192, 3, 2056, False, True, "1"), (96, 181, 448, 7, 1792, False, False, "01")])
def test_forward_block(B, T, D, H, Dm, gate, skip, kinds):
    gen = torch.Generator(device="cuda").manual_seed(B * T)

    def rand(*shape, mean=0.0, std=0.02):
        return (torch.randn(shape, generator=gen, device="cuda") * std + mean).to(torch.bfloat16)

    w = {"ln1_g": rand(D, mean=1.0), "ln1_b": rand(D), "w_qkv": rand(3, H, 64, D), "b_qkv": rand(3, H, 64), "w_o": rand(D, 64 * H),
         "b_o": rand(D), "ln2_g": rand(D, mean=1.0), "ln2_b": rand(D), "w1": rand(Dm, D), "b1": rand(Dm), "w2": rand(D, Dm), "b2": rand(D)}
    x = rand(B, T, D, std=1.0)
    ops = np.array([[P.OP_FULL if h % 3 != 1 or not skip else P.OP_SKIP for h in range(H)]], dtype=np.uint8)
    desc = P.make_desc(B, T, D, H, Dm, "bf16", flags=P.FLAG_GATE_FFN if gate else 0)
    st = P.BlockStack(desc, [w], "bf16", [])
    P.d2ft_timing_enable(True)
    try:
        y = st.forward(x, ops)
        labels = [r["name"] for r in P.d2ft_timing_read()]
    finally:
        P.d2ft_timing_enable(False)
    for kind in kinds:   # 0: the projections to Q, K, V; 1: the first feed-forward product with its GELU
        assert any(n.startswith("gemm_pair_kernel<" + kind) for n in labels), labels

    # the block in fp32, with the bf16 results that the block stores rounded as it rounds them
    def r16(t):
        return t.to(torch.bfloat16).float()

    f = {k: v.float() for k, v in w.items()}
    xf = x.float().reshape(-1, D)
    live = [h for h in range(H) if ops[0, h] != P.OP_SKIP]
    u = r16(torch.nn.functional.layer_norm(xf, (D,), f["ln1_g"], f["ln1_b"], 1e-6))
    o = torch.zeros(B * T, 64 * H, device="cuda")
    for h in live:
        q, k, v = (r16(u @ f["w_qkv"][i, h].T + f["b_qkv"][i, h]).reshape(B, T, 64) for i in range(3))
        s = torch.softmax(q @ k.transpose(1, 2).contiguous() / 8.0, -1)
        o[:, 64 * h:64 * h + 64] = r16(s @ v).reshape(-1, 64)
    x1 = r16(xf + o @ f["w_o"].T + f["b_o"])
    v2 = r16(torch.nn.functional.layer_norm(x1, (D,), f["ln2_g"], f["ln2_b"], 1e-6))
    hid = torch.arange(Dm, device="cuda")
    if gate:
        hid = torch.cat([torch.arange(h * Dm // H, (h + 1) * Dm // H, device="cuda") for h in live])
    g = r16(torch.nn.functional.gelu(v2 @ f["w1"][hid].T + f["b1"][hid]))
    ref = (x1 + g @ f["w2"][:, hid].T + f["b2"]).reshape(B, T, D)
    # eight roundings of 2^-9 on the way to y, of terms no larger than it: in the norm they add in quadrature (below 2^-9 * 3);
    # a row, column or slab in the wrong place is off by its whole share
    err = (y.float() - ref).norm() / ref.norm()
    assert err < 6e-3, float(err)
    rows = (y.float() - ref).abs().amax(-1) / ref.pow(2).mean().sqrt()
    assert rows.max() < 0.1, float(rows.max())
