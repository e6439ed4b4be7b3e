"""The bf16 attention backward of up to 224 tokens with more pairs than the chip holds at once, so that workgroups take a second
and third one, at token counts on and beside the edges of its 32-token tiles."""
import pytest

import d2ft_inputs as di
from test_gpu_block import run_case
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
