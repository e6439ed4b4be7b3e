"""GPU parity of the bf16 attention forward of 225 to 256 tokens: with few pairs of image and head, whose query tiles two
workgroups share, and with more."""
import pytest

import d2ft_inputs as di
from test_gpu_block import run_case

pytestmark = pytest.mark.gpu

FULL, FWD, SKIP = di.OP_FULL, di.OP_FWD, di.OP_SKIP


@pytest.mark.parametrize("tokens", [225, 256])
@pytest.mark.parametrize("batch", [1, 65])   # 2 and 130 live pairs
def test_query_tile_edges(tokens, batch):
    w = di.Workload("attn_pairs", batch, tokens, 64, 3, 64, 64, 1, "bf16")
    run_case(w, [FWD, SKIP, FULL], seed=91)


def test_last_call_with_two_workgroups_per_pair():
    w = di.Workload("attn_pairs_line", 64, 240, 64, 2, 64, 64, 1, "bf16")   # 128 pairs
    run_case(w, [FULL, FWD], seed=92)
