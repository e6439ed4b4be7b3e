"""GPU parity of the bf16 attention forward of 225 to 256 tokens: with few pairs of image and head, whose query tiles two
workgroups share, and with more."""
import pytest

import d2ft_inputs as di
from test_gpu_block import run_case
from test_gpu_ln_product import kernels_of

pytestmark = pytest.mark.gpu

FULL, FWD, SKIP = di.OP_FULL, di.OP_FWD, di.OP_SKIP


@pytest.mark.parametrize("tokens", [225, 256])
@pytest.mark.parametrize("batch", [1, 65])   # 2 and 130 live pairs
def test_query_tile_edges(tokens, batch):
    w = di.Workload("attn_pairs", batch, tokens, 64, 3, 64, 64, 1, "bf16")
    names = kernels_of(lambda: run_case(w, [FWD, SKIP, FULL], seed=91))
    assert ("attn_fwd_mfma" if batch == 65 else "attn_fwd_mfma, two per pair") in names, names


def test_last_call_with_two_workgroups_per_pair():
    w = di.Workload("attn_pairs_line", 64, 240, 64, 2, 64, 64, 1, "bf16")   # 128 pairs
    names = kernels_of(lambda: run_case(w, [FULL, FWD], seed=92))
    assert "attn_fwd_mfma, two per pair" in names, names
