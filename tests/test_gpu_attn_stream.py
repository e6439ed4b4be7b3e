"""GPU parity of the streaming attention kernels (kernels_attn_stream.hip) through one block forward + backward: token
counts at and beside the edges of tiles, stages and workgroups, the smallest and the largest."""
import pytest

import d2ft_inputs as di
from test_gpu_block import run_case

pytestmark = pytest.mark.gpu

FULL, FWD, SKIP = di.OP_FULL, di.OP_FWD, di.OP_SKIP


@pytest.mark.parametrize("tokens", [1, 31, 32, 33, 64, 127, 128, 129, 257])
def test_fp32_token_edges(tokens):
    run_case(di.Workload("stream_f32", 2, tokens, 128, 3, 64, 64, 1, "f32"), [FULL, FWD, FULL], seed=81)


@pytest.mark.parametrize("tokens", [225, 256, 257, 289, 320, 577])
def test_bf16_token_edges(tokens):
    run_case(di.Workload("stream_bf16", 2, tokens, 128, 3, 64, 64, 1, "bf16"), [FWD, FULL, FULL], seed=82)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_most_tokens(dtype):
    run_case(di.Workload("stream_max", 1, 1024, 64, 2, 64, 64, 1, dtype), [FULL, FWD], seed=83)


@pytest.mark.parametrize("tokens", [17, 64, 65, 128, 129, 197, 224])
def test_bf16_few_pairs_below_225_tokens(tokens):
    run_case(di.Workload("stream_few", 3, tokens, 128, 3, 64, 64, 1, "bf16"), [FULL, FWD, FULL], seed=84)
