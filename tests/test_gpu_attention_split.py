"""GPU parity of both forms of the prefill attention kernel: a query's keys split over two waves (few
workgroups) at the edges of its 32-key tiles, and the unsplit form (many workgroups) with and without the
causal mask. Every output element against the oracle."""
import pytest

import synth
from test_gpu_attention import check_full, run
from gpu_util import torch_or_skip

pytestmark = pytest.mark.gpu

SPLIT = [(1, S, 3, 3, D) for S in (31, 32, 33, 63, 65, 95, 96, 97, 161) for D in (64, 128)]
# more than 400 (causal, 640 with D = 64) and 256 workgroups of 128 rows; the last one at the limit
MANY = [(9, 130, 36, 4, 128), (9, 130, 36, 4, 64), (5, 129, 66, 11, 64), (5, 257, 27, 3, 128), (5, 129, 64, 8, 64)]


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,S,H,Hkv,D", SPLIT + MANY)
def test_attention_forms(B, S, H, Hkv, D, causal):
    torch = torch_or_skip()
    case = synth.attn_case(f"attn_forms_{B}x{S}x{H}/{Hkv}x{D}_{'c' if causal else 'f'}", B, S, H, Hkv, D, causal,
                           seed=91, stream=(B, S, H, Hkv, D), q_std=4.0)
    check_full(torch, case)
    assert torch.equal(run(torch, case), run(torch, case))
