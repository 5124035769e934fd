"""GPU parity of both forms of the prefill attention kernel: a query's keys split over two waves (few
workgroups) at the edges of its 32-key tiles, and the unsplit form (many workgroups) with and without the
causal mask. Every output element against the oracle."""
import pytest

import synth
from test_gpu_attention import check_full, run
from gpu_util import torch_or_skip

pytestmark = pytest.mark.gpu

SPLIT_BOTH = [(1, S, 3, 3, D) for S in (73, 95, 96, 97, 127, 161) for D in (64, 128)]   # with and without the mask
SPLIT = SPLIT_BOTH + [(1, S, 3, 3, D) for S in (31, 32, 33, 63, 64, 65) for D in (64, 128)]   # split from 65 on if causal
# too many workgroups to split, and at a limit with the mask (split)
MANY = [(9, 130, 36, 4, 128), (10, 130, 36, 4, 64), (5, 129, 72, 12, 64), (5, 257, 27, 3, 128)]
LIMIT = [(9, 130, 36, 4, 64), (5, 129, 66, 11, 64), (5, 129, 64, 8, 64), (2, 129, 88, 11, 128), (8, 300, 12, 3, 128)]


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,S,H,Hkv,D", SPLIT + MANY + LIMIT)
def test_attention_forms(B, S, H, Hkv, D, causal):
    torch = torch_or_skip()
    case = synth.attn_case(f"attn_forms_{B}x{S}x{H}/{Hkv}x{D}_{'c' if causal else 'f'}", B, S, H, Hkv, D, causal,
                           seed=91, stream=(B, S, H, Hkv, D), q_std=4.0)
    check_full(torch, case)
    assert torch.equal(run(torch, case), run(torch, case))


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,S,H,Hkv,D", [(1, 40, 3, 3, 64), (1, 97, 3, 3, 64), (1, 97, 3, 3, 128), (5, 129, 66, 11, 64), (9, 130, 36, 4, 128)])
def test_attention_keys_scoring_minus_infinity(B, S, H, Hkv, D, causal):
    """Keys 32..63 score -inf for every query (their first element is -inf, the queries' is positive): they
    take no weight in either form, also where they are all that one of two waves has seen."""
    import paper_2607_19438_amd as qg
    torch = torch_or_skip()
    gen = torch.Generator().manual_seed(7)
    q, k, v = (torch.randn((B, S, h, D), generator=gen).to(torch.bfloat16) for h in (H, Hkv, Hkv))
    q[..., 0] = q[..., 0].abs() + 0.5
    k[:, 32:64, :, 0] = -float("inf")
    o = qg.attention_prefill(q.cuda(), k.cuda(), v.cuda(), causal=causal)
    kk, vv = (t.double().repeat_interleave(H // Hkv, dim=2) for t in (k, v))
    s = torch.einsum("bqhd,bkhd->bhqk", q.double(), kk) / D ** 0.5
    if causal:
        s.masked_fill_(torch.ones(S, S, dtype=torch.bool).triu(1), -float("inf"))
    ref = torch.einsum("bhqk,bkhd->bqhd", torch.softmax(s, dim=-1), vv)
    # probabilities and outputs each rounded to bf16 (2^-9 relative), |sum p v| <= max |v|
    assert (o.cpu().double() - ref).abs().max().item() <= 2 ** -8 * float(vv.abs().max())
