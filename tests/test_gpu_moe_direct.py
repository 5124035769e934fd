"""GPU parity of the MoE kernel for few rows per expert, at the edges of its forms: 32-, 64- and
128-row groups (chosen by the mean rows per expert), K that is and is not whole stages, scale arrays
whose rows are not naturally aligned, ragged N and SwiGLU widths, and more experts than one launch
covers.

One routing runs in launches padded with different numbers of empty experts, which moves the mean and so
the kernel; every launch gives the same bits, and they meet the oracle's bar.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import check_levels, dev_i32, dev_x, torch_or_skip

pytestmark = pytest.mark.gpu

COUNTS = [129, 1, 32, 33, 0, 64, 65, 128, 31, 500]     # 983 rows
# experts in the launch -> mean rows 98 (staged tiles), 75, 40, 14, and two launches of 128 and 72
EXPERTS = [10, 13, 24, 70, 200]


@pytest.mark.parametrize("fmt", [synth.FMT_Q8, synth.FMT_Q4])
# K that is not whole stages ends on an odd or an even number of them: stages of four 64-wide steps (32- and
# 64-row groups) 32, 96, 160 one, 288, 416, 480 two, 544 three; of two (128-row groups) 32, 96 one, 160 two,
# 288 three, 416, 480 four, 544 five
@pytest.mark.parametrize("inter,K,misaligned", [(18, 32, False), (16, 96, False), (20, 160, False), (17, 256, False),
                                                (33, 288, False), (24, 416, False), (40, 480, False), (40, 544, False),
                                                (72, 768, False), (72, 768, True), (64, 2048, False)])
def test_direct_forms_bitwise(fmt, inter, K, misaligned):
    torch = torch_or_skip()
    import paper_2607_19438_amd as m
    rng = synth.rng_for(61, fmt, inter, K, *COUNTS)
    idx = np.repeat(np.arange(len(COUNTS), dtype=np.int32), COUNTS)
    rng.shuffle(idx)
    x = synth.make_x(rng, idx.size, K)
    ws = [synth.make_qweight(rng, 2 * inter, K, fmt) for _ in COUNTS]
    wq = [torch.from_numpy(w.wq).cuda() for w in ws]
    sc = []
    for w in ws:
        pad = torch.zeros(w.scales.size + 1, dtype=torch.float16, device="cuda")
        s = pad[1:] if misaligned else pad[:-1]
        s.copy_(torch.from_numpy(w.scales.reshape(-1)))
        sc.append(s.reshape(w.scales.shape))
    xd = dev_x(torch, x)
    ys, hs = [], []
    for E in EXPERTS:
        n = E - len(ws)
        table = m.ExpertTable(wq + [wq[0]] * n, sc + [sc[0]] * n, fmt)
        r = synth.routing_from_idx(idx, E, 1, np.ones(idx.size, np.float32))
        off = dev_i32(torch, r.expert_offsets)
        perm = m.moe_bucket(dev_i32(torch, r.token_expert_idx), off)
        y = m.moe_grouped(xd, perm, off, table, None, 1, fmt)
        h = m.moe_gate_up_swiglu(xd, perm, off, table, None, 1, fmt)
        torch.cuda.synchronize()
        ys.append(y.cpu().numpy())
        hs.append(h.cpu().view(torch.int16).numpy())
    for E, y, h in zip(EXPERTS, ys, hs):
        assert np.array_equal(y.view(np.uint32), ys[0].view(np.uint32)), E
        assert np.array_equal(h, hs[0]), E
    r = synth.routing_from_idx(idx, len(ws), 1, np.ones(idx.size, np.float32))
    args = (x, r.token_expert_idx, r.expert_offsets, [w.wq for w in ws], [w.scales for w in ws], 1, fmt)
    check_levels(f"moe direct inter={inter} K={K} {synth.FMT_NAMES[fmt]}", ys[-1], oracle.moe(*args),
                 oracle.moe(*args, bf16_weights=True), K, K >= 512)
