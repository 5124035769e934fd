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
# rows per group of four copies of the experts, from 130 columns on: narrower or fewer leave CUs without a
# workgroup and so take 32-row groups (Q4; and with Q8 128-row groups for means of 75 and 40 all the same)
FORMS = {synth.FMT_Q4: [0, 128, 64, 32, 32], synth.FMT_Q8: [0, 128, 128, 32, 32]}


@pytest.mark.parametrize("fmt", [synth.FMT_Q8, synth.FMT_Q4])
# K that is not whole stages ends on an odd or an even number of them: stages of four 64-wide steps (32- and
# 64-row groups) 32, 96, 160 one, 288, 416, 480 two, 544 three; of two (128-row groups) 32, 96 one, 160 two,
# 288 three, 416, 480 four, 544 five
@pytest.mark.parametrize("inter,K,misaligned", [(18, 32, False), (16, 96, False), (20, 160, False), (17, 256, False),
                                                (33, 288, False), (24, 416, False), (40, 480, False), (40, 544, False),
                                                (72, 768, False), (72, 768, True), (64, 2048, False)])
def test_direct_forms_bitwise(fmt, inter, K, misaligned):
    check_forms(fmt, inter, K, misaligned, 1)


@pytest.mark.parametrize("fmt", [synth.FMT_Q8, synth.FMT_Q4])
@pytest.mark.parametrize("inter,K,misaligned", [(130, 32, False), (144, 96, False), (131, 160, False), (145, 256, False),
                                                (137, 288, False), (152, 416, False), (168, 480, False), (160, 544, False),
                                                (136, 768, False), (136, 768, True), (130, 1024, False)])
def test_direct_forms_bitwise_all_heights(fmt, inter, K, misaligned):
    check_forms(fmt, inter, K, misaligned, 4)


def check_forms(fmt, inter, K, misaligned, copies):
    """The same rows in launches of every form; `copies` sets of the experts on the same weights."""
    torch = torch_or_skip()
    import paper_2607_19438_amd as m
    rng = synth.rng_for(61, fmt, inter, K, *COUNTS)
    idx = np.repeat(np.arange(len(COUNTS) * copies, dtype=np.int32), COUNTS * copies)
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
    for E in (e * copies for e in EXPERTS):
        n = E - copies * len(ws)
        table = m.ExpertTable(wq * copies + [wq[0]] * n, sc * copies + [sc[0]] * n, fmt)
        r = synth.routing_from_idx(idx, E, 1, np.ones(idx.size, np.float32))
        off = dev_i32(torch, r.expert_offsets)
        perm = m.moe_bucket(dev_i32(torch, r.token_expert_idx), off)
        y = m.moe_grouped(xd, perm, off, table, None, 1, fmt)
        h = m.moe_gate_up_swiglu(xd, perm, off, table, None, 1, fmt)
        torch.cuda.synchronize()
        ys.append(y.cpu().numpy())
        hs.append(h.cpu().view(torch.int16).numpy())
    for E, y, h in zip([e * copies for e in EXPERTS], ys, hs):
        assert np.array_equal(y.view(np.uint32), ys[0].view(np.uint32)), E
        assert np.array_equal(h, hs[0]), E
    r = synth.routing_from_idx(idx % len(ws), len(ws), 1, np.ones(idx.size, np.float32))
    args = (x, r.token_expert_idx, r.expert_offsets, [w.wq for w in ws], [w.scales for w in ws], 1, fmt)
    check_levels(f"moe direct inter={inter} K={K} {synth.FMT_NAMES[fmt]}", ys[-1], oracle.moe(*args),
                 oracle.moe(*args, bf16_weights=True), K, K >= 512)
