"""GPU dense GEMM inside a captured graph: a call that has run once leaves the workspace that the split-K
partials of another call of its range need, though it runs unsplit itself or with fewer splits, as a capture
cannot allocate it."""
import pytest

import synth
from gpu_util import torch_or_skip

pytestmark = pytest.mark.gpu


def inputs(torch, fmt, M, N, K, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((M, K), device="cuda", generator=gen).to(torch.bfloat16)
    if fmt == synth.FMT_Q8:
        wq = torch.randint(-127, 128, (N, K), dtype=torch.int8, device="cuda", generator=gen)
    else:
        wq = torch.randint(0, 256, (N, K // 2), dtype=torch.uint8, device="cuda", generator=gen)
    return x, wq, (0.005 + 0.01 * torch.rand((N, K // 32), device="cuda", generator=gen)).to(torch.float16)


@pytest.mark.parametrize("warm_fmt,warm,fmt,call", [
    (synth.FMT_Q4, (16, 2048, 2048), synth.FMT_Q4, (5, 2048, 8192)),       # unsplit, then four splits
    (synth.FMT_Q8, (128, 1024, 512), synth.FMT_Q8, (24, 1024, 4096)),      # unsplit, then eight
    (synth.FMT_Q8, (600, 4096, 4096), synth.FMT_Q4, (590, 4096, 4096)),    # two splits of 256x128, then three of 128x256
])
def test_capture_after_another_call(warm_fmt, warm, fmt, call):
    torch = torch_or_skip()
    import paper_2607_19438_amd as q
    first = inputs(torch, warm_fmt, *warm, 85)
    x, wq, scales = inputs(torch, fmt, *call, 86)
    x2 = inputs(torch, fmt, *call, 87)[0]
    xin = x.clone()
    y = torch.empty((call[0], call[1]), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    q.release()                                               # no workspace from earlier tests
    q.dense(*first, warm_fmt)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        q.dense(xin, wq, scales, fmt, out=y)
    for src in (x, x2, x):                                    # replays on new contents
        xin.copy_(src)
        y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, q.dense(src, wq, scales, fmt))
