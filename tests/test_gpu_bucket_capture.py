"""GPU bucketing inside a captured graph: a call that has run once, of one workgroup (up to 4096
assignments), leaves the workspace that the two-kernel form of the next sizes needs, as a capture cannot
allocate it."""
import numpy as np
import pytest

import synth
from gpu_util import dev_i32, torch_or_skip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("warm", [16, 4096])
def test_capture_after_a_smaller_call(warm):
    torch = torch_or_skip()
    import paper_2607_19438_amd as q
    E, n = 128, 16384
    rng = synth.rng_for(83, warm)
    idx = [rng.integers(0, E, m).astype(np.int32) for m in (warm, n, n)]
    off = [dev_i32(torch, synth.offsets_from_idx(i, E)) for i in idx]
    q.release()                                               # no workspace from earlier tests
    q.moe_bucket(dev_i32(torch, idx[0]), off[0])
    torch.cuda.synchronize()
    tab, offs, perm = dev_i32(torch, idx[1]), off[1].clone(), torch.empty(n, dtype=torch.int32, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        q.moe_bucket(tab, offs, out=perm)
    for i in (1, 2, 1):                                       # replays on new contents
        tab.copy_(dev_i32(torch, idx[i]))
        offs.copy_(off[i])
        perm.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(perm.cpu().numpy(), np.argsort(idx[i], kind="stable").astype(np.int32))
