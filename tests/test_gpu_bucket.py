"""GPU bucketing at the edges of its one-workgroup form (4096 assignments, 512 experts): whole and ragged
runs per wave, the first sizes of the two-kernel form, empty experts, and tables that disagree."""
import numpy as np
import pytest

import synth
from gpu_util import dev_i32, torch_or_skip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 65, 1023, 1024, 1025, 4095, 4096, 4097])
@pytest.mark.parametrize("E", [1, 2, 100, 512, 513])
def test_bucket_is_stable(n, E):
    torch = torch_or_skip()
    import paper_2607_19438_amd as q
    rng = synth.rng_for(81, n, E)
    idx = (E * rng.random(n) ** 2).astype(np.int32)          # skewed: late experts thin or empty
    perm = q.moe_bucket(dev_i32(torch, idx), dev_i32(torch, synth.offsets_from_idx(idx, E)))
    torch.cuda.synchronize()
    assert np.array_equal(perm.cpu().numpy(), np.argsort(idx, kind="stable").astype(np.int32))


@pytest.mark.parametrize("n", [700, 4097])
def test_bucket_of_disagreeing_tables(n):
    """An expert whose count is not its segment's length gets -1 entries; the others are bucketed."""
    torch = torch_or_skip()
    import paper_2607_19438_amd as q
    E = 6
    idx = (np.arange(n) % E).astype(np.int32)
    off = synth.offsets_from_idx(idx, E)
    bad = idx.copy()
    bad[6 * 20 + 2] = 3                                       # expert 2 one short, expert 3 one over
    bad[6 * 30 + 5] = E                                       # out of range: expert 5 one short
    perm = q.moe_bucket(dev_i32(torch, bad), dev_i32(torch, off))
    torch.cuda.synchronize()
    p = perm.cpu().numpy()
    for e in range(E):
        seg = p[off[e]:off[e + 1]]
        if e in (2, 3, 5):
            assert (seg == -1).all()
        else:
            assert np.array_equal(seg, np.nonzero(idx == e)[0])
