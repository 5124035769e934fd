"""GPU parity of the half-size dense tiles, 256x128 (most calls of 256 rows and more that few 256x256 tiles
would fill the chip for) and 128x256 (from 129 rows, and where 256x128 needs more rounds): partial row and
column tiles, K splits with ragged last steps, both formats."""
import pytest

import oracle
import synth
from gpu_util import check_levels, dev_w, dev_x, torch_or_skip

pytestmark = pytest.mark.gpu


# rows just past 256 and 512, columns just past a tile, K of whole and half steps; one, two and eight splits
@pytest.mark.parametrize("fmt", [synth.FMT_Q8, synth.FMT_Q4])
@pytest.mark.parametrize("M,N,K", [(256, 256, 64), (260, 300, 96), (257, 384, 800), (513, 260, 1568), (384, 257 * 4, 6176),
                                   (1024, 640, 2080)])
def test_tall_tiles(fmt, M, N, K):
    check_tile("tall", fmt, M, N, K)


# 128x256: two, five and eight splits; unsplit just past 128 and 129 rows, K of less than one step; one round where
# 256x128 needs two, with partial row tiles
@pytest.mark.parametrize("fmt", [synth.FMT_Q8, synth.FMT_Q4])
@pytest.mark.parametrize("M,N,K", [(132, 260, 1568), (200, 1000, 4128), (252, 512, 6176), (129, 256 * 130, 32), (250, 604, 96),
                                   (1028, 6912, 96)])
def test_wide_tiles(fmt, M, N, K):
    check_tile("wide", fmt, M, N, K)


def check_tile(name, fmt, M, N, K):
    torch = torch_or_skip()
    import paper_2607_19438_amd as q
    case = synth.dense_case(name, fmt, M, N, K, seed=71, stream=(M, N, K))
    x = dev_x(torch, case.x)
    wq, sc = dev_w(torch, case.w)
    y = torch.full((M + 2, N), 7.5, dtype=torch.float32, device="cuda")
    q.dense(x, wq, sc, fmt, out=y[1:M + 1])
    y2 = q.dense(x, wq, sc, fmt)
    torch.cuda.synchronize()
    assert torch.equal(y[1:M + 1], y2)
    assert bool((y[0] == 7.5).all()) and bool((y[M + 1] == 7.5).all())
    ref = oracle.dense(case.x, case.w.wq, case.w.scales, fmt)
    refb = oracle.dense(case.x, case.w.wq, case.w.scales, fmt, bf16_weights=True)
    check_levels(f"dense {name} {M}x{N}x{K} {synth.FMT_NAMES[fmt]}", y2.cpu().numpy(), ref, refb, K, K >= 512)
