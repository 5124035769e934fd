"""Host-side checks of the rules that pick a tile from a call's sizes (``tile_rules.hpp``), compiled by
itself with the host compiler. No test here touches a GPU.

Dense, 256 to 2048 rows: the half-size tile is 256x128 or 128x256, whichever needs fewer rounds of one
workgroup per CU and fewer K steps, so that a call does not pay a second round, or chains of K twice as long,
for the tile's shape alone.
"""
import os
import random
import subprocess
import sys

import pytest

from paper_2607_19438_amd import build

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

MAIN = """
#include <cstdio>
#include "tile_rules.hpp"
int main() {
  char what;
  long q4, a, b, c, d;
  while (std::scanf(" %c %ld %ld %ld %ld %ld", &what, &q4, &a, &b, &c, &d) == 6) {
    if (what == 'd') {
      const qg::DensePlan p = qg::dense_plan(q4 != 0, a, b, c);
      std::printf("%d %d\\n", (int)p.tile, p.splits);
    } else if (what == 'k') {
      const qg::DensePlan p = qg::dense_plan(q4 != 0, a, b, c);
      std::printf("%d %d\\n", p.splits, p.keep);
    } else if (what == 'a') {
      std::printf("%d 0\\n", (int)qg::attn_split(q4 != 0, a != 0, b, c));
    } else if (what == 's') {
      const qg::SmallPlan p = qg::small_plan(a <= 16 ? 1 : a <= 32 ? 2 : a <= 64 ? 4 : 8, (b + 31) / 32, c, q4 ? 128 : 64);
      std::printf("%ld %ld\\n", p.splits, p.keep);
    } else {
      const int rows = qg::moe_direct_rows(q4 != 0, d != 0, a, b, c);
      std::printf("%d %ld\\n", rows, rows ? qg::moe_direct_groups(rows, a, b) * qg::moe_direct_tiles(rows, d != 0, c) : 0);
    }
  }
}
"""
TILES = [(256, 256), (256, 128), (128, 256), (128, 128)]     # in the order of the enumeration


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "rules")
    subprocess.run(["g++", "-std=c++20", "-Wall", "-Werror", "-I", build.CSRC, str(d / "main.cpp"), "-o", exe], check=True)

    def run(what, calls):
        text = "".join(" ".join([what, *(str(int(v)) for v in c), *["0"] * (5 - len(c))]) + "\n" for c in calls)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split()
        return [(int(out[i]), int(out[i + 1])) for i in range(0, len(out), 2)]
    return run


@pytest.fixture(scope="module")
def plans(rules):
    return lambda calls: [(TILES[t], s) for t, s in rules("d", calls)]


@pytest.fixture(scope="module")
def direct(rules):
    """(rows per group, workgroups of one launch) of calls (q4, rows, experts, columns, fused gate/up)."""
    return lambda calls: rules("m", calls)


def cd(a, b):
    return -(-a // b)


def rounds_steps(tile, splits, M, N, K):
    items = cd(M, tile[0]) * cd(N, tile[1]) * splits
    return cd(items, 256), cd(cd(K, 64), splits)


@pytest.mark.parametrize("M,N,K", [(1100, 7168, 2048), (1904, 4285, 3040), (1028, 6912, 2048), (640, 11008, 4096),
                                   (785, 8448, 1984), (803, 8232, 8064)])
def test_dense_takes_one_round_where_a_half_size_tile_has_it(plans, M, N, K):
    for q4 in (False, True):
        ((tile, splits),) = plans([(q4, M, N, K)])
        assert tile == (128, 256) and rounds_steps(tile, splits, M, N, K)[0] == 1


@pytest.mark.parametrize("q4,M,N,K,tile,splits", [
    (True, 600, 4096, 4096, (128, 256), 3), (True, 576, 6340, 3360, (128, 256), 2),
    (False, 590, 5760, 7200, (128, 256), 2), (True, 590, 5760, 7200, (128, 256), 2),
    (False, 600, 4096, 4096, (256, 128), 2),                 # Q8: a 256x128 step is so much cheaper
    (True, 512, 8192, 3072, (256, 128), 2), (True, 1024, 4096, 4096, (256, 128), 2), (True, 768, 1536, 2048, (256, 128), 2),
    (True, 1536, 4096, 4096, (256, 128), 1), (False, 512, 2048, 2048, (256, 128), 2), (False, 2048, 4096, 2048, (256, 128), 1),
    (False, 300, 5000, 4096, (256, 128), 3), (False, 2048, 2048, 8192, (256, 256), 4), (False, 2048, 8192, 2048, (256, 256), 1),
    (False, 1506, 2688, 7616, (256, 128), 2), (True, 1154, 3088, 576, (128, 128), 1),
    (False, 200, 1000, 4128, (128, 256), 5), (False, 255, 257, 288, (128, 128), 1)])
def test_dense_measured_calls(plans, q4, M, N, K, tile, splits):
    assert plans([(q4, M, N, K)]) == [(tile, splits)]


def test_dense_half_size_tiles_never_add_a_round(plans):
    """Against the same call on the other half-size tile with the splits that it would get: no more rounds,
    and within one round no more than 1.5 times the K steps plus a split's cost."""
    rng = random.Random(5)
    calls = []
    while len(calls) < 4000:
        M, N, K = int(256 * 8 ** rng.random()), int(256 * 64 ** rng.random()), 32 * int(16 * 16 ** rng.random())
        if M * N % 4 == 0:
            calls.append((rng.random() < 0.5, M, N, K))
    seen = set()
    for (q4, M, N, K), (tile, splits) in zip(calls, plans(calls)):
        assert 1 <= splits <= 8 and (splits == 1 or cd(K, 64) // splits >= 12)
        if tile not in ((256, 128), (128, 256)):
            continue
        seen.add(tile)
        other = tile[::-1]
        S = max(1, min(8, 256 // (cd(M, other[0]) * cd(N, other[1]))))
        while S > 1 and cd(K, 64) // S < 12:
            S -= 1
        r, s = rounds_steps(tile, splits, M, N, K)
        r2, s2 = rounds_steps(other, S, M, N, K)
        sums = 6 + S * M * N / 2 ** 20 if S > 1 else 0
        assert r <= r2, (q4, M, N, K)
        if r == 1 and tile == (256, 128):
            assert s <= 1.5 * s2 + sums, (q4, M, N, K)
    assert seen == {(256, 128), (128, 256)}


@pytest.mark.parametrize("q4,T,E,topk,hidden,inter,rows", [
    # Q4: 32 rows up to a mean of 16 and below 4096 rows in all, 64 up to 48, 128 up to 80
    (True, 4, 128, 8, 2048, 768, (32, 32)), (True, 256, 128, 8, 2048, 768, (32, 32)), (True, 272, 128, 8, 2048, 768, (64, 64)),
    (True, 511, 256, 8, 4096, 2048, (32, 32)), (True, 512, 256, 8, 4096, 2048, (64, 64)), (True, 783, 128, 8, 2048, 768, (64, 64)), (True, 784, 128, 8, 2048, 768, (128, 128)),
    (True, 1295, 128, 8, 2048, 768, (128, 128)), (True, 1296, 128, 8, 2048, 768, (0, 0)),
    # and 32 rows on while 64 would leave CUs without a workgroup
    (True, 128, 8, 2, 4096, 2048, (32, 32)), (True, 256, 16, 2, 1024, 512, (32, 32)), (True, 512, 16, 2, 1024, 512, (32, 32)),
    (True, 128, 8, 2, 4096, 14336, (64, 32)),
    (True, 2876, 64, 1, 896, 384, (64, 64)), (True, 160, 8, 2, 2048, 1984, (64, 32)), (True, 160, 8, 2, 2048, 1920, (32, 32)),
    # Q8: 32 rows up to a mean of 20 (32 while 128 leaves CUs without a workgroup), 128 up to 96
    (False, 128, 64, 6, 2048, 1056, (32, 32)), (False, 223, 64, 6, 2048, 1056, (32, 32)), (False, 224, 64, 6, 2048, 1056, (128, 128)), (False, 512, 128, 8, 2048, 768, (128, 128)),
    (False, 192, 16, 2, 1024, 512, (32, 32)), (False, 300, 16, 2, 1024, 512, (128, 128)),
    (False, 777, 64, 6, 2048, 1056, (128, 128)), (False, 1034, 64, 6, 2048, 1056, (128, 128)), (False, 1035, 64, 6, 2048, 1056, (0, 0))])
def test_direct_rows(direct, q4, T, E, topk, hidden, inter, rows):
    """Rows per group of the gate/up and the down projection."""
    M = T * topk
    assert tuple(r for r, _ in direct([(q4, M, E, inter, True), (q4, M, E, hidden, False)])) == rows


@pytest.mark.parametrize("q4,M,E,cols,swi", [(False, 65536, 4096, 494400, True), (True, 128, 128, (1 << 23) + 64, True),
                                             (False, 128, 128, (1 << 24) + 128, False), (True, 4096, 128, 1 << 24, False)])
def test_direct_grid_of_2_to_the_32_threads_is_left_to_the_staged_tiles(direct, q4, M, E, cols, swi):
    """The runtime counts a grid's threads in 32 bits: more of them wrap, and part of the output stays unwritten."""
    assert direct([(q4, M, E, cols, swi)])[0][0] == 0
    (rows, groups), = direct([(q4, M, E, cols // 8, swi)])
    assert rows > 0 and 0 < groups * 64 * (8 if rows == 64 else 4) < 1 << 32


def test_direct_limits_that_the_gpu_tests_straddle(direct):
    import test_gpu_moe_direct as forms
    import test_gpu_moe_fewrows as few
    for fmt, inter, _, below, above, rows_below, rows_above in few.LIMITS:
        for (E, M), rows in ((below, rows_below), (above, rows_above)):
            q4 = fmt == few.synth.FMT_Q4
            got = direct([(q4, M, E, inter, True), (q4, M, E, 2 * inter, False)])
            assert [r for r, _ in got] == [rows, rows], (fmt, E, M)
    for fmt, rows in forms.FORMS.items():
        q4 = fmt == few.synth.FMT_Q4
        M, E = 4 * sum(forms.COUNTS), [4 * e for e in forms.EXPERTS]
        for inter in (130, 168):
            assert [direct([(q4, M, e, inter, True)])[0][0] for e in E] == rows
            assert [direct([(q4, M, e, 2 * inter, False)])[0][0] for e in E] == rows


def random_dense(rng, m_lo, m_hi, n):
    out = []
    while len(out) < n:
        M, N, K = int(m_lo * (m_hi / m_lo) ** rng.random()), int(64 * 128 ** rng.random()), 32 * int(4 * 100 ** rng.random())
        out.append((rng.random() < 0.5, M, N, K))
    return out


def test_small_workspace_holds_the_split_that_fills_the_chip(rules):
    """A short K runs unsplit, but the call leaves the partials' workspace of the split over 256 workgroups, as a
    later capture cannot allocate it."""
    assert rules("s", [(True, 16, 2048, 2048), (False, 128, 1024, 512), (False, 1, 8192, 2048)]) == [(1, 4), (1, 2), (1, 1)]
    calls = random_dense(random.Random(6), 1, 128, 2000)
    fewer = 0
    for (q4, M, N, K), (splits, keep) in zip(calls, rules("s", calls)):
        nc = cd(K, 128 if q4 else 64)
        S = min(nc, cd(256, cd(N, 32)))
        if M > 16:
            S = min(S, max(1, nc // 4))
        S = max(S, cd(nc, 64))
        assert 1 <= splits <= keep == max(splits, cd(nc, cd(nc, S))), (q4, M, N, K)
        fewer += splits < keep
    assert fewer > 200


def test_dense_workspace_holds_the_splits_of_the_other_tiles(rules):
    """256x128 tiles take fewer splits of K than the tiles that they replace; the workspace is sized for those."""
    assert rules("k", [(True, 576, 1024, 4096), (False, 2048, 2048, 8192), (True, 1100, 7168, 2048)]) == [(5, 5), (4, 4), (1, 1)]
    calls = random_dense(random.Random(7), 129, 4096, 4000)
    fewer = 0
    for (q4, M, N, K), (splits, keep) in zip(calls, rules("k", calls)):
        big, wide, S = cd(M, 256) * cd(N, 256), cd(M, 128) * cd(N, 256), 1
        if M * N % 4 == 0 and N >= 256 and not (M >= 256 and big >= 200):
            if M <= 1024 or (M <= 2048 and wide > 128):
                S = min(8, 256 // wide)
            elif M >= 256:
                S = min(8, cd(256, big))
        while S > 1 and cd(K, 64) // S < 12:
            S -= 1
        assert keep == max(splits, S, 1), (q4, M, N, K)
        fewer += splits < keep
    assert fewer


@pytest.mark.parametrize("D,causal,S,heads,split", [
    # one key block, or a second one of a few keys: nothing to halve
    (128, True, 64, 64, 0), (64, False, 64, 8, 0), (128, True, 65, 64, 1), (128, False, 72, 64, 0), (128, False, 73, 64, 1),
    # one 64-row workgroup per CU, and one head more
    (128, False, 96, 128, 1), (128, False, 96, 129, 0), (128, True, 96, 128, 1), (128, True, 96, 136, 0), (64, True, 96, 136, 1),
    # two (four) per CU
    (128, True, 300, 96, 1), (128, True, 300, 120, 0), (128, True, 192, 128, 0), (128, True, 512, 64, 1), (128, True, 512, 62, 0),
    (128, False, 512, 64, 1), (128, False, 512, 72, 0), (64, True, 96, 384, 1), (64, True, 96, 392, 0), (64, True, 300, 204, 1),
    # long causal chains
    (128, True, 700, 48, 1), (128, True, 700, 64, 0), (128, True, 1024, 48, 1), (128, True, 2048, 25, 1), (128, True, 2048, 32, 0),
    (64, True, 2048, 32, 1), (64, True, 4096, 32, 0)])
def test_attention_split(rules, D, causal, S, heads, split):
    assert rules("a", [(D == 64, causal, S, heads)]) == [(split, 0)]


def test_attention_forms_that_the_gpu_tests_name(rules):
    import test_gpu_attention_split as forms
    for cases, split in ((forms.SPLIT_BOTH, 1), (forms.MANY, 0)):
        for B, S, H, _, D in cases:
            for causal in (False, True):
                assert rules("a", [(D == 64, causal, S, B * H)]) == [(split, 0)], (B, S, H, D, causal)
