"""Which tiles a weight gradient takes, from the header that the library plans with, compiled for the host.

Every case names the ways that were measured within 5 % of the fastest one on that share of the CUs (masked
streams, microseconds: pieces of 256x256 tiles / of 128x128 tiles / chained, or 256x256 tiles with eight /
four waves / 128x128 tiles / mixed).  Plans that priced a whole 256x256 tile below the 128x128 tiles, or chose
the pieces for the whole device alone, took up to 1.6 times as long on a share."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_18710_amd", "csrc")
PIECES_LARGE, PIECES_SMALL, CHAINED, WHOLE8, WHOLE4, SMALL, MIXED8, MIXED4 = range(8)

PROGRAM = r"""
#include <stdio.h>
#include "gemm_plan.h"
int main() {
  long M, N, K; int cus, cut, four;
  long T, k, n;
  if (scanf("pair %ld %ld %ld %d", &T, &k, &n, &cus) == 4) {
    const PairPlan p = pair_plan(T, k, n, cus, wgrad_plan(k, n, T, cus, true, T >= 128));
    printf("%d %d %d\n", (int)p.pair, p.wgs_d, p.wgs_w);
    return 0;
  }
  if (scanf("rows %ld %ld %d", &K, &M, &cus) == 3) { printf("%d\n", row_block_for(K, M, cus)); return 0; }
  while (scanf("%ld %ld %ld %d %d %d", &M, &N, &K, &cus, &cut, &four) == 6) {
    const WgradPlan p = wgrad_plan(M, N, K, cus, cut, four);
    printf("%d %d %d %d\n", p.pieces, p.first, p.kper, (int)p.way);
  }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "plan.cpp"), "-o", str(d / "plan")], check=True)

    def call(line):
        out = subprocess.run([str(d / "plan")], input=line + "\n", capture_output=True, text=True, check=True).stdout
        return tuple(int(v) for v in out.split())

    def ask(T, k, n, cus, cut=1, four=1):
        return call("%d %d %d %d %d %d" % (k, n, T, cus, cut, four))
    ask.rows = lambda K, M, rows: call("rows %d %d %d" % (K, M, rows))[0]
    ask.pair = lambda T, k, n, cus: call("pair %d %d %d %d" % (T, k, n, cus))
    return ask


@pytest.mark.parametrize("T,k,n,cus,ways", [
    (1568, 768, 2304, 64, {SMALL}),                     # 32.7 / 34.4 / 22.4
    (1568, 768, 3072, 128, {SMALL}),                    # 32.6 / 34.7 / 22.5
    (1568, 2048, 2048, 192, {SMALL}),                   # 32.9 / 34.6 / 23.0
    (1568, 2048, 2048, 64, {WHOLE8, WHOLE4}),           # 33.5 / 35.2 / 43.3
    (502, 1344, 3456, 256, {SMALL}),                    # 16.9 / 17.4 / 12.9
    (175, 1920, 1664, 192, {SMALL}),                    # 10.4 / 11.1 / 8.5
    (4608, 4096, 12288, 256, {WHOLE4, MIXED4}),         # 350 / 320 / 422 / 318
    (2048, 4096, 4096, 256, {WHOLE4}),                  # 59.5 / 53.4 / 68.2
    (8192, 2048, 11264, 256, {MIXED4}),                 # 341 / 322 / 356 / 315 (eight waves), 290 (four)
    (8192, 2048, 2048, 256, {CHAINED, PIECES_LARGE}),   # 80 / 89 / 77
    (8192, 2048, 2048, 224, {PIECES_SMALL}),            # 109 / 93 / 107
    (8192, 2048, 2048, 192, {PIECES_LARGE, PIECES_SMALL, CHAINED}),   # 104 / 100 / 100
    (8192, 2048, 2048, 128, {PIECES_LARGE, CHAINED}),   # 99 / 123 / 103
    (8192, 2048, 2048, 64, {PIECES_LARGE}),             # 176 / 238 / 206
    (9216, 1024, 4096, 224, {PIECES_SMALL}),            # 118 / 101 / 122
    (9216, 1024, 4096, 128, {PIECES_LARGE}),            # 106 / 134 / 114
    (9216, 1024, 1024, 256, {PIECES_SMALL}),            # 40 / 33 / 66
    (9216, 1024, 1024, 64, {PIECES_LARGE, CHAINED}),    # 61 / 77 / 63
    (24000, 240, 1280, 256, {PIECES_SMALL}),            # 62 / 30 / 152
    (24000, 240, 1280, 64, {PIECES_LARGE, PIECES_SMALL}),   # 61 / 64 / 151
    (9216, 1024, 3072, 256, {PIECES_LARGE}),            # 70 / 81 / 76
    (9216, 1024, 3072, 192, {CHAINED}),                 # 97 / 83 / 73
    (2048, 1024, 2048, 64, {CHAINED}),                  # 44 / 52 / 33
    (5000, 1024, 3072, 128, {PIECES_LARGE}),            # 61 / 74 / 66
    (12000, 1280, 1280, 64, {PIECES_LARGE}),            # 133 / 144 / 151
])
def test_way_is_among_the_fastest_on_this_share(plan, T, k, n, cus, ways):
    assert plan(T, k, n, cus)[3] in ways


@pytest.mark.parametrize("T,k,n", [(8192, 2048, 2048), (9216, 600, 1024), (12000, 1280, 1280), (32768, 4096, 22016), (2056, 128, 128), (1568, 768, 768)])
def test_pieces_do_not_follow_the_share(plan, T, k, n):
    """The contraction is cut in the same places whatever the CUs and the way: the bits cannot follow them."""
    got = [plan(T, k, n, cus) for cus in (1, 8, 31, 32, 64, 96, 128, 160, 192, 224, 256)]
    assert len({g[:3] for g in got}) == 1
    pieces, first, kper, _ = got[0]
    assert kper % 32 == 0 and (pieces == 1 or (pieces - 1) * kper < T <= pieces * kper)


def test_without_scratch_or_four_waves(plan):
    assert all(plan(T, 2048, 2048, cus, cut=0)[0] == 1 for T in (8192, 100) for cus in (1, 64, 256))
    assert all(plan(T, 4096, 12288, cus, four=0)[3] not in (WHOLE4, MIXED4) for T in (100, 4608) for cus in (1, 64, 256))


@pytest.mark.parametrize("rows", [128, 160, 192, 224, 256])
def test_tile_rows_of_a_super_block(plan, rows):
    """The tile order is cut by the rows of the matrix, not by how many tile rows they make: no cut up to 16384 rows,
    above that whole 4-row patches whose operand is as near to 128 MB at every tile height."""
    for K in (128, 4096, 11008):
        for M in (1, 8192, 10496, 16384):
            assert plan.rows(K, M, rows) >= -(-M // rows), (K, M)
        for M in (16385, 32768, 100000):
            rb = plan.rows(K, M, rows)
            assert rb % 4 == 0 and rb >= 4
            if rb < -(-M // rows):
                per = rows * K * 2
                assert rb * per <= 128 << 20 < (rb + 4) * per, (K, M)


@pytest.mark.parametrize("T,k,n,pairs", [
    (1568, 768, 768, {256, 192, 64}), (1568, 768, 3072, {256, 192, 64}), (600, 1024, 1024, {256, 192}), (2048, 128, 2048, {256, 192, 64}),
    (2112, 768, 768, set()),            # pieces of 544 k-values are no whole 64-deep K-tiles
    (9216, 1024, 4096, set()), (32768, 4096, 22016, set()), (8192, 2048, 2048, set())])
def test_products_of_a_backward_pass_in_one_launch(plan, T, k, n, pairs):
    for cus in (8, 31, 32, 64, 192, 256):
        pair, d, w = plan.pair(T, k, n, cus)
        if pair:
            assert d >= 8 and w >= 8 and d % 8 == 0 and w % 8 == 0 and d + w <= cus, (cus, d, w)
        if cus in (192, 256, 64):
            assert bool(pair) == (cus in pairs), (cus, d, w)
        if cus == 8:
            assert not pair
