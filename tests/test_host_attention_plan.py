"""How the key tiles of dK and dV are dealt to the workgroups of a share of the CUs, from the header that the library plans with.

The deal is played through: static rounds or the queue's eight lists, one per XCD, with the cost of a tile under a causal mask the
number of query blocks that it streams.  With one workgroup to a CU nothing hides an uneven deal, so the last workgroup may not be
done much later than the longest tile, or an equal share of all tiles, takes."""
import heapq
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_18710_amd", "csrc")
PROGRAM = r"""
#include <stdio.h>
#include "attention_plan.h"
int main() {
  long heads, tiles, resident, items, query_tiles; int causal, one, group;
  if (scanf("deal %ld %ld %ld %d %d ", &heads, &tiles, &resident, &causal, &one) == 5) {
    const AttnDeal d = attn_deal(heads, (int)tiles, resident, causal, one);
    printf("%d %d %d\n", (int)d.queue, d.hb, d.unit);
    return 0;
  }
  if (scanf("parts %ld %ld %d %d", &items, &query_tiles, &group, &causal) == 4) printf("%d\n", (int)dkv_in_parts(items, query_tiles, group, causal));
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "plan.cpp"), "-o", str(d / "plan")], check=True)
    return lambda *line: tuple(int(v) for v in subprocess.run([str(d / "plan")], input=" ".join(map(str, line)) + "\n", capture_output=True, text=True,
                                                              check=True).stdout.split())


def tile_of(item, heads, tiles, hb):
    blk, within = divmod(item, hb * tiles)
    return within // min(hb, heads - blk * hb)


def finish(heads, tiles, G, queue, hb, chunk, cost):
    """When the last of G workgroups is done."""
    items = heads * tiles
    if not queue:
        done = [0.0] * G
        for r in range(-(-items // G)):
            cnt = min(G, items - r * G)
            per = -(-cnt // 8)
            flip = r % 2 and G // 8 % tiles == 0
            for b in range(G):
                local = b % 8 * per + b // 8
                if b // 8 < per and local < cnt:
                    t = (r * G + local) % tiles
                    done[b] += cost(tiles - 1 - t if flip else t)
        return max(done)
    full = items // (8 * chunk) * 8 * chunk
    tail = -(-(items - full) // 8)
    lists = [[i for c in range(x, full // chunk, 8) for i in range(c * chunk, (c + 1) * chunk)] +
             [i for i in range(full + x * tail, min(full + (x + 1) * tail, items))] for x in range(8)]
    assert sorted(sum(lists, [])) == list(range(items))
    at, free, end = [0] * 8, [(0.0, b, b % 8) for b in range(G)], 0.0
    heapq.heapify(free)
    while free:
        now, b, x = heapq.heappop(free)
        end = max(end, now)
        for d in range(8):
            if at[(x + d) % 8] < len(lists[(x + d) % 8]):
                x = (x + d) % 8
                heapq.heappush(free, (now + cost(tile_of(lists[x][at[x]], heads, tiles, hb)), b, x))
                at[x] += 1
                break
    return end


@pytest.mark.parametrize("B,N,H,Hkv", [(8, 1024, 16, 4), (5, 1024, 16, 4), (6, 1024, 32, 4), (7, 1024, 16, 4), (8, 768, 16, 4), (2, 2048, 32, 8), (1, 4096, 32, 8),
                                       (4, 2048, 16, 2), (8, 1000, 24, 3), (7, 900, 12, 3), (3, 1600, 40, 5), (1, 2600, 24, 6), (1, 1024, 16, 16)])
def test_two_groups_of_waves_share_a_causal_problem_evenly(plan, B, N, H, Hkv):
    heads, tiles, group = B * Hkv, -(-N // 128), H // Hkv
    blocks = -(-N // 32)
    assert plan("parts", heads * tiles, group * blocks, group, 1) == (1,)
    cost = lambda t: group * (blocks - 4 * t)
    total = heads * sum(cost(t) for t in range(tiles))
    for cus in (256, 192, 160, 128, 96, 64, 32):
        queue, hb, unit = plan("deal", heads, tiles, cus, 1, 1)
        end = finish(heads, tiles, cus, queue and heads * tiles > cus, hb, unit, cost)
        assert end <= 1.25 * max(cost(0), total / cus), (cus, queue, hb, unit, end, cost(0), total / cus)


def test_other_kernels_keep_their_deal(plan):
    for heads, tiles, resident, causal, deal in [(32, 8, 384, 1, (0, 4, 32)), (32, 8, 64, 1, (1, 2, 16)), (160, 12, 512, 0, (1, 1, 12)), (160, 12, 768, 0, (0, 1, 12)),
                                                 (8, 32, 512, 1, (0, 1, 32)), (256, 32, 512, 1, (1, 4, 128))]:
        assert plan("deal", heads, tiles, resident, causal, 0) == deal


@pytest.mark.parametrize("items,query_tiles,group,causal,parts", [(128, 8, 1, 0, 1), (128, 7, 1, 0, 0), (129, 32, 1, 1, 0), (256, 32, 4, 1, 1), (256, 32, 4, 0, 0), (256, 32, 3, 1, 0),
                                                                  (257, 32, 8, 1, 0)])
def test_where_a_key_tile_takes_two_groups(plan, items, query_tiles, group, causal, parts):
    assert plan("parts", items, query_tiles, group, causal) == (parts,)
