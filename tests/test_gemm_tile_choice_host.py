"""Tile choice of the bf16 GEMM (no GPU needed: the plan is host arithmetic), against shapes whose three tiles were measured."""
import subprocess

import pytest

from paper_1909_08053_amd import build as BLD
from test_gpu_bf16_gemm_k import LARGE_TILES

MAIN = """#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include "gemm_bf16_v2.h"
namespace mlm {
int gemm_cu_count() { return 256; }
int gemm_v2_forced_bn() { return 0; }
}
using namespace mlm;
int main(int argc, char** argv) {          // "layout M N K" -> tile width; "g T H p" -> tile width of the grouped launch
  char kind[8];
  int x, y, z;
  while (scanf("%7s %d %d %d", kind, &x, &y, &z) == 4) {
    if (kind[0] == 'g') {
      const int T = x, H = y, Hl = y / z, Fl = 4 * y / z;
      GemmArgs a[4];
      memset(a, 0, sizeof(a));
      const int mn[4][2] = {{Fl, H}, {H, Fl}, {H, 3 * Hl}, {Hl, H}};
      for (int q = 0; q < 4; ++q) { a[q].M = mn[q][0]; a[q].N = mn[q][1]; a[q].K = T; }
      printf("%d\\n", v2_group_cost(a, 4, V2_SMALL) < v2_group_cost(a, 4, V2_B) ? V2_SMALL : V2_B);
    } else if (!strcmp(kind, "fwd")) printf("%d\\n", v2_pick_bn<true, false, EPI_STORE>(x, y, z, false));
    else if (!strcmp(kind, "dgrad")) printf("%d\\n", v2_pick_bn<true, true, EPI_STORE>(x, y, z, false));
    else printf("%d\\n", v2_pick_bn<false, false, EPI_STORE>(x, y, z, kind[5] == 's'));   // "wgrads": with a k-split
  }
  return 0;
}
"""

# layout, M, N, K and the microseconds of a call with the 128-, 192- and 256-wide tile forced, tiles walked in strips where that pays
MEASURED = [
    ("wgrad", 1920, 25600, 8192, 789, 740, 715), ("fwd", 1920, 12800, 6144, 260, 312, 255), ("wgrad", 3200, 7680, 8192, 362, 417, 342),
    ("wgrad", 1920, 12800, 8192, 373, 419, 350), ("fwd", 3200, 7680, 6144, 258, 311, 247), ("wgrad", 8064, 1024, 8192, 127, 131, 152),
    ("wgrad", 3968, 2048, 8192, 122, 127, 151),
    # kernels of one weight gradient with a k-split where the plan has one (256 wide: 240 half-length pieces and the fix-up)
    ("wgrads", 3840, 1920, 8192, 149, 155, 136), ("wgrads", 1920, 3840, 8192, 149, 155, 136),
    # where the small tile is the better one it stays
    ("wgrad", 2048, 3840, 8192, 122, 122, 151), ("wgrad", 2560, 2560, 4096, 58, 64, 79), ("wgrad", 960, 1920, 8192, 60, 117, 145),
    ("fwd", 4096, 1920, 2560, 40, 47, 53), ("dgrad", 2048, 3072, 1024, 18.5, 20.3, 23.3),
]
# Odd numbers of tile rows, or few: the small tile's price there is from ids that went straight to tiles (v2_small_slice), and a large
# tile is taken though the small one is the faster one in strips.
CAUTIOUS = [
    ("dgrad", 8064, 1024, 6144, 85, 102, 104), ("fwd", 8064, 1024, 1536, 26.4, 32.3, 32.3), ("fwd", 768, 10240, 6144, 86, 96, 108),
    ("dgrad", 1024, 7680, 6144, 83, 88, 104), ("fwd", 896, 7552, 6144, 80, 91, 107), ("fwd", 768, 6400, 6144, 74, 90, 106),
]
# tokens, width, ways of the split and the microseconds of the grouped weight gradients of a layer shard, 128- and 256-wide tile, last
# round whole (test_shared_launch_rules_host.py: split)
GROUPS = [(8192, 1920, 2, 379, 355), (5000, 1920, 2, 233, 223), (8192, 1536, 1, 466, 386), (8192, 2304, 4, 256, 205),
          (8192, 3072, 8, 251, 199), (4096, 3072, 4, 216, 188), (4096, 2560, 4, 159, 177), (8192, 1536, 8, 76, 143),
          (3000, 1536, 4, 49, 62), (8192, 1536, 4, 115, 153)]

LAYOUTS = ("fwd", "dgrad", "wgrad")


@pytest.fixture(scope="module")
def picks(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, exe = d / "plan.hip", d / "plan"
    src.write_text(MAIN)
    subprocess.run([BLD._hipcc(), *BLD.FLAGS, str(src), "-o", str(exe)], check=True, capture_output=True, timeout=180)
    lines = [f"{m[0]} {m[1]} {m[2]} {m[3]}" for m in MEASURED + CAUTIOUS] + [f"g {g[0]} {g[1]} {g[2]}" for g in GROUPS]
    lines += [f"{l} {M} {N} {K}" for M, N, K in LARGE_TILES[192] + LARGE_TILES[256] for l in LAYOUTS]
    out = subprocess.run([str(exe)], input="\n".join(lines), text=True, check=True, capture_output=True, timeout=60).stdout.split()
    return [int(x) for x in out]


def test_chosen_tile_is_within_five_percent_of_the_best(picks):
    for m, bn in zip(MEASURED, picks):
        us = dict(zip((128, 192, 256), m[4:]))
        assert us[bn] <= 1.05 * min(us.values()), (m, bn)


def test_cautious_choice_loses_at_most_a_quarter(picks):
    for m, bn in zip(CAUTIOUS, picks[len(MEASURED):]):
        us = dict(zip((128, 192, 256), m[4:]))
        assert us[bn] <= 1.25 * us[128] and us[128] == min(us.values()), (m, bn)


def test_grouped_weight_gradients_take_the_better_tile(picks):
    first = len(MEASURED) + len(CAUTIOUS)
    for g, bn in zip(GROUPS, picks[first:first + len(GROUPS)]):
        assert g[3 if bn == 128 else 4] <= 1.05 * min(g[3:]), (g, bn)


def test_shapes_of_the_large_tiles_test_take_the_large_tiles(picks):
    large = picks[len(MEASURED) + len(CAUTIOUS) + len(GROUPS):]
    n = 3 * len(LARGE_TILES[192])
    assert set(large[:n]) == {192} and set(large[n:]) == {256}, large
