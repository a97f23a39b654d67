"""Walk of the bf16 GEMM over its tiles (no GPU needed): every tile once, and an XCD's tiles close together."""
import subprocess

import pytest

from paper_1909_08053_amd import build as BLD

MAIN = """#include <stdio.h>
#include <set>
#include <utility>
#include "gemm_bf16_v2.h"
namespace mlm {
int gemm_cu_count() { return 256; }
int gemm_v2_forced_bn() { return 0; }
}
using namespace mlm;
int main() {                               // "tiles_m tiles_n window" -> wrong tiles, most operand panels of an XCD
  int R, N, W;
  while (scanf("%d %d %d", &R, &N, &W) == 3) {
    V2Plan p{};
    p.tiles_m = R; p.tiles_n = N; p.bm = p.bn = 256;
    p.split = 1; p.full_tiles = R * N;
    v2_set_walk(&p, W, 4096);
    const int n = R * N;
    std::set<std::pair<int, int>> seen;
    int wrong = 0;
    size_t panels = 0;
    for (int base = 0; base < n; base += W)
      for (int x = 0; x < 8; ++x) {
        std::set<int> rows, cols;
        for (int id = base + x; id < base + W && id < n; id += 8) {
          int m, c;
          v2_tile_of(p, p.strip ? v2_xcd_order(id, n, W) : id, &m, &c);
          wrong += m < 0 || m >= R || c < 0 || c >= N || !seen.insert({m, c}).second;
          rows.insert(m);
          cols.insert(c);
        }
        if (rows.size() + cols.size() > panels) panels = rows.size() + cols.size();
      }
    printf("%d %zu\\n", wrong, panels);
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("walk")
    src, exe = d / "walk.hip", d / "walk"
    src.write_text(MAIN)
    subprocess.run([BLD._hipcc(), *BLD.FLAGS, str(src), "-o", str(exe)], check=True, capture_output=True, timeout=180)

    def run(cases):
        text = "\n".join("%d %d %d" % c for c in cases)
        out = subprocess.run([str(exe)], input=text, text=True, check=True, capture_output=True, timeout=60).stdout.split()
        return list(zip(map(int, out[::2]), map(int, out[1::2])))
    return run


def test_every_tile_is_walked_once(walk):
    cases = [(m, n, w) for m in (1, 2, 3, 7, 8, 12, 13, 31, 32, 33, 64) for n in (1, 2, 5, 8, 9, 25, 40, 100) for w in (8, 240, 256, 512)]
    assert all(wrong == 0 for wrong, _ in walk(cases))


def test_tiles_of_an_xcd_share_panels(walk):
    """32 tiles have at least 12 panels in whole patches; a strip's end inside a share adds a few.  (Tile row fastest: 33 for
    15, 33 or 63 rows.)"""
    cases = [(32, 25, 256), (32, 12, 256), (16, 14, 256), (4, 100, 256), (15, 50, 256), (33, 17, 256), (63, 8, 256), (20, 20, 256)]
    for c, (_, panels) in zip(cases, walk(cases)):
        assert panels <= 16, (c, panels)


RULE = """#include <stdio.h>
#include <string.h>
#include "gemm_bf16_v2.h"
namespace mlm {
int gemm_cu_count() { return 256; }
int gemm_v2_forced_bn() { return 0; }
}
using namespace mlm;
int main() {                               // "layout M N K split" -> strips, k-pieces, part by part of k
  char lay[8];
  int M, N, K, sp;
  while (scanf("%7s %d %d %d %d", lay, &M, &N, &K, &sp) == 5) {
    const int bn = !strcmp(lay, "fwd") ? v2_pick_bn<true, false, EPI_STORE>(M, N, K, sp)
                 : !strcmp(lay, "dgrad") ? v2_pick_bn<true, true, EPI_STORE>(M, N, K, sp) : v2_pick_bn<false, false, EPI_STORE>(M, N, K, sp);
    V2Plan p = v2_plan(M, N, K, sp, bn);
    v2_set_walk(&p, bn == V2_SMALL && !p.deep() ? 512 : 256, K);
    printf("%d %d %d\\n", p.strip != 0, p.tail_tiles * p.split, p.long_pieces);
  }
  return 0;
}
"""

# layout, M, N, K; us with ids straight to tiles and in strips.  The last three are the first product of a call, with the call's time.
STRIPS = [
    ("dgrad", 280, 5040, 1872, 20.5, 15.8), ("fwd", 360, 6440, 3968, 37.0, 29.1), ("fwd", 600, 5520, 2416, 30.8, 25.4),
    ("fwd", 5776, 1064, 3808, 71.6, 59.3), ("dgrad", 1608, 1824, 1352, 18.1, 15.2), ("wgrad", 528, 3496, 4992, 41.8, 38.0),
    ("wgrad", 1488, 3248, 1720, 30.1, 27.3), ("dgrad", 2416, 3616, 80, 9.0, 9.3), ("fwd", 1432, 816, 216, 5.8, 6.0),
    ("wgrad", 928, 1208, 224, 5.2, 5.4), ("wgrad", 736, 480, 88, 4.0, 4.2), ("dgrad", 3440, 3104, 120, 9.9, 10.3),
    ("fwd", 520, 2000, 864, 28.4, 31.1), ("fwd", 1068, 2016, 448, 24.9, 27.3), ("fwd", 2400, 1440, 480, 27.9, 29.7),
]
# layout, M, N, K of products in k-pieces only; us of their call with the pieces spread over the XCDs and part by part of k
PIECES = [
    ("dgrad", 7343, 112, 14688, 161.0, 174.6), ("dgrad", 5519, 208, 3160, 72.1, 75.0), ("dgrad", 863, 512, 22616, 99.3, 78.8),
    ("dgrad", 2111, 360, 27072, 167.0, 133.1), ("fwd", 1332, 680, 9184, 74.0, 62.5), ("dgrad", 1399, 432, 26168, 138.6, 120.1),
    ("dgrad", 2230, 144, 12928, 73.6, 65.4), ("fwd", 336, 1320, 11760, 79.2, 70.8), ("dgrad", 3970, 136, 13952, 102.5, 114.0),
]


def test_walk_takes_the_faster_order(tmp_path):
    """Short launches keep the plain order, whose tiles cost one division, and k-pieces are ordered only where that shares more panels."""
    (tmp_path / "rule.hip").write_text(RULE)
    subprocess.run([BLD._hipcc(), *BLD.FLAGS, str(tmp_path / "rule.hip"), "-o", str(tmp_path / "rule")], check=True, capture_output=True,
                   timeout=180)
    lines = ["%s %d %d %d 0" % c[:4] for c in STRIPS] + ["%s %d %d %d 1" % c[:4] for c in PIECES]
    out = subprocess.run([str(tmp_path / "rule")], input="\n".join(lines), text=True, check=True, capture_output=True, timeout=60).stdout
    got = [tuple(map(int, l.split())) for l in out.splitlines()]
    for c, (strips, _, _) in zip(STRIPS, got):
        assert c[4 + strips] == min(c[4:]), (c, strips)
    for c, (_, pieces, parts) in zip(PIECES, got[len(STRIPS):]):
        assert pieces and c[4 + parts] == min(c[4:]), (c, pieces, parts)
