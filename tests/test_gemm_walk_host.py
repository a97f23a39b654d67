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
