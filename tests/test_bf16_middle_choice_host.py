"""Which bf16 products go to 128 x 192 tiles (no GPU needed: host arithmetic), against measured products and groups of weight gradients; and that the
shapes of the GPU tests reach every kernel of that tile."""
import subprocess

import pytest

from paper_1909_08053_amd import build as BLD
from test_gpu_bf16_middle_tile import KS, LAYERS, MN

MAIN = """#include <stdio.h>
#include <string.h>
#include "gemm_bf16_split.h"
namespace mlm {
int gemm_cu_count() { return 256; }
int gemm_v2_forced_bn() { return 0; }
bool gemm_v2_group_off() { return false; }
}
using namespace mlm;
template <bool A_KC, bool B_KC, int EPI> void one(int M, int N, int K, bool scratch) {
  const int form = split_pick_alone<A_KC, B_KC, EPI>(M, N, K, scratch).form;
  const V2Choice c = v2_choose<A_KC, B_KC, EPI>(M, N, K, scratch);
  printf("%s %d\\n", form ? "split" : c.middle ? "middle" : "plan", form ? form : c.bn);
}
int main() {          // "layout scratch M N K" -> kind and width of a product's tiles; "group T H p" -> of a shard's weight gradients
  char kind[8];
  int scratch, x, y, z;
  while (scanf("%7s %d %d %d %d", kind, &scratch, &x, &y, &z) == 5) {
    if (!strcmp(kind, "group")) {
      GemmArgs a[4];
      memset(a, 0, sizeof(a));
      const int Hl = y / z, Fl = 4 * y / z;
      const int mn[4][2] = {{Fl, y}, {y, Fl}, {y, 3 * Hl}, {Hl, y}};
      for (int q = 0; q < 4; ++q) { a[q].M = mn[q][0]; a[q].N = mn[q][1]; a[q].K = x; a[q].epi = EPI_STORE; }
      const V2GroupPlan p = v2_group_plan(a, 4, true);
      const bool middle = v2_group_middle(a, 4, p);
      const int form = middle ? 0 : split_group_pick(a, 4, p);
      printf("%s %d\\n", middle ? "middle" : form ? "split" : "plan", middle ? 192 : form ? form : p.bn);
    } else if (!strcmp(kind, "fwd")) one<true, false, EPI_STORE>(x, y, z, scratch);
    else if (!strcmp(kind, "gelu")) one<true, false, EPI_BIAS_GELU>(x, y, z, scratch);
    else if (!strcmp(kind, "dgrad")) one<true, true, EPI_STORE>(x, y, z, scratch);
    else if (!strcmp(kind, "dgelu")) one<true, true, EPI_DGELU>(x, y, z, scratch);
    else one<false, false, EPI_STORE>(x, y, z, scratch);
  }
  return 0;
}
"""

# layout, whether the large tiles may split k, M, N, K; us in 128 x 192 tiles and in those that are taken otherwise, the fix-up of pieces included
MEASURED = [
    ("dgrad", 1, 3000, 1536, 30592, 305, 255), ("dgrad", 1, 6600, 544, 23928, 354, 250), ("wgrad", 1, 992, 4144, 1800, 26.0, 36.5),
    ("wgrad", 1, 1080, 4280, 11145, 140, 113), ("wgrad", 1, 21144, 168, 12352, 165, 128),
    ("dgrad", 1, 4416, 1200, 3304, 53.1, 58.0), ("fwd", 1, 2352, 1792, 1728, 20.5, 33.2), ("fwd", 1, 7168, 640, 2560, 28.6, 31.7),
    ("dgrad", 1, 3000, 1536, 1536, 17.9, 20.7), ("gelu", 1, 3000, 1536, 1536, 22.5, 24.3), ("dgelu", 1, 3000, 1536, 1536, 22.3, 24.2),
    ("fwd", 1, 8192, 768, 1536, 20.9, 21.8), ("dgelu", 1, 8192, 768, 1536, 24.4, 25.0), ("dgrad", 1, 6152, 696, 648, 14.6, 19.9),
    ("dgelu", 1, 1144, 5024, 256, 14.0, 12.6), ("dgelu", 1, 2648, 2192, 272, 15.1, 13.8), ("gelu", 1, 2552, 2104, 256, 12.8, 12.2),
    ("dgrad", 0, 3000, 1536, 30592, 305, 395), ("fwd", 0, 3448, 1216, 10944, 101.3, 123.7), ("wgrad", 0, 880, 5512, 7616, 87.4, 111.2),
    # ... of the whole step of a layer shard: k-pieces leave partial tiles in the memory-side cache, where the next launches' operands were
    ("dgrad", 1, 3000, 1536, 7648, 541, 551), ("dgrad", 1, 5000, 1152, 10944, 706, 717), ("dgrad", 1, 2400, 1920, 8544, 646, 658),
    ("dgrad", 1, 4000, 1344, 9600, 771, 781), ("dgrad", 1, 3000, 1536, 11264, 690, 684), ("dgrad", 1, 3000, 1536, 15296, 1289, 1242),
    ("dgrad", 1, 7000, 640, 20000, 1271, 1222),
    # the four weight gradients of a shard, tokens, width, ways of the split
    ("group", 1, 1376, 640, 1, 25.2, 29.7), ("group", 1, 1646, 1312, 4, 34.0, 27.9), ("group", 1, 1600, 1856, 8, 27.9, 24.6),
    ("group", 1, 1648, 1184, 4, 28.5, 36.0), ("group", 1, 5400, 1184, 4, 67.0, 75.7), ("group", 1, 11156, 848, 2, 132, 160),
    ("group", 1, 17024, 528, 1, 259, 195), ("group", 1, 23288, 1248, 4, 342, 276), ("group", 1, 20202, 552, 1, 309, 258),
]


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("middle")
    src, exe = d / "middle.hip", d / "middle"
    src.write_text(MAIN)
    subprocess.run([BLD._hipcc(), *BLD.FLAGS, str(src), "-o", str(exe)], check=True, capture_output=True, timeout=180)

    def run(queries):
        text = "\n".join(" ".join(map(str, q)) for q in queries)
        out = subprocess.run([str(exe)], input=text, text=True, check=True, capture_output=True, timeout=60).stdout
        return [tuple(l.split()) for l in out.splitlines()]
    return run


def test_middle_tile_is_taken_where_it_is_faster(ask):
    for m, (kind, _) in zip(MEASURED, ask([m[:5] for m in MEASURED])):
        assert kind == ("middle" if m[5] < m[6] else "plan"), (m, kind)


def test_shapes_of_the_gpu_test_take_the_middle_tile(ask):
    queries = [(l, 0, M, N, K) for M, N in MN for K in KS for l in ("fwd", "dgrad", "wgrad")]
    for q, (kind, _) in zip(queries, ask(queries)):
        assert kind == "middle", q


def test_layers_of_the_gpu_test_reach_every_middle_kernel(ask):
    """Of a layer's products, those that the GPU test names; between them every epilogue, the column sums beside an input gradient (whose blocks are
    about one a compute unit) and the joint launch."""
    seen = set()
    for (b, s, H, _, _, p, _), expected in LAYERS.items():
        T, Hl, Fl = b * s, H // p, 4 * H // p
        products = {"qkv": ("fwd", 1, T, 3 * Hl, H), "proj": ("fwd", 1, T, H, Hl), "fc1": ("gelu", 1, T, Fl, H), "fc2": ("fwd", 1, T, H, Fl),
                    "dg": ("dgelu", 1, T, Fl, H), "dfc1": ("dgrad", 1, T, H, Fl), "dctx": ("dgrad", 1, T, Hl, H), "dqkv": ("dgrad", 1, T, H, 3 * Hl),
                    "wgrads": ("group", 1, T, H, p)}
        taken = {name for name, (kind, _) in zip(products, ask(products.values())) if kind == "middle"}
        assert taken == set(expected.split()), (b, s, H, taken)
        seen |= {name + " beside" if name in ("dfc1", "dqkv") and -(-T // 64) * -(-products[name][4] // 512) <= 320 else name for name in taken}
    assert {"qkv", "fc1", "dg", "proj", "fc2", "dctx", "dfc1", "dqkv beside", "wgrads"} <= seen, seen
