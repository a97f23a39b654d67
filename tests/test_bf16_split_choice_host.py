"""Which bf16 products take the tiles whose k is dealt to the waves of a workgroup (no GPU needed: host arithmetic), against measured
products; and that the shapes of the GPU tests take the form that they are meant for."""
import subprocess

import pytest

from paper_1909_08053_amd import build as BLD
from test_gpu_bf16_split import DUALS, GROUPS, SHAPES

MAIN = """#include <stdio.h>
#include <string.h>
#include "gemm_bf16_split.h"
namespace mlm {
int gemm_cu_count() { return 256; }
int gemm_v2_forced_bn() { return 0; }
bool gemm_v2_group_off() { return false; }
}
using namespace mlm;
int main() {          // "layout M N K" -> form of a product; "group T H p", "dual T H V" -> form of a joint launch
  char kind[8];
  int x, y, z;
  while (scanf("%7s %d %d %d", kind, &x, &y, &z) == 4) {
    GemmArgs a[4];
    memset(a, 0, sizeof(a));
    if (!strcmp(kind, "group")) {
      const int Hl = y / z, Fl = 4 * y / z;
      const int mn[4][2] = {{Fl, y}, {y, Fl}, {y, 3 * Hl}, {Hl, y}};
      for (int q = 0; q < 4; ++q) { a[q].M = mn[q][0]; a[q].N = mn[q][1]; a[q].K = x; }
      printf("%d\\n", split_group_pick(a, 4, v2_group_plan(a, 4, true)));
      continue;
    }
    if (!strcmp(kind, "dual")) {
      a[0].M = y; a[0].N = z; a[0].K = x;
      a[1].M = x; a[1].N = y; a[1].K = z;
      printf("%d\\n", split_dual_pick(a[0], a[1], v2_dual(a[0], a[1])));
      continue;
    }
    const bool split = kind[strlen(kind) - 1] == 's';
    const int form = !strncmp(kind, "fwd", 3) ? split_pick_alone<true, false, EPI_STORE>(x, y, z, split).form
                     : kind[0] == 'd'         ? split_pick_alone<true, true, EPI_STORE>(x, y, z, split).form
                     : kind[0] == 'c'         ? split_pick_alone<true, false, EPI_CE>(x, y, z, true).form
                                              : split_pick_alone<false, false, EPI_STORE>(x, y, z, split).form;
    printf("%d\\n", form);
  }
  return 0;
}
"""

# layout (with an s: the large tiles may split k), M, N, K and the microseconds in the large tiles, in 64 x 64, 32 x 64 and 32 x 32
MEASURED = [
    ("fwds", 5397, 216, 648, 10.4, 11.1, 12.1, 11.7), ("dgrads", 3951, 1264, 632, 17.5, 23.0, 29.2, 26.8), ("dgrads", 494, 1224, 4896, 21.1, 22.6, 31.7, 33.7),
    ("fwds", 1024, 1920, 960, 10.3, 12.2, 17.1, 17.8), ("fwds", 272, 2528, 1264, 14.0, 8.2, 10.7, 10.4), ("wgrads", 368, 1472, 2868, 17.1, 13.5, 18.5, 21.6),
    ("dgrads", 355, 1464, 2928, 18.8, 16.0, 20.3, 18.9), ("fwds", 8056, 96, 784, 10.7, 7.1, 8.9, 8.4), ("dgrads", 841, 472, 1888, 17.4, 10.8, 8.4, 9.3),
    ("wgrads", 1104, 368, 1415, 14.8, 9.6, 8.1, 10.7), ("dgrads", 70, 4680, 1560, 16.9, 9.8, 8.7, 9.6), ("wgrads", 80, 672, 301, 5.2, 3.8, 3.2, 2.8),
    ("dgrads", 1058, 192, 192, 4.4, 3.6, 3.0, 2.7), ("fwds", 70, 2312, 3464, 19.2, 17.9, 14.6, 12.2), ("wgrads", 624, 416, 4059, 19.5, 19.1, 16.1, 23.7),
    ("wgrads", 1272, 216, 4916, 21.7, 23.5, 18.5, 29.3), ("wgrads", 264, 976, 3443, 16.5, 14.6, 12.7, 19.6), ("wgrads", 184, 1432, 3288, 17.2, 15.7, 14.1, 20.3),
]


@pytest.fixture(scope="module")
def picks(tmp_path_factory):
    d = tmp_path_factory.mktemp("split")
    src, exe = d / "split.hip", d / "split"
    src.write_text(MAIN)
    subprocess.run([BLD._hipcc(), *BLD.FLAGS, str(src), "-o", str(exe)], check=True, capture_output=True, timeout=180)

    def ask(lines):
        out = subprocess.run([str(exe)], input="\n".join(lines), text=True, check=True, capture_output=True, timeout=60).stdout.split()
        return [int(x) for x in out]
    return ask


def test_chosen_form_is_within_a_seventh_of_the_best(picks):
    for m, form in zip(MEASURED, picks([f"{m[0]} {m[1]} {m[2]} {m[3]}" for m in MEASURED])):
        assert m[4 + form] <= 1.15 * min(m[4:]), (m, form)


def test_shapes_of_the_gpu_tests_take_their_form(picks):
    for form, shapes in SHAPES.items():
        lines = [f"{l} {M} {N} {K}" for M, N, K in shapes for l in ("fwds", "dgrad", "wgrad")]
        assert set(picks(lines)) == {form}, (form, list(zip(lines, picks(lines))))
    assert picks([f"group {T} {H} {p}" for T, H, p, _ in GROUPS]) == [f for *_, f in GROUPS]
    assert picks([f"dual {T} {H} {V}" for T, H, V, _ in DUALS]) == [f for *_, f in DUALS]


def test_partials_of_the_loss_fit_the_workspace(picks):
    """Column tiles of 64 write more partials than the 128-wide ones; what they take of the k-split scratch is far below its 64 MB."""
    taken = 0
    for T in (8, 64, 333, 1024, 5000, 65536, 1 << 21):
        for V in (8, 264, 1024, 8192, 51200, 1 << 20):
            for H in (8, 192, 3072):
                if picks([f"ce {T} {V} {H}"])[0]:
                    taken += 1
                    assert 8 * T * ((V + 63) // 64 - (V + 127) // 128) < 8 << 20
    assert taken > 10
