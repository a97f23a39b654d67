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
    ("fwds", 400, 288, 192, 4.5, 3.8, 3.1, 2.7), ("fwds", 123, 1888, 1888, 15.9, 11.9, 9.2, 7.2), ("fwds", 1024, 1920, 960, 10.3, 16.3, 17.2, 20.7),
    ("dgrads", 400, 192, 512, 6.0, 6.2, 4.9, 3.9), ("dgrads", 915, 928, 464, 8.3, 6.1, 6.2, 7.1), ("dgrads", 1068, 848, 848, 12.1, 7.8, 9.3, 10.9),
    ("wgrads", 192, 512, 400, 6.2, 4.8, 5.0, 3.1), ("wgrads", 688, 168, 2166, 15.6, 13.4, 10.7, 8.6), ("fwds", 3000, 1536, 384, 9.4, 20.7, 17.6, 19.2),
    ("dgrads", 3277, 768, 768, 9.6, 22.1, 22.7, 28.9), ("wgrads", 1648, 6592, 1175, 34.9, 85, 74, 121), ("fwds", 448, 896, 896, 9.1, 8.6, 6.2, 7.1),
    ("wgrads", 2536, 2536, 289, 11.1, 26.8, 29.3, 28.8), ("dgrads", 1233, 768, 1152, 10.5, 11.3, 12.5, 13.9), ("fwds", 4020, 144, 592, 9.2, 6.1, 6.6, 6.8),
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
