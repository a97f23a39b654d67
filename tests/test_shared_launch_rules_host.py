"""Which products share a launch, and in which tiles, and how the pass over stored logits is divided (no GPU needed: the rules are host
arithmetic): for the shapes of the GPU tests, whose names claim it, and against measured launches."""
import subprocess

import pytest

import test_gpu_ce_bwd_joint as BCE
import test_gpu_fp32_ce_bwd_joint as FCE
import test_gpu_fp32_wgrad_group as FWG
import test_gpu_wgrad_group_split as BWG
from paper_1909_08053_amd import build as BLD

F32 = """#include <stdio.h>
#include "gemm_f32_pick.h"
int mlm::gemm_cu_count() { return 256; }
using namespace mlm;
int main() {                       // "w T H F p" -> tile, chains, 128-wide ones apart; "d T H V" -> tile, chains
  char kind[4];
  int T, H, F, p;
  while (scanf("%3s %d %d %d", kind, &T, &H, &F) == 4) {
    if (kind[0] == 'w') {
      if (scanf("%d", &p) != 1) return 1;
      const int Hl = H / p, Fl = F / p, M[4] = {Fl, H, H, Hl}, N[4] = {H, Fl, 3 * Hl, H};
      const F32GroupPlan g = f32_group_plan(M, N, 4, T);
      int kinds = 0;                                    // tiles that the four take alone, one bit each
      for (int q = 0; q < 4; ++q) kinds |= f32_pick(M[q], N[q], T) / 32;
      printf("%d %d %d %d\\n", g.tile, g.chains, g.wide_apart, kinds);
    } else {
      const F32DualPick d = f32_dual_pick(H, F, T, T, H, F);
      printf("%d %d 0 0\\n", d.tile, d.chains);
    }
  }
  return 0;
}
"""

# fp32 weight gradients, tokens, width, ways of the split; us with a launch each, in one launch of 64-wide tiles with sums of as many
# chains as needed, with the 128-wide ones in a launch of their own (all four: the same), the others in 64-wide tiles or a launch each
F32_GROUPS = [
    (16, 2048, 1, 66.5, 131.6, 54.1), (108, 2048, 1, 139.1, 204.8, 127.6), (1024, 2048, 1, 784.8, 921.0, 764.1), (16, 1568, 1, 54.5, 80.1, 38.4),
    (211, 1544, 1, 163.0, 151.1, 150.2), (80, 1712, 1, 105.6, 112.3, 97.4), (841, 984, 1, 189.6, 186.6, 175.6), (204, 912, 1, 69.2, 59.4, 59.8),
    (23, 904, 1, 29.8, 32.3, 24.8), (1147, 1104, 1, 320.1, 299.2, 295.4), (372, 1912, 1, 318.9, 310.1, 285.6), (955, 1872, 1, 709.6, 689.4, 689.9),
    (2063, 1120, 1, 565.2, 530.6, 556.9), (68, 776, 1, 41.8, 37.2, 40.3), (37, 832, 1, 34.3, 26.2, 30.6), (14, 632, 1, 27.9, 16.1, 22.0),
    (29, 680, 1, 30.2, 19.4, 26.6), (49, 1920, 4, 37.4, 26.8, 29.9), (27, 1464, 1, 60.2, 52.1, 53.4), (44, 1520, 2, 49.5, 41.7, 46.5),
]
# both fp32 gradients of the logits, tokens, width, vocabulary; us of the call in two launches, in one of 64-wide tiles
F32_DUALS = [
    (805, 200, 3176, 60.5, 64.7), (6097, 1968, 440, 202.5, 192.0), (613, 568, 17880, 425.3, 352.3), (390, 672, 16032, 421.1, 277.7),
    (4554, 216, 1168, 123.9, 90.0), (128, 2232, 21512, 632.6, 372.8), (6000, 1024, 256, 90.3, 108.6), (3792, 192, 248, 46.4, 72.3),
    (64, 1024, 30000, 317.5, 496.4), (22, 784, 38944, 422.3, 639.2), (512, 1024, 4096, 114.8, 94.4), (271, 2000, 25784, 691.6, 583.4),
    (406, 1008, 18416, 462.3, 373.3), (593, 712, 1016, 39.7, 36.6), (1737, 1032, 4592, 316.6, 311.5), (2010, 1808, 3480, 467.6, 444.3),
]


@pytest.fixture(scope="module")
def f32(tmp_path_factory):
    d = tmp_path_factory.mktemp("f32")
    (d / "f32.cpp").write_text(F32)
    subprocess.run(["g++", "-std=c++17", "-I" + BLD.CSRC, str(d / "f32.cpp"), "-o", str(d / "f32")], check=True, timeout=60)

    def run(lines):
        out = subprocess.run([str(d / "f32")], input="\n".join(lines), text=True, check=True, capture_output=True, timeout=60).stdout
        return [tuple(map(int, l.split())) for l in out.splitlines()]
    return run


def test_fp32_shapes_of_the_gpu_tests_share_launches(f32):
    plans = f32(["w %d %d %d %d" % s for s in FWG.SHAPES])
    assert {(64, 2, 0), (64, 8, 0), (128, 1, 0), (64, 2, 1), (0, 0, 1)} <= {p[:3] for p in plans}, plans
    assert all(tile or wide for tile, _, wide, _ in plans), plans
    duals = f32(["d %d %d %d" % s for s in FCE.SHAPES])
    assert [d[:2] for d in duals] == [(64, 2)] * (len(duals) - 1) + [(64, 8)]


def test_fp32_sums_keep_their_chains(f32):
    """Two in the 64-wide tiles are enough only where nothing takes the split kernel alone; 128-wide tiles only where all do."""
    sizes = [(T, H, 4 * H, p) for T in (5, 24, 55, 123, 333, 1024, 4096) for H in (64, 320, 768, 1032, 1536, 2048) for p in (1, 2, 4, 8)]
    for s, (tile, chains, wide, kinds) in zip(sizes, f32(["w %d %d %d %d" % s for s in sizes])):
        assert tile != 64 or chains == (8 if kinds & 1 else 2), s
        assert tile != 128 or kinds == 4, s


def test_fp32_rules_take_the_faster_form(f32):
    for m, (tile, _, wide, _) in zip(F32_GROUPS, f32(["w %d %d %d %d" % (*m[:2], 4 * m[1], m[2]) for m in F32_GROUPS])):
        assert m[3 + (2 if wide or tile == 128 else 1 if tile else 0)] <= 1.04 * min(m[3:]), (m, tile, wide)
    for m, (tile, _, _, _) in zip(F32_DUALS, f32(["d %d %d %d" % m[:3] for m in F32_DUALS])):
        assert m[4 if tile else 3] <= 1.04 * min(m[3:]), (m, tile)


# rows, 16-byte vectors of a row of bf16 logits; us with a vector per thread and with a workgroup per row
DLOGITS = [(16, 800, 2.56, 3.08), (40, 800, 2.60, 3.16), (64, 1024, 2.96, 3.52), (128, 800, 3.08, 3.48), (300, 800, 4.88, 5.24),
           (512, 800, 7.08, 6.36), (1000, 257, 6.68, 5.52), (2048, 800, 13.48, 10.08), (8192, 800, 37.23, 32.32), (8192, 257, 19.32, 14.64),
           (8192, 6400, 266.0, 279.0)]


def test_pass_over_logits_takes_the_faster_form(tmp_path):
    (tmp_path / "dl.cpp").write_text("""#include <stdio.h>
#include "schedule.h"
int main() { int t, nv; while (scanf("%d %d", &t, &nv) == 2) printf("%d\\n", mlm::dlogits_vectors(t, nv, 256)); return 0; }
""")
    subprocess.run(["g++", "-std=c++17", "-I" + BLD.CSRC, str(tmp_path / "dl.cpp"), "-o", str(tmp_path / "dl")], check=True, timeout=60)
    text = "\n".join("%d %d" % m[:2] for m in DLOGITS)
    out = subprocess.run([str(tmp_path / "dl")], input=text, text=True, check=True, capture_output=True, timeout=60).stdout.split()
    for m, v in zip(DLOGITS, map(int, out)):
        assert m[3 if v == 4 else 2] == min(m[2:]), (m, v)


BF16 = """#include <stdio.h>
#include <string.h>
#include "gemm_bf16_v2.h"
namespace mlm {
int forced = 0, off = 0;
int gemm_cu_count() { return 256; }
int gemm_v2_forced_bn() { return forced; }
bool gemm_v2_group_off() { return off != 0; }
}
using namespace mlm;
int main() {                       // "o BN OFF 0" sets the overrides; "d T H V" -> tile, whether dhf leads; "g T H p F / H" -> tile, the split problem, its pieces
  char kind[4];
  int T, H, x, f;
  while (scanf("%3s %d %d %d", kind, &T, &H, &x) == 4) {
    GemmArgs a[4];
    memset(a, 0, sizeof(a));
    if (kind[0] == 'o') { forced = T; off = H; continue; }
    auto set = [&](int q, int M, int N, int K) { a[q].M = M; a[q].N = N; a[q].K = K; a[q].epi = EPI_STORE; };
    if (kind[0] == 'd') {
      set(0, H, x, T);
      set(1, T, H, x);
      const V2Dual d = v2_dual(a[0], a[1]);
      printf("%d %d 0\\n", d.bn, d.first_is_1);
    } else {
      if (scanf("%d", &f) != 1) return 1;
      const int Hl = H / x, Fl = f * H / x;
      set(0, Fl, H, T); set(1, H, Fl, T); set(2, H, 3 * Hl, T); set(3, Hl, H, T);
      const V2GroupPlan p = v2_group_plan(a, 4, true);
      printf("%d %d %d\\n", p.bn, p.split.last, p.split.split);
    }
  }
  return 0;
}
"""

# both bf16 gradients of the logits, tokens, width, vocabulary; us of the call in two launches, in one
BF16_DUALS = [
    (8192, 3072, 6400, 490, 458), (8192, 1536, 51200, 2154, 2030), (3008, 3072, 12800, 424, 353), (1536, 3072, 2048, 53.5, 45.7),
    (6144, 2560, 3072, 166, 145), (320, 1920, 1000, 19.3, 15.0), (704, 384, 512, 16.4, 10.9), (3008, 3072, 4096, 131, 138),
    (4096, 1920, 6400, 182, 186), (8192, 1536, 6400, 273, 266), (8192, 1920, 25600, 1307, 1406), (4096, 2560, 7648, 276, 260),
    (2048, 1024, 4096, 53.3, 77.6), (4096, 3072, 6400, 249, 235), (8192, 2560, 12800, 806, 842), (1024, 1536, 6400, 58.5, 112.9),
    (512, 1536, 7648, 46.4, 154.7), (4096, 1536, 25600, 571, 634), (2048, 3072, 25600, 517, 620), (8192, 768, 3200, 101.5, 166.5),
    (400, 768, 3000, 28.5, 34.3), (1000, 512, 1024, 30.8, 14.6), (8192, 1536, 25600, 1104, 1070), (72, 384, 1000, 16.9, 12.0),
]
# bf16 weight gradients of a layer shard, tokens, width, ways of the split; us in whole tiles or a launch each, with a split last round
BF16_GROUPS = [
    (4096, 2560, 4, 154.2, 143.0), (3360, 2304, 3, 147.7, 130.0), (6176, 2560, 4, 249.4, 212.0), (7000, 2304, 3, 298.8, 260.1),
    (8192, 1920, 2, 351.9, 320.9), (6000, 1152, 1, 238.7, 186.0), (4096, 1056, 1, 172.0, 123.1), (8192, 1216, 1, 341.7, 263.4),
    (1536, 1056, 1, 49.1, 61.0), (2000, 1152, 1, 68.6, 82.0),
]


@pytest.fixture(scope="module")
def bf16(tmp_path_factory):
    d = tmp_path_factory.mktemp("bf16")
    src, exe = d / "bf16.hip", d / "bf16"
    src.write_text(BF16)
    subprocess.run([BLD._hipcc(), *BLD.FLAGS, str(src), "-o", str(exe)], check=True, capture_output=True, timeout=180)

    def run(lines):
        out = subprocess.run([str(exe)], input="\n".join(lines), text=True, check=True, capture_output=True, timeout=60).stdout
        return [tuple(map(int, l.split())) for l in out.splitlines()]
    return run


def test_overrides_change_what_they_name(bf16):
    """A forced tile width leaves it open which products share a launch; ungrouped weight gradients leave the logits' alone."""
    duals, groups = ["d 8192 3072 6400", "d 200 192 520"], ["g 8192 3072 8 4", "g 4096 2560 4 4"]
    assert [bn for bn, _, _ in bf16(duals)] == [256, 128]
    free = bf16(groups)
    assert [bn for bn, _, _ in free] == [256, 256] and [split > 0 for _, _, split in free] == [False, True]
    assert [bn for bn, _, _ in bf16(["o 256 0 0"] + duals)] == [256, 0]
    assert [bn for bn, _, _ in bf16(["o 128 0 0"] + duals)] == [0, 128]
    assert [bn for bn, _, _ in bf16(["o 0 1 0"] + duals)] == [256, 128]
    assert bf16(["o 256 0 0"] + groups) == free
    assert [g[::2] for g in bf16(["o 0 1 0"] + groups)] == [(0, 0)] * 2
    assert [split for _, _, split in bf16(["o 128 0 0"] + groups)] == [0, 0]


def test_bf16_rules(bf16):
    lines = ["d %d %d %d" % s for s in BCE.SHAPES] + ["g %d %d %d %d" % s for s in BWG.SHAPES]
    lines += ["d %d %d %d" % m[:3] for m in BF16_DUALS] + ["g %d %d %d 4" % m[:3] for m in BF16_GROUPS]
    got = bf16(lines)
    take = lambda n: [got.pop(0) for _ in range(n)]
    # the shapes of the GPU tests: small tiles, then large ones with either gradient leading; a split problem in first and middle place
    duals = take(len(BCE.SHAPES))
    assert [d[0] for d in duals] == [128, 128, 128, 256, 256, 256, 256] and {d[1] for d in duals[3:]} == {0, 1}, duals
    groups = take(len(BWG.SHAPES))
    assert all(bn == 256 and split > 1 for bn, _, split in groups), groups
    assert {0, 2} <= {last for _, last, _ in groups} and len({split for _, _, split in groups}) > 2, groups
    for m, (bn, _, _) in zip(BF16_DUALS, take(len(BF16_DUALS))):
        assert m[4 if bn else 3] <= 1.04 * min(m[3:]), (m, bn)
    for m, (_, _, split) in zip(BF16_GROUPS, take(len(BF16_GROUPS))):
        assert m[4 if split else 3] <= 1.04 * min(m[3:]), (m, split)
