"""How the bf16 attention kernels divide a launch (no GPU needed: the rule is host arithmetic), against measured launches."""
import subprocess

import pytest

from paper_1909_08053_amd import build as BLD

MAIN = """#include <stdio.h>
#include "attention_modes.h"
int mlm::gemm_cu_count() { return 256; }
int main() {
  int causal, d, s, pairs;
  while (scanf("%d %d %d %d", &causal, &d, &s, &pairs) == 4)
    printf("%d %d\\n", (int)mlm::attn_mode(s, pairs, causal != 0, d), causal || d > 96 ||
           mlm::attn_bwd_mode(s, pairs, false, 1) != mlm::ATTN_BWD_TWO ? -1 : (int)mlm::attn_dkv_split(s, pairs));   // -1: not asked
  return 0;
}
"""

# causal, head size, sequence, (batch, head) pairs; us of forward + dQ as WIDE, PAIR (d = 192: WIDE), SPLIT; of dK / dV in 128- and
# 64-key workgroups
MEASURED = [
    # long causal sequences on every compute unit; few long or uneven pairs, whose halved blocks queue on one XCD
    (1, 64, 4096, 9, 181, 125, 159, 87, 99), (1, 96, 4096, 16, 243, 180, 231, 122, 145), (1, 96, 2048, 24, 126, 107, 123, 69, 76),
    (1, 128, 8192, 8, 492, 386, 533, 447, 570), (0, 96, 4096, 4, 170, 152, 197, 104, 127), (0, 64, 768, 20, 32, 30, 43, 19, 25),
    (0, 128, 1536, 9, 87, 72, 107, 81, 86), (0, 192, 4096, 1, 352, 343, 447, 657, 660), (1, 128, 8192, 1, 434, 328, 458, 377, 487),
    (0, 128, 2048, 1, 107, 84, 69, 53, 71), (1, 128, 4096, 1, 209, 156, 144, 112, 147), (0, 96, 3072, 4, 125, 110, 145, 74, 91),
    # few workgroups
    (1, 96, 1024, 8, 47, 44, 34, 28, 19), (1, 96, 3072, 4, 120, 103, 77, 69, 47), (1, 192, 4096, 4, 340, 340, 265, 376, 371),
    (0, 64, 1024, 16, 39, 35, 28, 23, 17), (0, 96, 1024, 8, 46, 44, 34, 27, 20), (0, 128, 512, 4, 36, 34, 30, 19, 16),
    # one per compute unit and more
    (1, 96, 1024, 32, 51, 50, 63, 30, 36), (1, 96, 1024, 64, 76, 91, 112, 59, 64), (1, 96, 2048, 32, 132, 135, 143, 89, 86),
    (0, 96, 1024, 128, 166, 193, 272, 129, 162), (1, 64, 512, 48, 25, 25, 33, 15, 18), (1, 64, 4096, 20, 230, 228, 248, 160, 157),
]


@pytest.fixture(scope="module")
def chosen(tmp_path_factory):
    d = tmp_path_factory.mktemp("modes")
    (d / "modes.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I" + BLD.CSRC, str(d / "modes.cpp"), "-o", str(d / "modes")], check=True, timeout=60)
    lines = "\n".join(" ".join(map(str, m[:4])) for m in MEASURED)
    out = subprocess.run([str(d / "modes")], input=lines, text=True, check=True, capture_output=True, timeout=60).stdout
    return [tuple(map(int, l.split())) for l in out.splitlines()]


def test_forward_and_dq_take_the_fastest_division(chosen):
    for m, (mode, _) in zip(MEASURED, chosen):
        assert m[4 + mode] <= 1.06 * min(m[4:7]), (m, mode)


def test_dkv_takes_the_better_workgroup(chosen):
    """Where dK / dV is a launch of its own that has both forms: without a mask, up to 96."""
    asked = [(m, split) for m, (_, split) in zip(MEASURED, chosen) if split >= 0]
    assert len(asked) >= 4 and {split for _, split in asked} == {0, 1}, asked
    for m, split in asked:
        assert m[7 + split] <= 1.06 * min(m[7:9]), (m, split)
