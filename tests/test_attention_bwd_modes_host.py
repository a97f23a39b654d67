"""How the bf16 attention backward is launched (no GPU needed: the rule is host arithmetic), against measured launches."""
import subprocess

import pytest

import test_gpu_attention_bwd_two_launches as TWO
from paper_1909_08053_amd import build as BLD

MAIN = """#include <stdio.h>
#include "attention_modes.h"
int mlm::gemm_cu_count() { return 256; }
int main() {
  int causal, d, s, pairs;
  while (scanf("%d %d %d %d", &causal, &d, &s, &pairs) == 4)
    printf("%d %d\\n", (int)mlm::attn_bwd_mode(s, pairs, causal != 0, d >= 128 ? 2 : 1), (int)mlm::attn_mode(s, pairs, causal != 0, d));
  return 0;
}
"""

# causal, head size, sequence, (batch, head) pairs; us of the backward call (its GEMMs included) in two launches, in one with
# 128-row workgroups, in one with 64-row ones
MEASURED = [
    (1, 96, 200, 1, 33.1, 30.3, 27.9), (1, 96, 1024, 2, 55.0, 48.4, 40.9), (1, 96, 2048, 8, 91.3, 86.4, 78.1),
    (1, 96, 1024, 24, 83.4, 64.2, 77.8), (1, 96, 1024, 64, 153.4, 135.3, 167.3), (1, 96, 4096, 8, 196.2, 151.5, 175.1),
    (1, 96, 4096, 12, 245.6, 254.8, 297.8), (1, 64, 512, 24, 45.8, 42.3, 43.6), (1, 64, 4096, 16, 192.5, 199.7, 235.1),
    (1, 64, 1024, 96, 144.6, 124.8, 163.5), (1, 128, 512, 32, 78.4, 72.4, 83.1), (1, 128, 768, 6, 68.9, 59.2, 56.3),
    (1, 128, 2048, 8, 127.3, 99.3, 114.8), (0, 96, 1024, 8, 66.5, 66.2, 56.0), (0, 96, 768, 12, 61.7, 55.6, 63.5),
    (0, 96, 2048, 6, 89.8, 98.2, 106.0), (0, 96, 1024, 32, 94.1, 99.3, 114.7), (0, 64, 4096, 24, 427.8, 469.7, 545.0),
    (0, 128, 512, 12, 62.2, 55.6, 64.1), (0, 128, 1024, 12, 90.4, 95.8, 99.5),
]


@pytest.fixture(scope="module")
def modes(tmp_path_factory):
    d = tmp_path_factory.mktemp("modes")
    (d / "modes.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I" + BLD.CSRC, str(d / "modes.cpp"), "-o", str(d / "modes")], check=True, timeout=60)

    def run(cases):
        lines = "\n".join(" ".join(map(str, c)) for c in cases)
        out = subprocess.run([str(d / "modes")], input=lines, text=True, check=True, capture_output=True, timeout=60).stdout
        return [tuple(map(int, l.split())) for l in out.splitlines()]
    return run


def test_backward_takes_the_fastest_form(modes):
    for m, (mode, _) in zip(MEASURED, modes([m[:4] for m in MEASURED])):
        assert m[4 + mode] <= 1.04 * min(m[4:]), (m, mode)


def test_long_sequences_of_the_gpu_test_take_two_launches(modes):
    for d in (64, 96, 128):
        got = modes([(1, d, s, b * h) for b, h, s in TWO.SHAPES])
        assert [mode for mode, _ in got] == [0, 0], (d, got)                     # two launches
        assert [dq for _, dq in got] == [1, 0], (d, got)                         # dQ in paired wave groups, and in single ones
