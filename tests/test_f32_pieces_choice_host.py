"""Which fp32 products are formed in bf16 pieces (no GPU needed: the rule is host arithmetic)."""
import subprocess

import pytest

import test_gpu_fp32_pieces as P
from paper_1909_08053_amd import build as BLD

MAIN = """#include <stdio.h>
#include "gemm_f32_pick.h"
int mlm::gemm_cu_count() { return 256; }
int main() {
  int M, N, K;
  while (scanf("%d %d %d", &M, &N, &K) == 3) printf("%d\\n", mlm::f32_pieces_pick(M, N, K));
  return 0;
}
"""

# M, N, K; us on the fp32 matrix cores, in pieces with 128-wide and with 64-wide tiles (forward layout)
MEASURED = [
    (1024, 1024, 256, 8.4, 15.0, 10.1), (1024, 1024, 1024, 21.2, 41.3, 20.3), (1024, 1024, 4096, 71.6, 147.0, 65.7), (512, 512, 1024, 11.3, 41.2, 17.9),
    (512, 1024, 4096, 69.9, 146.5, 58.8), (256, 1024, 4096, 35.6, 147.6, 56.6), (256, 256, 4096, 31.7, 148.9, 54.2), (768, 2048, 4096, 135.1, 149.1, 117.3),
    (768, 2048, 256, 12.8, 15.4, 17.3), (1024, 2048, 4096, 139.1, 153.8, 128.7), (1024, 2560, 512, 30.1, 25.1, 34.2), (1024, 3072, 1024, 54.2, 46.1, 56.3),
    (1024, 3072, 128, 12.8, 11.8, 20.2), (1024, 4096, 1024, 71.8, 52.1, 74.8), (1536, 4096, 256, 33.7, 27.3, 47.1), (2048, 4096, 128, 24.1, 21.2, 49.1),
    (2048, 6144, 1024, 194.5, 142.5, 222.4), (4096, 4096, 512, 133.7, 100.0, 177.1), (4096, 4096, 1024, 251.3, 186.1, 286.2),
]


@pytest.fixture(scope="module")
def pick(tmp_path_factory):
    d = tmp_path_factory.mktemp("pieces")
    (d / "pick.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I" + BLD.CSRC, str(d / "pick.cpp"), "-o", str(d / "pick")], check=True, timeout=60)

    def run(shapes):
        text = "\n".join("%d %d %d" % tuple(s[:3]) for s in shapes)
        out = subprocess.run([str(d / "pick")], input=text, text=True, check=True, capture_output=True, timeout=60).stdout
        return [int(x) for x in out.split()]
    return run


def test_shapes_of_the_gpu_tests(pick):
    for tile, shapes in P.SHAPES.items():
        assert pick(shapes) == [tile] * len(shapes), tile


def test_rule_takes_the_faster_form(pick):
    for m, bt in zip(MEASURED, pick(MEASURED)):
        assert m[{0: 3, 128: 4, 64: 5}[bt]] <= 1.05 * min(m[3:]), (m, bt)


def test_steps_lie_inside_k(pick):
    """What is fetched ahead of the last step needs 64 k."""
    assert pick([(4096, 4096, 56), (8192, 8192, 8), (4096, 4096, 64)]) == [0, 0, 128]
