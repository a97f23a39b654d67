"""Which fp32 GEMM kernel the shapes of the GPU tests take (no GPU needed: the rule is host arithmetic)."""
import subprocess

import pytest

from paper_1909_08053_amd import build as BLD
from test_gpu_fp32_kernels import F32_KERNELS, F32_LAYERS

MAIN = """#include <stdio.h>
#include "gemm_f32_pick.h"
int mlm::gemm_cu_count() { return 256; }
int main() {
  int M, N, K;
  while (scanf("%d %d %d", &M, &N, &K) == 3) printf("%d\\n", mlm::f32_pick(M, N, K));
  return 0;
}
"""


@pytest.fixture(scope="module")
def pick(tmp_path_factory):
    d = tmp_path_factory.mktemp("pick")
    (d / "pick.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I" + BLD.CSRC, str(d / "pick.cpp"), "-o", str(d / "pick")], check=True, timeout=60)

    def run(shapes):
        text = "\n".join(" ".join(map(str, s)) for s in shapes)
        out = subprocess.run([str(d / "pick")], input=text, text=True, check=True, capture_output=True, timeout=60).stdout
        return [int(x) for x in out.split()]
    return run


def test_gemm_shapes_take_the_kernels_they_are_listed_under(pick):
    for tile, shapes in F32_KERNELS.items():
        assert pick(shapes) == [tile] * len(shapes), tile


def test_layers_reach_the_fused_epilogues_of_the_tile_kernels(pick):
    for tile, (T, c) in F32_LAYERS.items():
        # bias + GeLU, GeLU' (both [T, F] over H), the recomputed logits [T, V] over H
        assert pick([(T, c["F"], c["H"]), (T, c["V"], c["H"])]) == [tile, tile]
        # weight gradients over the tokens (T is odd)
        assert set(pick([(c["H"], c["F"], T), (c["F"], c["H"], T)])) <= {64, 128}
    assert pick([(256, 32768, 133)]) == [128]
