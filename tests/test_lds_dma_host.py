"""Assembly of the copies into LDS (no GPU needed: hipcc only compiles)."""
import os
import subprocess

from paper_1909_08053_amd import build as BLD

SRC = """#include "lds_dma.h"
__global__ void copies(const mlm::bf16* a, const float* b, float* out, unsigned at) {
  extern __shared__ float lds[];
  mlm::dma16(a + threadIdx.x * 8, __builtin_amdgcn_readfirstlane(at));
  mlm::dma4(b + threadIdx.x, __builtin_amdgcn_readfirstlane(at + 1024));
  mlm::wait_vmcnt<0>();
  __syncthreads();
  out[threadIdx.x] = lds[threadIdx.x];
}
"""


def test_copies_into_lds_wait_one_state_behind_the_write_of_m0(tmp_path):
    """A copy into LDS takes its LDS address from M0, and gfx950 wants one wait state between a scalar write of M0 and the
    copy; the compiler puts it between instructions of its own, inside inline assembly it does not."""
    src, asm = tmp_path / "copies.hip", tmp_path / "copies.s"
    src.write_text(SRC)
    subprocess.run([BLD._hipcc(), *BLD.FLAGS, "--cuda-device-only", "-S", str(src), "-o", str(asm)], check=True,
                   capture_output=True, timeout=120)
    code = [l.strip() for l in asm.read_text().splitlines()]
    code = [l for l in code if l and l[0] not in ";." and not l.endswith(":")]
    copies = [i for i, l in enumerate(code) if l.startswith("global_load_lds")]
    assert len(copies) == 2
    for i in copies:
        assert "m0" not in code[i - 1], code[i - 2:i + 1]
        assert any(l.startswith("s_mov_b32 m0") for l in code[i - 2:i]), code[i - 2:i + 1]
