"""fp32 products in small tiles whose k is dealt to the eight waves of a workgroup, each with a ring of its own: remainders of k, more and
fewer slices than stages, edges of tiles, all layouts, and what lies behind the operands."""
import pytest
import torch

from paper_1909_08053_amd import binding as B
from paper_1909_08053_amd import synth
from test_gpu_parity import run_layer_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# 32 x 32 tiles (k in chunks of 8): fewer chunks than waves, one, an uneven deal, two and three slices of 16 a wave with and without a half one,
# many; one tile and ragged ones.  16 x 16 (chunks of 16): one to nine slices a wave, uneven.
S32 = [(M, N, K) for M, N in ((264, 200), (8, 8)) for K in (8, 40, 64, 72, 136, 200, 264, 328, 392, 1000)] + [(40, 1000, 248), (872, 104, 2216)]
S16 = [(M, N, K) for M, N in ((264, 200), (24, 8)) for K in (128, 256, 384, 512, 640, 784, 1136)] + [(248, 504, 512), (504, 232, 1040)]


@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", S32 + S16)
def test_fp32_split_tiles(layout, M, N, K):
    ta, tb = layout
    g = torch.Generator(device=DEV)
    g.manual_seed(M + K)

    def operand(rows, cols):
        # what lies behind the operand in memory must never enter a sum
        t = torch.full((rows + 64, cols), float("nan"), device=DEV)
        t[:rows] = torch.randn(rows, cols, generator=g, device=DEV)
        return t[:rows]

    A = operand(K, M) if ta else operand(M, K)
    W = operand(N, K) if tb else operand(K, N)
    bias = torch.randn(N, generator=g, device=DEV)
    C = torch.full((M + 1, N), float("nan"), device=DEV)
    a, w = (A.t() if ta else A).double(), (W.t() if tb else W).double()
    for b in (None, bias):
        B.mlm_gemm(B.MLM_F32, ta, tb, M, N, K, A, W, C[:M], b)
        ref, mag = a @ w, a.abs() @ w.abs()
        if b is not None:
            ref, mag = ref + b.double(), mag + b.double().abs()
        # fp32 products and sums in any order: K products, K + 1 sums, u = 2^-24 each
        assert bool((C[:M].double() - ref).abs().le((K + 2) * 2.0 ** -24 * mag).all())
        assert bool(C[M].isnan().all())


# all epilogues, column sums beside, joint launches: token counts (k of the weight gradients) of no multiple of anything
@pytest.mark.parametrize("b,s,H,h,V,p,causal", [(1, 3, 64, 2, 264, 1, True), (1, 33, 192, 2, 264, 1, True), (2, 131, 256, 4, 528, 2, False)])
def test_fp32_layer_in_split_tiles(b, s, H, h, V, p, causal):
    run_layer_parity(synth.small_config(name=f"split{b * s}_{H}", dtype="fp32", b=b, s=s, H=H, h=h, F=4 * H, V=V, p=p, causal=causal,
                                        masked_lm=not causal))
