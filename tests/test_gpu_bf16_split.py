"""bf16 products in tiles whose k is dealt to the eight waves of a workgroup: remainders of k, edges of tiles, every form and layout, joint
launches; and the 128 x 128 tile at the remainders of k, where outputs are just large enough for it."""
import pytest
import torch

from paper_1909_08053_amd import binding as B
from paper_1909_08053_amd import synth
from test_gpu_parity import run_layer_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# form (1: 64 x 64, 2: 32 x 64, 3: 32 x 32, 0: large tiles) -> M, N, K.  One unit of 8, one short of / one past a slice of 32, fewer slices than
# waves, a slice more or less than a round of the eight waves, two and three slices a wave, long ragged k; one tile, ragged tiles.
SHAPES = {
    3: [(M, N, K) for M, N in ((264, 200), (8, 8)) for K in (8, 24, 40, 256, 264, 488, 520, 1000)] + [(32, 64, 32), (264, 200, 1384)],
    2: [(456, 1000, 256), (488, 904, 488), (424, 1000, 520), (488, 904, 744), (488, 872, 1000), (1096, 392, 776)],
    1: [(904, 904, K) for K in (8, 40, 256, 264, 488, 520, 744, 1384)] + [(968, 872, 72)],
    0: [(1800, 1800, K) for K in (8, 40, 72, 96, 1000)],
}
# tokens, width, ways of the split, form of the four weight gradients in one launch; tokens, width, vocabulary, form of the logits' gradients
GROUPS = [(33, 192, 1, 3), (262, 192, 1, 2), (210, 256, 1, 1), (210, 256, 4, 3)]
DUALS = [(33, 192, 264, 3), (800, 256, 1096, 2), (800, 448, 1096, 1), (420, 768, 1096, 1)]


@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", [s for f in SHAPES.values() for s in f])
def test_bf16_gemm_forms(layout, M, N, K):
    ta, tb = layout
    g = torch.Generator(device=DEV)
    g.manual_seed(M + K)

    def operand(rows, cols):
        # what lies behind the operand in memory must never enter a sum
        t = torch.full((rows + 64, cols), float("nan"), device=DEV, dtype=torch.bfloat16)
        t[:rows] = torch.randn(rows, cols, generator=g, device=DEV).to(torch.bfloat16)
        return t[:rows]

    A = operand(K, M) if ta else operand(M, K)
    W = operand(N, K) if tb else operand(K, N)
    bias = torch.randn(N, generator=g, device=DEV).to(torch.bfloat16)
    C = torch.full((M + 1, N), float("nan"), device=DEV, dtype=torch.bfloat16)
    a, w = (A.t() if ta else A).double(), (W.t() if tb else W).double()
    for b in (None, bias):
        B.mlm_gemm(B.MLM_BF16, ta, tb, M, N, K, A, W, C[:M], b)
        ref, mag = a @ w, a.abs() @ w.abs()
        if b is not None:
            ref, mag = ref + b.double(), mag + b.double().abs()
        # fp32 accumulation of exact products in any order, then one rounding to bf16 (u = 2^-8)
        bound = 2.0 ** -8 * ref.abs() + (K + 2) * 2.0 ** -24 * mag
        assert bool((C[:M].double() - ref).abs().le(bound * 1.01).all())
        assert bool(C[M].isnan().all())


# all epilogues, the bias gradients beside and the joint launches above: token counts of no multiple of anything, all shards
@pytest.mark.parametrize("b,s,H,h,V,p,causal", [(1, 33, 192, 2, 264, 1, True), (2, 131, 192, 3, 1096, 1, False), (2, 105, 256, 4, 528, 1, True),
                                                (2, 105, 256, 4, 544, 4, True), (2, 210, 768, 8, 1096, 1, False), (1, 800, 448, 7, 1096, 1, True),
                                                (2, 400, 256, 4, 1096, 1, True)])
def test_bf16_layer_in_split_tiles(b, s, H, h, V, p, causal):
    run_layer_parity(synth.small_config(name=f"split{b * s}_{H}", dtype="bf16", b=b, s=s, H=H, h=h, F=4 * H, V=V, p=p, causal=causal,
                                        masked_lm=not causal), scale_w=3.0)
