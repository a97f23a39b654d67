"""bf16 products in 128 x 192 tiles, at most one a compute unit: remainders of k around pairs of slices and the eight-slice ring, ragged tiles at
every edge, all layouts, every epilogue and the column sums beside; the four weight gradients of a shard in one launch, of token counts that are no multiple of anything."""
import pytest
import torch

from paper_1909_08053_amd import binding as B
from paper_1909_08053_amd import synth
from test_gpu_parity import run_layer_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# more than 256 tiles of 128 x 128, at most 256 of 128 x 192: whole tiles (256 of them), a last column tile of 8, 64 and 184 columns, of one row
# and of 120; rows in one tile row, columns in two tile columns
MN = [(8192, 768), (3000, 1544), (5256, 952), (4360, 1240), (120, 33016), (16384, 264)]
KS = [192, 200, 224, 248, 256, 264, 320, 504, 520, 1032]


@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", [(M, N, K) for M, N in MN for K in ((192, 264) if M * N > 2 ** 22 else KS[:4])] + [(3000, 1544, K) for K in KS[4:]])
def test_bf16_middle_tile(layout, M, N, K):
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


# (b, s, H, h, V, p, causal) -> which of the layer's products take the tile (test_bf16_middle_choice_host.py): bias + GeLU, GeLU', plain products, the column
# sums beside an input gradient, and the weight gradients of token counts that are no multiple of anything
LAYERS = {
    (2, 1100, 512, 8, 528, 1, True): "", (2, 724, 768, 8, 528, 1, False): "fc1 dg", (64, 133, 512, 8, 264, 1, True): "proj fc2 dfc1 dctx dqkv",
    (1, 193, 576, 6, 264, 1, True): "wgrads", (3, 211, 640, 5, 264, 1, False): "wgrads", (7, 257, 576, 9, 264, 1, True): "wgrads",
    (1, 1900, 768, 12, 264, 1, True): "qkv fc1 dg", (20, 380, 640, 10, 528, 2, True): "proj fc2 dfc1 dqkv",
}


@pytest.mark.parametrize("b,s,H,h,V,p,causal", LAYERS)
def test_bf16_layer_in_middle_tiles(b, s, H, h, V, p, causal):
    run_layer_parity(synth.small_config(name=f"middle{b * s}_{H}", dtype="bf16", b=b, s=s, H=H, h=h, F=4 * H, V=V, p=p, causal=causal,
                                        masked_lm=not causal), scale_w=3.0)
