"""fp32 matrix-core kernels at the edges of their tiles: the three GEMM kernels, and attention at every kind of head size."""
import pytest
import torch

from paper_1909_08053_amd import binding as B
from paper_1909_08053_amd import synth
from test_gpu_parity import run_layer_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (M, N, K): split-k kernel with fewer k chunks than waves, uneven eighths, one row past a 32-tile; 64-tile kernel on
# ragged tiles, with a last k tile of 8 and exactly one k tile; 128-tile kernel with a ragged last tile column
F32_SHAPES = [(8, 8, 8), (40, 72, 136), (264, 256, 520), (1000, 1544, 328), (1032, 2048, 64), (4096, 4088, 136)]


@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("shape", F32_SHAPES)
def test_f32_gemm_kernels(shape, layout):
    M, N, K = shape
    ta, tb = layout
    g = torch.Generator(device=DEV)
    g.manual_seed(M + 3 * N + 7 * K)
    A = torch.randn((K, M) if ta else (M, K), generator=g, device=DEV)
    W = torch.randn((N, K) if tb else (K, N), generator=g, device=DEV)
    bias = torch.randn(N, generator=g, device=DEV)
    C = torch.full((M + 1, N), 7.0, device=DEV)          # one canary row after the output
    B.mlm_gemm(B.MLM_F32, ta, tb, M, N, K, A, W, C, bias)
    a, w = (A.t() if ta else A).double(), (W.t() if tb else W).double()
    ref = a @ w + bias.double()
    # forward error of any summation order of K fp32 products and the bias: (K + 1) u sum |a| |w|, u = 2^-24
    bound = (K + 2) * 2.0 ** -24 * (a.abs() @ w.abs() + bias.double().abs())
    assert bool((C[:M].double() - ref).abs().le(bound).all())
    assert bool((C[M] == 7.0).all()), "write past the end of C"


# (the weight gradients' k is the token count: 62, 33, 261 leave a last chunk of 6, 1 and 5 of its 8)
# sequence lengths around the 32-row tiles and the four waves that share them; head sizes that do and do not fill 32 columns
F32_ATTN = {
    "d16_one_tile": dict(b=2, s=31, H=64, h=4, p=2),
    "d48_two_tiles": dict(b=1, s=33, H=192, h=4, p=2),
    "d80_bert": dict(b=3, s=130, H=320, h=4, p=2, causal=False, masked_lm=True),
    "d112_five_tiles": dict(b=1, s=136, H=224, h=2, p=1),
    "d128_nine_tiles": dict(b=1, s=261, H=256, h=2, p=2),
}


@pytest.mark.parametrize("name", sorted(F32_ATTN))
def test_f32_attention_tiles(name):
    kw = dict(F32_ATTN[name], dtype="fp32", V=256)
    kw["F"] = 4 * kw["H"]
    run_layer_parity(synth.small_config(name=name, **kw), scale_w=4.0)
