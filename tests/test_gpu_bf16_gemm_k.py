"""bf16 GEMM: a contraction length that is no multiple of the 64-deep pairs its loop walks, and the 128 x 128 tile."""
import pytest
import torch

from paper_1909_08053_amd import binding as B
from paper_1909_08053_amd import synth
from test_gpu_parity import run_layer_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# one unit of 8, one short of / one past a slice of 32 and a pair of 64, an odd number of slices, a long ragged k
@pytest.mark.parametrize("K", [8, 24, 40, 56, 72, 96, 120, 136, 1000])
@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 0)])
def test_bf16_gemm_k_remainders(layout, K):
    M, N = 264, 200
    ta, tb = layout
    g = torch.Generator(device=DEV)
    g.manual_seed(K)

    def operand(rows, cols):
        # what lies behind the operand in memory must never enter a sum: rows past K (k-major) / past the end are NaN
        t = torch.full((rows + 64, cols), float("nan"), device=DEV, dtype=torch.bfloat16)
        t[:rows] = torch.randn(rows, cols, generator=g, device=DEV).to(torch.bfloat16)
        return t[:rows]

    A = operand(K, M) if ta else operand(M, K)
    W = operand(N, K) if tb else operand(K, N)
    C = torch.empty(M, N, device=DEV, dtype=torch.bfloat16)
    B.mlm_gemm(B.MLM_BF16, ta, tb, M, N, K, A, W, C, None)
    a, w = (A.t() if ta else A).double(), (W.t() if tb else W).double()
    ref = a @ w
    # fp32 accumulation of exact products in any order, then one rounding to bf16 (u = 2^-8)
    bound = 2.0 ** -8 * ref.abs() + (K + 2) * 2.0 ** -24 * (a.abs() @ w.abs())
    assert bool((C.double() - ref).abs().le(bound * 1.01).all())


@pytest.mark.parametrize("s", [33, 131, 261])
def test_bf16_layer_with_an_odd_token_count(s):
    """The weight gradients sum over the tokens: K = 33, 131, 261, one by one and through the grouped launch."""
    run_layer_parity(synth.small_config(name=f"s{s}", dtype="bf16", b=1, s=s, H=192, h=2, F=768, V=264, p=1), scale_w=3.0)


# more than one 128 x 128 tile per compute unit but at most two (the four-wave form of the small tile), ragged in every
# direction; and a contraction long and an output small enough for its k-split
@pytest.mark.parametrize("M,N,K", [(2056, 2008, 72), (4096, 1032, 136), (1960, 3000, 64), (264, 392, 4104)])
@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 0)])
def test_bf16_gemm_small_tiles(layout, M, N, K):
    ta, tb = layout
    g = torch.Generator(device=DEV)
    g.manual_seed(M + K)
    A = torch.randn((K, M) if ta else (M, K), generator=g, device=DEV).to(torch.bfloat16)
    W = torch.randn((N, K) if tb else (K, N), generator=g, device=DEV).to(torch.bfloat16)
    C = torch.full((M + 1, N), float("nan"), device=DEV, dtype=torch.bfloat16)
    B.mlm_gemm(B.MLM_BF16, ta, tb, M, N, K, A, W, C[:M], None)
    a, w = (A.t() if ta else A).double(), (W.t() if tb else W).double()
    ref = a @ w
    bound = 2.0 ** -8 * ref.abs() + (K + 2) * 2.0 ** -24 * (a.abs() @ w.abs())
    assert bool((C[:M].double() - ref).abs().le(bound * 1.01).all())
    assert bool(C[M].isnan().all())


@pytest.mark.parametrize("H,h,V", [(768, 12, 520), (256, 4, 2600)])
def test_bf16_layer_on_small_tiles(H, h, V):
    """432 tiles in the grouped weight gradients (H = 768); cross-entropy partials of 128 columns with a ragged last tile."""
    run_layer_parity(synth.small_config(name=f"h{H}", dtype="bf16", b=1, s=264, H=H, h=h, F=4 * H, V=V, p=1), scale_w=3.0)
