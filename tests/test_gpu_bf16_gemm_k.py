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


@pytest.mark.parametrize("s", [33, 131, 261, 1001])
def test_bf16_layer_with_an_odd_token_count(s):
    """The weight gradients sum over the tokens: K = 33, 131, 261, 1001, one by one and through the grouped launch; those of
    the output embedding with a k-split from 1001 on."""
    run_layer_parity(synth.small_config(name=f"s{s}", dtype="bf16", b=1, s=s, H=192, h=2, F=768, V=264, p=1), scale_w=3.0)


# more than one 128 x 128 tile per compute unit but at most two (the four-wave form of the small tile), ragged in every
# direction; and a long ragged contraction
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


# large tiles, 192 and 256 wide, ragged, with an odd number of 32-deep slices and with a K of any length
LARGE_TILES = {192: [(4088, 3064, 96), (1656, 2936, 1056), (4088, 3064, 1000)], 256: [(4088, 4088, 96), (4088, 4088, 160), (4088, 4088, 168)]}


@pytest.mark.parametrize("M,N,K", LARGE_TILES[192] + LARGE_TILES[256])
@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 0)])
def test_bf16_gemm_large_tiles_at_the_end_of_k(layout, M, N, K):
    ta, tb = layout
    g = torch.Generator(device=DEV)
    g.manual_seed(M + K)
    A = torch.randn((K, M) if ta else (M, K), generator=g, device=DEV).to(torch.bfloat16)
    W = torch.randn((N, K) if tb else (K, N), generator=g, device=DEV).to(torch.bfloat16)
    # an infinite operand in the slice that an odd count of slices copies twice is multiplied once: never 0 x Inf
    inf_at = K - 48
    (A[inf_at] if ta else A[:, inf_at])[7] = float("inf")
    C = torch.full((M + 1, N), float("nan"), device=DEV, dtype=torch.bfloat16)
    B.mlm_gemm(B.MLM_BF16, ta, tb, M, N, K, A, W, C[:M], None)
    a, w = (A.t() if ta else A).double(), (W.t() if tb else W).double()
    col = w[inf_at]
    assert torch.equal(C[7][col != 0].double(), torch.sign(col[col != 0]) * float("inf"))
    rows = torch.arange(M, device=DEV) != 7
    a, got = a[rows], C[:M][rows].double()
    ref = a @ w
    bound = 2.0 ** -8 * ref.abs() + (K + 2) * 2.0 ** -24 * (a.abs() @ w.abs())
    assert bool((got - ref).abs().le(bound * 1.01).all())
    assert bool(C[M].isnan().all())


def test_bf16_weight_gradients_of_large_tiles_split_along_an_odd_number_of_slices():
    """8224 = 257 x 32 tokens: the 256-wide tile in two k-pieces and a fix-up (dA, dB of 1920 x 3840)."""
    b, s, H, p = 8, 1028, 1920, 2
    T, Fl = b * s, 4 * H // p
    d = B.make_dims(b, s, H, 20, 4 * H, 16, p, 0, B.MLM_BF16)
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    r = lambda *sh, std=1.0: (torch.randn(*sh, generator=g, device=DEV) * std).to(torch.bfloat16)
    dx2, u2, A, W, pre, y = r(T, H), r(T, H), r(H, Fl, std=0.02), r(Fl, H, std=0.02), r(T, Fl), r(T, Fl)
    e = lambda *sh: torch.full(sh, float("nan"), device=DEV, dtype=torch.bfloat16)
    dA, da, dB, du, dg, da2, du2 = e(H, Fl), e(Fl), e(Fl, H), e(T, H), e(T, Fl), e(Fl), e(T, H)
    ws = torch.empty(B.mlm_workspace_bytes(d, B.WS_MLP_BWD), device=DEV, dtype=torch.uint8)
    B.mlm_mlp_shard_bwd(d, dx2, u2, A, W, pre, y, dA, da, dB, du, ws)
    B.mlm_mlp_shard_bwd_input(d, dx2, A, W, pre, dg, da2, du2, ws)           # dg: what dA is formed from
    for got, x, z in ((dB, y, dx2), (dA, u2, dg)):
        ref, mag = x.double().t() @ z.double(), x.double().abs().t() @ z.double().abs()
        assert bool((got.double() - ref).abs().le((2.0 ** -8 * ref.abs() + (T + 2) * 2.0 ** -24 * mag) * 1.01).all())


@pytest.mark.parametrize("H,h,V", [(768, 12, 520), (256, 4, 2600)])
def test_bf16_layer_on_small_tiles(H, h, V):
    """432 tiles in the grouped weight gradients (H = 768); cross-entropy partials of 128 columns with a ragged last tile."""
    run_layer_parity(synth.small_config(name=f"h{H}", dtype="bf16", b=1, s=264, H=H, h=h, F=4 * H, V=V, p=1), scale_w=3.0)
