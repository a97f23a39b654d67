"""fp32 matrix-core kernels at the edges of their tiles: the three GEMM kernels, and attention at every kind of head size."""
import pytest
import torch

from paper_1909_08053_amd import binding as B
from paper_1909_08053_amd import synth
from test_gpu_parity import run_layer_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (M, N, K) by kernel: split-k (32) with fewer k chunks than waves, uneven eighths, one row past a 32-tile; 64-tile on ragged
# tiles, with a last k tile of 8 and with one k tile, whole and not; 128-tile with few k and a ragged last tile column
F32_KERNELS = {32: [(8, 8, 8), (40, 72, 136), (264, 256, 520)], 64: [(1000, 1544, 328), (1000, 1016, 64), (1000, 1016, 40)],
               128: [(1032, 2048, 64), (4096, 4088, 136)]}
F32_SHAPES = [s for k in sorted(F32_KERNELS) for s in F32_KERNELS[k]]


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


# Layers whose GEMMs take the tile kernels, so that every fused epilogue of theirs (bias + GeLU with the saved pre-activation,
# GeLU', the recomputed logits' gradient) and weight gradients over a ragged token count are checked: (tokens, config)
F32_LAYERS = {64: (261, dict(b=1, s=261, H=512, h=4, F=2048, V=2048, p=1)), 128: (2001, dict(b=3, s=667, H=256, h=4, F=4096, V=4096, p=1))}


@pytest.mark.parametrize("tile", sorted(F32_LAYERS))
@pytest.mark.parametrize("store_logits", [True, False])
def test_f32_layer_on_the_tile_kernels(tile, store_logits):
    kw = dict(F32_LAYERS[tile][1], dtype="fp32")
    run_layer_parity(synth.small_config(name=f"tile{tile}", **kw), store_logits=store_logits, scale_w=2.0)


def test_f32_ragged_weight_gradient_on_the_128_tile_kernel():
    """dE of 256 x 32768 over 133 tokens, the logits recomputed."""
    b, s, H, V = 1, 133, 256, 32768
    T = b * s
    d = B.make_dims(b, s, H, 4, 4 * H, V, 1, 0, B.MLM_F32)
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    hf, E = torch.randn(T, H, generator=g, device=DEV), torch.randn(H, V, generator=g, device=DEV) * 0.1
    tgt = torch.randint(0, V, (T,), generator=g, device=DEV).int()
    w = torch.rand(T, generator=g, device=DEV)
    z = torch.empty(1, T, device=DEV)
    m, su, t = z, torch.empty_like(z), torch.empty_like(z)
    ws = torch.empty(max(B.mlm_workspace_bytes(d, k) for k in (B.WS_VOCAB_CE_FWD, B.WS_VOCAB_CE_BWD)), device=DEV, dtype=torch.uint8)
    ce, M, S, loss = (torch.empty(n, device=DEV) for n in (T, T, T, 2))
    B.mlm_vocab_ce_shard_fwd(d, hf, E, tgt, m, su, t, None, ws)
    B.mlm_vocab_ce_merge(d, m, su, t, 1, w, ce, M, S, loss)
    dE, dhf = torch.full((H, V), float("nan"), device=DEV), torch.full((T, H), float("nan"), device=DEV)
    B.mlm_vocab_ce_shard_bwd(d, hf, E, tgt, w, M, S, loss, None, dE, dhf, ws)
    L = hf.double() @ E.double()
    dL = torch.softmax(L, -1)
    dL[torch.arange(T, device=DEV), tgt.long()] -= 1.0
    dL *= (w.double() / w.double().sum())[:, None]
    # logits of 256 terms (and the maxima and sums formed from them) are off by at most 1e-5 of their terms' magnitude, which
    # exp passes on as a relative error of the probabilities; then one more fp32 sum
    err = 2e-5 * (hf.double().abs() @ E.double().abs()).max() * (torch.softmax(L, -1) * (w.double() / w.double().sum())[:, None])
    for got, ref, bound in ((dE, hf.double().t() @ dL, hf.double().abs().t() @ err), (dhf, dL @ E.double().t(), err @ E.double().abs().t())):
        assert bool(((got.double() - ref).abs() <= bound + 1e-5 * ref.abs() + 1e-9).all())
