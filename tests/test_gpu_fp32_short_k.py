"""fp32 products over few k: the split kernel's ranges of chunks, and the tile kernels where a k is too short for anything else."""
import pytest
import torch

from paper_1909_08053_amd import binding as B
from paper_1909_08053_amd import synth
from test_gpu_parity import run_layer_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (M, N, K).  Eight waves share a tile's chunks of 8 k, four chunks a step: waves with none, with one chunk, with a whole step, with
# one and with two steps, of which the last is not whole, with an odd and an even number of whole ones, with more than two
SPLIT = [(40, 72, K) for K in (8, 56, 72, 256, 296, 512, 520, 768, 1024, 1096, 1544)]
# (where 16 x 16 tiles find a compute unit each and K is a multiple of 128, or two a unit and K is one of 16 from 512 on, those: the
# same, with chunks of 16 k, and either side of the rule)
SPLIT += [(M, N, K) for M, N in ((16, 8), (24, 264)) for K in (112, 128, 256, 512, 528, 640, 1040, 1552, 2064)]
SPLIT += [(256, 256, 128), (264, 256, 256), (256, 512, 496), (256, 512, 512), (264, 512, 512)]
# the 64- and 128-tile kernels below the shortest k that is multiplied in pieces
TILES = [(1000, 1016, 56), (1032, 2048, 48), (4096, 4088, 56), (4088, 4096, 8)]


@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("shape", SPLIT + TILES)
def test_products(shape, layout):
    M, N, K = shape
    ta, tb = layout
    g = torch.Generator(device=DEV)
    g.manual_seed(M + N + K)
    A = torch.randn((K, M) if ta else (M, K), generator=g, device=DEV)
    W = torch.randn((N, K) if tb else (K, N), generator=g, device=DEV)
    C = torch.full((M + 1, N), 7.0, device=DEV)          # one canary row after the output
    B.mlm_gemm(B.MLM_F32, ta, tb, M, N, K, A, W, C, None)
    a, w = (A.t() if ta else A).double(), (W.t() if tb else W).double()
    # forward error of any summation order of K fp32 products: (K + 1) u sum |a| |w|, u = 2^-24
    assert bool(((C[:M].double() - a @ w).abs() <= (K + 1) * 2.0 ** -24 * (a.abs() @ w.abs())).all())
    assert bool((C[M] == 7.0).all()), "write past the end of C"


@pytest.mark.parametrize("T", [1, 7, 63, 100, 257, 515])
def test_weight_gradients_over_any_number_of_tokens(T):
    """The k of a weight gradient counts tokens: a wave whose last chunk is not whole reads its rows one by one."""
    H, V = 64, 128
    d = B.make_dims(1, T, H, 2, 4 * H, V, 1, 0, B.MLM_F32)
    g = torch.Generator(device=DEV)
    g.manual_seed(T)
    hf, E = torch.randn(T, H, generator=g, device=DEV), torch.randn(H, V, generator=g, device=DEV) * 0.1
    tgt = torch.randint(0, V, (T,), generator=g, device=DEV).int()
    w = torch.rand(T, generator=g, device=DEV) + 0.1
    m, su, t = (torch.empty(1, T, device=DEV) for _ in range(3))
    ws = torch.empty(max(B.mlm_workspace_bytes(d, k) for k in (B.WS_VOCAB_CE_FWD, B.WS_VOCAB_CE_BWD)), device=DEV, dtype=torch.uint8)
    ce, M, S, loss = (torch.empty(n, device=DEV) for n in (T, T, T, 2))
    B.mlm_vocab_ce_shard_fwd(d, hf, E, tgt, m, su, t, None, ws)
    B.mlm_vocab_ce_merge(d, m, su, t, 1, w, ce, M, S, loss)
    dE, dhf = torch.full((H, V), float("nan"), device=DEV), torch.full((T, H), float("nan"), device=DEV)
    B.mlm_vocab_ce_shard_bwd(d, hf, E, tgt, w, M, S, loss, None, dE, dhf, ws)
    dL = torch.softmax(hf.double() @ E.double(), -1)
    err = dL.clone()
    dL[torch.arange(T, device=DEV), tgt.long()] -= 1.0
    scale = (w.double() / w.double().sum())[:, None]
    # logits of 64 terms, off by at most 65 u of their terms' magnitude (as are the maxima), then exp (2 ulp) and four roundings: a
    # relative error of the probabilities of at most 2 * 65 u max sum |hf| |E| + 10 u, and one more sum of T (dE) or V (dhf) terms
    u = 2.0 ** -24
    rel = 2 * 65 * u * float((hf.double().abs() @ E.double().abs()).max()) + 10 * u
    dL, err = dL * scale, err * scale * rel
    for got, ref, bound, n in ((dE, hf.double().t() @ dL, hf.double().abs().t() @ err, T), (dhf, dL @ E.double().t(), err @ E.double().abs().t(), V)):
        mag = hf.double().abs().t() @ dL.abs() if got is dE else dL.abs() @ E.double().abs().t()
        assert bool(((got.double() - ref).abs() <= bound + (n + 4) * u * mag + 1e-12).all())


# narrow layers over many tokens: the fused epilogues of the 64- and 128-tile kernels at such k
LAYERS = {64: dict(b=1, s=1000, H=48, h=3, F=1024, V=1024), 128: dict(b=3, s=667, H=32, h=2, F=4096, V=4096)}


@pytest.mark.parametrize("tile", sorted(LAYERS))
@pytest.mark.parametrize("store_logits", [True, False])
def test_layer_on_the_tile_kernels(tile, store_logits):
    run_layer_parity(synth.small_config(name=f"narrow{tile}", dtype="fp32", p=1, **LAYERS[tile]), store_logits=store_logits, scale_w=2.0)
