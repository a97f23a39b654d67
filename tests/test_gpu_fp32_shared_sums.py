"""fp32 products that share a launch are no further from float64 than each of them alone."""
import pytest
import torch

from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def no_further(name, got, trans_a, trans_b, X, Y):
    """X, Y as stored; got: their product as the shared launch left it."""
    a, b = X.double().t() if trans_a else X.double(), Y.double().t() if trans_b else Y.double()
    M, K, N = a.shape[0], a.shape[1], b.shape[1]
    alone = torch.empty(M, N, device=DEV)
    B.mlm_gemm(B.MLM_F32, trans_a, trans_b, M, N, K, X, Y, alone)
    ref = a @ b
    err = lambda t: float((t.double() - ref).norm())
    # sums of as many chains of the same length or shorter ones: 2-norms over 10^4 rounding errors and more, 3 % of spread each
    assert err(got) <= 1.1 * err(alone), (name, err(got) / float(ref.norm()), err(alone) / float(ref.norm()))


# tokens, width, ways of the split: products that alone take the split kernel beside 64- and 128-wide ones
@pytest.mark.parametrize("T,H,p", [(56, 768, 1), (48, 1600, 4), (120, 1512, 1), (176, 1880, 1), (1024, 1024, 1)])
def test_weight_gradients(T, H, p):
    d = B.make_dims(1, T, H, H // 8, 4 * H, 8 * p, p, 0, B.MLM_F32)
    Hl, F = H // p, 4 * H // p
    g = torch.Generator(device=DEV)
    g.manual_seed(T)
    x = {k: torch.randn(T, n, generator=g, device=DEV) for k, n in dict(u=H, dqkv=3 * Hl, ctx=Hl, dz1=H, u2=H, dg=F, y=F, dz2=H).items()}
    out = [torch.empty(m, n, device=DEV) for m, n in ((H, 3 * Hl), (Hl, H), (H, F), (F, H))]
    ws = torch.empty(16, device=DEV, dtype=torch.uint8)
    B.mlm_layer_shard_wgrads(d, *(x[k] for k in ("u", "dqkv", "ctx", "dz1", "u2", "dg", "y", "dz2")), *out, ws)
    for o, (a, b) in zip(out, (("u", "dqkv"), ("ctx", "dz1"), ("u2", "dg"), ("y", "dz2"))):
        no_further(a + b, o, 1, 0, x[a], x[b])


@pytest.mark.parametrize("T,H,V", [(1000, 144, 2328), (704, 1920, 2560), (512, 1024, 4096)])
def test_gradients_of_the_logits(T, H, V):
    d = B.make_dims(1, T, H, 1, 8, V, 1, 0, B.MLM_F32)
    g = torch.Generator(device=DEV)
    g.manual_seed(V)
    hf, E, L = (torch.randn(*sh, generator=g, device=DEV) for sh in ((T, H), (H, V), (T, V)))
    targets = torch.randint(0, V, (T,), generator=g, device=DEV, dtype=torch.int32)
    M = L.max(1).values
    S = torch.exp(L - M[:, None]).sum(1)
    ws = torch.empty(B.mlm_workspace_bytes(d, B.WS_VOCAB_CE_BWD), device=DEV, dtype=torch.uint8)
    dE, dh = torch.empty(H, V, device=DEV), torch.empty(T, H, device=DEV)
    B.mlm_vocab_ce_shard_bwd(d, hf, E, targets, None, M, S, torch.tensor([1.0, float(T)], device=DEV), L, dE, dh, ws)   # L: now dL
    no_further("dE", dE, 1, 0, hf, L)
    no_further("dhf", dh, 0, 1, L, E)
