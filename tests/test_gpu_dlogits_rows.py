"""Gradients of stored logits, formed in place: every vector of every row, in both forms of the pass, against float64."""
import pytest
import torch

from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# rows around the line between the forms and around none; rows of one vector, of one workgroup's vectors and one more, of 1024 and 1025
@pytest.mark.parametrize("T", [1, 40, 511, 512, 1000])
@pytest.mark.parametrize("nv", [1, 255, 257, 800, 1024, 1025])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("weighted", [True, False])
def test_every_vector_once(T, nv, dtype, weighted):
    td, code, vn = (torch.bfloat16, B.MLM_BF16, 8) if dtype == "bf16" else (torch.float32, B.MLM_F32, 4)
    V, H = (nv + nv % 2 * (vn == 4)) * vn, 16                      # (a vocabulary is a multiple of eight)
    d = B.make_dims(1, T, H, 2, 16, 2 * V, 2, 1, code)             # the second of two shards: targets from V on are its own
    g = torch.Generator(device=DEV)
    g.manual_seed(T + nv)
    L = torch.full((T + 1, V), float("nan"), device=DEV, dtype=td)
    L[:T] = torch.randn(T, V, generator=g, device=DEV) * 2
    targets = torch.randint(0, 2 * V, (T,), generator=g, device=DEV, dtype=torch.int32)
    targets[0] = 2 * V - 1
    w = torch.rand(T, generator=g, device=DEV) if weighted else None
    x = L[:T].double()
    M = x.max(1).values.float()
    S = torch.exp(x - M.double()[:, None]).sum(1).float()
    stats = torch.tensor([1.0, 3.0], device=DEV)
    hf, E = torch.randn(T, H, generator=g, device=DEV).to(td), torch.randn(H, V, generator=g, device=DEV).to(td)
    dE, dh = torch.empty(H, V, device=DEV, dtype=td), torch.empty(T, H, device=DEV, dtype=td)
    ws = torch.empty(B.mlm_workspace_bytes(d, B.WS_VOCAB_CE_BWD), device=DEV, dtype=torch.uint8)
    B.mlm_vocab_ce_shard_bwd(d, hf, E, targets, w, M, S, stats, L[:T], dE, dh, ws)
    coef = ((w.double() if weighted else torch.ones(T, device=DEV, dtype=torch.float64)) / 3.0)[:, None]
    p = torch.exp(x - M.double()[:, None]) / S.double()[:, None] * coef
    hot = torch.arange(V, 2 * V, device=DEV)[None, :] == targets[:, None]
    want = p - coef * hot
    # u = 2^-24: the difference L - M and its product with log2 e are rounded, each an error of |L - M| u in the exponent; exponential,
    # factor, its two divisions and the last subtraction some 8 u of either term; one rounding to bf16
    arg = M.double()[:, None] - x
    bound = (p * (2 * arg + 8) + coef * hot * 8) * 2.0 ** -24 + (want.abs() * 2.0 ** -8 if dtype == "bf16" else 0.0)
    assert bool(((L[:T].double() - want).abs() <= bound + 1e-30).all())
    assert bool(L[T].isnan().all())
