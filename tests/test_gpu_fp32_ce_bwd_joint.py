"""The two fp32 gradients of the logits in one launch of 64 x 64 tiles, against float64 products of the same dL."""
import pytest
import torch

from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# tokens, width, vocabulary of the shard: either gradient's tiles leading, ragged edges in all three, last k tiles of 5 and of 8; sums of
# eight chains (the last)
SHAPES = [(512, 1024, 4096), (1101, 1032, 1024), (709, 1928, 2568), (1101, 1024, 1032), (389, 680, 16040)]


@pytest.mark.parametrize("T,H,V", SHAPES)
def test_logits_gradients_in_one_launch(T, H, V):
    dm = B.make_dims(1, T, H, 1, 8, V, 1, 0, B.MLM_F32)
    g = torch.Generator(device=DEV)
    g.manual_seed(T + V)
    hf, E, L = (torch.randn(*sh, generator=g, device=DEV) for sh in ((T, H), (H, V), (T, V)))
    targets = torch.randint(0, V, (T,), generator=g, device=DEV, dtype=torch.int32)
    M = L.max(1).values
    S = torch.exp(L - M[:, None]).sum(1)
    stats = torch.tensor([1.0, float(T)], device=DEV)
    ws = torch.empty(B.mlm_workspace_bytes(dm, B.WS_VOCAB_CE_BWD), device=DEV, dtype=torch.uint8)
    dE, dh = (torch.full(sh, float("nan"), device=DEV) for sh in ((H + 1, V), (T + 1, H)))
    B.mlm_vocab_ce_shard_bwd(dm, hf, E, targets, None, M, S, stats, L, dE[:H], dh[:T], ws)       # L now holds dL
    for got, a, b in ((dE, hf.t(), L), (dh, L, E.t())):
        a, b = a.double(), b.double()
        # forward error of any summation order of K fp32 products: (K + 1) u sum |a| |b|, u = 2^-24
        assert bool(((got[:-1].double() - a @ b).abs() <= (a.shape[1] + 1) * 2.0 ** -24 * (a.abs() @ b.abs())).all())
        assert bool(got[-1].isnan().all()), "write past the end"
