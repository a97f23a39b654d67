"""fp32 weight gradients of a layer shard, in one launch of the tile kernels' tiles, against float64."""
import pytest
import torch

from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# tokens, width, FFN width, ways of the split: 64-wide tiles with whole and ragged edges, a last k tile of 5, a single k tile, sums of two
# and of eight chains; 128-wide tiles, whole and ragged, for all and for some of the four; fewer tokens than a k tile
SHAPES = [(261, 512, 2048, 1), (517, 1000, 2000, 5), (64, 768, 768, 1), (33, 1032, 2056, 1), (1024, 1024, 4096, 1), (1021, 2064, 8208, 2),
          (77, 1000, 4000, 1), (5, 1032, 2056, 1), (77, 1032, 4104, 1), (33, 2040, 8160, 1), (72, 2048, 8192, 1), (218, 968, 3872, 1)]


@pytest.mark.parametrize("T,H,F,p", SHAPES)
def test_weight_gradients_in_one_launch(T, H, F, p):
    d = B.make_dims(1, T, H, H // 8, F, 8 * p, p, 0, B.MLM_F32)
    Hl, F = H // p, F // p
    g = torch.Generator(device=DEV)
    g.manual_seed(T + H)
    x = {k: torch.randn(T, n, generator=g, device=DEV) for k, n in
         dict(u=H, dqkv=3 * Hl, ctx=Hl, dz1=H, u2=H, dg=F, y=F, dz2=H).items()}
    out = [torch.full((m + 1, n), float("nan"), device=DEV) for m, n in ((H, 3 * Hl), (Hl, H), (H, F), (F, H))]
    ws = torch.empty(16, device=DEV, dtype=torch.uint8)                # fp32 needs none
    B.mlm_layer_shard_wgrads(d, *(x[k] for k in ("u", "dqkv", "ctx", "dz1", "u2", "dg", "y", "dz2")), *(o[:-1] for o in out), ws)
    for o, (a, b) in zip(out, (("u", "dqkv"), ("ctx", "dz1"), ("u2", "dg"), ("y", "dz2"))):
        a, b = x[a].double(), x[b].double()
        # forward error of any summation order of T fp32 products: (T + 1) u sum |a| |b|, u = 2^-24
        assert bool(((o[:-1].double() - a.t() @ b).abs() <= (T + 1) * 2.0 ** -24 * (a.abs().t() @ b.abs())).all())
        assert bool(o[-1].isnan().all()), "write past the end"
