"""Input embedding at the edges of its 64 x 64 (gradient of few tokens: 16 x 16) tiles: one token, ragged tokens and rows, runs of equal ids that cross the 16
positions of a wave and the 64 of a tile, ids of other shards."""
import pytest
import torch

from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("T,H,Vl,distinct", [(1, 16, 8, 8), (64, 64, 64, 1), (257, 80, 40, 2),
                                                (1000, 144, 512, 1024), (700, 64, 24, 30),
                                                # gradient with four waves per workgroup: 65 x 17 and 47 x 8 tiles
                                                (4100, 1040, 64, 3), (3000, 512, 704, 1400)])
def test_embedding_tiles(dtype, T, H, Vl, distinct):
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    p, r = 2, 1                                       # the shard owns ids [Vl, 2 Vl)
    d = B.make_dims(1, T, H, 1, 16, 2 * Vl, 1, 0, B.MLM_BF16 if dtype == "bf16" else B.MLM_F32)
    d.p, d.r, d.h, d.F = p, r, 2, 16
    g = torch.Generator(device=DEV)
    g.manual_seed(T)
    lo = 0 if distinct > Vl else Vl
    ids = (lo + torch.randint(0, min(distinct, 2 * Vl - lo), (T,), generator=g, device=DEV)).int()
    E = torch.randn(H, Vl, generator=g, device=DEV).to(dt)
    dE = torch.randn(H, Vl, generator=g, device=DEV).to(dt)
    dz = torch.randn(T, H, generator=g, device=DEV).to(dt)
    perm = torch.empty(T, device=DEV, dtype=torch.int32)
    out = torch.full((T + 1, H), float("nan"), device=DEV, dtype=dt)
    B.mlm_embed_shard_fwd(d, ids, E, perm, out[:T])
    loc = ids.long() - Vl
    own = loc >= 0
    want = torch.where(own[:, None], E.t()[loc.clamp(min=0)], torch.zeros((), device=DEV, dtype=dt))
    assert torch.equal(out[:T], want) and bool(out[T].isnan().all())
    key = torch.where(own, loc, Vl)
    assert torch.equal(perm.long(), torch.sort(key, stable=True).indices)
    got = dE.clone()
    B.mlm_embed_shard_bwd(d, ids, perm, dz, got)
    ref = dE.double().t().contiguous()
    ref.index_add_(0, loc[own], dz.double()[own])
    mag = dE.double().abs().t().contiguous()
    mag.index_add_(0, loc[own], dz.double().abs()[own])
    u = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -23
    # fp32 sums of at most T terms, one rounding to the storage type
    assert bool(((got.t().double() - ref).abs() <= u * ref.abs() + (T + 2) * 2.0 ** -24 * mag).all())
    untouched = torch.ones(Vl, dtype=torch.bool, device=DEV)
    untouched[loc[own]] = False
    assert torch.equal(got[:, untouched], dE[:, untouched])
