"""Layer-norm backward with four rows a workgroup (few bf16 rows, and fp32): widths around a lane's vectors, partials two at a time."""
import numpy as np
import pytest
import torch

from oracle import layer_oracle as O
from oracle import rng_embed_oracle as R
from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# rows: one, one more than a workgroup's, the most; widths: one vector, whole and ragged vectors of one wave, of two; fp32 also several rows a wave
@pytest.mark.parametrize("dtype,T,H", [("bf16", 1, 8), ("bf16", 5, 192), ("bf16", 333, 520), ("bf16", 767, 1536), ("bf16", 6, 1544), ("bf16", 130, 3072),
                                       ("fp32", 3, 8), ("fp32", 257, 264), ("fp32", 66, 768), ("fp32", 1025, 776), ("fp32", 5, 1536), ("fp32", 4099, 256)])
@pytest.mark.parametrize("n,p_drop", [(1, 0.0), (2, 0.0), (3, 0.1)])
def test_few_rows(dtype, T, H, n, p_drop):
    td, u = (torch.bfloat16, 2.0 ** -8) if dtype == "bf16" else (torch.float32, 2.0 ** -23)
    d = B.make_dims(1, T, H, 1, 8, 8, 1, 0, B.MLM_BF16 if dtype == "bf16" else B.MLM_F32)
    g = torch.Generator(device=DEV)
    g.manual_seed(T + H + n)
    parts = [torch.randn(T, H, generator=g, device=DEV).to(td) for _ in range(n)]
    x, res = [torch.randn(T, H, generator=g, device=DEV).to(td) for _ in range(2)]
    gam = (1 + 0.2 * torch.randn(H, generator=g, device=DEV)).to(td)
    mean, rstd = x.float().mean(1).contiguous(), (x.float().var(1, unbiased=False) + 1e-5).rsqrt().contiguous()
    ws = torch.full((B.mlm_workspace_bytes(d, B.WS_LAYERNORM_BWD),), 255, device=DEV, dtype=torch.uint8)
    nan = lambda *sh: torch.full(sh, float("nan"), device=DEV, dtype=td)
    dy, dx, dz = (nan(T + 1, H) for _ in range(3))
    dg, db, cs = (nan(H + 8) for _ in range(3))
    out = (dg[:H], db[:H], cs[:H], ws)
    if p_drop:
        drop = B.make_dropout(p_drop, 5, 3)
        B.mlm_combine_layernorm_bwd_dropout(d, parts, x, gam, mean, rstd, res, drop, dy[:T], dx[:T], dz[:T], *out)
    else:
        B.mlm_combine_layernorm_bwd(d, parts, x, gam, mean, rstd, res, dy[:T], dx[:T], *out)
    f = lambda t: t.double().cpu().numpy()
    total = parts[0].float()
    for p in parts[1:]:
        total = total + p.float()                                  # in the order of the partials, fp32
    dyv = f(total.to(td))
    assert np.array_equal(f(dy[:T]), dyv)
    rdx, rdg, rdb = O.layernorm_bwd(dyv, f(x), f(gam), f(mean), f(rstd))
    rdx = rdx + f(res)
    got = f(dx[:T])
    assert (np.abs(got - rdx) <= u * np.abs(rdx) + (1e-4 if dtype == "bf16" else 1e-5) * np.abs(rdx).max()).all()
    summed = got
    if p_drop:
        ref = np.where(R.keep_mask(5, 3, (T, H), p_drop), got / (1.0 - np.float32(p_drop)), 0.0)
        summed = f(dz[:T])
        assert (np.abs(summed - ref) <= 1.01 * u * np.abs(ref) + 1e-6 * np.abs(ref)).all()
    xhat = (f(x) - f(mean)[:, None]) * f(rstd)[:, None]
    e32 = (T + 8) * 2.0 ** -24                        # fp32 sums in any order (at most T terms), one rounding to the storage type
    for v, ref, mag in ((dg, rdg, np.abs(dyv * xhat).sum(0)), (db, rdb, np.abs(dyv).sum(0)), (cs, summed.sum(0), np.abs(summed).sum(0))):
        assert (np.abs(f(v[:H]) - ref) <= u * np.abs(ref) + (e32 + 1e-5) * mag).all()
    for t in (dy[T], dx[T], dg[H:], db[H:], cs[H:]):
        assert bool(t.isnan().all()), "write past the end"
