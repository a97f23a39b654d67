"""Layer-norm backward at the edges of its workgroup count: one batch of rows, a ragged last batch, a second batch per
workgroup, and the smallest workspace the call accepts (which runs fewer workgroups than the workspace query asks for)."""
import numpy as np
import pytest
import torch

from oracle import layer_oracle as O
from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype,T,H", [("fp32", 1, 8), ("fp32", 2050, 1024), ("fp32", 1029, 2048), ("bf16", 4, 64),
                                       ("bf16", 5, 192), ("bf16", 2051, 1536), ("bf16", 1025, 3072), ("bf16", 1030, 3080)])
def test_ln_bwd_block_counts(dtype, T, H):
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    d = B.make_dims(1, T, H, 1, 8, 8, 1, 0, B.MLM_BF16 if dtype == "bf16" else B.MLM_F32)
    g = torch.Generator(device=DEV)
    g.manual_seed(T + H)
    dy, x, res = [torch.randn(T, H, generator=g, device=DEV).to(dt) for _ in range(3)]
    gam = (1 + 0.2 * torch.randn(H, generator=g, device=DEV)).to(dt)
    mean, rstd = x.float().mean(1).contiguous(), (x.float().var(1, unbiased=False) + 1e-5).rsqrt().contiguous()
    small = -(-((T + 31) // 32 * 3 * H * 4) // 256) * 256          # one partial per 32 rows
    full = B.mlm_workspace_bytes(d, B.WS_LAYERNORM_BWD)
    assert full >= small
    got = []
    for nbytes in (full, small):
        ws = torch.full((nbytes,), 255, device=DEV, dtype=torch.uint8)
        dx, dg, db, cs = torch.empty_like(x), torch.empty_like(gam), torch.empty_like(gam), torch.empty_like(gam)
        B.mlm_combine_layernorm_bwd(d, [dy], x, gam, mean, rstd, res, None, dx, dg, db, cs, ws)
        got.append([t.double().cpu().numpy() for t in (dx, dg, db, cs)])
    with pytest.raises(B.MlmError):
        B.mlm_combine_layernorm_bwd(d, [dy], x, gam, mean, rstd, res, None, dx, dg, db, cs,
                                    torch.empty(small - 256, device=DEV, dtype=torch.uint8) if small > 256 else None)
    f = lambda t: t.double().cpu().numpy()
    rdx, rdg, rdb = O.layernorm_bwd(f(dy), f(x), f(gam), f(mean), f(rstd))
    rdx = rdx + f(res)
    u = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -23
    assert np.array_equal(got[0][0], got[1][0])                    # a row's dx does not depend on the split
    xhat = (f(x) - f(mean)[:, None]) * f(rstd)[:, None]
    # fp32 sums in any order (at most T terms), one rounding to the storage type
    e32 = (T + 8) * 2.0 ** -24
    for dx, dg, db, cs in got:
        assert (np.abs(dx - rdx) <= u * np.abs(rdx) + 1e-4 * np.abs(rdx).max()).all()
        for v, ref, mag in ((dg, rdg, np.abs(f(dy) * xhat).sum(0)), (db, rdb, np.abs(f(dy)).sum(0)),
                            (cs, dx.sum(0), np.abs(dx).sum(0))):
            assert (np.abs(v - ref) <= u * np.abs(ref) + (e32 + 1e-5) * mag).all()
