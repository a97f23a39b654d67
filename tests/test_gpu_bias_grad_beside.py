"""Bias gradients that are summed beside the input gradient's tiles, against the stored gradients that they sum."""
import pytest
import torch

from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# tokens, width, FFN width: one chunk of rows, a ragged one, ragged column blocks; small tiles alone and two a compute unit, the narrow
# and the large tile, a k-split; sums in a launch of their own (the last)
@pytest.mark.parametrize("T,H,F", [(40, 64, 72), (200, 192, 520), (704, 2048, 2048), (3000, 1536, 1536), (2048, 3072, 640), (4096, 4096, 1000),
                                   (8192, 512, 2048)])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_mlp_bias_gradient(T, H, F, dtype):
    td, code = (torch.bfloat16, B.MLM_BF16) if dtype == "bf16" else (torch.float32, B.MLM_F32)
    dm = B.make_dims(1, T, H, 1, F, 8, 1, 0, code)
    g = torch.Generator(device=DEV)
    g.manual_seed(T + F)
    n = lambda *sh, std: (torch.randn(*sh, generator=g, device=DEV) * std).to(td)
    dx2, A, Bm, pre = n(T, H, std=1.0), n(H, F, std=0.02), n(F, H, std=0.02), n(T, F, std=1.0)
    dg, da, du = (torch.full(sh, float("nan"), device=DEV, dtype=td) for sh in ((T, F), (F + 8,), (T, H)))
    ws = torch.empty(B.mlm_workspace_bytes(dm, B.WS_MLP_BWD), device=DEV, dtype=torch.uint8)
    B.mlm_mlp_shard_bwd_input(dm, dx2, A, Bm, pre, dg, da[:F], du, ws)
    eps = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -23
    want, mag = dg.double().sum(0), dg.double().abs().sum(0)
    # rounded once; chunks of 64 rows in slices of at most 16, then the chunks in slices: some 30 + T / 1024 additions in a row
    assert bool(((da[:F].double() - want).abs() <= eps * want.abs() + mag * 2.0 ** -24 * (30 + T / 1024)).all())
    assert bool(da[F:].isnan().all())
    ref, mag = dg.double() @ A.double().t(), dg.double().abs() @ A.double().abs().t()
    assert bool(((du.double() - ref).abs() <= eps * ref.abs() + mag * 2.0 ** -24 * 4 * F ** 0.5).all())
