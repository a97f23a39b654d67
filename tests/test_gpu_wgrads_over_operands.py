"""Weight gradients of a layer shard written over operands that only an earlier one of them reads, against float64."""
import pytest
import torch

from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# sizes that share a launch where nothing overlaps: in small, in 64-wide and (bf16) in large tiles with a split last round
@pytest.mark.parametrize("T,H", [(256, 256), (1024, 1024), (4096, 1056)])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_outputs_over_operands_read_before(T, H, dtype):
    td, code = (torch.bfloat16, B.MLM_BF16) if dtype == "bf16" else (torch.float32, B.MLM_F32)
    F = 4 * H
    d = B.make_dims(1, T, H, H // 8, F, 8, 1, 0, code)
    g = torch.Generator(device=DEV)
    g.manual_seed(T)
    x = {k: torch.randn(T, n, generator=g, device=DEV).to(td) for k, n in dict(u=H, dqkv=3 * H, ctx=H, dz1=H, u2=H, dg=F, y=F, dz2=H).items()}
    pairs = (("y", "dz2"), ("u2", "dg"), ("u", "dqkv"), ("ctx", "dz1"))          # the order in which they are formed
    ref = [x[a].double().t() @ x[b].double() for a, b in pairs]
    mag = [x[a].double().abs().t() @ x[b].double().abs() for a, b in pairs]
    over = lambda t, m, n: t.view(-1)[:m * n].view(m, n)
    dB, dA, dWqkv, dWo = torch.empty(F, H, device=DEV, dtype=td), over(x["y"], H, F), over(x["dg"], H, 3 * H), over(x["u"], H, H)
    ws = torch.empty(256 * 256 * 256 * 4, device=DEV, dtype=torch.uint8)
    B.mlm_layer_shard_wgrads(d, *(x[k] for k in ("u", "dqkv", "ctx", "dz1", "u2", "dg", "y", "dz2")), dWqkv, dWo, dA, dB, ws)
    eps = 2.0 ** -8 if dtype == "bf16" else 0.0
    for name, o, r, m in zip(("dB", "dA", "dWqkv", "dWo"), (dB, dA, dWqkv, dWo), ref, mag):
        # one rounding to bf16, and the forward error of any summation order of T fp32 products
        assert bool(((o.double() - r).abs() <= eps * r.abs() + (T + 1) * 2.0 ** -24 * m).all()), name
