"""Cross-entropy partials of a vocabulary shard: column tiles fewer and more than a slice takes at a time (bf16), rows shorter and longer than what
a thread keeps of one (fp32), token counts that are no multiple of a block's, targets on and off the shard; rows that overflow an exp."""
import pytest
import torch

from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

V = [8, 64, 520, 1016, 4096, 4104, 8192, 8200, 8704, 25608]


@pytest.mark.parametrize("dtype", [B.MLM_BF16, B.MLM_F32])
@pytest.mark.parametrize("T", [1, 33, 264])
@pytest.mark.parametrize("V", V)
def test_partials(dtype, T, V):
    H = 128
    dims = B.make_dims(1, T, H, 2, 4 * H, 2 * V, 2, 1, dtype, True)            # the second of two shards
    g = torch.Generator(device=DEV)
    g.manual_seed(T + V)
    td = torch.bfloat16 if dtype == B.MLM_BF16 else torch.float32
    hf = (torch.randn(T, H, generator=g, device=DEV) * 3).to(td)
    E = torch.randn(H, V, generator=g, device=DEV).to(td)
    targets = torch.randint(0, 2 * V, (T,), generator=g, device=DEV, dtype=torch.int32)
    m, s, t = (torch.full((T + 1,), float("nan"), device=DEV) for _ in range(3))
    logits = torch.empty(T, V, device=DEV, dtype=td)
    ws = torch.empty(B.mlm_workspace_bytes(dims, B.WS_VOCAB_CE_FWD), dtype=torch.uint8, device=DEV)
    for scale in (1.0, 16.0):                                                  # (exp(16 x 24 ..) is beyond fp32)
        x = (hf.double() * scale).to(td)
        B.mlm_vocab_ce_shard_fwd(dims, x, E, targets, m, s, t, logits, ws)
        ref = x.double() @ E.double()
        mag = (x.double().abs() @ E.double().abs()).max(1).values
        # logits: fp32 sums of H products, u = 2^-24 of their magnitude; the exponential and its argument: as much again of |logit|, doubled; V sums
        u = 2.0 ** -24
        eps = (2 * H + 8) * u * mag + 4 * u * ref.abs().max(1).values + 1e-6
        assert bool((m[:T].double() - ref.max(1).values).abs().le(eps).all())
        got = m[:T].double() + s[:T].double().log()
        # (shares of V / 256 terms a thread, or of 64 .. 256 columns a tile and V / 512 tiles a slice, then a tree)
        assert bool((got - torch.logsumexp(ref, 1)).abs().le(2 * eps + (V / 256 + 300) * u + 3e-6).all())
        on = targets >= V
        want = torch.where(on, ref.gather(1, (targets.long() - V).clamp(min=0)[:, None])[:, 0], torch.zeros((), device=DEV, dtype=torch.double))
        assert bool((t[:T].double() - want).abs().le(eps).all())
        assert bool(m[T].isnan() and s[T].isnan() and t[T].isnan())
