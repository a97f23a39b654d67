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


LOWEST = {B.MLM_BF16: -3.3895313892515355e38, B.MLM_F32: -3.4028234663852886e38}
# tokens, columns, width: 64 x 64 and 32 x 64 tiles whose k is dealt to the waves, 128 x 128 tiles (one and two a compute unit, k whole and in
# pieces), 256 x 256 (k whole and in pieces); fp32 rows shorter and longer than what a thread keeps
MINUS_INF = [(B.MLM_BF16, 40, 8784, 1608), (B.MLM_BF16, 400, 1024, 192), (B.MLM_BF16, 33, 1032, 128), (B.MLM_BF16, 80, 10144, 80),
             (B.MLM_BF16, 272, 12008, 144), (B.MLM_BF16, 224, 5536, 2032), (B.MLM_BF16, 264, 25608, 128), (B.MLM_BF16, 488, 8240, 1616),
             (B.MLM_F32, 33, 1024, 128), (B.MLM_F32, 65, 8712, 128)]


def minus_inf_case(dtype, T, V, H):
    """Every third row overflows to -inf in all columns but the first quarter, every other third in none; V a whole number of tiles or not."""
    g = torch.Generator(device=DEV)
    g.manual_seed(T + V)
    td = torch.bfloat16 if dtype == B.MLM_BF16 else torch.float32
    hf = (torch.randn(T, H, generator=g, device=DEV)).to(td)
    E = torch.randn(H, V, generator=g, device=DEV).to(td)
    hf[:, :2] = 0
    hf[::3, 0] = 4.0
    E[:2] = 0
    E[0, V // 4:] = LOWEST[dtype]
    targets = torch.randint(0, V, (T,), generator=g, device=DEV, dtype=torch.int32)
    dims = B.make_dims(1, T, H, 1, 4 * H, V, 1, 0, dtype, True)
    out = [torch.full((T,), float("nan"), device=DEV) for _ in range(3)]
    logits = torch.empty(T, V, device=DEV, dtype=td)
    ws = torch.empty(B.mlm_workspace_bytes(dims, B.WS_VOCAB_CE_FWD), dtype=torch.uint8, device=DEV)
    return hf, E, lambda: (B.mlm_vocab_ce_shard_fwd(dims, hf, E, targets, *out, logits, ws), *out, logits)[1:]


@pytest.mark.parametrize("dtype,T,V,H", MINUS_INF)
def test_logits_at_minus_infinity(dtype, T, V, H):
    hf, E, run = minus_inf_case(dtype, T, V, H)
    m, s, t, logits = run()
    ref = hf.double() @ E.double()
    ref[ref < -3.5e38] = float("-inf")
    assert bool((logits[::3, V // 4:] == float("-inf")).all() and logits[::3, :V // 4].isfinite().all() and logits[1::3].isfinite().all())
    u, small = 2.0 ** -24, E.double()
    small[0] = 0                                                               # (no part of a finite logit)
    eps = (2 * H + 8) * u * (hf.double().abs() @ small.abs()).max(1).values + 4 * u * ref[ref.isfinite()].abs().max() + 1e-6
    assert bool((m.double() - ref.max(1).values).abs().le(eps).all())
    assert bool((m.double() + s.double().log() - torch.logsumexp(ref, 1)).abs().le(2 * eps + (V / 256 + 300) * u + 3e-6).all())


@pytest.mark.parametrize("dtype,T,V,H", MINUS_INF)
def test_a_nan_among_logits_at_minus_infinity_shows(dtype, T, V, H):
    hf, E, run = minus_inf_case(dtype, T, V, H)
    E[1, V // 2 + 5] = float("nan")                                            # one column of every row
    m, s, _, _ = run()
    assert bool(s.isnan().all() and not m[1::3].isnan().any())


@pytest.mark.parametrize("dtype,T,V,H", MINUS_INF)
def test_a_shard_at_minus_infinity(dtype, T, V, H):
    """All of a row's logits in the shard: its sum is 0, so that the merge with another shard's finite logits stays exact."""
    hf, E, run = minus_inf_case(dtype, T, V, H)
    E[0] = LOWEST[dtype]
    m, s, _, _ = run()
    assert bool((m[::3] == float("-inf")).all() and (s[::3] == 0).all() and m[1::3].isfinite().all() and (s[1::3] > 0).all())
