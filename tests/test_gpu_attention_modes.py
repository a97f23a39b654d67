"""bf16 attention kernels in each of the ways their waves divide the work (by the number of 128-row workgroups), against
float64 on the same bf16 inputs."""
import pytest
import torch

from oracle import rng_embed_oracle as R
from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# s = 136: a second block of 8 queries, a third tile of 8 keys; 2, 136 and 272 workgroups of 128 rows
@pytest.mark.parametrize("b,h", [(1, 1), (4, 17), (8, 17)])
@pytest.mark.parametrize("d", [64, 96, 128, 192])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("p_drop", [0.0, 0.1])
def test_attention_modes(b, h, d, causal, p_drop):
    s, H, T = 136, h * d, b * 136
    dm = B.make_dims(b, s, H, h, 8, 8, 1, 0, B.MLM_BF16, causal=causal)
    g = torch.Generator(device=DEV)
    g.manual_seed(d + b)
    n = lambda *sh, std=1.0: (torch.randn(*sh, generator=g, device=DEV) * std).to(torch.bfloat16)
    u, Wqkv, Wo, dx1 = n(T, H), n(H, 3 * H, std=H ** -0.5), torch.eye(H, device=DEV).to(torch.bfloat16), n(T, H)
    key_len = torch.tensor([(s, 1, 33, 97, 64, 130, 7, 135)[i % 8] for i in range(b)], device=DEV, dtype=torch.int32)
    e = lambda *sh: torch.full(sh, float("nan"), device=DEV, dtype=torch.bfloat16)
    qkv, ctx, part, dqkv, dbqkv, du = e(T, 3 * H), e(T, H), e(T, H), e(T, 3 * H), e(3 * H), e(T, H)
    lse = torch.full((b, h, s), float("nan"), device=DEV)
    ws = torch.empty(max(B.mlm_workspace_bytes(dm, w) for w in (B.WS_ATTN_FWD, B.WS_ATTN_BWD)), device=DEV, dtype=torch.uint8)
    drop, kb, keep = None, None, 1.0
    if p_drop:
        drop, kb = B.make_dropout(p_drop, 77, 5), torch.empty(B.mlm_attn_keep_words(dm), device=DEV, dtype=torch.int32)
        keep = torch.from_numpy(R.keep_mask(77, 5, (b * h, s, s), p_drop)).to(DEV).double() / (1 - p_drop)
        B.mlm_attn_shard_fwd_dropout(dm, u, Wqkv, None, Wo, key_len, drop, qkv, ctx, lse, kb, part, ws)
    else:
        B.mlm_attn_shard_fwd(dm, u, Wqkv, None, Wo, key_len, qkv, ctx, lse, part, ws)
    B.mlm_attn_shard_bwd_input(dm, dx1, Wqkv, Wo, key_len, drop, qkv, ctx, lse, kb, dqkv, dbqkv, du, ws)

    heads = lambda t: t.double().view(b, s, h, d).permute(0, 2, 1, 3).reshape(b * h, s, d).contiguous()
    q, k, v = (heads(qkv[:, i * H:(i + 1) * H].contiguous()) for i in range(3))
    do, o = heads(dx1), heads(ctx)
    mm = lambda x, y: torch.bmm(x.contiguous(), y.contiguous())
    t = lambda x: x.transpose(1, 2)
    i = torch.arange(s, device=DEV)
    ok = (i[None, None, :] < key_len.repeat_interleave(h)[:, None, None]) & ((i[None, None, :] <= i[None, :, None]) | (not causal))
    sc = d ** -0.5
    S = torch.where(ok, mm(q, t(k)) * sc, float("-inf"))
    P = torch.softmax(S, -1)
    Pd = P * keep                        # the probabilities that multiply V
    ref = mm(Pd, v)
    u8 = 2.0 ** -8                      # one rounding to bf16 (half of it) and a margin for the fp32 arithmetic

    def close(name, got, want, bound):
        err = (got - want).abs() - bound * 1.05 - 1e-5
        assert bool((err <= 0).all()), (name, float(err.max()))

    close("lse", lse.double().view(b * h, s), torch.logsumexp(S, -1), 1e-4)
    close("ctx", o, ref, u8 * (ref.abs() + mm(Pd, v.abs())))             # P and ctx are rounded
    delta = (do * o).sum(-1, keepdim=True)                               # from the rounded ctx, as the kernels form it
    dS = P * (mm(do, t(v)) * keep - delta)
    dP_err = 1e-5 * mm(do.abs(), t(v.abs())) * keep
    sl = dS.abs() * u8 + P * dP_err                                      # dS is rounded before the second product
    dq, dk, dv = (heads(dqkv[:, j * H:(j + 1) * H].contiguous()) for j in range(3))
    rq, rk, rv = mm(dS, k) * sc, mm(t(dS), q) * sc, mm(t(Pd), do)
    close("dq", dq, rq, u8 * rq.abs() + sc * mm(sl, k.abs()))
    close("dk", dk, rk, u8 * rk.abs() + sc * mm(t(sl), q.abs()))
    close("dv", dv, rv, u8 * rv.abs() + u8 * mm(t(Pd), do.abs()))
