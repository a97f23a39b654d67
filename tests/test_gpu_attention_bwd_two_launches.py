"""bf16 attention backward of long causal sequences, whose dQ and dK/dV are kernels of their own, against float64 on the same inputs."""
import pytest
import torch

from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# batch, heads, sequence: nine pairs of 26 and of 34 blocks with a ragged last one; dQ in paired wave groups, and in single ones
SHAPES = [(3, 3, 3208), (3, 3, 4232)]


@pytest.mark.parametrize("b,h,s", SHAPES)
@pytest.mark.parametrize("d", [64, 96, 128])
@pytest.mark.parametrize("p_drop", [0.0, 0.1])
def test_long_causal_sequences(b, h, s, d, p_drop):
    H, T = h * d, b * s
    dm = B.make_dims(b, s, H, h, 8, 8, 1, 0, B.MLM_BF16, causal=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(d + s)
    n = lambda *sh, std=1.0: (torch.randn(*sh, generator=g, device=DEV) * std).to(torch.bfloat16)
    u, Wqkv, Wo, dx1 = n(T, H), n(H, 3 * H, std=H ** -0.5), torch.eye(H, device=DEV).to(torch.bfloat16), n(T, H)
    key_len = torch.tensor([s, 1041, s - 70], device=DEV, dtype=torch.int32)
    e = lambda *sh: torch.full(sh, float("nan"), device=DEV, dtype=torch.bfloat16)
    qkv, ctx, part, dqkv, dbqkv, du = e(T, 3 * H), e(T, H), e(T, H), e(T, 3 * H), e(3 * H), e(T, H)
    lse = torch.full((b, h, s), float("nan"), device=DEV)
    ws = torch.empty(max(B.mlm_workspace_bytes(dm, w) for w in (B.WS_ATTN_FWD, B.WS_ATTN_BWD)), device=DEV, dtype=torch.uint8)
    drop, kb = None, None
    if p_drop:
        drop, kb = B.make_dropout(p_drop, 77, 5), torch.empty(B.mlm_attn_keep_words(dm), device=DEV, dtype=torch.int32)
        B.mlm_attn_shard_fwd_dropout(dm, u, Wqkv, None, Wo, key_len, drop, qkv, ctx, lse, kb, part, ws)
    else:
        B.mlm_attn_shard_fwd(dm, u, Wqkv, None, Wo, key_len, qkv, ctx, lse, part, ws)
    B.mlm_attn_shard_bwd_input(dm, dx1, Wqkv, Wo, key_len, drop, qkv, ctx, lse, kb, dqkv, dbqkv, du, ws)

    i, sc, u8 = torch.arange(s, device=DEV), d ** -0.5, 2.0 ** -8
    t = lambda x: x.t().contiguous()
    for bi in range(b):
        for hd in range(h):
            col = lambda x, j: x[bi * s:(bi + 1) * s, j * H + hd * d:j * H + (hd + 1) * d].double().contiguous()
            q, k, v, do, o = col(qkv, 0), col(qkv, 1), col(qkv, 2), col(dx1, 0), col(ctx, 0)
            ok = (i[None, :] < key_len[bi]) & (i[None, :] <= i[:, None])
            S = torch.where(ok, q @ t(k) * sc, float("-inf"))
            P = torch.softmax(S, -1)
            keep = 1.0
            if p_drop:                   # the saved decisions, one bit a key (the generator has its own tests)
                words = kb.view(b, h, s, -1)[bi, hd]
                bits = (words[:, :, None] >> torch.arange(32, device=DEV, dtype=torch.int32)) & 1
                keep = bits.view(s, -1)[:, :s].double() / (1 - p_drop)
            Pd = P * keep
            ref = Pd @ v
            dS = P * ((do @ t(v)) * keep - (do * o).sum(-1, keepdim=True))
            sl = dS.abs() * u8 + P * (1e-5 * (do.abs() @ t(v.abs())) * keep)        # dS is rounded before the second product
            for name, got, want, bound in (
                    ("ctx", o, ref, u8 * (ref.abs() + Pd @ v.abs())),
                    ("dq", col(dqkv, 0), dS @ k * sc, u8 * (dS @ k * sc).abs() + sc * (sl @ k.abs())),
                    ("dk", col(dqkv, 1), t(dS) @ q * sc, u8 * (t(dS) @ q * sc).abs() + sc * (t(sl) @ q.abs())),
                    ("dv", col(dqkv, 2), t(Pd) @ do, u8 * (t(Pd) @ do).abs() + u8 * (t(Pd) @ do.abs()))):
                # (bounds of the other attention tests: one rounding to bf16 of each stored value, a margin for fp32 arithmetic)
                err = (got - want).abs() - bound * 1.05 - 1e-5
                assert bool((err <= 0).all()), (name, bi, hd, float(err.max()))
