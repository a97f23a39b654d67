"""fp32 attention: every block of every (batch, head) pair is worked on, whichever XCD order the launch takes."""
import pytest
import torch

from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# (batch, heads, sequence): pairs that fill no XCD evenly and leave units idle; 9 pairs of 33 blocks in plain order (whole pairs would
# leave an XCD twice the work); 24 pairs of 33 blocks in one group; 264 pairs of one block; 64 pairs of 48 in groups of three, three and two an XCD
@pytest.mark.parametrize("b,h,s", [(3, 1, 50), (1, 9, 1030), (2, 12, 1030), (24, 11, 20), (8, 8, 1510)])
@pytest.mark.parametrize("causal", [True, False])
def test_blocks(b, h, s, causal):
    d, T = 16, b * s
    H = h * d
    dm = B.make_dims(b, s, H, h, 8, 8, 1, 0, B.MLM_F32, causal=causal)
    g = torch.Generator(device=DEV)
    g.manual_seed(s + h)
    n = lambda *sh, std=1.0: torch.randn(*sh, generator=g, device=DEV) * std
    u, Wqkv, Wo, dx1 = n(T, H), n(H, 3 * H, std=H ** -0.5), torch.eye(H, device=DEV), n(T, H)
    e = lambda *sh: torch.full(sh, float("nan"), device=DEV)
    qkv, ctx, part, dqkv, dbqkv, du, lse = e(T, 3 * H), e(T, H), e(T, H), e(T, 3 * H), e(3 * H), e(T, H), e(b, h, s)
    ws = torch.empty(max(B.mlm_workspace_bytes(dm, w) for w in (B.WS_ATTN_FWD, B.WS_ATTN_BWD)), device=DEV, dtype=torch.uint8)
    B.mlm_attn_shard_fwd(dm, u, Wqkv, None, Wo, None, qkv, ctx, lse, part, ws)
    B.mlm_attn_shard_bwd_input(dm, dx1, Wqkv, Wo, None, None, qkv, ctx, lse, None, dqkv, dbqkv, du, ws)
    heads = lambda t: t.double().view(b, s, h, d).permute(0, 2, 1, 3).reshape(b * h, s, d).contiguous()
    q, k, v = (heads(qkv[:, i * H:(i + 1) * H].contiguous()) for i in range(3))
    do = heads(dx1)
    mm = lambda x, y: torch.bmm(x.contiguous(), y.contiguous())
    t = lambda x: x.transpose(1, 2)
    i = torch.arange(s, device=DEV)
    S = mm(q, t(k)) * d ** -0.5
    if causal:
        S = torch.where(i[None, None, :] <= i[None, :, None], S, float("-inf"))
    P = torch.softmax(S, -1)
    o = mm(P, v)
    dS = P * (mm(do, t(v)) - (do * o).sum(-1, keepdim=True)) * d ** -0.5

    def close(name, got, want):
        # fp32 sums of up to s terms of order one: a few hundred roundings of 2^-24
        assert float((got - want).abs().max()) <= 2e-5 * max(1.0, float(want.abs().max())), name

    close("ctx", heads(ctx), o)
    for name, j, want in (("dq", 0, mm(dS, k)), ("dk", 1, mm(t(dS), q)), ("dv", 2, mm(t(P), do))):
        close(name, heads(dqkv[:, j * H:(j + 1) * H].contiguous()), want)
