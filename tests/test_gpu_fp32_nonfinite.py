"""fp32 attention: a value that is not finite reaches only the rows whose key or query it is, never a pair that the causal
mask or the key length excludes."""
import pytest
import torch

from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _run(dm, b, s, h, d, u, Wqkv, dx1, key_len, drop):
    H, T = h * d, b * s
    e = lambda *sh: torch.full(sh, 7.0, device=DEV)
    qkv, ctx, part, dqkv, dbqkv, du, lse = e(T, 3 * H), e(T, H), e(T, H), e(T, 3 * H), e(3 * H), e(T, H), e(b, h, s)
    ws = torch.empty(max(B.mlm_workspace_bytes(dm, w) for w in (B.WS_ATTN_FWD, B.WS_ATTN_BWD)), device=DEV, dtype=torch.uint8)
    eye = torch.eye(H, device=DEV)
    kb = torch.zeros(B.mlm_attn_keep_words(dm), device=DEV, dtype=torch.int32) if drop else None
    if drop:
        B.mlm_attn_shard_fwd_dropout(dm, u, Wqkv, None, eye, key_len, drop, qkv, ctx, lse, kb, part, ws)
    else:
        B.mlm_attn_shard_fwd(dm, u, Wqkv, None, eye, key_len, qkv, ctx, lse, part, ws)
    B.mlm_attn_shard_bwd_input(dm, dx1, Wqkv, eye, key_len, drop, qkv, ctx, lse, kb, dqkv, dbqkv, du, ws)
    dq, dk, dv = (dqkv[:, i * H:(i + 1) * H].reshape(b, s, H) for i in range(3))
    return ctx.view(b, s, H), dq, dk, dv


# token 70 lies in the third 32-row tile (64 .. 95); s = 136 leaves a last tile of 8 rows, key length 77 cuts the third tile
@pytest.mark.parametrize("d", [16, 48, 64, 128])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("p_drop", [0.0, 0.1])
def test_nonfinite_tokens_stay_out_of_excluded_pairs(d, causal, p_drop):
    b, s, h = 2, 136, 2
    bad = 70 if causal else 90
    klen = s if causal else 77
    dm = B.make_dims(b, s, h * d, h, 8, 8, 1, 0, B.MLM_F32, causal=causal)
    g = torch.Generator(device=DEV)
    g.manual_seed(d)
    n = lambda *sh, std=1.0: torch.randn(*sh, generator=g, device=DEV) * std
    u, Wqkv, dx1 = n(b * s, h * d), n(h * d, 3 * h * d, std=(h * d) ** -0.5), n(b * s, h * d)
    key_len = torch.full((b,), klen, device=DEV, dtype=torch.int32)
    drop = B.make_dropout(p_drop, 5, 1) if p_drop else None
    clean = _run(dm, b, s, h, d, u, Wqkv, dx1, key_len, drop)
    dirty_u = u.clone().view(b, s, -1)
    dirty_u[0, bad] = float("inf")                   # q, k and v of this token: Inf or NaN
    dirty = _run(dm, b, s, h, d, dirty_u.view_as(u), Wqkv, dx1, key_len, drop)
    # forward and dQ of a query: only the keys it may look at.  dK, dV of a key: only the queries that may look at it (causal:
    # the last query, which looks at the token, looks at every key)
    rows = torch.arange(s, device=DEV)
    reached_q = (rows >= bad) if causal else (rows == bad)
    reached_k = (rows >= 0) if causal else (rows < klen)
    for name, x, y, reached in (("ctx", clean[0], dirty[0], reached_q), ("dq", clean[1], dirty[1], reached_q),
                                ("dk", clean[2], dirty[2], reached_k), ("dv", clean[3], dirty[3], reached_k)):
        assert torch.equal(x[1], y[1]), name         # the other sequence
        assert not bool(y[0][reached].isfinite().all()), name
        ok = ~reached
        # the same products in another order
        assert bool((x[0][ok] - y[0][ok]).abs().le(1e-5 * x[0].abs().max()).all()), name
    if not causal:
        for y in (dirty[2], dirty[3]):
            assert bool((y[:, klen:] == 0).all())    # a padded key's gradient is exactly zero


@pytest.mark.parametrize("d", [32, 128])
def test_nonfinite_output_gradient_stays_out_of_excluded_pairs(d):
    """An output gradient that is not finite at one query: the keys behind it (causal) keep their gradients."""
    b, s, h, bad = 1, 100, 2, 40
    dm = B.make_dims(b, s, h * d, h, 8, 8, 1, 0, B.MLM_F32, causal=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(d)
    n = lambda *sh, std=1.0: torch.randn(*sh, generator=g, device=DEV) * std
    u, Wqkv, dx1 = n(b * s, h * d), n(h * d, 3 * h * d, std=(h * d) ** -0.5), n(b * s, h * d)
    clean = _run(dm, b, s, h, d, u, Wqkv, dx1, None, None)
    dx1[bad] = float("nan")
    dirty = _run(dm, b, s, h, d, u, Wqkv, dx1, None, None)
    for name, x, y in (("dk", clean[2], dirty[2]), ("dv", clean[3], dirty[3])):
        assert bool((x[0, bad + 1:] - y[0, bad + 1:]).abs().le(1e-5 * x[0].abs().max()).all()), name
        assert bool(y[0, :bad + 1].isnan().all()), name
    keep = torch.arange(s, device=DEV) != bad
    assert torch.equal(clean[1][0][keep], dirty[1][0][keep]) and bool(dirty[1][0, bad].isnan().all())
