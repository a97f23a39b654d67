"""fp32 attention backward beyond a block a compute unit, where dQ and dK/dV are kernels of their own: dropout, key lengths, head sizes up
to 128 against float64, and values that are not finite."""
import pytest
import torch

import test_gpu_fp32_nonfinite as N
from oracle import rng_embed_oracle as R
from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BATCH, HEADS, SEQ = 2, 13, 168                        # 26 pairs of 6 blocks (the last of 8 rows), for either kind
assert 2 * BATCH * HEADS * ((SEQ + 31) // 32) > 256


@pytest.mark.parametrize("d", [16, 64, 80, 128])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("p_drop", [0.0, 0.1])
def test_backward(d, causal, p_drop):
    b, h, s = BATCH, HEADS, SEQ
    H = h * d
    dm = B.make_dims(b, s, H, h, 8, 8, 1, 0, B.MLM_F32, causal=causal)
    g = torch.Generator(device=DEV)
    g.manual_seed(d)
    n = lambda *sh, std=1.0: torch.randn(*sh, generator=g, device=DEV) * std
    u, Wqkv, dx1 = n(b * s, H), n(H, 3 * H, std=H ** -0.5), n(b * s, H)
    key_len = torch.tensor([s, 77], device=DEV, dtype=torch.int32)
    drop = B.make_dropout(p_drop, 5, 1) if p_drop else None
    ctx, dq, dk, dv = N._run(dm, b, s, h, d, u, Wqkv, dx1, key_len, drop)
    heads = lambda x: x.double().reshape(b, s, h, d).permute(0, 2, 1, 3).reshape(b * h, s, d).contiguous()
    q, k, v = (heads(x) for x in (u.double() @ Wqkv.double()).view(b, s, 3, H).unbind(2))
    do = heads(dx1.view(b, s, H))
    mm = lambda x, y: torch.bmm(x.contiguous(), y.contiguous())
    t = lambda x: x.transpose(1, 2)
    i = torch.arange(s, device=DEV)
    ok = (i[None, None, :] < key_len.repeat_interleave(h)[:, None, None]) & ((i[None, None, :] <= i[None, :, None]) | (not causal))
    keep = torch.from_numpy(R.keep_mask(5, 1, (b * h, s, s), p_drop)).to(DEV).double() / (1 - p_drop) if p_drop else 1.0
    P = torch.softmax(torch.where(ok, mm(q, t(k)) * d ** -0.5, float("-inf")), -1)
    o = mm(P * keep, v)
    dS = P * (mm(do, t(v)) * keep - (do * o).sum(-1, keepdim=True)) * d ** -0.5
    for name, got, want in (("ctx", ctx, o), ("dq", dq, mm(dS, k)), ("dk", dk, mm(t(dS), q)), ("dv", dv, mm(t(P * keep), do))):
        # fp32 sums of up to H and s terms of order one, one after the other: a few hundred roundings of 2^-24
        assert float((heads(got) - want).abs().max()) <= 2e-5 * max(1.0, float(want.abs().max())), name


@pytest.mark.parametrize("d", [32, 128])
@pytest.mark.parametrize("p_drop", [0.0, 0.1])
def test_nonfinite_token_stays_out_of_excluded_pairs(d, p_drop):
    b, h, s, bad, klen = BATCH, HEADS, SEQ, 90, 77
    dm = B.make_dims(b, s, h * d, h, 8, 8, 1, 0, B.MLM_F32, causal=False)
    g = torch.Generator(device=DEV)
    g.manual_seed(d)
    n = lambda *sh, std=1.0: torch.randn(*sh, generator=g, device=DEV) * std
    u, Wqkv, dx1 = n(b * s, h * d), n(h * d, 3 * h * d, std=(h * d) ** -0.5), n(b * s, h * d)
    key_len = torch.full((b,), klen, device=DEV, dtype=torch.int32)
    drop = B.make_dropout(p_drop, 5, 1) if p_drop else None
    clean = N._run(dm, b, s, h, d, u, Wqkv, dx1, key_len, drop)
    dirty_u = u.clone().view(b, s, -1)
    dirty_u[0, bad] = float("inf")                   # a padded token: as a query it reaches every key, as a key nothing
    dirty = N._run(dm, b, s, h, d, dirty_u.view_as(u), Wqkv, dx1, key_len, drop)
    rows = torch.arange(s, device=DEV)
    for name, x, y, reached in (("ctx", clean[0], dirty[0], rows == bad), ("dq", clean[1], dirty[1], rows == bad),
                                ("dk", clean[2], dirty[2], rows < klen), ("dv", clean[3], dirty[3], rows < klen)):
        assert torch.equal(x[1], y[1]), name         # the other sequence
        assert not bool(y[0][reached].isfinite().all()), name
        assert bool((x[0][~reached] - y[0][~reached]).abs().le(1e-5 * x[0].abs().max()).all()), name   # the same products in another order
    for y in dirty[2:]:
        assert bool((y[:, klen:] == 0).all())        # a padded key's gradient is exactly zero


def test_nonfinite_output_gradient_stays_out_of_excluded_pairs():
    """An output gradient that is not finite at one query: the keys behind it (causal) keep their gradients."""
    b, h, s, d, bad = BATCH, HEADS, SEQ, 64, 40
    dm = B.make_dims(b, s, h * d, h, 8, 8, 1, 0, B.MLM_F32, causal=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(d)
    n = lambda *sh, std=1.0: torch.randn(*sh, generator=g, device=DEV) * std
    u, Wqkv, dx1 = n(b * s, h * d), n(h * d, 3 * h * d, std=(h * d) ** -0.5), n(b * s, h * d)
    clean = N._run(dm, b, s, h, d, u, Wqkv, dx1, None, None)
    dx1[bad] = float("nan")
    dirty = N._run(dm, b, s, h, d, u, Wqkv, dx1, None, None)
    for name, x, y in (("dk", clean[2], dirty[2]), ("dv", clean[3], dirty[3])):
        assert bool((x[0, bad + 1:] - y[0, bad + 1:]).abs().le(1e-5 * x[0].abs().max()).all()), name
        assert bool(y[0, :bad + 1].isnan().all()), name
    keep = torch.arange(s, device=DEV) != bad
    assert torch.equal(clean[1][0][keep], dirty[1][0][keep]) and bool(dirty[1][0, bad].isnan().all())
