"""bf16 attention forward under a causal mask with half a block of rows from either end per workgroup, against float64."""
import subprocess

import pytest
import torch

from oracle import rng_embed_oracle as R
from paper_1909_08053_amd import binding as B
from paper_1909_08053_amd import build as BLD

DEV = "cuda:0"
# sequence, batch, heads: an odd number of 32- and of 64-row halves (the middle one once), a last half of 8 rows, whole blocks
SHAPES = {"split": [(520, 1, 3), (512, 3, 2), (544, 2, 1)], "pair": [(576, 16, 3), (520, 16, 3), (1024, 4, 8)]}


def test_shapes_are_folded(tmp_path):
    """(no GPU needed) ... and launches whose workgroups queue on an XCD, or of few tiles, are not."""
    (tmp_path / "f.cpp").write_text("""#include <stdio.h>
#include "attention_modes.h"
int mlm::gemm_cu_count() { return 256; }
int main() { int s, n; while (scanf("%d %d", &s, &n) == 2) { auto m = mlm::attn_mode(s, n, true, 96); printf("%d%d\\n", (int)m, (int)mlm::attn_fwd_fold(m, s, n)); } return 0; }
""")
    subprocess.run(["g++", "-std=c++17", "-I" + BLD.CSRC, str(tmp_path / "f.cpp"), "-o", str(tmp_path / "f")], check=True, timeout=60)
    run = lambda shapes: subprocess.run([str(tmp_path / "f")], input="\n".join("%d %d" % x for x in shapes), text=True, check=True,
                                        capture_output=True, timeout=60).stdout.split()
    for mode, shapes in SHAPES.items():
        assert run([(s, b * h) for s, b, h in shapes]) == [{"pair": "11", "split": "21"}[mode]] * len(shapes), mode
    assert [x[1] for x in run([(4096, 16), (2048, 24), (8192, 8), (3072, 4), (200, 12), (320, 6)])] == ["0"] * 6


@pytest.mark.gpu
@pytest.mark.parametrize("s,b,h", SHAPES["split"] + SHAPES["pair"])
@pytest.mark.parametrize("d", [64, 96, 128])
@pytest.mark.parametrize("p_drop", [0.0, 0.1])
def test_forward(s, b, h, d, p_drop):
    H, T = h * d, b * s
    dm = B.make_dims(b, s, H, h, 8, 8, 1, 0, B.MLM_BF16, causal=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(d + s)
    n = lambda *sh, std=1.0: (torch.randn(*sh, generator=g, device=DEV) * std).to(torch.bfloat16)
    u, Wqkv, Wo = n(T, H), n(H, 3 * H, std=2 * H ** -0.5), torch.eye(H, device=DEV).to(torch.bfloat16)
    key_len = torch.tensor([(s, 1, s - 7, 300, 64)[i % 5] for i in range(b)], device=DEV, dtype=torch.int32)
    e = lambda *sh: torch.full(sh, float("nan"), device=DEV, dtype=torch.bfloat16)
    qkv, ctx, part, lse = e(T, 3 * H), e(T + 1, H), e(T, H), torch.full((b * h * s + 1,), float("nan"), device=DEV)
    ws = torch.empty(B.mlm_workspace_bytes(dm, B.WS_ATTN_FWD), device=DEV, dtype=torch.uint8)
    keep = 1.0
    if p_drop:
        kb = torch.empty(B.mlm_attn_keep_words(dm), device=DEV, dtype=torch.int32)
        keep = torch.from_numpy(R.keep_mask(77, 5, (b * h, s, s), p_drop)).to(DEV).double() / (1 - p_drop)
        B.mlm_attn_shard_fwd_dropout(dm, u, Wqkv, None, Wo, key_len, B.make_dropout(p_drop, 77, 5), qkv, ctx[:T], lse[:-1], kb, part, ws)
    else:
        B.mlm_attn_shard_fwd(dm, u, Wqkv, None, Wo, key_len, qkv, ctx[:T], lse[:-1], part, ws)
    heads = lambda t: t.double().view(b, s, h, d).permute(0, 2, 1, 3).reshape(b * h, s, d).contiguous()
    q, k, v = (heads(qkv[:, i * H:(i + 1) * H].contiguous()) for i in range(3))
    i = torch.arange(s, device=DEV)
    allowed = (i[None, :] <= i[:, None])[None] & (i[None, None, :] < key_len.repeat_interleave(h)[:, None, None])
    S = torch.where(allowed, (q @ k.transpose(1, 2).contiguous()) * d ** -0.5, -torch.inf)
    P = torch.softmax(S, -1)
    ref, mag = (P * keep) @ v, (P * keep) @ v.abs()
    # probabilities rounded to bf16 before the second product (2^-9 of a term), the result once more; scores of d fp32 terms
    assert bool(((heads(ctx[:T]) - ref).abs() <= 2.0 ** -8 * ref.abs() + 2.0 ** -8 * mag + 1e-5).all())
    assert bool(((lse[:-1].view(b * h, s).double() - torch.logsumexp(S, -1)).abs() <= 1e-4).all())
    assert bool(ctx[T].isnan().all()) and bool(lse[-1].isnan()), "write past the end"
