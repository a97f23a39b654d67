"""bf16 weight gradients of a layer shard in one launch whose last round is split along k, against float64."""
import pytest
import torch

from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# tokens, width, ways of the split, FFN width over width: K ending on a pair of slices, on half a pair and anywhere; few and many pieces;
# ragged tiles in both directions; the split problem first and (the last two) third of the four
SHAPES = [(4096, 2560, 4, 4), (3360, 2304, 3, 4), (3333, 2560, 4, 4), (2016, 1056, 1, 4), (6000, 1152, 1, 4), (4096, 1920, 2, 4),
          (3333, 2560, 2, 1), (2048, 1536, 1, 2)]


@pytest.mark.parametrize("T,H,p,f", SHAPES)
def test_weight_gradients_with_a_split_last_round(T, H, p, f):
    Hl, F = H // p, f * H // p
    d = B.make_dims(1, T, H, p, f * H, 8 * p, p, 0, B.MLM_BF16)
    g = torch.Generator(device=DEV)
    g.manual_seed(T + H)
    x = {k: torch.randn(T, n, generator=g, device=DEV).bfloat16() for k, n in
         dict(u=H, dqkv=3 * Hl, ctx=Hl, dz1=H, u2=H, dg=F, y=F, dz2=H).items()}
    out = [torch.full((m + 1, n), float("nan"), device=DEV, dtype=torch.bfloat16) for m, n in ((H, 3 * Hl), (Hl, H), (H, F), (F, H))]
    ws = torch.empty(256 * 256 * 256 * 4, device=DEV, dtype=torch.uint8)
    for _ in range(2):                                   # the second time over the partial tiles of the first
        B.mlm_layer_shard_wgrads(d, *(x[k] for k in ("u", "dqkv", "ctx", "dz1", "u2", "dg", "y", "dz2")), *(o[:-1] for o in out), ws)
    for o, (a, b) in zip(out, (("u", "dqkv"), ("ctx", "dz1"), ("u2", "dg"), ("y", "dz2"))):
        a, b = x[a].double(), x[b].double()
        ref, mag = a.t() @ b, a.abs().t() @ b.abs()
        # one rounding to bf16, and fp32 sums of T products: 2^-24 of the sum of magnitudes a step, of which errors of either sign
        # leave about the square root
        assert bool(((o[:-1].double() - ref).abs() <= ref.abs() * 2.0 ** -8 + mag * 2.0 ** -24 * 4 * T ** 0.5).all())
        assert bool(o[-1].isnan().all()), "write past the end"
