"""The two gradients of the logits in one launch (bf16), against float64 products of the same dL."""
import pytest
import torch

from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# tokens, width, vocabulary of the shard: small tiles (token count and vocabulary that are no multiples of a slice; one tile each),
# large tiles with either gradient's tiles leading, and with a vocabulary that ends on half a pair of slices
SHAPES = [(200, 192, 520), (24, 128, 128), (72, 384, 1000), (2048, 2304, 2048), (1536, 3072, 2048), (5056, 1024, 5024), (3008, 1920, 5024)]


def setup(T, H, V):
    dm = B.make_dims(1, T, H, 1, 8, V, 1, 0, B.MLM_BF16)
    g = torch.Generator(device=DEV)
    g.manual_seed(T + V)
    n = lambda *sh, std: (torch.randn(*sh, generator=g, device=DEV) * std).to(torch.bfloat16)
    hf, E, logits = n(T, H, std=1.0), n(H, V, std=0.02), n(T, V, std=2.0)
    targets = torch.randint(0, V, (T,), generator=g, device=DEV, dtype=torch.int32)
    M = logits.float().max(1).values
    S = torch.exp(logits.float() - M[:, None]).sum(1)
    stats = torch.tensor([1.0, float(T)], device=DEV)
    ws = torch.empty(B.mlm_workspace_bytes(dm, B.WS_VOCAB_CE_BWD), device=DEV, dtype=torch.uint8)
    return dm, hf, E, logits, targets, M, S, stats, ws


def close(name, got, A, W):
    ref, mag = A.double() @ W.double(), A.double().abs() @ W.double().abs()
    # one rounding to bf16, and fp32 sums of K products: 2^-24 of the sum of magnitudes a step, of which errors of either sign
    # leave about the square root
    bound = ref.abs() * 2.0 ** -8 + mag * 2.0 ** -24 * 4 * A.shape[1] ** 0.5
    err = (got.double() - ref).abs() - bound
    assert bool((err <= 1e-12).all()), (name, float(err.max()))


@pytest.mark.parametrize("T,H,V", SHAPES)
def test_logits_gradients_in_one_launch(T, H, V):
    dm, hf, E, logits, targets, M, S, stats, ws = setup(T, H, V)
    dE = torch.full((H + 1, V), float("nan"), device=DEV, dtype=torch.bfloat16)
    dh = torch.full((T + 1, H), float("nan"), device=DEV, dtype=torch.bfloat16)
    B.mlm_vocab_ce_shard_bwd(dm, hf, E, targets, None, M, S, stats, logits, dE[:H], dh[:T], ws)
    close("dE", dE[:H], hf.t(), logits)                  # `logits` now holds dL
    close("dhf", dh[:T], logits, E.t())
    assert bool(dE[H:].isnan().all()) and bool(dh[T:].isnan().all())


@pytest.mark.parametrize("T,H,V", [(200, 192, 520), (2048, 2304, 2048)])
def test_gradient_over_its_input_keeps_the_order(T, H, V):
    dm, hf, E, logits, targets, M, S, stats, ws = setup(T, H, V)
    x, dE = hf.clone(), torch.empty(H, V, device=DEV, dtype=torch.bfloat16)
    B.mlm_vocab_ce_shard_bwd(dm, x, E, targets, None, M, S, stats, logits, dE, x, ws)       # dhf over hf
    close("dE", dE, hf.t(), logits)
    close("dhf", x, logits, E.t())
