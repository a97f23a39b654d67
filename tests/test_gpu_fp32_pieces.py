"""fp32 products in bf16 pieces at the edges of their tiles, and with values that are not finite, at the ends of the range or far apart."""
import pytest
import torch

from paper_1909_08053_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (M, N, K) by tile: ragged last tiles of either side, a last step of 8 k, whole steps, an odd number of them; nine rows of tiles
SHAPES = {128: [(1160, 4088, 264), (2056, 4096, 1000), (1024, 3072, 1008)], 64: [(1000, 1016, 2056), (520, 1032, 4096), (776, 2040, 3000)]}
LAYOUTS = [(0, 0), (0, 1), (1, 0)]


def _operands(M, N, K, layout, seed, std_w=1.0):
    ta, tb = layout
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    A = torch.randn((K, M) if ta else (M, K), generator=g, device=DEV)
    W = torch.randn((N, K) if tb else (K, N), generator=g, device=DEV) * std_w
    return A, W, (A.t() if ta else A), (W.t() if tb else W)


def _run(M, N, K, layout, A, W):
    C = torch.full((M + 1, N), 7.0, device=DEV)          # one canary row after the output
    B.mlm_gemm(B.MLM_F32, *layout, M, N, K, A, W, C, None)
    assert bool((C[M] == 7.0).all()), "write past the end of C"
    return C[:M].double()


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("shape", SHAPES[128] + SHAPES[64])
def test_products(shape, layout):
    M, N, K = shape
    A, W, a, w = _operands(M, N, K, layout, M + N + K)
    got, ref = _run(M, N, K, layout, A, W), a.double() @ w.double()
    # forward error of any summation order of K fp32 products: (K + 1) u sum |a| |w|, u = 2^-24
    assert bool(((got - ref).abs() <= (K + 1) * 2.0 ** -24 * (a.abs().double() @ w.abs().double())).all())
    # and no further off than ONE chain of K / 4 fp32 additions is on average: its rounding errors u |partial sum| add up like a random
    # walk over partial sums of 2-norm sqrt(k): u sqrt(sum of k) = u K / sqrt(8), against a result of sqrt(K)
    assert float((got - ref).norm() / ref.norm()) <= 2.0 ** -24 * (K / 8.0) ** 0.5


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("shape", [SHAPES[128][0], SHAPES[64][0]])
def test_values_that_are_not_finite_or_round_to_infinity(shape, layout):
    M, N, K = shape
    A, W, a, w = _operands(M, N, K, layout, 3)
    clean = _run(M, N, K, layout, A, W)
    a[5, 3], a[M - 1, K - 1], w[1, N - 1] = float("inf"), float("nan"), float("-inf")
    a[77] *= 2.0 ** -60
    a[77, 11] = torch.finfo(torch.float32).max           # finite, but no bf16 value is nearer than infinity
    got, ref = _run(M, N, K, layout, A, W), a.double() @ w.double()
    ref[77] = torch.where(ref[77].abs() > torch.finfo(torch.float32).max, ref[77].sign() * float("inf"), ref[77])
    nan, inf = ref.isnan(), ref.isinf()
    assert bool((got.isnan() == nan).all()) and bool((got[inf] == ref[inf]).all())
    ok = ~(nan | inf)
    bound = (K + 1) * 2.0 ** -24 * (a.abs().double() @ w.abs().double())
    assert bool(((got - ref).abs()[ok] <= bound[ok]).all())
    far = torch.ones(M, N, dtype=torch.bool, device=DEV)              # tiles that hold none of these rows and columns: unchanged
    for r in (5, 77, M - 1):
        far[r // 128 * 128:r // 128 * 128 + 128] = False
    far[:, (N - 1) // 128 * 128:] = False
    assert torch.equal(got[far], clean[far])


@pytest.mark.parametrize("shape", [SHAPES[128][0], SHAPES[64][0]])
def test_magnitudes_far_apart(shape):
    """Rows of 2^-100 .. 2^60, columns of 2^-20 .. 2^20: an operand's smaller pieces are as exact as its largest."""
    M, N, K = shape
    A, W, a, w = _operands(M, N, K, (0, 0), 9)
    A *= torch.pow(2.0, torch.linspace(-100, 60, M, device=DEV).round())[:, None]
    W *= torch.pow(2.0, torch.linspace(-20, 20, N, device=DEV).round())[None, :]
    got, ref = _run(M, N, K, (0, 0), A, W), a.double() @ w.double()
    assert bool(((got - ref).abs() <= (K + 1) * 2.0 ** -24 * (a.abs().double() @ w.abs().double())).all())
