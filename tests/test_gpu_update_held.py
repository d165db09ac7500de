"""GPU parity of the fp32 product Y whose weights stay in LDS (many rows, 128 or 256 columns): it takes the steps of the other tall
tiles in the same order, so its results are bit for bit those of the same rows in calls of few rows, which the other tests compare
with the oracle; and one product against float64."""
import pytest
import torch

from test_gpu_guard_bands import Guarded
from paper_2409_14939_amd import binding as B

pytestmark = pytest.mark.gpu


def data(M, K, N, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return [torch.empty(s, device="cuda").normal_(generator=g) for s in ((M, K), (K, N), (N,))]


def in_parts(H, W, bias, relu):
    """The same rows in calls of at most 60 000, below the line."""
    return torch.cat([B.fastgl_update_fwd(h, W, bias, relu) for h in H.chunk((H.shape[0] - 1) // 60_000 + 1)])


def held(M, K, N):
    """Does the kernel take it?  The rule of held_fits, in tiles of 32 rows and rounds of 2 048 of them."""
    tiles = -(-M // 32)
    rounds = -(-tiles // 2048)
    if -(-K // 8) * N * 3 * 16 + 16 > 160 * 1024:
        return False
    if N == 128:
        return rounds >= 9 and K > 144
    if rounds == 2:
        return 2 * tiles <= 3 * 2048 or K > 96
    return rounds > 2 and K > 64 and 20 * tiles >= 17 * rounds * 2048


# K: each number of steps of the last turn and its edges, the smallest and the largest that LDS holds and the first beyond; M:
# remainders of a tile of 32 rows, one tile more than one round, a round and a half, two that are full, rounds that are just full enough
CASES = ([(65_537, K, 256, True) for K in (4, 8, 16, 17, 32, 33, 47, 49, 64, 65, 80, 81, 100, 101, 104)] + [(65_537, 105, 256, False)] +
         [(65_568, 100, 256, True), (98_304, 60, 256, True), (98_305, 60, 256, False), (98_305, 97, 256, True)] +
         [(131_072, 100, 256, True), (131_073, 100, 256, False), (196_607, 100, 256, True), (300_001, 65, 256, True), (300_001, 64, 256, False)] +
         [(524_289, K, 128, True) for K in (145, 160, 161, 176, 177, 192, 193)] + [(524_288, 200, 128, False), (524_320, 144, 128, False)] +
         [(524_320, 208, 128, True), (524_320, 209, 128, False), (530_001, 150, 128, True)])


@pytest.mark.parametrize("M,K,N,takes", CASES)
def test_same_bits(M, K, N, takes):
    assert held(M, K, N) == takes
    print(f"case held M={M} K={K} N={N}", flush=True)
    H, W, bias = data(M, K, N, M + K)
    relu = K % 2 == 0
    bias = None if K % 3 == 0 else bias
    assert torch.equal(B.fastgl_update_fwd(H, W, bias, relu), in_parts(H, W, bias, relu))


def test_against_float64():
    H, W, bias = data(70_003, 100, 256, 5)
    ref = H.double() @ W.double() + bias.double()
    size = H.abs().double() @ W.abs().double() + bias.abs().double()
    err = (B.fastgl_update_fwd(H, W, bias, False).double() - ref).abs()
    # a chain of 101 fp32 additions and the rounding of the result; the planes that are dropped stay below 2^-23 of the products
    assert bool((err <= (101 + 2) * 2.0 ** -24 * size).all())


def test_elements_that_are_not_finite():
    """Rows and columns that hold them, and nothing else, are what the other kernel makes of them."""
    H, W, bias = data(65_600, 100, 256, 6)
    H[3, 99], H[40_000, 0], H[65_599, 50] = float("inf"), float("nan"), -float("inf")
    W[99, 255], W[0, 7] = float("nan"), float("inf")
    got, ref = B.fastgl_update_fwd(H, W, bias, False), in_parts(H, W, bias, False)
    assert torch.equal(got.isfinite(), ref.isfinite()) and torch.equal(got.nan_to_num(), ref.nan_to_num())
    assert bool(got[5, :7].isfinite().all()) and not bool(got[:, 7].isfinite().any())


@pytest.mark.parametrize("M,K,N", [(65_537, 101, 256), (524_319, 153, 128)])
def test_between_guard_bands(M, K, N):
    """The result's neighbours stay as they are; what lies around the operands is NaN and reaches no result."""
    assert held(M, K, N)
    around = []
    for t in data(M, K, N, 7)[:2]:
        around.append(Guarded(*t.shape, torch.float32))
        around[-1].t.copy_(t)
    Y = Guarded(M, N, torch.float32)
    B.fastgl_update_fwd(around[0].t, around[1].t, None, False, Y=Y.t)
    Y.check("held")
    assert torch.equal(Y.t, in_parts(around[0].t.clone(), around[1].t.clone(), None, False))
