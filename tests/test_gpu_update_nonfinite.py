"""Elements that are not finite in the update phase: every result that one enters is not finite, every other result has
the bits it has without them.  One shape for each kernel and tile width: few columns (multiply-adds), small tiles,
tall tiles of 32 to 256 columns with whole and ragged ends, dW tiles of 64 and 128 columns."""
import pytest
import torch

from paper_2409_14939_amd import binding as B

pytestmark = pytest.mark.gpu
INF, NAN = float("inf"), float("nan")
SHAPES = [(1000, 64, 1), (1001, 30, 3), (999, 65, 8), (20001, 20, 1), (20001, 33, 6),         # few columns
          (300, 100, 47), (1000, 256, 256), (17, 7, 9),                                     # small tiles
          (17001, 37, 31), (17001, 100, 64), (31001, 33, 100), (31001, 18, 255)]             # tall tiles


def spoiled(t, at):
    out = t.clone()
    for (r, c), v in zip(at, (INF, -INF, NAN)):
        out[r, c] = v
    return out


def same_but(got, clean, rows, cols, what):
    """got is not finite in the given rows and columns and equals clean everywhere else."""
    hit = torch.zeros(got.shape, dtype=torch.bool, device="cuda")
    if rows is not None:
        hit[rows] = True
    if cols is not None:
        hit[:, cols] = True
    assert not bool(torch.isfinite(got[hit]).any()), what
    assert torch.equal(got[~hit], clean[~hit]), what


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("M,K,N", SHAPES)
def test_a_non_finite_element_spoils_what_it_enters(M, K, N, dtype):
    g = torch.Generator(device="cuda").manual_seed(M + K + N)
    H, W, dY = (torch.randn(s, generator=g, device="cuda").to(dtype) for s in ((M, K), (K, N), (M, N)))
    print(f"non-finite update M={M} K={K} N={N} {dtype}", flush=True)
    Y = B.fastgl_update_fwd(H, W, None, False)
    dH, dW, db = B.fastgl_update_bwd(H, W, None, dY, False)
    # rows: the first, one inside, the last; contracted indices and columns: the last, the first, one inside
    m, k, n = [0, M // 2, M - 1], [K - 1, 0, K // 2], [N - 1, 0, N // 2]

    Hx = spoiled(H, list(zip(m, k)))
    same_but(B.fastgl_update_fwd(Hx, W, None, False), Y, m, None, "Y of H")
    same_but(B.fastgl_update_bwd(Hx, W, None, dY, False)[1], dW, k, None, "dW of H")

    Wx = spoiled(W, list(zip(k, n)))
    same_but(B.fastgl_update_fwd(H, Wx, None, False), Y, None, n, "Y of W")
    same_but(B.fastgl_update_bwd(H, Wx, None, dY, False, want=("dH",))[0], dH, None, k, "dH of W")

    dYx = spoiled(dY, list(zip(m, n)))
    got = B.fastgl_update_bwd(H, W, None, dYx, False)
    same_but(got[0], dH, m, None, "dH of dY")
    same_but(got[1], dW, None, n, "dW of dY")
    same_but(got[2][None], db[None], None, n, "db of dY")

    # behind a closed gate it does not enter
    gate = torch.ones_like(dY)
    for r, c in zip(m, n):
        gate[r, c] = 0
    for a, b in zip(B.fastgl_update_bwd(H, W, gate, dYx, True), B.fastgl_update_bwd(H, W, gate, dY, True)):
        assert torch.equal(a, b)


def test_large_elements_are_nan_from_pieces_and_finite_from_multiply_adds():
    big = 3.4e38                                               # between the largest bf16 and the largest fp32
    H = torch.zeros((40, 16), device="cuda")
    H[3, 5] = big
    for N, nan in ((4, False), (9, True)):
        Y = B.fastgl_update_fwd(H, torch.full((16, N), 0.5, device="cuda"), None, False)
        assert bool(torch.isnan(Y[3]).all()) if nan else torch.equal(Y[3], torch.full((N,), 0.5 * big, device="cuda"))
        assert not Y[torch.arange(40, device="cuda") != 3].any()
