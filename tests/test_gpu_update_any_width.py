"""GPU parity of the weight gradient at widths whose quads end with a row, start early or do not exist (rows of fewer than
four elements go element by element), around the tiles' edges, and of operands at any element's address."""
import numpy as np
import pytest
import torch

from paper_2409_14939_amd import binding as B
from test_gpu_update import run_case, test_update_parity_bf16 as bf16_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N", [(33, 1, 9), (50, 2, 70), (70, 3, 12), (17, 4, 11), (1000, 126, 65), (1001, 127, 66), (999, 129, 67),
                                   (515, 130, 127), (514, 131, 129), (300, 257, 130), (64, 259, 131), (16, 5, 10), (15, 6, 257)])
@pytest.mark.parametrize("relu", [False, True])
def test_widths(M, K, N, relu):
    run_case(M, K, N, relu, bias=True, seed=M + K + N, what="any width")
    bf16_case(M, K, N, relu)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("K,N", [(100, 64), (99, 131)])
@pytest.mark.parametrize("by", [1, 3])
def test_any_alignment(dtype, K, N, by):
    """The same bits wherever the operands start."""
    g = torch.Generator(device="cuda")
    g.manual_seed(K + N)
    M = 777

    def both(rows, cols):
        a = torch.randn(rows, cols, generator=g, device="cuda").to(dtype)
        room = torch.full((rows * cols + 2 * by + 8,), float("nan"), dtype=dtype, device="cuda")
        room[by:by + rows * cols] = a.reshape(-1)
        return a, room[by:by + rows * cols].reshape(rows, cols)

    (H, Hs), (W, Ws), (Y, Ys), (dY, dYs) = both(M, K), both(K, N), both(M, N), both(M, N)
    plain = B.fastgl_update_bwd(H, W, Y, dY, True, want=("dW", "db"))
    shifted = B.fastgl_update_bwd(Hs, Ws, Ys, dYs, True, want=("dW", "db"))
    assert all(torch.equal(a, b) for a, b in zip(plain, shifted) if a is not None)
    assert torch.isfinite(plain[1]).all()
