"""GPU parity of the update phase at sizes where the tall tiles of the row products run (more than 512 tiles of
32 x 64 results): each tile width, ragged last tiles of rows and columns, contracted lengths that are no whole
chunk, rows of odd length (loads aligned to a dword only), both data types; and at the largest sizes of the
small tiles."""
import pytest

from test_gpu_update import run_case, test_update_parity_bf16 as bf16_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N", [(17001, 36, 61), (17001, 3, 64), (17000, 101, 9), (9003, 130, 100), (31001, 33, 129),
                                   (31000, 100, 256), (31001, 17, 255), (8001, 70, 330), (16353, 256, 47)])
def test_tall_update_parity(M, K, N):
    run_case(M, K, N, relu=M % 2 == 1, bias=K % 2 == 0, seed=M + K + N, what="tall update")


@pytest.mark.parametrize("M,K,N", [(17001, 36, 61), (17000, 101, 47), (9003, 130, 101), (31001, 33, 130), (31000, 9, 255)])
def test_tall_update_parity_bf16(M, K, N):
    bf16_case(M, K, N, M % 2 == 1)
