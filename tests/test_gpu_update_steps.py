"""GPU parity of the tall tiles of the update phase where the loop over contracted indices can end: behind each of the four
steps of 16 that a turn holds, one index before and after, and within the first turn; each width of tile, forward
and backward, both data types."""
import pytest

from test_gpu_update import run_case, test_update_parity_bf16 as bf16_case

pytestmark = pytest.mark.gpu

FEW = [(K, N) for K in (48, 65, 112) for N in (32, 128)] + [(80, 256)]


@pytest.mark.parametrize("K,N", [(K, 64) for K in (16, 31, 32, 33, 48, 49, 63, 64, 65, 97, 128)] + FEW)
def test_last_step_fp32(K, N):
    M = 31000 if N == 256 else 16500
    run_case(M, K, N, relu=K % 2 == 0, bias=True, seed=K + N, what="last step")


@pytest.mark.parametrize("K,N", [(48, 64), (100, 97), (112, 128)])
def test_last_step_of_the_input_gradient_fp32(K, N):
    run_case(31000 if N == 128 else 16500, K, N, relu=True, bias=False, seed=K + N, what="last step of dH")


@pytest.mark.parametrize("K,N", [(48, 32), (65, 64), (112, 256)])
def test_last_step_bf16(K, N):
    bf16_case(31000 if N == 256 else 16500, K, N, True)
