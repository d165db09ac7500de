"""GPU parity of the update phase around the width of the weight gradient's narrow tile (64 columns): widths whose pairs
are whole, cut and missing, with and without the gate, few and many rows, both data types."""
import pytest

from test_gpu_update import run_case, test_update_parity_bf16 as bf16_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N", [(1, 5, 9), (31, 129, 10), (33, 128, 32), (1000, 100, 63), (1001, 100, 64), (4097, 37, 64),
                                   (4096, 260, 33), (1001, 100, 65)])
@pytest.mark.parametrize("relu", [False, True])
def test_half_tile(M, K, N, relu):
    run_case(M, K, N, relu, bias=True, seed=M + K + N, what="half tile")
    bf16_case(M, K, N, relu)
