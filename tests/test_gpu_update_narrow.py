"""GPU parity of the update phase with few result columns (its own kernels up to 8 columns), at the edges of
their lane groups: K around the lanes of a group and beyond one column block of dW, rows around the rows in
flight and beyond one slab, quads and single elements, both data types."""
import pytest

from test_gpu_update import run_case, test_update_parity_bf16 as bf16_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N", [(1, 1, 1), (3, 4, 2), (4, 3, 3), (5, 64, 1), (63, 255, 5), (65, 256, 8), (66, 260, 7),
                                   (129, 1030, 4), (70001, 20, 1), (70001, 7, 6), (1025, 100, 9),
                                   (20001, 64, 1), (20000, 65, 3), (20001, 3, 8), (20001, 130, 6)])
def test_narrow_update_parity(M, K, N):
    run_case(M, K, N, relu=M % 2 == 0, bias=M % 4 != 1, seed=M + K + N, what="narrow update")


@pytest.mark.parametrize("M,K,N", [(1500, 64, 1), (300, 18, 7), (257, 260, 8)])
def test_narrow_update_parity_bf16(M, K, N):
    bf16_case(M, K, N, M % 2 == 0)
