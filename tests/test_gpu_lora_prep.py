"""More than 128 rows with an adapter: its down-projection in the launch that prepares the rows, K in ranges that the next launch
adds.  Each row length's kernel (4, 8 and 16 waves, rows of one to eight passes) with each count of rank tiles, one range and
several, a last range that is shorter, a last tile of rows that is not full; against the oracle as in test_gpu_lora."""
import pytest

from test_gpu_lora import check_lora, rand_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,r", [(129, 1008, 72, 64), (129, 1040, 72, 8), (130, 2064, 264, 24), (145, 4048, 136, 40), (200, 4112, 136, 64),
                                     (129, 8208, 72, 16), (137, 16368, 40, 56), (129, 20496, 24, 32), (129, 32752, 8, 48)])
def test_ranges_next_to_the_preparation(M, K, N, r):
    X, W, A, B = rand_case(M + K, M, K, N, r, outlier_cols=(3, K - 1))
    check_lora(X, W, A, B, 6.0)
