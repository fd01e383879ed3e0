"""K shared out between workgroups on 128 x 128 tiles (K of at most 6144): ranges that do not divide K evenly, the last one short, ragged
rows and columns, the longest K of the rule and the next, weights requested once and not; few critical columns, more than the
first slabs hold, and so many that the walk with both products takes them; against the oracle, integers exactly."""
import numpy as np
import pytest

from paper_2407_19775_amd import workloads as wl
from gpu_util import critical_column_plan, gemm_splits
from test_gpu_linear import check_linear, exactly_n_critical

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_crit", [0, 270, "walk"])
@pytest.mark.parametrize("M,K,N", [(129, 2944, 264), (200, 4112, 1000), (257, 6144, 520), (130, 6160, 72), (256, 4992, 4104)])
def test_ranges_on_small_tiles(M, K, N, n_crit):
    assert gemm_splits(M, K, N) > 1
    dense_from = critical_column_plan(M, K, N)[1]
    if n_crit == 270:
        n_crit = min(n_crit, dense_from - 1)
    rng = np.random.default_rng([M, K, N])
    X, _ = exactly_n_critical(rng, M, K, dense_from if n_crit == "walk" else n_crit)
    check_linear(X, wl.gaussian_weight(K, N, 0.05, rng), 6.0, bias=wl.gaussian_bias(N, 0.1, rng))
