"""K shared out between workgroups on 128 x 128 tiles and, where the ranges of those do not fit one round, on 128 x 256: ranges that do
not divide K evenly, the last one short, ragged rows and columns, weights requested once and not; few critical columns, more
than the first slabs hold, and so many that the walk with both products takes them; against the oracle, integers exactly."""
import numpy as np
import pytest

from paper_2407_19775_amd import workloads as wl
from gpu_util import critical_column_plan, gemm_splits, ranges_on_small_tiles
from test_gpu_linear import check_linear, exactly_n_critical

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,ranges,small", [(129, 2944, 264, 10, True), (200, 4112, 1000, 6, True), (257, 6144, 520, 12, True),
                                                (130, 6160, 72, 20, True), (256, 4992, 4104, 3, True), (1200, 4112, 520, 4, True),
                                                (1000, 8192, 1000, 4, True), (129, 5008, 8200, 3, False)])
@pytest.mark.parametrize("n_crit", [0, 257, 400, "walk"])
def test_ranges_and_their_tiles(M, K, N, ranges, small, n_crit):
    """257 and 400 columns are further slabs where 1000 rows and more put the line to the walk beyond them (one slab and five, shared out
    among the ranges), elsewhere the smallest counts that take the walk."""
    assert gemm_splits(M, K, N) == ranges and ranges_on_small_tiles(M, K, N) == small
    dense_from = critical_column_plan(M, K, N)[1]
    assert dense_from == 257 if M < 1000 else dense_from > 400
    rng = np.random.default_rng([M, K, N])
    X, _ = exactly_n_critical(rng, M, K, max(dense_from, 700) if n_crit == "walk" else n_crit)
    rows = np.concatenate([np.arange(0, 260), np.arange(M - 140, M)]) if M > 400 else None
    check_linear(X, wl.gaussian_weight(K, N, 0.05, rng), 6.0, bias=wl.gaussian_bias(N, 0.1, rng), rows=rows)
