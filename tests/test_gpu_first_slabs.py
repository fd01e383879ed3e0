"""The slabs that a tiled GEMM's workgroup requests before it knows the count of critical columns: K of two slabs (fewer than the
rings hold), every tile configuration, a last range of K of a single slab; with few critical columns and with so many that
the walk with both products takes over the slabs on their way."""
import numpy as np
import pytest

from oracle import mixed_linear as ml
from paper_2407_19775_amd import binding, workloads as wl
from gpu_util import assert_y_close, critical_column_plan, gemm_splits, to_gpu, to_np
from test_gpu_linear import check_linear, check_weight

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [16, 128, 144, 320])
@pytest.mark.parametrize("variant", [0, 1, 2, 3, 4, 5])
@pytest.mark.parametrize("tau", [6.0, 0.5])
def test_few_slabs(K, variant, tau):
    M, N = 260, 264
    rng = np.random.default_rng([K, variant])
    X = wl.to_fp16(rng.standard_t(3.0, size=(M, K)).astype(np.float32))
    pw, Wq, c = check_weight(wl.gaussian_weight(K, N, 0.05, rng))
    Y, taps = binding.mixed_int8_linear(to_gpu(X), pw, tau, taps=True, tuning=binding.tune_gemm_tiles(variant))
    o = ml.mixed_int8_linear(X, Wq, c, tau, None)
    assert np.array_equal(to_np(taps["acc"]), o["acc"])
    assert_y_close(to_np(Y), o["Y"])


@pytest.mark.parametrize("walk", [False, True])
def test_last_range_of_one_slab(walk):
    M, K, N = 129, 2944, 264
    assert gemm_splits(M, K, N) == 10                                # 46 slabs: nine ranges of five
    rng = np.random.default_rng([M, walk])
    X = wl.to_fp16(rng.standard_t(3.0, size=(M, K)).astype(np.float32) if walk else rng.standard_normal((M, K)).astype(np.float32))
    assert (int(ml.outlier_mask(X, 6.0).sum()) >= critical_column_plan(M, K, N)[1]) == walk
    check_linear(X, wl.gaussian_weight(K, N, 0.05, rng), 6.0, bias=wl.gaussian_bias(N, 0.1, rng))
