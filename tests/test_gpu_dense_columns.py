"""The tiled GEMM's walk over K for inputs with very many critical columns: ragged ends of K, rows and columns, rows
with unreadable numbers behind their end, and K beyond the masks that fit in LDS at a time."""
import numpy as np
import pytest
import torch

from oracle import mixed_linear as ml
from paper_2407_19775_amd import binding, workloads as wl
from gpu_util import assert_y_close, critical_column_plan, to_np
from test_gpu_linear import check_weight

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [None, 0, 1, 4])
@pytest.mark.parametrize("M,K,N", [(129, 1040, 72), (257, 2096, 264), (130, 16400, 40), (300, 16448, 520)])
def test_ragged_ends(M, K, N, variant):
    """The numbers between the end of a row and the next row are NaN: the last slab of K must not let them in."""
    rng = np.random.default_rng([M, K, 5])
    x = wl.to_fp16(rng.standard_t(3.0, size=(M, K)).astype(np.float32))
    x[5, 3] = np.float16(65504.0)
    tau = 0.75
    flag = ml.outlier_mask(x, tau)
    assert critical_column_plan(M, K, N)[1] <= int(flag.sum())
    padded = torch.full((M, K + 24), float("nan"), dtype=torch.float16, device="cuda")
    X = padded[:, :K]
    X.copy_(torch.from_numpy(x))
    pw, Wq, c = check_weight(wl.gaussian_weight(K, N, 0.05, rng))
    tuning = 0 if variant is None else binding.tune_gemm_tiles(variant)
    Y, taps = binding.mixed_int8_linear(X, pw, tau, taps=True, tuning=tuning)
    o = ml.mixed_int8_linear(x, Wq, c, tau, None)
    assert np.array_equal(to_np(taps["acc"]), o["acc"])
    assert_y_close(to_np(Y), o["Y"])
