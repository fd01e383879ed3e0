"""More than 128 rows prepared with a row per workgroup: each row length's kernel (4, 8 and 16 waves, one and two passes, a last
piece that is not whole), counts of rows around the 256 that the compute units' order repeats with, rows apart by more than
their length, the last size before four rows share a workgroup and the first one after, at each end of the rule; integers against the oracle."""
import numpy as np
import pytest
import torch

from oracle import mixed_linear as ml
from paper_2407_19775_amd import binding, workloads as wl
from gpu_util import assert_y_close, to_np
from test_gpu_linear import check_weight

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K", [(129, 1024), (129, 1040), (255, 2064), (257, 4096), (512, 4112), (512, 8208), (513, 8208), (130, 8192), (200, 16368), (131, 16400),
                                 (129, 32752), (1586, 4096), (1587, 4096), (1024, 1040), (1025, 1040), (2800, 2064), (2801, 2064)])
def test_row_per_workgroup(M, K):
    N = 24
    rng = np.random.default_rng([M, K])
    x = rng.standard_normal((M, K)).astype(np.float32)
    x[:, rng.integers(0, K, 5)] *= 20.0
    x[M - 1, K - 1], x[3] = 100.0, 0.0                               # a critical entry at the very end; a row of zeros
    x = wl.to_fp16(x)
    padded = torch.full((M, K + 24), float("nan"), dtype=torch.float16, device="cuda")
    X = padded[:, :K]
    X.copy_(torch.from_numpy(x))
    pw, Wq, c = check_weight(wl.gaussian_weight(K, N, 0.05, rng))
    Y, taps = binding.mixed_int8_linear(X, pw, 6.0, taps=True)
    o = ml.mixed_int8_linear(x, Wq, c, 6.0, None)
    assert np.array_equal(to_np(taps["outlier_mask"]).astype(bool), o["flag"])
    assert np.array_equal(to_np(taps["xq"]), o["Xq"])
    assert np.array_equal(to_np(taps["acc"]), o["acc"])
    assert_y_close(to_np(Y), o["Y"])
