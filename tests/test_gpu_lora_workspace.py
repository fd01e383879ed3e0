"""An adapter in a workspace that has no room for the sums of its split down-projection, nor (a size down) for those of the
layer: served with one range of K each, T and Y as the oracle has them."""
import numpy as np
import pytest
import torch

from oracle import lora, mixed_linear as ml
from paper_2407_19775_amd import binding
from gpu_util import assert_y_close, gemm_splits, lora_ranges_in, to_gpu, to_np
from test_gpu_lora import rand_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,r", [(130, 2064, 264, 16), (300, 4112, 136, 64), (145, 8208, 72, 24)])
def test_one_range_of_the_down_projection(M, K, N, r):
    X, W, A, B = rand_case(M + K, M, K, N, r, outlier_cols=(3, K - 1))
    pw, Xg, Ag, Bg = binding.prequantize_weight(to_gpu(W)), to_gpu(X), to_gpu(A), to_gpu(B)
    o = lora.mixed_int8_linear_lora(X, *ml.prequantize_weight(W), 6.0, A, B)
    full = binding.linear_workspace(M, K, N, Xg.device, r)
    assert lora_ranges_in(full.numel(), M, K, N, r) > 1 and gemm_splits(M, K, N) > 1
    sizes = [n for n in range(full.numel(), 0, -256) if lora_ranges_in(n, M, K, N, r)]
    for n in (next(n for n in sizes if lora_ranges_in(n, M, K, N, r) == 1), sizes[-1]):
        assert n < full.numel() and lora_ranges_in(n, M, K, N, r) == 1
        T = torch.full((M, r), float("nan"), dtype=torch.float16, device="cuda")
        Y = binding.mixed_int8_linear(Xg, pw, 6.0, lora=(Ag, Bg, T), workspace=full[:n])
        Tg, To = to_np(T).astype(np.float64), o["T"].astype(np.float64)
        # as in test_gpu_lora: fp32 sums of K products, one rounding
        slack = 2.0 ** -10 * np.abs(To) + K * 2.0 ** -24 * (np.abs(X.astype(np.float64)) @ np.abs(A.astype(np.float64)).T) + 2.0 ** -24
        assert np.all(np.abs(Tg - To) <= slack)
        assert_y_close(to_np(Y), o["Y"])
    with pytest.raises(binding.Mmd8Error):
        binding.mixed_int8_linear(Xg, pw, 6.0, lora=(Ag, Bg), workspace=full[:sizes[-1] - 256])
