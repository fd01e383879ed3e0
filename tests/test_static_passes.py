"""The entry point without a workspace at 65 to 128 rows whose partial outputs do not fit in its array all at once: served in two
passes, as large as ever."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import mixed_linear as ml
from paper_2407_19775_amd import binding, workloads as wl
from gpu_util import static_decode_plan


@pytest.mark.parametrize("M,K,N", [(128, 8192, 57344), (100, 64, 77824), (128, 28672, 8192)])
def test_sizes_are_accepted(M, K, N):
    """The size check comes before that of the layout tag, which ends the call here: no pointer is used."""
    L = binding.lib()
    fake, y = ctypes.c_void_p(0x1000), ctypes.c_void_p(0x40000000)
    assert L.mmd8_mixed_int8_linear_static(fake, M, K, K, fake, L.mmd8_packed_weight_layout() + 1, fake, N, None, 6.0, y, N, None, None) == -5


@pytest.mark.parametrize("M,K,N", [(128, 36864, 8192), (128, 5120, 20480), (112, 10240, 32768), (128, 2304, 21504)])
def test_passes_of_64_rows_come_before_an_unsplit_k(M, K, N):
    """All rows at once do not fit, half of them do with as many ranges of K as a call of half the rows has: unsplit, 128 x 36864
    -> 8192 would be 32 workgroups."""
    splits, pass_rows = static_decode_plan(M, K, N)
    assert splits > 1 and (splits, 64) == static_decode_plan(64, K, N) and pass_rows == 64


@pytest.mark.parametrize("M,K,N,plan", [(128, 8192, 57344, (1, 64)), (128, 832, 30720, (1, 128)), (128, 4096, 4096, None), (64, 63776, 29960, (1, 64)), (128, 63776, 29960, (1, 64))])
def test_what_else_the_array_holds(M, K, N, plan):
    """Room for everything: one pass.  A short K, or no room for 64 rows with the ranges: K in one, as many rows a pass as fit."""
    splits, pass_rows = static_decode_plan(M, K, N)
    assert (splits, pass_rows) == plan if plan else (splits > 1 and pass_rows == M)


@pytest.mark.gpu
def test_two_passes_with_a_split_k():
    """Split K in both passes: the layer of the entry point with a workspace to another order of fp32 additions (64-row tiles share a
    slab's k-steps out), the same bits again on the next call."""
    from gpu_util import assert_y_close, to_gpu, to_np
    M, K, N = 128, 2304, 21504
    assert static_decode_plan(M, K, N) == (3, 64)
    rng = np.random.default_rng(M)
    X, W = wl.to_fp16(rng.standard_t(3.0, size=(M, K)).astype(np.float32)), wl.gaussian_weight(K, N, 0.02, rng)
    pw, Xg, bias = binding.prequantize_weight(to_gpu(W)), to_gpu(X), wl.gaussian_bias(N, 0.3, rng)
    got = [torch.zeros((M, N), dtype=torch.float16, device="cuda") for _ in range(2)]
    for out in got:
        binding.mixed_int8_linear_static(Xg, pw, wl.TAU, out, bias=to_gpu(bias))
    want = binding.mixed_int8_linear(Xg, pw, wl.TAU, bias=to_gpu(bias))
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[1])
    assert_y_close(to_np(got[0]), to_np(want), rel=2e-3)            # as where other kernels' sums are compared
    cols = np.arange(0, N, 97)
    assert_y_close(to_np(got[0])[:, cols], ml.mixed_int8_linear(X, *ml.prequantize_weight(W[:, cols]), wl.TAU, bias[cols])["Y"])


@pytest.mark.gpu
@pytest.mark.parametrize("M", [65, 100, 128])
def test_two_passes_give_the_same_layer(M):
    """Against one pass over all rows another order of fp32 additions (64-row tiles share a slab's k-steps out), the oracle to the
    usual bar, and the same bits again on the next call: the flags are zero after the second pass."""
    from gpu_util import assert_y_close, to_gpu, to_np
    K, N = 80, 90112                                                # 128 rows of partial outputs: 46 MB
    rng = np.random.default_rng(M)
    X, W = wl.to_fp16(rng.standard_t(3.0, size=(M, K)).astype(np.float32)), wl.gaussian_weight(K, N, 0.02, rng)
    pw, Xg, bias = binding.prequantize_weight(to_gpu(W)), to_gpu(X), wl.gaussian_bias(N, 0.3, rng)
    want = binding.mixed_int8_linear(Xg, pw, wl.TAU, bias=to_gpu(bias))
    got = [torch.zeros((M, N), dtype=torch.float16, device="cuda") for _ in range(2)]
    for out in got:
        binding.mixed_int8_linear_static(Xg, pw, wl.TAU, out, bias=to_gpu(bias))
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[1])
    assert_y_close(to_np(got[0]), to_np(want), rel=2e-3)            # as where other kernels' sums are compared
    assert_y_close(to_np(got[0]), ml.mixed_int8_linear(X, *ml.prequantize_weight(W), wl.TAU, bias)["Y"])
