"""129 to 512 rows with large weights, requested as bytes that nothing else reads: at the line of the rule, on both tile widths, with
and without a split K, few and very many critical columns, and behind the layer: what the plain requests give, bit for bit,
and the oracle's integers and outputs on some of the columns."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import mixed_linear as ml
from paper_2407_19775_amd import binding, workloads as wl
from gpu_util import assert_y_close, gemm_splits, to_gpu, to_np


def read_once(M, K, N):
    f = binding.lib()._ZN4mmd817weights_read_onceEiii
    f.argtypes, f.restype = [ctypes.c_int] * 3, ctypes.c_bool
    return f(M, (K + 127) // 128 * 128, N)


@pytest.mark.parametrize("M,K,N,once", [(256, 3072, 9216, True), (129, 4096, 12288, True), (512, 2048, 11008, True), (128, 4096, 12288, False),
                                        (513, 4096, 12288, False), (333, 1536, 4608, False), (512, 4096, 4096, False)])
def test_rule_follows_the_measured_sides(M, K, N, once):
    assert read_once(M, K, N) == once


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,tile", [(129, 2496, 8192, 0), (300, 1296, 16392, 5), (512, 2560, 8192, 0), (200, 8192, 2560, None), (384, 11024, 2056, None)])
@pytest.mark.parametrize("heavy", [False, True])
def test_same_layer_as_with_plain_requests(M, K, N, tile, heavy):
    assert read_once(M, K, N) and (gemm_splits(M, K, N) > 1) == (tile is None)
    rng = np.random.default_rng([M, K, N])
    x = (rng.standard_t(3.0, size=(M, K)) if heavy else rng.standard_normal((M, K))).astype(np.float32)
    x[:, rng.integers(0, K, 4)] *= 20.0
    X, bias = wl.to_fp16(x), wl.gaussian_bias(N, 0.3, rng)
    W = torch.randn((K, N), generator=torch.Generator(device="cuda").manual_seed(M), device="cuda", dtype=torch.float16) * 0.02
    pw, Xg, bg = binding.prequantize_weight(W), to_gpu(X), to_gpu(bias)
    Y = binding.mixed_int8_linear(Xg, pw, wl.TAU, bias=bg)
    Y_tap, t = binding.mixed_int8_linear(Xg, pw, wl.TAU, bias=bg, taps=("acc",))      # plain requests
    assert torch.equal(Y, Y_tap)
    cols = torch.unique(torch.cat([torch.linspace(0, N - 1, 60).long(), torch.tensor([127, 128, 255, 256, N - 8])]))
    o = ml.mixed_int8_linear(X, *ml.prequantize_weight(to_np(W[:, cols.cuda()].contiguous())), wl.TAU, bias[to_np(cols)])
    assert np.array_equal(to_np(t["acc"][:, cols.cuda()]), o["acc"])
    assert_y_close(to_np(Y[:, cols.cuda()]), o["Y"])
    R = to_gpu(wl.to_fp16(rng.standard_t(3.0, size=(M, N)).astype(np.float32)))
    H = torch.empty((M, N), dtype=torch.float16, device="cuda")
    codes, absmax = binding.mixed_int8_linear_to_codes(Xg, pw, wl.TAU, 64, bias=bg, residual=R, H=H)
    want = binding.quantize_blockwise(H, 64)
    assert torch.equal(H, binding.mixed_int8_linear(Xg, pw, wl.TAU, bias=bg, residual=R)) and torch.equal(codes, want[0]) and torch.equal(absmax, want[1])
    if tile is not None:
        tune = binding.tune_gemm_tiles(tile)
        assert torch.equal(Y, binding.mixed_int8_linear(Xg, pw, wl.TAU, bias=bg, tuning=tune))
        assert torch.equal(H, binding.mixed_int8_linear(Xg, pw, wl.TAU, bias=bg, residual=R, tuning=tune))
