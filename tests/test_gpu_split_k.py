"""The tiled GEMM with K shared out between workgroups (more than 128 rows, few tiles, long K): ranges that do not divide
K evenly, every kind of slab in the last range, and each way the sums can leave."""
import numpy as np
import pytest
import torch

from oracle import blockwise_codec as bc
from oracle import boundary_exit as be
from oracle import mixed_linear as ml
from paper_2407_19775_amd import binding, workloads as wl
from gpu_util import assert_y_close, critical_column_plan, gemm_splits, to_gpu, to_np
from test_gpu_linear import check_linear, exactly_n_critical

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,n_crit", [(129, 8208, 264, 5), (130, 11008, 1000, 0), (1000, 8192, 520, 300), (129, 32768, 72, 2400)])
def test_ranges_of_k(M, K, N, n_crit):
    """300 of 8192 columns: further slabs, shared out between the ranges; 2400 of 32768: the walk over K, in ranges."""
    rng = np.random.default_rng([M, K, N])
    X, _ = exactly_n_critical(rng, M, K, n_crit)
    assert gemm_splits(M, K, N) > 1 and (n_crit >= critical_column_plan(M, K, N)[1]) == (n_crit == 2400)
    check_linear(X, wl.gaussian_weight(K, N, 0.05, rng), 6.0, bias=wl.gaussian_bias(N, 0.1, rng))


def test_columns_beyond_the_slabs_in_a_split_call():
    """2350 of 8192 columns: more than the fp16 slabs hold, fewer than the walk over all of K takes: gathered by the
    last range."""
    M, K, N = 6000, 8192, 264
    in_slabs, dense_from = critical_column_plan(M, K, N)
    assert gemm_splits(M, K, N) > 1 and in_slabs == 2304 and 2350 < dense_from
    rng = np.random.default_rng([M, K, N])
    X, _ = exactly_n_critical(rng, M, K, 2350)
    rows = np.concatenate([np.arange(0, 260), np.arange(M - 200, M)])
    check_linear(X, wl.gaussian_weight(K, N, 0.05, rng), 6.0, bias=wl.gaussian_bias(N, 0.1, rng), rows=rows)


@pytest.mark.parametrize("tau", [6.0, 0.75])
def test_ways_out(tau):
    M, K, N = 200, 8208, 512
    rng = np.random.default_rng([M, K])
    x = rng.standard_normal((M, K)).astype(np.float32)
    x[:, ::400] *= 20.0
    X, W, b = wl.to_fp16(x), wl.gaussian_weight(K, N, 0.02, rng), wl.gaussian_bias(N, 0.3, rng)
    R = wl.to_fp16(rng.standard_t(3.0, size=(M, N)).astype(np.float32))
    pw, Xg, bg, Rg = binding.prequantize_weight(to_gpu(W)), to_gpu(X), to_gpu(b), to_gpu(R)
    Y = binding.mixed_int8_linear(Xg, pw, tau, bias=bg)
    H = binding.mixed_int8_linear(Xg, pw, tau, bias=bg, residual=Rg, out=Rg.clone())
    want = be.add_residual(to_np(Y), R)
    assert np.array_equal(to_np(H).view(np.uint16), want.view(np.uint16))
    codes, absmax = binding.mixed_int8_linear_to_codes(Xg, pw, tau, 128, bias=bg, residual=Rg)
    oc, oa = bc.quantize_blockwise(want.reshape(-1), 128)
    assert np.array_equal(to_np(codes).reshape(-1), oc) and np.array_equal(to_np(absmax).reshape(-1), oa)
    # GELU of a zero-weight layer's bias and of the layer itself: one fp16 step from the activation of the plain output
    G = binding.mixed_int8_linear(Xg, pw, tau, bias=bg, gelu=True)
    g = torch.nn.functional.gelu(Y.double()).cpu().numpy()
    assert np.all(np.abs(to_np(G).astype(np.float64) - g) <= 2.0 ** -10 * np.abs(g) + 2.0 ** -24)
    # an adapter: one plus its term, T rounded to fp16 as the definition says
    r = 24
    A, B = wl.gaussian_weight(r, K, 0.02, rng), wl.gaussian_weight(N, r, 0.05, rng)
    L = binding.mixed_int8_linear(Xg, pw, tau, bias=bg, lora=(to_gpu(A), to_gpu(B)))
    T = (X.astype(np.float64) @ A.astype(np.float64).T).astype(np.float16).astype(np.float64)
    assert_y_close(to_np(L), to_np(Y).astype(np.float64) + T @ B.astype(np.float64).T)


def test_workspace_of_an_unsplit_call_still_serves():
    """A workspace that was sized for more rows than the split is for: the call goes through without the split."""
    M, K, N = 129, 8192, 1024
    rng = np.random.default_rng(3)
    X, W = wl.to_fp16(rng.standard_normal((M, K)).astype(np.float32)), wl.gaussian_weight(K, N, 0.02, rng)
    pw, Xg = binding.prequantize_weight(to_gpu(W)), to_gpu(X)
    full = binding.linear_workspace(M, K, N, Xg.device)
    Y = binding.mixed_int8_linear(Xg, pw, wl.TAU, workspace=full)
    out = binding.mixed_int8_linear(Xg, pw, wl.TAU, workspace=full[:-256])      # 256 bytes short of the split's sums
    Wq, c = ml.prequantize_weight(W)
    ref = ml.mixed_int8_linear(X, Wq, c, wl.TAU, None)["Y"]
    assert_y_close(to_np(Y), ref)
    assert_y_close(to_np(out), ref)


def test_workspace_of_more_rows_gives_the_same_bits():
    """1025 rows are not split and need less for themselves than 129 to 256 rows with the sums of their ranges."""
    K, N = 11008, 4096
    rng = np.random.default_rng(4)
    X, _ = exactly_n_critical(rng, 256, K, 40)
    pw, Xg = binding.prequantize_weight(to_gpu(wl.gaussian_weight(K, N, 0.02, rng))), to_gpu(X)
    ws = binding.linear_workspace(1025, K, N, Xg.device)
    for M in (129, 200, 256):
        assert torch.equal(binding.mixed_int8_linear(Xg[:M], pw, wl.TAU, workspace=ws), binding.mixed_int8_linear(Xg[:M], pw, wl.TAU))
