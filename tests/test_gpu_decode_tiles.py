"""Nine to 128 rows: integers equal to the oracle's and outputs to the fp16 bar where the tiles and the ring can go wrong: the
smallest and largest number of rows of each tile height, a K that ends inside a slab or leaves a slab of padding only, ranges
shorter than the ring, one that outlives the masks held at a time (a workspace without room for the split), ragged columns."""
import numpy as np
import pytest
import torch

from oracle import mixed_linear as ml
from paper_2407_19775_amd import binding, workloads as wl
from gpu_util import assert_y_close, to_gpu, to_np

pytestmark = pytest.mark.gpu


def inputs(M, K, N):
    rng = np.random.default_rng([M, K, N])
    X = rng.standard_t(3.0, size=(M, K)).astype(np.float32)
    X[:, K - 1], X[M - 1, : K // 2] = 30.0, 0.0
    return wl.to_fp16(X), wl.gaussian_weight(K, N, 0.02, rng)


@pytest.mark.parametrize("M,K,N", [(9, 16, 8), (9, 4096, 264), (32, 1040, 520), (33, 144, 256), (33, 4096, 4096), (64, 2096, 776), (65, 64, 72),
                                   (65, 4112, 1032), (127, 528, 264), (128, 1168, 3080)])
def test_edges_of_the_tiles(M, K, N):
    X, W = inputs(M, K, N)
    pw, Wide = binding.prequantize_weight(to_gpu(W)), torch.zeros((M, K + 24), dtype=torch.float16, device="cuda")
    Xg = Wide[:, :K]                                                # rows further apart than they are long
    Xg.copy_(to_gpu(X))
    Wq, c = ml.prequantize_weight(W)
    for tau in (wl.TAU, 0.0, np.inf):
        o = ml.mixed_int8_linear(X, Wq, c, tau)
        Y, t = binding.mixed_int8_linear(Xg, pw, tau, taps=("acc",))
        Y_all, t_all = binding.mixed_int8_linear(Xg, pw, tau, taps=True)
        assert np.array_equal(to_np(t["acc"]), o["acc"]) and np.array_equal(to_np(t_all["acc"]), o["acc"]), tau
        assert_y_close(to_np(Y), o["Y"])
        assert torch.equal(Y, Y_all) and torch.equal(Y, binding.mixed_int8_linear(Xg, pw, tau)), tau


@pytest.mark.parametrize("M", [12, 40, 100])
def test_range_longer_than_the_masks(M):
    K, N = 33040, 72                                                # 518 slabs, masks of 256 at a time
    X, W = inputs(M, K, N)
    pw, Xg = binding.prequantize_weight(to_gpu(W)), to_gpu(X)
    ws = binding.linear_workspace(M, K, N, Xg.device)
    Y = binding.mixed_int8_linear(Xg, pw, wl.TAU, workspace=ws)
    out, t = binding.mixed_int8_linear(Xg, pw, wl.TAU, workspace=ws[:-256], taps=("acc",))      # 256 bytes short of the split's sums
    o = ml.mixed_int8_linear(X, *ml.prequantize_weight(W), wl.TAU)
    assert np.array_equal(to_np(t["acc"]), o["acc"])
    assert_y_close(to_np(out), o["Y"])
    assert_y_close(to_np(Y), o["Y"])


@pytest.mark.parametrize("M,K,N", [(9, 4112, 72), (33, 1072, 264), (100, 2096, 72), (128, 16, 8)])
def test_an_infinite_last_column_stays_infinite(M, K, N):
    """K is no multiple of the padded length: what stands in for the columns beyond it meets weights of zero and must be finite.
    Row 2 has an infinity among its last eight entries: its outputs are infinite with the sign of the weight (not a number where
    the weight is zero), the other rows are what they are without it."""
    X, W = inputs(M, K, N)
    W[K - 3] = np.where(W[K - 3] == 0, np.float16(0.01), W[K - 3])
    X[2, K - 3] = np.inf
    pw, Wq = binding.prequantize_weight(to_gpu(W)), ml.prequantize_weight(W)
    Y = to_np(binding.mixed_int8_linear(to_gpu(X), pw, wl.TAU))
    q = Wq[0][K - 3].astype(np.float32)
    want = np.where(q == 0, np.float32(np.nan), np.copysign(np.float32(np.inf), q))
    assert np.array_equal(Y[2].astype(np.float32), want, equal_nan=True)
    rest = np.arange(M) != 2
    X[2, K - 3] = 30.0                                              # (critical as before)
    assert_y_close(Y[rest], ml.mixed_int8_linear(X, *Wq, wl.TAU)["Y"][rest])
