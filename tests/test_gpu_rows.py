"""A few rows, the whole layer in one kernel: integers equal to the oracle's and outputs to the fp16 bar where its shares can go
wrong: fewer slabs of K than waves, the most chunks of the rows a thread holds and one more (then another kernel serves), as many
column tiles as workgroups and one more, a ragged last tile, one to eight rows; with the outputs of a call that asks for
every tap equal bit for bit."""
import numpy as np
import pytest
import torch

from oracle import mixed_linear as ml
from paper_2407_19775_amd import binding, workloads as wl
from gpu_util import assert_y_close, to_gpu, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N", [(1, 64, 8), (1, 49152, 24), (1, 49168, 24), (2, 8192, 4096), (2, 16400, 4104), (3, 1040, 8200), (4, 11008, 72),
                                   (4, 12304, 40), (5, 1040, 6160), (6, 5456, 4112), (7, 528, 264), (8, 2048, 12304), (8, 6160, 48)])
def test_edges_of_the_shares(M, K, N):
    rng = np.random.default_rng([M, K, N])
    X = rng.standard_t(3.0, size=(M, K)).astype(np.float32)
    X[:, K - 1] = 30.0                                              # the last column is critical
    if M > 1:
        X[M - 1, :K // 2] = 0.0
    X = wl.to_fp16(X)
    W = wl.gaussian_weight(K, N, 0.02, rng)
    pw, Xg = binding.prequantize_weight(to_gpu(W)), to_gpu(X)
    Wq, c = ml.prequantize_weight(W)
    for tau in (wl.TAU, 0.0, np.inf):
        o = ml.mixed_int8_linear(X, Wq, c, tau)
        Y, t = binding.mixed_int8_linear(Xg, pw, tau, taps=("acc",))
        Y_all, t_all = binding.mixed_int8_linear(Xg, pw, tau, taps=True)
        assert np.array_equal(to_np(t["acc"]), o["acc"]) and np.array_equal(to_np(t_all["acc"]), o["acc"]), tau
        assert_y_close(to_np(Y), o["Y"])
        assert torch.equal(Y, Y_all) and torch.equal(Y, binding.mixed_int8_linear(Xg, pw, tau)), tau
