"""A few rows whose operands do not fit in LDS: the kernel that prepares its own operands for a range of K.  Integers equal to the
oracle's and outputs to the fp16 bar where it can go wrong: K in one range (the whole layer in one kernel) and in many, ranges
of eight slabs and of the most there are, a last range that is shorter, a K that ends inside a slab, ragged columns, one to
eight rows; with the outputs of a call that asks for every tap equal bit for bit, with what can follow the layer, and at the
lines of its dispatch."""
import numpy as np
import pytest
import torch

from oracle import boundary_exit as be
from oracle import lora, mixed_linear as ml
from paper_2407_19775_amd import binding, workloads as wl
from gpu_util import assert_y_close, panel_plan, rows_kernel_fits, to_gpu, to_np

CASES = [(1, 65536, 24), (2, 112, 57352), (2, 24592, 1032), (3, 20496, 264), (3, 96, 33016), (5, 528, 65544), (6, 12304, 4104), (7, 16400, 72),
         (8, 5136, 776)]


@pytest.mark.parametrize("M,K,N,here", [(8, 11008, 4096, True), (3, 16384, 2048, True), (5, 512, 57344, True), (2, 36864, 8192, True),
                                        (8, 24576, 2048, True), (3, 17920, 6656, True), (4, 20480, 8192, True), (8, 4096, 24576, False),
                                        (8, 65536, 1024, False), (4, 24576, 8192, False), (2, 49152, 8192, False), (9, 11008, 4096, False)])
def test_dispatch_follows_the_measured_sides(M, K, N, here):
    """Where this kernel measured faster than k_prep_rows and k_gemm_decode, or slower (256 compute units)."""
    assert not rows_kernel_fits(M, K, N) and (panel_plan(M, K, N)[0] > 0) == here


@pytest.mark.parametrize("M,K,N,single", [(3, 512, 57344, False), (3, 512, 28672, True), (5, 8192, 8192, False), (6, 6144, 8192, True),
                                          (4, 11008, 8192, True), (2, 24576, 1024, False), (2, 24576, 4096, True), (2, 24576, 8192, False)])
def test_single_kernel_where_it_measured_faster(M, K, N, single):
    assert rows_kernel_fits(M, K, N) == single


def inputs(M, K, N):
    rng = np.random.default_rng([M, K, N])
    X = rng.standard_t(3.0, size=(M, K)).astype(np.float32)
    X[:, K - 1] = 30.0                                              # the last column is critical
    if M > 1:
        X[M - 1, :K // 2] = 0.0
    return wl.to_fp16(X), wl.gaussian_weight(K, N, 0.02, rng), rng


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", CASES)
def test_edges_of_the_ranges(M, K, N):
    assert not rows_kernel_fits(M, K, N) and panel_plan(M, K, N)[0] > 0
    X, W, rng = inputs(M, K, N)
    Wide = torch.zeros((M, K + 8), dtype=torch.float16, device="cuda")
    Xg, pw, bias = Wide[:, :K], binding.prequantize_weight(to_gpu(W)), wl.gaussian_bias(N, 0.3, rng)
    Xg.copy_(to_gpu(X))                                             # rows further apart than they are long
    bg, (Wq, c) = to_gpu(bias), ml.prequantize_weight(W)
    for tau in (wl.TAU, 0.0, np.inf):
        o = ml.mixed_int8_linear(X, Wq, c, tau, bias)
        Y, t = binding.mixed_int8_linear(Xg, pw, tau, bias=bg, taps=("acc",))
        Y_all, t_all = binding.mixed_int8_linear(Xg, pw, tau, bias=bg, taps=True)
        assert np.array_equal(to_np(t["acc"]), o["acc"]) and np.array_equal(to_np(t_all["acc"]), o["acc"]), tau
        assert np.array_equal(to_np(t_all["outlier_mask"]).astype(bool), o["flag"]) and np.array_equal(to_np(t_all["xq"]), o["Xq"])
        assert_y_close(to_np(Y), o["Y"])
        assert torch.equal(Y, Y_all) and torch.equal(Y, binding.mixed_int8_linear(Xg, pw, tau, bias=bg)), tau
        other = binding.mixed_int8_linear(Xg, pw, tau, bias=bg, tuning=binding.TUNE_NO_ROWS_KERNEL)
        assert_y_close(to_np(Y), to_np(other), rel=2e-3)            # another order of fp32 additions


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(3, 96, 33016), (8, 5136, 776)])
def test_what_follows_the_layer(M, K, N):
    X, W, rng = inputs(M, K, N)
    Wq, c = ml.prequantize_weight(W)
    pw, Xg = binding.prequantize_weight(to_gpu(W)), to_gpu(X)
    plain = to_np(binding.mixed_int8_linear(Xg, pw, wl.TAU))
    R = wl.to_fp16(rng.standard_t(3.0, size=(M, N)).astype(np.float32))
    H = be.add_residual(plain, R)
    assert np.array_equal(to_np(binding.mixed_int8_linear(Xg, pw, wl.TAU, residual=to_gpu(R))).view(np.uint16), H.view(np.uint16))
    Hg = torch.zeros((M, N), dtype=torch.float16, device="cuda")
    codes, absmax = binding.mixed_int8_linear_to_codes(Xg, pw, wl.TAU, 64, residual=to_gpu(R), H=Hg)
    want = binding.quantize_blockwise(to_gpu(H), 64)
    assert np.array_equal(to_np(Hg).view(np.uint16), H.view(np.uint16)) and torch.equal(codes, want[0]) and torch.equal(absmax, want[1])
    gelu = to_np(binding.mixed_int8_linear(Xg, pw, wl.TAU, gelu=True))
    z = torch.from_numpy(plain).double()
    assert_y_close(gelu, (0.5 * z * torch.special.erfc(-z / 2 ** 0.5)).numpy(), rel=2e-3)
    A, B = (wl.to_fp16(rng.standard_normal(s).astype(np.float32) * 0.05) for s in ((16, K), (N, 16)))
    T = torch.zeros((M, 16), dtype=torch.float16, device="cuda")
    Y = binding.mixed_int8_linear(Xg, pw, wl.TAU, lora=(to_gpu(A), to_gpu(B), T))
    o = lora.mixed_int8_linear_lora(X, Wq, c, wl.TAU, A, B)
    assert_y_close(to_np(Y), o["Y"])
    assert_y_close(to_np(T), o["T"])


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(8, 2048, 59144), (2, 32768, 16384)])
def test_the_longest_ranges(M, K, N):
    """As many columns of the rows in LDS as there is room for, and a range of more slabs than a word of flags; the oracle on some of
    the columns."""
    splits, slabs = panel_plan(M, K, N)
    assert not rows_kernel_fits(M, K, N) and splits > 0 and (M * slabs == 256 or slabs == 128)
    X = inputs(M, K, 8)[0]
    W = torch.randn((K, N), generator=torch.Generator(device="cuda").manual_seed(M), device="cuda", dtype=torch.float16) * 0.02
    pw, Xg = binding.prequantize_weight(W), to_gpu(X)
    cols = torch.unique(torch.cat([torch.linspace(0, N - 1, 250).long(), torch.tensor([255, 256, N - 8])]))
    Wq, c = ml.prequantize_weight(to_np(W[:, cols.cuda()].contiguous()))
    for tau in (wl.TAU, np.inf):
        Y, t = binding.mixed_int8_linear(Xg, pw, tau, taps=("acc",))
        o = ml.mixed_int8_linear(X, Wq, c, tau)
        assert np.array_equal(to_np(t["acc"][:, cols.cuda()]), o["acc"])
        assert_y_close(to_np(Y[:, cols.cuda()]), o["Y"])
