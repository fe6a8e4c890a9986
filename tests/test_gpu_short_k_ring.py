"""GPU parity of the short-K kernels, on the one with its rows in an LDS ring wherever it fits (shortk_ring.h), on the one with
fragments from global memory (shortk.h), and by the dispatcher's choice: launches with fewer and with more steps per
workgroup than the ring has blocks, in each of its widths (one wave's columns, 32 to 128 of them, and four waves side by side),
with and without the residual add and weight zero-points; weights, row pitches and outputs that are not 16-byte aligned; strided
1x1 convolutions whose 32 rows span several images."""
import numpy as np
import pytest
import torch

import oracle
import paper_1806_08342_amd as qnn

from gpu_util import assert_same, dev, host

pytestmark = pytest.mark.gpu


# QNN_SHORTK_ALDS: the ring kernel wherever it fits, by shape, never
ROUTES = pytest.mark.parametrize("route", ["2", "1", "0"])


def _case(M, N, K, bits, seed):
    rng = np.random.default_rng(seed)
    lim = 8 if bits == 4 else 128
    A = rng.integers(0, 256, (M, K)).astype(np.uint8)
    B = rng.integers(-lim, lim, (N, K)).astype(np.int8)
    mult, shift = oracle.quantize_multipliers(10 ** rng.uniform(-3.9, -3.2, N) * (16 if bits == 4 else 1))
    bias = rng.integers(-20000, 20000, N).astype(np.int32)
    rows = np.arange(M) if M < 300 else np.unique(np.r_[0:40, M - 140:M, rng.integers(0, M, 200)])
    return rng, A, oracle.pack_int4(B) if bits == 4 else B, mult, shift, bias, rows


@ROUTES
@pytest.mark.parametrize("M", [129, 2049, 300001])
@pytest.mark.parametrize("N,K", [(16, 256), (32, 16), (64, 128), (48, 32), (128, 64), (96, 208), (512, 64), (512, 256), (224, 96), (160, 224), (72, 160)])
@pytest.mark.parametrize("bits", [8, 4])
def test_walks(tuning, route, M, N, K, bits):
    tuning.setenv("QNN_SHORTK_ALDS", route)
    rng, A, B, mult, shift, bias, rows = _case(M, N, K, bits, M + 3 * N + K + bits)
    dA, dB, dm, ds, db = dev(A), dev(B), dev(mult), dev(shift), dev(bias)
    for z_a, z_out, lo in ((0, 0, 0), (128, 120, 3)):
        want = oracle.qgemm(A[rows], z_a, B, mult, shift, z_out, lo, 250, bias=bias, weight_bits=bits)
        got = host(qnn.qgemm(dA, z_a, dB, dm, ds, z_out, lo, 250, bias=db, weight_bits=bits))
        assert_same(got[rows], want, f"{M}x{N}x{K} z_a={z_a}")
    R = rng.integers(0, 256, (M, N)).astype(np.uint8)
    p = oracle.qadd_params(0.02, 0.031, 0.04)
    got = host(qnn.qgemm_add(dA, z_a, dB, dm, ds, z_out, lo, 250, dev(R), 7, p, 3, 0, 255, bias=db, weight_bits=bits))
    assert_same(got[rows], oracle.qadd(want, z_out, R[rows], 7, p, 3, 0, 255), f"{M}x{N}x{K} add")
    zw = rng.integers(-8, 8, N).astype(np.int32)
    want = oracle.qgemm(A[rows], z_a, B, mult, shift, z_out, lo, 250, bias=bias, weight_bits=bits, z_w=zw)
    got = host(qnn.qgemm_asym(dA, z_a, dB, dev(zw), dm, ds, z_out, lo, 250, bias=db, weight_bits=bits))
    assert_same(got[rows], want, f"{M}x{N}x{K} asym")


@ROUTES
@pytest.mark.parametrize("M", [200, 150001])
@pytest.mark.parametrize("N,K", [(40, 48), (136, 256), (512, 128)])
def test_pitches_and_alignment(tuning, route, M, N, K):
    tuning.setenv("QNN_SHORTK_ALDS", route)
    rng, A, B, mult, shift, bias, rows = _case(M, N, K, 8, 77 + M + N + K)
    dm, ds, db = dev(mult), dev(shift), dev(bias)
    wide = torch.zeros((M, K + 32), dtype=torch.uint8, device="cuda:0")
    wide[:, 16:16 + K] = dev(A)
    flat = torch.zeros(N * K + 16, dtype=torch.int8, device="cuda:0")
    flat[4:4 + N * K] = dev(B).reshape(-1)  # 4-byte aligned weights
    out = torch.full((M, N + 24), 77, dtype=torch.uint8, device="cuda:0")
    qnn.qgemm(wide[:, 16:16 + K], 9, flat[4:4 + N * K].view(N, K), dm, ds, 0, 0, 255, bias=db, out=out[:, 8:8 + N])
    got = host(out)
    assert_same(got[rows, 8:8 + N], oracle.qgemm(A[rows], 9, B, mult, shift, 0, 0, 255, bias=bias), f"{M}x{N}x{K}")
    assert (got[:, :8] == 77).all() and (got[:, 8 + N:] == 77).all(), "bytes beside the output"


@ROUTES
@pytest.mark.parametrize("batch,H,W,cin,cout,stride", [(3, 29, 31, 64, 200, 2), (40, 3, 2, 32, 32, 2), (70, 1, 1, 256, 512, 3), (9, 56, 7, 128, 64, 3),
                                                       (2, 5, 300, 16, 96, 2), (64, 28, 28, 256, 130, 2), (200, 27, 27, 64, 448, 2)])
@pytest.mark.parametrize("bits", [8, 4])
def test_strided_convolutions(tuning, route, batch, H, W, cin, cout, stride, bits):
    tuning.setenv("QNN_SHORTK_ALDS", route)
    rng, _, B, mult, shift, bias, _ = _case(100, cout, cin, bits, batch + H + W + cin + bits)
    x = rng.integers(0, 256, (batch, H, W, cin)).astype(np.uint8)
    w = B.reshape(cout, 1, 1, -1)
    want = oracle.qconv2d(x, 5, w, (stride, stride), (0, 0), mult, shift, 0, 0, 255, bias=bias, weight_bits=bits)
    got = host(qnn.qconv2d(dev(x), 5, dev(w), (stride, stride), (0, 0), dev(mult), dev(shift), 0, 0, 255, bias=dev(bias), weight_bits=bits))
    assert_same(got, want, f"strided {batch}x{H}x{W}x{cin}->{cout}")
    R = rng.integers(0, 256, want.shape).astype(np.uint8)
    p = oracle.qadd_params(0.02, 0.031, 0.04)
    got = host(qnn.qconv2d_add(dev(x), 5, dev(w), (stride, stride), (0, 0), dev(mult), dev(shift), 0, 0, 255, dev(R), 7, p, 3, 0, 255, bias=dev(bias),
                               weight_bits=bits))
    assert_same(got, oracle.qadd(want, 0, R, 7, p, 3, 0, 255), f"strided {batch}x{H}x{W}x{cin}->{cout} add")


@ROUTES
@pytest.mark.parametrize("M,N,K,bits", [(26310, 640, 208, 8), (5003, 640, 208, 4), (9000, 1100, 64, 8), (3001, 2300, 32, 4), (20011, 700, 128, 8),
                                        (300, 20000, 96, 8)])
def test_sets_that_do_not_divide_the_cus(tuning, route, M, N, K, bits):
    tuning.setenv("QNN_SHORTK_ALDS", route)
    # three, five, seven and more sets of column groups, more sets than workgroups of an XCD: walkers of unequal numbers of steps
    rng, A, B, mult, shift, bias, rows = _case(M, N, K, bits, 5 * M + N + K)
    z_a, z_out = 128, 120
    want = oracle.qgemm(A[rows], z_a, B, mult, shift, z_out, 3, 250, bias=bias, weight_bits=bits)
    got = host(qnn.qgemm(dev(A), z_a, dev(B), dev(mult), dev(shift), z_out, 3, 250, bias=dev(bias), weight_bits=bits))
    assert_same(got[rows], want, f"{M}x{N}x{K}")
    R = rng.integers(0, 256, (M, N)).astype(np.uint8)
    p = oracle.qadd_params(0.02, 0.031, 0.04)
    got = host(qnn.qgemm_add(dev(A), z_a, dev(B), dev(mult), dev(shift), z_out, 3, 250, dev(R), 7, p, 3, 0, 255, bias=dev(bias), weight_bits=bits))
    assert_same(got[rows], oracle.qadd(want, z_out, R[rows], 7, p, 3, 0, 255), f"{M}x{N}x{K} add")


@pytest.mark.parametrize("lda", [(1 << 26) - 16, 1 << 26, (1 << 26) + 8])
@pytest.mark.parametrize("N,K", [(200, 64), (48, 240)])
def test_rows_far_apart(tuning, lda, N, K):
    # 32 rows at the edge of the ring kernel's 31-bit offsets and beyond it
    tuning.setenv("QNN_SMALL", "0")  # 65 rows take the short-K kernels only on request
    M = 65
    rng, A, B, mult, shift, bias, rows = _case(M, N, K, 8, N + K)
    far = torch.empty((M - 1) * lda + K, dtype=torch.uint8, device="cuda:0").as_strided((M, K), (lda, 1))
    far.copy_(dev(A))
    want = oracle.qgemm(A, 9, B, mult, shift, 0, 0, 255, bias=bias)
    assert_same(host(qnn.qgemm(far, 9, dev(B), dev(mult), dev(shift), 0, 0, 255, bias=dev(bias))), want, f"lda {lda} {N}x{K}")
    zw = rng.integers(-8, 8, N).astype(np.int32)
    want = oracle.qgemm(A, 9, B, mult, shift, 0, 0, 255, bias=bias, z_w=zw)
    assert_same(host(qnn.qgemm_asym(far, 9, dev(B), dev(zw), dev(mult), dev(shift), 0, 0, 255, bias=dev(bias))), want, f"lda {lda} {N}x{K} asym")


@pytest.mark.parametrize("N,K", [(512, 64), (512, 128), (512, 256), (1024, 96)])
def test_waves_of_a_workgroup_in_different_rescale_forms(tuning, N, K):
    # four waves side by side share a barrier per step: some take the fused rescale, one the general one in range (shift 25), one
    # the one beyond (bias 2^28), one with a left shift
    tuning.setenv("QNN_SHORTK_ALDS", "2")
    M = 20000
    rng, A, B, mult, shift, bias, rows = _case(M, N, K, 8, N + K)
    mult[130], shift[130] = 2 ** 30 + 12345, -3
    bias[150] = 2 ** 28
    shift[300], shift[310] = 25, 31
    bias[N - 1], bias[N - 2] = 2 ** 28, -(2 ** 28)
    zw = rng.integers(-8, 8, N).astype(np.int32)
    R = rng.integers(0, 256, (M, N)).astype(np.uint8)
    p = oracle.qadd_params(0.02, 0.031, 0.04)
    for z_a, z_out, lo, hi in ((0, 0, 0, 255), (128, 120, 3, 250)):
        want = oracle.qgemm(A[rows], z_a, B, mult, shift, z_out, lo, hi, bias=bias)
        got = host(qnn.qgemm(dev(A), z_a, dev(B), dev(mult), dev(shift), z_out, lo, hi, bias=dev(bias)))
        assert_same(got[rows], want, f"{M}x{N}x{K} z_a={z_a}")
        got = host(qnn.qgemm_add(dev(A), z_a, dev(B), dev(mult), dev(shift), z_out, lo, hi, dev(R), 7, p, 3, 0, 255, bias=dev(bias)))
        assert_same(got[rows], oracle.qadd(want, z_out, R[rows], 7, p, 3, 0, 255), f"{M}x{N}x{K} z_a={z_a} add")
        want = oracle.qgemm(A[rows], z_a, B, mult, shift, z_out, lo, hi, bias=bias, z_w=zw)
        got = host(qnn.qgemm_asym(dev(A), z_a, dev(B), dev(zw), dev(mult), dev(shift), z_out, lo, hi, bias=dev(bias)))
        assert_same(got[rows], want, f"{M}x{N}x{K} z_a={z_a} asym")
