"""Every kernel that takes weight zero-points, at the edges of what it accepts, against the oracle: the depthwise patch,
matrix-unit and multiply-add forms, the few-row, short-K, stem, staged and large-tile dense kernels.  The zero-points
include -128, which the depthwise kernels treat apart, and both ends of the weight range meet it."""
import numpy as np
import pytest

import oracle
import paper_1806_08342_amd as qnn

from gpu_util import assert_same, dev, host

pytestmark = pytest.mark.gpu


def _rescale(rng, channels, terms, lim):
    return oracle.quantize_multipliers(rng.uniform(40.0, 120.0, channels) / (terms * 255.0 * lim))


def _zero_points(rng, channels, lim):
    z = rng.integers(-lim, lim, channels).astype(np.int32)
    z[::3] = -lim
    z[1::5] = lim - 1
    return z


@pytest.mark.parametrize("N,H,W,C,stride,pad", [
    (1, 3, 3, 4, 1, 1), (2, 9, 7, 12, 1, 1), (2, 10, 13, 20, 2, 1), (1, 8, 8, 512, 1, 1), (3, 17, 5, 8, 2, 0),
    (2, 33, 21, 68, 1, 0),           # patch kernel: ragged patches, tall and short
    (2, 112, 112, 96, 1, 1), (3, 113, 115, 80, 1, 0), (4, 113, 112, 176, 2, 1), (3, 131, 129, 176, 2, 0),  # matrix-unit kernel
    (65537, 3, 3, 4, 1, 1), (65537, 3, 3, 4, 2, 1),  # more images than a grid dimension takes: multiply-add form
])
def test_depthwise_routes(N, H, W, C, stride, pad):
    rng = np.random.default_rng(N + H * W + C + stride)
    x = rng.integers(0, 256, (N, H, W, C)).astype(np.uint8)
    w = rng.integers(-128, 128, (3, 3, C)).astype(np.int8)
    z_w = _zero_points(rng, C, 128)
    w[:, :, ::6] = 127  # z_w = -128: the largest effective weight, 255
    w[:, :, 3::6] = -128
    x[:, :, :, ::6] = 255
    mult, shift = _rescale(rng, C, 9, 128)
    bias = rng.integers(-2000, 2000, C).astype(np.int32)
    general = shift.copy()
    general[0] = 27  # outside the 32-bit rescale
    for z_x, sh, act_min in ((131, shift, 120), (0, shift, 0), (255, general, 3)):
        want = oracle.qdwconv2d(x, z_x, w, (stride, stride), (pad, pad), mult, sh, 120, act_min, 250, bias=bias, z_w=z_w)
        got = host(qnn.qdwconv2d_asym(dev(x), z_x, dev(w), dev(z_w), (stride, stride), (pad, pad), dev(mult), dev(sh), 120, act_min,
                                      250, bias=dev(bias)))
        assert_same(got, want, f"z_x={z_x}")
    assert len(np.unique(want)) > 16


@pytest.mark.parametrize("N,H,W,C,stride,pad", [
    (2, 9, 7, 12, 1, 1), (1, 17, 22, 68, 2, 0),            # patch kernel
    (2, 113, 115, 112, 1, 0), (4, 113, 112, 176, 2, 1),    # matrix-unit kernel, C no multiple of 32
    (65537, 3, 3, 4, 1, 1),                                # multiply-add form
])
def test_depthwise_zero_points_beyond_a_byte(N, H, W, C, stride, pad):
    rng = np.random.default_rng(N + H * W + C)
    x = rng.integers(0, 256, (N, H, W, C)).astype(np.uint8)
    w = rng.integers(-128, 128, (3, 3, C)).astype(np.int8)
    mult, shift = _rescale(rng, C, 9, 128)
    bias = rng.integers(-2000, 2000, C).astype(np.int32)
    z_w = _zero_points(rng, C, 128)
    z_w[C // 2] = 128               # one channel only: its neighbours stay on the byte form
    z_w[-1] = -129
    for z in (z_w, rng.integers(0, 256, C).astype(np.int32), rng.integers(-70000, 70000, C).astype(np.int32)):
        want = oracle.qdwconv2d(x, 131, w, (stride, stride), (pad, pad), mult, shift, 120, 0, 255, bias=bias, z_w=z)
        got = host(qnn.qdwconv2d_asym(dev(x), 131, dev(w), dev(z), (stride, stride), (pad, pad), dev(mult), dev(shift), 120, 0, 255,
                                      bias=dev(bias)))
        assert_same(got, want, f"z_w in [{z.min()}, {z.max()}]")
    assert len(np.unique(want)) > 1


@pytest.mark.parametrize("M,N,K,bits", [
    (1, 16, 16, 8), (64, 70, 129, 8), (33, 40, 258, 4), (700, 48, 384, 8),      # few rows, with tails in K
    (9, 20, 208, 8), (500, 48, 80, 8), (90, 33, 96, 4), (40, 50, 1120, 4),       # ... of whole 16-byte pieces
    (5000, 30, 8, 8), (5001, 33, 24, 4), (4100, 96, 40, 8), (3000, 200, 72, 4), (2999, 130, 120, 8), (7001, 260, 256, 8),
    (6000, 131, 248, 4),                                                         # short K, partial steps
    (3000, 700, 320, 8), (2500, 900, 640, 4), (9000, 2100, 448, 8),              # large tiles
    (1500, 1100, 323, 8), (2100, 1300, 402, 4),                                  # staged tiles
])
def test_matrix_routes(M, N, K, bits):
    rng = np.random.default_rng(M + N + K)
    lim = 8 if bits == 4 else 128
    A = rng.integers(0, 256, (M, K)).astype(np.uint8)
    Bt = rng.integers(-lim, lim, (N, K)).astype(np.int8)
    z_w = _zero_points(rng, N, lim)
    mult, shift = _rescale(rng, N, K, lim)
    bias = rng.integers(-2000, 2000, N).astype(np.int32)
    Bo = oracle.pack_int4(Bt) if bits == 4 else Bt
    rows = np.unique(np.r_[0:min(M, 150), M // 2:min(M, M // 2 + 150), max(0, M - 150):M])
    general = shift.copy()
    general[N // 2] = 27
    for z_a, sh in ((131, shift), (0, general), (255, shift)):
        want = oracle.qgemm(A[rows], z_a, Bo, mult, sh, 120, 0, 255, bias=bias, weight_bits=bits, z_w=z_w)
        got = host(qnn.qgemm_asym(dev(A), z_a, dev(Bo), dev(z_w), dev(mult), dev(sh), 120, 0, 255, bias=dev(bias), weight_bits=bits))
        assert_same(got[rows], want, f"z_a={z_a}")
    assert len(np.unique(want)) > 8


@pytest.mark.parametrize("N,H,W,Cin,Cout,k,stride,pad,bits", [
    (8, 65, 67, 3, 32, 3, 2, 1, 8), (4, 64, 61, 3, 64, 7, 2, 3, 8), (8, 50, 41, 4, 40, 3, 1, 1, 8), (2, 57, 33, 1, 24, 5, 1, 2, 8),  # stems
    (1, 7, 7, 48, 33, 3, 1, 1, 8), (2, 9, 9, 80, 24, 3, 2, 1, 4),               # few positions, window longer than whole steps
    (8, 30, 29, 64, 200, 3, 1, 1, 8), (8, 31, 31, 128, 72, 3, 2, 1, 4),         # large tiles
    (6, 33, 35, 20, 100, 3, 1, 1, 8),                                            # staged tiles
    (6, 40, 40, 64, 90, 1, 2, 0, 8),                                             # strided 1x1
])
def test_convolution_routes(N, H, W, Cin, Cout, k, stride, pad, bits):
    rng = np.random.default_rng(N + H * W + Cin + Cout)
    lim = 8 if bits == 4 else 128
    x = rng.integers(0, 256, (N, H, W, Cin)).astype(np.uint8)
    w = rng.integers(-lim, lim, (Cout, k, k, Cin)).astype(np.int8)
    z_w = _zero_points(rng, Cout, lim)
    mult, shift = _rescale(rng, Cout, k * k * Cin, lim)
    bias = rng.integers(-2000, 2000, Cout).astype(np.int32)
    wo = oracle.pack_int4(w) if bits == 4 else w
    for z_x in (131, 0, 255):
        want = oracle.qconv2d(x, z_x, wo, (stride, stride), (pad, pad), mult, shift, 120, 0, 255, bias=bias, weight_bits=bits, z_w=z_w)
        got = host(qnn.qconv2d_asym(dev(x), z_x, dev(wo), dev(z_w), (stride, stride), (pad, pad), dev(mult), dev(shift), 120, 0, 255,
                                    bias=dev(bias), weight_bits=bits))
        assert_same(got, want, f"z_x={z_x}")
    assert len(np.unique(want)) > 8
