"""GPU parity of the pipelined tiles on convolutions whose taps outside the image read as zeros outside a buffer (code z_x = 0, or
no padding) and on their neighbours that gather a constant chunk (z_x != 0 with padding, more than 32 taps, Cin % 64 != 0):
images smaller than a tile, tiles across images, every tile form."""
import numpy as np
import pytest

import oracle
import paper_1806_08342_amd as qnn

from gpu_util import assert_same, dev, host

pytestmark = pytest.mark.gpu

TILES = ["dma128x128", "dma256x256", "dma256x64", "dma256x128", "p128x256", "p256x128", "dma128x128s3"]


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("batch,H,W,cin,cout,k,stride,pad,z_x", [
    (2, 13, 11, 128, 72, 3, 1, 1, 0), (2, 13, 11, 128, 72, 3, 1, 1, 91), (40, 3, 2, 64, 130, 3, 2, 1, 0), (3, 9, 10, 64, 64, 5, 1, 2, 0),
    (1, 12, 12, 64, 40, 6, 1, 2, 0), (3, 10, 7, 192, 256, 1, 2, 0, 200), (2, 8, 8, 64, 96, 3, 2, 0, 17), (2, 9, 9, 48, 64, 3, 1, 1, 0),
    (2, 7, 7, 64, 64, 4, 3, 3, 0)])
def test_conv_taps(tuning, tile, batch, H, W, cin, cout, k, stride, pad, z_x):
    tuning.setenv("QNN_FORCE_TILE", tile)
    rng = np.random.default_rng(batch + H + W + cin + cout + k + stride + z_x)
    x = rng.integers(0, 256, (batch, H, W, cin)).astype(np.uint8)
    w = rng.integers(-128, 128, (cout, k, k, cin)).astype(np.int8)
    mult, shift = oracle.quantize_multipliers(10 ** rng.uniform(-4.0, -3.4, cout))
    bias = rng.integers(-20000, 20000, cout).astype(np.int32)
    for z_out in (0, 120):
        want = oracle.qconv2d(x, z_x, w, (stride, stride), (pad, pad), mult, shift, z_out, 0, 255, bias=bias)
        got = host(qnn.qconv2d(dev(x), z_x, dev(w), (stride, stride), (pad, pad), dev(mult), dev(shift), z_out, 0, 255, bias=dev(bias)))
        assert_same(got, want, f"{tile} {batch}x{H}x{W}x{cin}->{cout} k={k} s={stride} p={pad} z_x={z_x} z_out={z_out}")
