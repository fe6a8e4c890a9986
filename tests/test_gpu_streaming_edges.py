"""Element-wise passes at the edges of their tiles: lengths around a vector, a tile and several tiles, pointers that are
only aligned to their element, channel counts that do and do not divide a tile row, rows shorter than a vector."""
import numpy as np
import pytest
import torch

import oracle
import paper_1806_08342_amd as qnn

from gpu_util import assert_same, dev, host

pytestmark = pytest.mark.gpu

LENGTHS = [1, 3, 5, 1023, 4096, 4099, 8192 * 4 + 7, 300_001]


def _shifted(a, by):
    """The same values at a device address that is `by` elements past an aligned one."""
    t = dev(np.concatenate([np.zeros(by, a.dtype), a]))
    return t[by:]


@pytest.mark.parametrize("n", LENGTHS)
@pytest.mark.parametrize("by", [0, 1])
def test_quantize_and_dequantize(n, by):
    x = np.random.default_rng(n).normal(0, 2, n).astype(np.float32)
    x[:1] = np.nan
    xd, s, z = _shifted(x, by), 0.031, 120
    q = oracle.quantize(x, s, z)
    out = torch.zeros(n + by, dtype=torch.uint8, device="cuda:0")
    assert_same(host(qnn.quantize(xd, s, z, out=out[by:])), q, "quantize")
    back = torch.zeros(n + by, dtype=torch.float32, device="cuda:0")
    assert_same(host(qnn.dequantize(out[by:], s, z, out=back[by:])), oracle.dequantize(q, s, z), "dequantize")
    wide = oracle.quantize_wide(x, 1e-4, 30000, 0, 65535)
    assert_same(host(qnn.quantize_u16(xd, 1e-4, 30000)), wide, "quantize u16")
    assert_same(host(qnn.dequantize_u16(_shifted(wide, by), 1e-4, 30000)), oracle.dequantize_wide(wide, 1e-4, 30000), "dequantize u16")
    g = np.random.default_rng(n + 1).normal(0, 1, n).astype(np.float32)
    assert_same(host(qnn.simquant(xd, s, z)), oracle.simquant(x, s, z, 0, 255), "simquant")
    assert_same(host(qnn.simquant_backward(xd, _shifted(g, by), s, z)), oracle.simquant_backward(x, g, s, z, 0, 255), "backward")
    st = qnn.new_range_state()
    codes = host(qnn.quantize_dynamic(xd, st))
    lo, hi = oracle.finite_range(x)
    r = qnn.read_range_state(st)
    assert (r["xmin"], r["xmax"]) == (np.float32(lo), np.float32(hi))
    assert_same(codes, oracle.quantize(x, r["scale"], r["zero_point"]), "dynamic")


@pytest.mark.parametrize("rows,channels", [(1, 1), (3, 2), (700, 3), (1000, 7), (513, 16), (300, 100), (257, 256), (65, 1000), (40, 1024), (33, 3000)])
@pytest.mark.parametrize("per_channel", [True, False])
def test_requantize(rows, channels, per_channel):
    rng = np.random.default_rng(rows + channels)
    acc = rng.integers(-300000, 300000, (rows, channels)).astype(np.int32)
    mult, shift = oracle.quantize_multipliers(10 ** rng.uniform(-4, -2.5, channels))
    if channels > 5:
        shift[5] = 0  # a channel on the general form
    acc[0, 0] = 2 ** 31 - 1
    m, s = (mult, shift) if per_channel else (mult[:1], shift[:1])
    want = oracle.requantize(acc, m, s, per_channel, 100, 2, 250)
    assert_same(host(qnn.requantize(dev(acc), dev(m), dev(s), per_channel, 100, 2, 250)), want, "requantize")
    shifted = _shifted(acc.reshape(-1), 1).view(rows, channels)
    assert_same(host(qnn.requantize(shifted, dev(m), dev(s), per_channel, 100, 2, 250)), want, "requantize, 4-byte aligned")


@pytest.mark.parametrize("rows,cols", [(1, 1), (5, 15), (700, 16), (333, 17), (64, 1000), (1000, 33), (3, 5000)])
def test_add_and_concat_rescale(rows, cols):
    rng = np.random.default_rng(rows * cols)
    a, b = (rng.integers(0, 256, (rows, cols)).astype(np.uint8) for _ in range(2))
    p = oracle.qadd_params(0.02, 0.031, 0.04)
    want = oracle.qadd(a, 120, b, 131, p, 3, 3, 250)
    assert_same(host(qnn.qadd(dev(a), 120, dev(b), 131, p, 3, 3, 250)), want, "qadd")
    flat = qnn.qadd(_shifted(a.reshape(-1), 3), 120, _shifted(b.reshape(-1), 5), 131, p, 3, 3, 250)
    assert_same(host(flat).reshape(rows, cols), want, "qadd at odd addresses")
    mult, shift = oracle.quantize_multiplier(0.7)
    one = np.array([mult], np.int32), np.array([shift], np.int32)
    ref = oracle.requantize(a.astype(np.int32) - 9, *one, False, 128, 1, 254)
    cat = torch.full((rows, 2 * cols + 3), 77, dtype=torch.uint8, device="cuda:0")
    qnn.rescale_u8(dev(a), 9, mult, shift, 128, 1, 254, out=cat[:, 1:1 + cols])
    assert_same(host(cat[:, 1:1 + cols].contiguous()), ref, "concat slice")
    assert bool((cat[:, 0] == 77).all()) and bool((cat[:, 1 + cols:] == 77).all())


@pytest.mark.parametrize("rows,cols,spaced", [(7, 15, 0), (300, 17, 0), (300, 17, 3), (2000, 31, 16), (64, 1000, 8), (3, 70_001, 1), (50, 48, 0)])
def test_concat_rescale_in_place(rows, cols, spaced):
    # each code is rescaled once, whatever pieces the rows are cut into
    rng = np.random.default_rng(rows + cols)
    a = rng.integers(0, 256, (rows, cols + spaced)).astype(np.uint8)
    mult, shift = oracle.quantize_multiplier(0.7)
    one = np.array([mult], np.int32), np.array([shift], np.int32)
    want = a.copy()
    want[:, :cols] = oracle.requantize(np.ascontiguousarray(a[:, :cols]).astype(np.int32) - 9, *one, False, 128, 1, 254)
    t = dev(a)
    qnn.rescale_u8(t[:, :cols], 9, mult, shift, 128, 1, 254, out=t[:, :cols])
    assert_same(host(t), want, "in place")
