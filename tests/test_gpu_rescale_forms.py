"""GPU parity of the epilogue's forms of the rescale: every combination of output range (0 ... 255 or narrower) and tie
term (act_min below z_out or not), with per-channel multipliers and shifts at the edges of what the 64-bit
multiply-add takes and beyond them (those channels go through the general form), on every kernel family."""
import numpy as np
import pytest

import oracle
import paper_1806_08342_amd as qnn

from gpu_util import assert_same, dev, host

pytestmark = pytest.mark.gpu

RANGES = [(0, 0, 255), (128, 0, 255), (10, 10, 200), (100, 20, 230), (255, 0, 255), (0, 0, 0)]
INSIDE = [(1 << 30, 9), ((1 << 31) - 1, 10), (1518500250, 8), (1 << 30, 1), ((1 << 31) - 1, 20), (1 << 30, 20), (1234567891, 11)]
OUTSIDE = [((1 << 30) - 1, 9), (5, 3), (0, 1), (-(1 << 30), 9), (1 << 30, 0), (1 << 30, 21), (1 << 30, -2)]


def _params(n, edge, rng):
    """Multipliers and shifts of n channels; `edge`: some channels outside the fused forms as well"""
    pool = INSIDE + (OUTSIDE if edge else [])
    pick = [pool[i] for i in rng.integers(0, len(pool), n)]
    return np.array([p[0] for p in pick], np.int32), np.array([p[1] for p in pick], np.int32)


def _bias(n, shift, rng):
    # values around zero and around the ends of the range, exact ties of negative values among them
    return (rng.integers(-400, 400, n) * (1 << np.clip(shift, 0, 11)) // 2).astype(np.int32)


@pytest.mark.parametrize("z_out,lo,hi", RANGES)
@pytest.mark.parametrize("edge", [False, True])
@pytest.mark.parametrize("M,N,K,tile", [(9, 48, 64, ""), (2085, 272, 64, ""), (1063, 272, 256, ""), (700, 192, 320, "dma64x64"),
                                        (300, 272, 320, "dma256x256"), (257, 144, 320, "p256x128"), (200, 80, 72, "64x64"), (33000, 80, 288, "")])
def test_product(z_out, lo, hi, edge, M, N, K, tile):
    rng = np.random.default_rng(M + N + K + z_out)
    A = rng.integers(0, 256, (M, K)).astype(np.uint8)
    B = rng.integers(-2, 3, (N, K)).astype(np.int8)
    mult, shift = _params(N, edge, rng)
    bias = _bias(N, shift, rng)
    rows = np.arange(M) if M < 4000 else np.sort(rng.choice(M, 500, replace=False))
    want = oracle.qgemm(A[rows], 77, B, mult, shift, z_out, lo, hi, bias=bias)
    if tile:
        qnn.tuning_set("QNN_FORCE_TILE", tile)
    try:
        got = host(qnn.qgemm(dev(A), 77, dev(B), dev(mult), dev(shift), z_out, lo, hi, bias=dev(bias)))
    finally:
        qnn.tuning_set("QNN_FORCE_TILE")
    assert_same(got[rows], want, f"product {M}x{N}x{K} {tile}")


@pytest.mark.parametrize("z_out,lo,hi", RANGES)
@pytest.mark.parametrize("edge", [False, True])
@pytest.mark.parametrize("asym", [False, True])
@pytest.mark.parametrize("variant,stride,C,H,W", [("0", 1, 20, 9, 13), ("0", 2, 8, 12, 11), ("3", 1, 48, 9, 33), ("3", 2, 32, 11, 61)])
def test_depthwise(z_out, lo, hi, edge, asym, variant, stride, C, H, W):
    rng = np.random.default_rng(C + H + W + z_out)
    x = rng.integers(0, 256, (2, H, W, C)).astype(np.uint8)
    w = rng.integers(-20, 21, (3, 3, C)).astype(np.int8)
    mult, shift = _params(C, edge, rng)
    bias = _bias(C, shift, rng)
    zw = rng.integers(-3, 4, C).astype(np.int32)
    qnn.tuning_set("QNN_DW_VARIANT", variant)
    try:
        if asym:
            want = oracle.qdwconv2d(x, 31, w, (stride, stride), (1, 1), mult, shift, z_out, lo, hi, bias=bias, z_w=zw)
            got = host(qnn.qdwconv2d_asym(dev(x), 31, dev(w), dev(zw), (stride, stride), (1, 1), dev(mult), dev(shift), z_out, lo, hi, bias=dev(bias)))
        else:
            want = oracle.qdwconv2d(x, 31, w, (stride, stride), (1, 1), mult, shift, z_out, lo, hi, bias=bias)
            got = host(qnn.qdwconv2d(dev(x), 31, dev(w), (stride, stride), (1, 1), dev(mult), dev(shift), z_out, lo, hi, bias=dev(bias)))
    finally:
        qnn.tuning_set("QNN_DW_VARIANT")
    assert_same(got, want, f"depthwise {variant} {C}")


@pytest.mark.parametrize("z_out,lo,hi", RANGES)
@pytest.mark.parametrize("edge", [False, True])
@pytest.mark.parametrize("k,cout", [(3, 32), (7, 48)])
def test_stem(z_out, lo, hi, edge, k, cout):
    rng = np.random.default_rng(k + z_out)
    x = rng.integers(0, 256, (2, 37, 45, 3)).astype(np.uint8)
    w = rng.integers(-8, 9, (cout, k, k, 3)).astype(np.int8)
    mult, shift = _params(cout, edge, rng)
    bias = _bias(cout, shift, rng)
    want = oracle.qconv2d(x, 90, w, (2, 2), (k // 2, k // 2), mult, shift, z_out, lo, hi, bias=bias)
    got = host(qnn.qconv2d(dev(x), 90, dev(w), (2, 2), (k // 2, k // 2), dev(mult), dev(shift), z_out, lo, hi, bias=dev(bias)))
    assert_same(got, want, f"stem {k}")


@pytest.mark.parametrize("z_out,lo,hi", RANGES)
@pytest.mark.parametrize("mult_o,shift_o", [(1 << 30, 18), ((1 << 31) - 1, 20), ((1 << 30) - 1, 18), (1 << 30, 22)])
def test_table_of_code_pairs(z_out, lo, hi, mult_o, shift_o):
    """The 65536-entry table of the add (2^24 outputs and more): all pairs of codes, in a product that passes its codes on"""
    M, N, K = 65536, 256, 16
    A = np.zeros((M, K), np.uint8)
    A[:, 0] = np.arange(M) & 255
    B = np.zeros((N, K), np.int8)
    B[:, 0] = 64
    R = ((np.arange(M) >> 8)[:, None] + np.arange(N)[None, :]).astype(np.uint8)
    mult, shift = np.full(N, 1 << 30, np.int32), np.full(N, 5, np.int32) # 64 x / 64
    p = dict(left_shift=20, mult_a=1 << 30, shift_a=1, mult_b=(1 << 31) - 1, shift_b=1, mult_o=mult_o, shift_o=shift_o)
    mid = np.broadcast_to(A[:, :1], (M, N))
    # codes pass through with z_mid = 0
    want = oracle.qadd(np.ascontiguousarray(mid), 0, R, 5, p, z_out, lo, hi)
    got = host(qnn.qgemm_add(dev(A), 0, dev(B), dev(mult), dev(shift), 0, 0, 255, dev(R), 5, p, z_out, lo, hi))
    assert_same(got, want, "pairs")


SMALL = [((1 << 30) - 1, 9), (5, 3), (0, 1), (-(1 << 30), 9), (1 << 29, 20), (-(1 << 31), 12), (1 << 30, 9), ((1 << 31) - 1, 10)]


def _small_params(n, rng):
    """Shifts inside the fused forms' range, multipliers of any size and sign: channels beyond N aside, all waves meet both kinds"""
    pick = [SMALL[i] for i in rng.integers(0, len(SMALL), n)]
    return np.array([p[0] for p in pick], np.int32), np.array([p[1] for p in pick], np.int32)


@pytest.mark.parametrize("z_out,lo,hi", RANGES)
@pytest.mark.parametrize("kind", ["few", "shortk", "shortk8", "bres", "tile64", "dma128", "dma256", "p256x128", "staged", "patch", "patch2",
                                  "matrix", "matrix2", "patch_asym", "matrix_asym", "stem", "stem7"])
def test_multipliers_below_the_encoding(kind, z_out, lo, hi):
    """Multipliers that are no encoding of a real number in [0.5, 1): the tie term's form does not take them"""
    rng = np.random.default_rng(z_out + lo + len(kind))
    products = dict(few=(9, 48, 64, ""), shortk=(2085, 272, 64, ""), shortk8=(1063, 272, 200, ""), bres=(33000, 80, 288, ""), tile64=(700, 190, 320, "dma64x64"),
                    dma128=(300, 272, 320, "dma128x128"), dma256=(300, 272, 320, "dma256x256"), p256x128=(257, 144, 320, "p256x128"),
                    staged=(200, 80, 72, "64x64"))
    if kind in products:
        M, N, K, tile = products[kind]
        A, B = rng.integers(0, 256, (M, K)).astype(np.uint8), rng.integers(-2, 3, (N, K)).astype(np.int8)
        mult, shift = _small_params(N, rng)
        bias = _bias(N, shift, rng)
        rows = np.arange(M) if M < 4000 else np.sort(rng.choice(M, 500, replace=False))
        want = oracle.qgemm(A[rows], 77, B, mult, shift, z_out, lo, hi, bias=bias)
        if tile:
            qnn.tuning_set("QNN_FORCE_TILE", tile)
        try:
            got = host(qnn.qgemm(dev(A), 77, dev(B), dev(mult), dev(shift), z_out, lo, hi, bias=dev(bias)))[rows]
        finally:
            qnn.tuning_set("QNN_FORCE_TILE")
    elif kind.startswith("stem"):
        k, cout = (7, 48) if kind == "stem7" else (3, 32)
        x, w = rng.integers(0, 256, (2, 37, 45, 3)).astype(np.uint8), rng.integers(-8, 9, (cout, k, k, 3)).astype(np.int8)
        mult, shift = _small_params(cout, rng)
        bias = _bias(cout, shift, rng)
        want = oracle.qconv2d(x, 90, w, (2, 2), (k // 2, k // 2), mult, shift, z_out, lo, hi, bias=bias)
        got = host(qnn.qconv2d(dev(x), 90, dev(w), (2, 2), (k // 2, k // 2), dev(mult), dev(shift), z_out, lo, hi, bias=dev(bias)))
    else:
        s, C = (2 if "2" in kind else 1), (48 if "matrix" in kind else 20)
        x, w = rng.integers(0, 256, (2, 11, 61, C)).astype(np.uint8), rng.integers(-20, 21, (3, 3, C)).astype(np.int8)
        mult, shift = _small_params(C, rng)
        bias = _bias(C, shift, rng)
        zw = rng.integers(-3, 4, C).astype(np.int32)
        qnn.tuning_set("QNN_DW_VARIANT", "3" if "matrix" in kind else "0")
        try:
            if "asym" in kind:
                want = oracle.qdwconv2d(x, 31, w, (s, s), (1, 1), mult, shift, z_out, lo, hi, bias=bias, z_w=zw)
                got = host(qnn.qdwconv2d_asym(dev(x), 31, dev(w), dev(zw), (s, s), (1, 1), dev(mult), dev(shift), z_out, lo, hi, bias=dev(bias)))
            else:
                want = oracle.qdwconv2d(x, 31, w, (s, s), (1, 1), mult, shift, z_out, lo, hi, bias=bias)
                got = host(qnn.qdwconv2d(dev(x), 31, dev(w), (s, s), (1, 1), dev(mult), dev(shift), z_out, lo, hi, bias=dev(bias)))
        finally:
            qnn.tuning_set("QNN_DW_VARIANT")
    assert_same(got, want, kind)
