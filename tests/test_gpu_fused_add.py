"""GPU parity of the add fused behind a product (qnn_qgemm_add / qnn_qconv2d_add): the expected
value is the oracle's layer followed by the oracle's rescaling add -- no arithmetic of its own.
Every route of the dispatcher is forced once: kernels that apply the add on the way out of their
LDS tile (short-K, pipelined and staged tiles) and kernels followed by the in-place second pass."""
import numpy as np
import pytest
import torch

import oracle
import paper_1806_08342_amd as qnn
import workloads
from workloads import synth

from gpu_util import assert_same, dev, host

pytestmark = pytest.mark.gpu


def _add_setup(rng, shape, act="relu", odd=False):
    """Residual tensor + add parameters; `odd` picks scales that leave the fused 32-bit form."""
    R = rng.integers(0, 256, shape).astype(np.uint8)
    z_mid = int(rng.integers(90, 170))
    z_r = int(rng.integers(0, 256))
    if odd:
        s_mid, s_r, s_o = 0.03, 0.041, 0.3  # shift_o = 22: beyond the fused 32-bit form, the general output rescale
    else:
        s_mid = float(rng.uniform(0.02, 0.05))
        s_r = s_mid * float(rng.uniform(0.5, 2.0))
        s_o = float(rng.uniform(0.03, 0.08))
    z_o = 0 if act == "relu" else int(rng.integers(100, 150))
    lo, hi = (z_o, 255) if act == "relu" else (0, 255)
    return R, z_mid, z_r, oracle.qadd_params(s_mid, s_r, s_o), z_o, lo, hi


def _gemm_inputs(rng, M, N, K, bits=8):
    A = rng.integers(0, 256, (M, K)).astype(np.uint8)
    lim = 8 if bits == 4 else 128
    Bt = rng.integers(-lim, lim, (N, K)).astype(np.int8)
    real = 10 ** rng.uniform(-4.2, -3.2, N) / np.sqrt(K / 64.0) * (16.0 if bits == 4 else 1.0)
    mult, shift = oracle.quantize_multipliers(real)
    bias = rng.integers(-20000, 20000, N).astype(np.int32)
    return A, Bt, bias, mult, shift


def _check_gemm_add(M, N, K, seed, what, bits=8, odd=False, act="relu", mid=(0, 255), z_a=None):
    rng = np.random.default_rng(seed)
    A, Bt, bias, mult, shift = _gemm_inputs(rng, M, N, K, bits)
    R, z_mid, z_r, p, z_o, lo, hi = _add_setup(rng, (M, N), act, odd)
    z_a = int(rng.integers(0, 256)) if z_a is None else z_a
    Bo = oracle.pack_int4(Bt) if bits == 4 else Bt
    t = oracle.qgemm(A, z_a, Bo, mult, shift, z_mid, mid[0], mid[1], bias=bias, weight_bits=bits)
    want = oracle.qadd(t, z_mid, R, z_r, p, z_o, lo, hi)
    got = host(qnn.qgemm_add(dev(A), z_a, dev(Bo), dev(mult), dev(shift), z_mid, mid[0], mid[1], dev(R), z_r, p, z_o, lo, hi,
                             bias=dev(bias), weight_bits=bits))
    assert_same(got, want, what)
    assert len(np.unique(want)) > 8, "parity would be vacuous"
    return A, Bo, bias, mult, shift, R, z_a, z_mid, z_r, p, z_o, lo, hi, want


@pytest.mark.parametrize("M,N,K", [(300, 130, 64), (1000, 256, 128), (4099, 512, 256), (97, 48, 32), (2048, 64, 96),
                                   (500, 200, 72)])  # K = 72: no 16-byte rows, the add runs as a second pass
@pytest.mark.parametrize("bits", [8, 4])
def test_qgemm_add_short_k(M, N, K, bits):
    assert qnn.qgemm_plan(M, N, K) == "shortk"
    _check_gemm_add(M, N, K, 4000 + M + N + K + bits, f"qgemm_add short-K {M}x{N}x{K} bits={bits}", bits=bits)
    _check_gemm_add(M, N, K, 4100 + M + N + K + bits, f"qgemm_add short-K {M}x{N}x{K} bits={bits}, general add rescale",
                    bits=bits, odd=True, act="none")


@pytest.mark.parametrize("M,N,K,bits", [(70001, 256, 64, 8), (33000, 512, 160, 4)])
def test_qgemm_add_pair_table(M, N, K, bits):
    # from 2^24 outputs on, the short-K kernel combines the two codes through a 65536-entry table
    assert M * N >= 2 ** 24 and qnn.qgemm_plan(M, N, K) == "shortk"
    _check_gemm_add(M, N, K, 4150 + K, f"qgemm_add pair table {M}x{N}x{K} bits={bits}", bits=bits, mid=(2, 251))
    _check_gemm_add(M, N, K, 4160 + K, f"qgemm_add pair table {M}x{N}x{K} bits={bits}, general add rescale", bits=bits, odd=True,
                    act="none")


@pytest.mark.parametrize("alds", [2, 1, 0])
@pytest.mark.parametrize("M,N,K,bits", [(1000, 512, 128, 8), (4099, 520, 256, 8), (133, 1030, 128, 4), (2500, 256, 256, 4),
                                         (9100, 320, 32, 8), (5000, 64, 128, 4), (70001, 24, 16, 4),  # tables of rescaled codes, on the ring kernel
                                         # 2^24 outputs: the table of code pairs
                                         (262200, 128, 64, 8), (131080, 256, 48, 4),  # 8 waves, each on rows of its own
                                         (16400, 1024, 256, 8),   # 8 waves, four side by side
                                         (24000, 720, 208, 4), (120000, 144, 192, 8),  # the same, and too few columns for it
                                         (33000, 1024, 128, 4), (33001, 512, 112, 8),  # 16 waves, eight side by side
                                         (82001, 208, 128, 8),    # 16 waves, four side by side
                                         (60003, 288, 104, 4)])   # no rows of whole 16-byte pieces
def test_qgemm_add_short_k_rows_through_lds(tuning, alds, M, N, K, bits):
    # short-K products with the add in either kernel: the one with its rows in an LDS ring wherever it has a form (2), by shape (1),
    # always the one with fragments from global memory (0); operands that are no whole aligned chunks take a second pass
    tuning.setenv("QNN_SHORTK_ALDS", str(alds))
    assert qnn.qgemm_plan(M, N, K) == "shortk"
    _check_gemm_add(M, N, K, 4300 + M + N + K + bits, f"qgemm_add short-K route={alds} {M}x{N}x{K} bits={bits}", bits=bits)
    _check_gemm_add(M, N, K, 4400 + M + N + K + bits, f"qgemm_add short-K route={alds} {M}x{N}x{K} bits={bits}, general add rescale",
                    bits=bits, odd=True, act="none")


@pytest.mark.parametrize("tile", ["dma128x128", "dma256x256", "dma256x64", "dma256x128", "dma128x128s3", "dma64x64",
                                  "dma256x64s3", "128x128", "64x64"])
@pytest.mark.parametrize("M,N,K", [(300, 270, 512), (513, 130, 320)])
def test_qgemm_add_every_tile(tuning, tile, M, N, K):
    tuning.setenv("QNN_FORCE_TILE", tile)
    _check_gemm_add(M, N, K, 4200 + M + K, f"qgemm_add tile={tile} {M}x{N}x{K}", mid=(3, 250))
    _check_gemm_add(M, N, K, 4300 + M + K, f"qgemm_add tile={tile} {M}x{N}x{K}, general add rescale", odd=True, act="none")


def test_qgemm_add_default_routes():
    # tiles chosen by the cost model, split-K, few rows, 4-bit weights through the unpack pass
    for (M, N, K, bits) in [(2048, 2048, 512, 8), (256, 512, 8192, 8), (16, 256, 512, 8), (64, 4096, 1024, 8),
                            (1500, 384, 1024, 4), (12544, 2048, 512, 8)]:
        _check_gemm_add(M, N, K, 4400 + M + N, f"qgemm_add {M}x{N}x{K} bits={bits} plan={qnn.qgemm_plan(M, N, K)}", bits=bits)


def test_qgemm_add_weight_resident(tuning):
    tuning.setenv("QNN_BRES", "1")
    _check_gemm_add(4500, 64, 512, 4500, "qgemm_add weight-resident kernel + second pass")


def test_qgemm_add_spaced_rows_and_unaligned_residual():
    # output and residual are column slices of wider matrices; the residual starts at an odd byte
    rng = np.random.default_rng(4600)
    M, N, K = 700, 96, 128
    A, Bt, bias, mult, shift = _gemm_inputs(rng, M, N, K)
    Rw, z_mid, z_r, p, z_o, lo, hi = _add_setup(rng, (M, N + 37))
    R = Rw[:, 5:5 + N]
    t = oracle.qgemm(A, 77, Bt, mult, shift, z_mid, 0, 255, bias=bias)
    want = oracle.qadd(t, z_mid, np.ascontiguousarray(R), z_r, p, z_o, lo, hi)
    Cw = torch.zeros((M, N + 16), dtype=torch.uint8, device="cuda:0")
    for r_dev, what in [(dev(Rw)[:, 5:5 + N], "odd offset"), (dev(np.ascontiguousarray(R)), "dense")]:
        out = Cw[:, 16:]
        qnn.qgemm_add(dev(A), 77, dev(Bt), dev(mult), dev(shift), z_mid, 0, 255, r_dev, z_r, p, z_o, lo, hi, bias=dev(bias),
                      out=out)
        assert_same(host(out.contiguous()), want, f"qgemm_add spaced rows, residual {what}")
    assert int(Cw[:, :16].max()) == 0


CONV_ADD_SHAPES = [
    # H, W, Cin, Cout, k, stride, pad, bits
    (14, 14, 64, 256, 1, 1, 0, 8),     # last 1x1 of a bottleneck: short-K
    (14, 14, 512, 2048, 1, 1, 0, 8),   # K = 512: tiles
    (28, 28, 64, 96, 1, 2, 0, 8),      # strided 1x1
    (12, 12, 32, 64, 3, 1, 1, 8),      # 3x3 convolution through the tile kernel
    (14, 14, 96, 24, 1, 1, 0, 4),      # MobileNetV2-style linear bottleneck, 4-bit weights
    (20, 20, 3, 32, 3, 2, 1, 8),       # stem kernel + second pass
    (9, 9, 20, 30, 3, 1, 1, 8),        # nothing aligned
]


@pytest.mark.parametrize("shape", CONV_ADD_SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("batch", [1, 5])
def test_qconv2d_add_matches_oracle(shape, batch):
    H, W, Cin, Cout, k, s, p_, bits = shape
    layer = workloads.Layer("t", "conv", H, W, Cin, Cout, k=k, stride=s, pad=p_, act="none", weight_bits=bits)
    c = synth.conv_case(layer, batch, 4700 + sum(shape) + batch, oracle)
    w_o = c.get("w_packed", c["w"])
    t = oracle.qconv2d(c["x"], c["z_x"], w_o, c["stride"], c["pad"], c["mult"], c["shift"], c["z_out"], c["act_min"],
                       c["act_max"], bias=c["bias"], weight_bits=bits)
    rng = np.random.default_rng(4800 + sum(shape))
    R, _, z_r, p, z_o, lo, hi = _add_setup(rng, t.shape)
    want = oracle.qadd(t, c["z_out"], R, z_r, p, z_o, lo, hi)
    got = host(qnn.qconv2d_add(dev(c["x"]), c["z_x"], dev(w_o), c["stride"], c["pad"], dev(c["mult"]), dev(c["shift"]),
                               c["z_out"], c["act_min"], c["act_max"], dev(R), z_r, p, z_o, lo, hi, bias=dev(c["bias"]),
                               weight_bits=bits))
    assert_same(got, want, f"qconv2d_add {shape} batch {batch}")
    assert len(np.unique(want)) > 8


def test_fused_add_equals_two_calls_on_the_gpu():
    # the documented identity, checked on the device side as well: layer into a temporary, then qnn_qadd
    A, Bo, bias, mult, shift, R, z_a, z_mid, z_r, p, z_o, lo, hi, want = _check_gemm_add(900, 256, 64, 4900, "identity case")
    t = qnn.qgemm(dev(A), z_a, dev(Bo), dev(mult), dev(shift), z_mid, 0, 255, bias=dev(bias))
    two = host(qnn.qadd(t, z_mid, dev(R), z_r, p, z_o, lo, hi))
    assert_same(two, want, "qgemm then qadd")


def _launches(fn):
    """Number of nodes that `fn` leaves in a captured graph."""
    import ctypes

    fn()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        fn()
    n = ctypes.c_size_t()
    assert ctypes.CDLL("libamdhip64.so").hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


# rows per workgroup 8, 16, 32 and 64; 4, 8 and 16 waves; N and K that are no multiple of 4; misaligned residual rows
@pytest.mark.parametrize("M,N,K,bits", [(1, 16, 64, 8), (8, 33, 2048, 8), (9, 21, 1030, 4), (16, 64, 4096, 4), (31, 47, 129, 8), (50, 4099, 300, 8),
                                        (64, 4112, 514, 4), (65, 18, 2304, 8), (97, 66, 6000, 4), (333, 35, 77, 8), (1570, 162, 960, 4), (3137, 25, 144, 4),
                                        (1571, 127, 1000, 8)])
def test_small_launches_add_in_one_kernel(M, N, K, bits):
    rng = np.random.default_rng(M + N + K)
    A, Bt, bias, mult, shift = _gemm_inputs(rng, M, N, K, bits)
    Bo = oracle.pack_int4(Bt) if bits == 4 else Bt
    for odd, act, spaced in ((False, "relu", 0), (False, "none", 3), (True, "none", 5)):
        Rw, z_mid, z_r, p, z_o, lo, hi = _add_setup(rng, (M, N + spaced), act, odd)
        R = Rw[:, spaced:]
        t = oracle.qgemm(A, 77, Bo, mult, shift, z_mid, 2, 252, bias=bias, weight_bits=bits)
        want = oracle.qadd(t, z_mid, np.ascontiguousarray(R), z_r, p, z_o, lo, hi)
        out = torch.full((M, N + spaced), 9, dtype=torch.uint8, device="cuda:0")
        args = [dev(v) for v in (A, Bo, mult, shift, Rw, bias)]

        def run():
            qnn.qgemm_add(args[0], 77, args[1], args[2], args[3], z_mid, 2, 252, args[4][:, spaced:], z_r, p, z_o, lo, hi, bias=args[5],
                          weight_bits=bits, out=out[:, spaced:])

        assert _launches(run) == 1
        out.fill_(9)
        run()
        assert_same(host(out[:, spaced:].contiguous()), want, f"{M}x{N}x{K} bits={bits} odd={odd} spaced={spaced}")
        assert spaced == 0 or bool((out[:, :spaced] == 9).all())
    assert M == 1 or len(np.unique(want)) > 8


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("batch,H,W,cin,cout,k,s", [(1, 7, 7, 512, 130, 3, 1), (2, 9, 11, 32, 33, 3, 2), (1, 28, 28, 32, 32, 3, 1), (2, 20, 20, 272, 63, 1, 2)])
def test_small_convolutions_add_in_one_kernel(batch, H, W, cin, cout, k, s, bits):
    layer = workloads.Layer("t", "conv", H, W, cin, cout, k=k, stride=s, pad=k // 2, act="none", weight_bits=bits)
    c = synth.conv_case(layer, batch, 4950 + cin + cout, oracle)
    w_o = c.get("w_packed", c["w"])
    t = oracle.qconv2d(c["x"], c["z_x"], w_o, c["stride"], c["pad"], c["mult"], c["shift"], c["z_out"], 0, 255, bias=c["bias"], weight_bits=bits)
    R, _, z_r, p, z_o, lo, hi = _add_setup(np.random.default_rng(cout), t.shape)
    want = oracle.qadd(t, c["z_out"], R, z_r, p, z_o, lo, hi)
    args = [dev(v) for v in (c["x"], w_o, c["mult"], c["shift"], R, c["bias"])]
    out = torch.empty(t.shape, dtype=torch.uint8, device="cuda:0")

    def run():
        qnn.qconv2d_add(args[0], c["z_x"], args[1], c["stride"], c["pad"], args[2], args[3], c["z_out"], 0, 255, args[4], z_r, p, z_o, lo, hi,
                        bias=args[5], weight_bits=bits, out=out)

    assert _launches(run) == 1
    out.fill_(9)
    run()
    assert_same(host(out), want, f"conv {batch}x{H}x{W}x{cin}->{cout} k{k} s{s} bits={bits}")
