"""GPU parity of the weight-resident kernel for matrices with its rows in an LDS ring (bres_ring.h): three and six slots, and weights
that leave no room for three (200 columns with K = 768: bres.h), one to four column blocks, the last block of rows whole, partial and missing, row-spaced operands, outputs that are no whole chunks."""
import numpy as np
import pytest
import torch

import oracle
import paper_1806_08342_amd as qnn

from gpu_util import assert_same, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [4096, 4129, 70003])
@pytest.mark.parametrize("N,K", [(24, 320), (64, 512), (128, 512), (200, 768), (256, 1024), (72, 384), (200, 448), (160, 512)])
@pytest.mark.parametrize("bits", [8, 4])
def test_rows_through_the_ring(tuning, M, N, K, bits):
    tuning.setenv("QNN_BRES", "1")  # shapes this small take the kernel only on request
    rng = np.random.default_rng(M + N + K + bits)
    lim = 8 if bits == 4 else 128
    A = rng.integers(0, 256, (M, K)).astype(np.uint8)
    B = rng.integers(-lim, lim, (N, K)).astype(np.int8)
    B = oracle.pack_int4(B) if bits == 4 else B
    mult, shift = oracle.quantize_multipliers(10 ** rng.uniform(-4.0, -3.4, N) * (16 if bits == 4 else 1))
    bias = rng.integers(-20000, 20000, N).astype(np.int32)
    rows = np.unique(np.r_[0:40, M - 140:M, rng.integers(0, M, 200)])
    wide = torch.zeros((M, K + 16), dtype=torch.uint8, device="cuda:0")
    wide[:, :K] = dev(A)
    out = torch.full((M, N + 5), 77, dtype=torch.uint8, device="cuda:0")
    for z_a, z_out, lo in ((0, 0, 0), (128, 120, 3)):
        want = oracle.qgemm(A[rows], z_a, B, mult, shift, z_out, lo, 250, bias=bias, weight_bits=bits)
        got = host(qnn.qgemm(dev(A), z_a, dev(B), dev(mult), dev(shift), z_out, lo, 250, bias=dev(bias), weight_bits=bits))
        assert_same(got[rows], want, f"{M}x{N}x{K} z_a={z_a}")
        qnn.qgemm(wide[:, :K], z_a, dev(B), dev(mult), dev(shift), z_out, lo, 250, bias=dev(bias), weight_bits=bits, out=out[:, 3:3 + N])
        got = host(out)
        assert_same(got[rows, 3:3 + N], want, f"{M}x{N}x{K} z_a={z_a} with pitches")
        assert (got[:, :3] == 77).all() and (got[:, 3 + N:] == 77).all(), "bytes beside the output"
