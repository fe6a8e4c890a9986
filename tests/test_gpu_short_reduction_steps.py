"""GPU parity of the short-K kernel (shortk.h) at every number of K sub-steps it has a form for, whole and partial last
ones, with one block of rows per wave and with several."""
import numpy as np
import pytest

import oracle
import paper_1806_08342_amd as qnn

from gpu_util import assert_same, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [16, 40, 64, 72, 80, 96, 112, 128, 136, 160, 176, 192, 200, 208, 224, 232, 240, 256])
@pytest.mark.parametrize("M,N", [(65, 33), (3001, 80), (70001, 48)])
@pytest.mark.parametrize("bits", [8, 4])
def test_every_number_of_sub_steps(K, M, N, bits):
    rng = np.random.default_rng(K + M + N + bits)
    A = rng.integers(0, 256, (M, K)).astype(np.uint8)
    B = rng.integers(-8 if bits == 4 else -128, 8 if bits == 4 else 128, (N, K)).astype(np.int8)
    mult, shift = oracle.quantize_multipliers(10 ** rng.uniform(-3.9, -3.2, N) * (16 if bits == 4 else 1))
    bias = rng.integers(-20000, 20000, N).astype(np.int32)
    zw = rng.integers(-8 if bits == 4 else -100, 8 if bits == 4 else 101, N).astype(np.int32)
    R = rng.integers(0, 256, (M, N)).astype(np.uint8)
    p = oracle.qadd_params(0.02, 0.031, 0.04)
    Bo = oracle.pack_int4(B) if bits == 4 else B
    rows = np.arange(M) if M < 100 else np.unique(np.r_[0:40, M - 40:M, rng.integers(0, M, 200)])
    dA, dB, dm, ds, db = dev(A), dev(Bo), dev(mult), dev(shift), dev(bias)
    for z_a in (128, 9):
        want = oracle.qgemm(A[rows], z_a, Bo, mult, shift, 120, 0, 255, bias=bias, weight_bits=bits)
        got = host(qnn.qgemm(dA, z_a, dB, dm, ds, 120, 0, 255, bias=db, weight_bits=bits))
        assert_same(got[rows], want, f"plain z_a={z_a}")
        got = host(qnn.qgemm_add(dA, z_a, dB, dm, ds, 120, 0, 255, dev(R), 7, p, 3, 0, 255, bias=db, weight_bits=bits))
        assert_same(got[rows], oracle.qadd(want, 120, R[rows], 7, p, 3, 0, 255), f"add z_a={z_a}")
        want = oracle.qgemm(A[rows], z_a, Bo, mult, shift, 120, 0, 255, bias=bias, weight_bits=bits, z_w=zw)
        got = host(qnn.qgemm_asym(dA, z_a, dB, dev(zw), dm, ds, 120, 0, 255, bias=db, weight_bits=bits))
        assert_same(got[rows], want, f"asym z_a={z_a}")
