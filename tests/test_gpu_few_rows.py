"""Few-row products (M <= 64) at the edges of their kernel: rows per load, partial K-steps, rows shorter than one
load, misaligned pitches, both weight widths, activation zero-points with and without the column-sum term."""
import numpy as np
import pytest
import torch

import oracle
import paper_1806_08342_amd as qnn
from workloads import synth

from gpu_util import assert_same, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,K", [(1, 1, 2), (1, 16, 14), (8, 5, 130), (9, 17, 128), (16, 1001, 256), (17, 33, 254), (32, 48, 1026),
                                   (33, 15, 2050), (64, 31, 2304), (64, 130, 384), (7, 40, 4222), (12, 100, 6400)])
def test_few_rows_any_k(M, N, K, bits):
    c = synth.gemm_case(M, N, K, 7 * M + N + K, oracle, weight_bits=bits)
    rng = np.random.default_rng(M + K)
    bias = rng.integers(-5000, 5000, N).astype(np.int32)
    for z_a in (128, 3):
        want = oracle.qgemm(c["A"], z_a, c["Bt"], c["mult"], c["shift"], c["z_out"], 0, 255, bias=bias)
        got = qnn.qgemm(dev(c["A"]), z_a, dev(c.get("Bt_packed", c["Bt"])), dev(c["mult"]), dev(c["shift"]), c["z_out"], 0, 255,
                        bias=dev(bias), weight_bits=bits)
        assert_same(host(got), want, f"few rows {M}x{N}x{K} bits={bits} z_a={z_a}")


def test_few_rows_misaligned_row_pitch():
    M, N, K = 20, 70, 515
    c = synth.gemm_case(M, N, K, 99, oracle)
    wide = torch.zeros((M, K + 6), dtype=torch.uint8, device="cuda:0")
    wide[:, 3:3 + K] = dev(c["A"])
    out = torch.full((M, N + 5), 9, dtype=torch.uint8, device="cuda:0")
    qnn.qgemm(wide[:, 3:3 + K], c["z_a"], dev(c["Bt"]), dev(c["mult"]), dev(c["shift"]), c["z_out"], 0, 255, out=out[:, 1:1 + N])
    assert_same(host(out[:, 1:1 + N].contiguous()), oracle.qgemm(c["A"], c["z_a"], c["Bt"], c["mult"], c["shift"], c["z_out"], 0, 255), "slices")
    assert bool((out[:, 0] == 9).all()) and bool((out[:, 1 + N:] == 9).all())


@pytest.mark.parametrize("small", ["1", "0"])
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,K", [(65, 16, 64), (300, 130, 256), (1000, 40, 72), (97, 100, 514), (800, 256, 1152), (129, 90, 2306),
                                   (200, 70, 16), (333, 50, 48), (90, 33, 176), (70, 20, 1056),  # partial K-steps of whole 16-byte pieces
                                   (6272, 64, 384), (6145, 60, 352), (6144, 64, 384), (1570, 250, 512)])  # around 768 workgroups of 4-bit weights
def test_small_launches_and_the_kernels_they_replace(tuning, small, M, N, K, bits):
    tuning.setenv("QNN_SMALL", small)
    c = synth.gemm_case(M, N, K, 11 * M + K, oracle, weight_bits=bits)
    bias = np.random.default_rng(N).integers(-5000, 5000, N).astype(np.int32)
    for z_a in (128, 250):
        want = oracle.qgemm(c["A"], z_a, c["Bt"], c["mult"], c["shift"], c["z_out"], 0, 255, bias=bias)
        got = qnn.qgemm(dev(c["A"]), z_a, dev(c.get("Bt_packed", c["Bt"])), dev(c["mult"]), dev(c["shift"]), c["z_out"], 0, 255,
                        bias=dev(bias), weight_bits=bits)
        assert_same(host(got), want, f"small={small} {M}x{N}x{K} bits={bits} z_a={z_a}")
