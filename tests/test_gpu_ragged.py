"""Products and convolutions whose sizes divide nothing: K that is no multiple of 64 (chunks beyond K), rows that are no
whole 16-byte chunks (zero-padded copies in the workspace, and the route without a workspace), stems on images of any
width."""
import numpy as np
import pytest
import torch

import oracle
import paper_1806_08342_amd as qnn
import workloads
from workloads import synth

from gpu_util import assert_same, dev, host

pytestmark = pytest.mark.gpu


def _gemm(M, N, K, bits, z_a, workspace=None, seed=0):
    c = synth.gemm_case(M, N, K, 5000 + M + N + K + seed, oracle, weight_bits=bits)
    bias = np.random.default_rng(K).integers(-9000, 9000, N).astype(np.int32)
    want = oracle.qgemm(c["A"], z_a, c["Bt"], c["mult"], c["shift"], c["z_out"], 0, 255, bias=bias)
    got = qnn.qgemm(dev(c["A"]), z_a, dev(c.get("Bt_packed", c["Bt"])), dev(c["mult"]), dev(c["shift"]), c["z_out"], 0, 255,
                    bias=dev(bias), weight_bits=bits, workspace=workspace)
    assert_same(host(got), want, f"{M}x{N}x{K} bits={bits} z_a={z_a}")


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,K", [(65, 1001, 1026), (129, 64, 608), (200, 333, 1040), (257, 130, 2082), (100, 700, 96), (1021, 501, 338),
                                   (700, 520, 800), (66, 2000, 8000), (1300, 700, 1031 * 2)])
def test_ragged_products(M, N, K, bits):
    for z_a in (128, 7):
        _gemm(M, N, K, bits, z_a)


def test_ragged_product_without_room_for_copies():
    K = 1027
    assert qnn.qgemm_workspace_bytes(1200, 700, K) >= (1200 + 700) * 1040
    _gemm(1200, 700, K, 8, 3, workspace=torch.empty(256, dtype=torch.uint8, device="cuda:0"))


@pytest.mark.parametrize("M,N,K", [(4100, 4100, 272), (5000, 2500, 1040), (70000, 100, 304), (2600, 2600, 784)])
def test_ragged_products_on_the_large_tiles(M, N, K):
    # too large for the oracle as a whole: the first, middle and last rows
    c = synth.gemm_case(M, N, K, 6000 + M, oracle)
    rows = np.r_[0:8, M // 2:M // 2 + 8, M - 8:M]
    want = oracle.qgemm(c["A"][rows], 9, c["Bt"], c["mult"], c["shift"], c["z_out"], 0, 255)
    got = qnn.qgemm(dev(c["A"]), 9, dev(c["Bt"]), dev(c["mult"]), dev(c["shift"]), c["z_out"], 0, 255)
    assert_same(host(got[torch.from_numpy(rows).to("cuda:0")]), want, f"{M}x{N}x{K}")


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("batch,H,W,cin,cout,k,s", [(1, 7, 7, 512, 130, 3, 1), (2, 14, 13, 36, 70, 3, 1), (3, 9, 11, 30, 33, 3, 2), (1, 28, 28, 32, 32, 3, 1),
                                                   (4, 15, 15, 144, 100, 3, 1), (2, 20, 20, 270, 64, 1, 2), (8, 12, 12, 302, 190, 1, 1), (40, 30, 31, 48, 130, 3, 1)])
def test_convolutions_with_any_channel_count(batch, H, W, cin, cout, k, s, bits):
    layer = workloads.Layer("t", "conv", H, W, cin, cout, k=k, stride=s, pad=k // 2, act="relu6", weight_bits=bits)
    c = synth.conv_case(layer, batch, 7000 + cin + cout, oracle)
    for z_x in (c["z_x"], 131):
        want = oracle.qconv2d(c["x"], z_x, c["w"], c["stride"], c["pad"], c["mult"], c["shift"], c["z_out"], c["act_min"], c["act_max"], bias=c["bias"])
        got = qnn.qconv2d(dev(c["x"]), z_x, dev(c.get("w_packed", c["w"])), c["stride"], c["pad"], dev(c["mult"]), dev(c["shift"]), c["z_out"],
                          c["act_min"], c["act_max"], bias=dev(c["bias"]), weight_bits=bits)
        assert_same(host(got), want, f"conv {batch}x{H}x{W}x{cin}->{cout} k{k} s{s} bits={bits} z_x={z_x}")


@pytest.mark.parametrize("H,W,cin,k,stride", [(20, 33, 3, 3, 2), (9, 2, 3, 3, 1), (30, 131, 3, 7, 2), (21, 70, 1, 3, 1), (16, 65, 2, 7, 2), (12, 101, 3, 3, 2)])
def test_stems_of_any_width(H, W, cin, k, stride):
    layer = workloads.Layer("t", "conv", H, W, cin, 40, k=k, stride=stride, pad=k // 2, act="relu")
    c = synth.conv_case(layer, 3, 7100 + W, oracle, in_range=(-2.0, 2.2))
    # a misaligned image as well: one byte into a larger buffer
    buf = torch.zeros(c["x"].size + 1, dtype=torch.uint8, device="cuda:0")
    buf[1:] = dev(c["x"]).view(-1)
    want = oracle.qconv2d(c["x"], c["z_x"], c["w"], c["stride"], c["pad"], c["mult"], c["shift"], c["z_out"], c["act_min"], c["act_max"], bias=c["bias"])
    for x in (dev(c["x"]), buf[1:].view(c["x"].shape)):
        got = qnn.qconv2d(x, c["z_x"], dev(c["w"]), c["stride"], c["pad"], dev(c["mult"]), dev(c["shift"]), c["z_out"], c["act_min"], c["act_max"],
                          bias=dev(c["bias"]))
        assert_same(host(got), want, f"stem {H}x{W}x{cin} k{k} s{stride}")


@pytest.mark.parametrize("z_a", [128, 7])
def test_split_products_with_a_partial_last_step(z_a):
    # the last of the K ranges ends in a partial step
    assert qnn.qgemm_workspace_bytes(66, 2000, 8016) > 0
    _gemm(66, 2000, 8016, 8, z_a)


@pytest.mark.parametrize("bits,K", [(8, 528), (8, 1056), (8, 1072), (4, 544), (4, 1056)])
@pytest.mark.parametrize("tile", ["dma64x64", "dma128x128", "dma256x256", "dma256x128", "dma256x64"])
def test_every_pipelined_tile_with_a_partial_step(tuning, tile, bits, K):
    tuning.setenv("QNN_FORCE_TILE", tile)
    _gemm(300, 270, K, bits, 9)
    if bits == 8 and tile in ("dma64x64", "dma128x128"):
        tuning.setenv("QNN_FORCE_SPLIT", "3")
        assert qnn.qgemm_workspace_bytes(300, 270, K) > 0
        _gemm(300, 270, K, bits, 9)


@pytest.mark.parametrize("tile", ["dma64x64", "dma128x128", "dma256x256", "dma256x128", "dma256x64"])
@pytest.mark.parametrize("bits,cin,split", [(8, 48, 1), (8, 112, 2), (4, 32, 1), (4, 96, 1)])
def test_convolutions_on_every_pipelined_tile_with_a_partial_step(tuning, tile, bits, cin, split):
    tuning.setenv("QNN_FORCE_TILE", tile)
    tuning.setenv("QNN_FORCE_SPLIT", str(split))
    layer = workloads.Layer("t", "conv", 13, 15, cin, 130, k=3, stride=1, pad=1, act="relu6", weight_bits=bits)
    c = synth.conv_case(layer, 2, 7300 + cin, oracle)
    assert (9 * cin) % 64 != 0
    for z_x in (c["z_x"], 131):
        want = oracle.qconv2d(c["x"], z_x, c["w"], c["stride"], c["pad"], c["mult"], c["shift"], c["z_out"], c["act_min"], c["act_max"], bias=c["bias"])
        got = qnn.qconv2d(dev(c["x"]), z_x, dev(c.get("w_packed", c["w"])), c["stride"], c["pad"], dev(c["mult"]), dev(c["shift"]), c["z_out"],
                          c["act_min"], c["act_max"], bias=dev(c["bias"]), weight_bits=bits)
        assert_same(host(got), want, f"{tile} bits={bits} cin={cin} z_x={z_x}")


@pytest.mark.parametrize("M,N,K", [(2600, 2100, 352), (5000, 2300, 544)])  # 4-bit weights on the 128x128 and 256x256 tiles by default
def test_ragged_4bit_products_on_the_large_tiles(M, N, K):
    c = synth.gemm_case(M, N, K, 6100 + M, oracle, weight_bits=4)
    rows = np.r_[0:8, M // 2:M // 2 + 8, M - 8:M]
    want = oracle.qgemm(c["A"][rows], 9, c["Bt"], c["mult"], c["shift"], c["z_out"], 0, 255)
    got = qnn.qgemm(dev(c["A"]), 9, dev(c["Bt_packed"]), dev(c["mult"]), dev(c["shift"]), c["z_out"], 0, 255, weight_bits=4)
    assert_same(host(got[torch.from_numpy(rows).to("cuda:0")]), want, f"{M}x{N}x{K}")
