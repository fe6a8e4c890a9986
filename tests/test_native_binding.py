"""The compiled binding: argument checks that need no GPU, and (on a GPU) allocation, caller-owned outputs and errors."""
import os
import re
import threading

import numpy as np
import pytest
import torch

import oracle
import paper_1806_08342_amd as qnn
from paper_1806_08342_amd import binding

from gpu_util import assert_same, dev, host


def test_binding_names_match_the_compiled_module():
    mod = binding._native()
    for name in ("quantize", "dequantize", "requantize", "qgemm", "qconv2d", "qdwconv2d", "qadd", "qgemm_add", "qconv2d_add",
                 "qgemm_asym", "qconv2d_asym", "qdwconv2d_asym", "minmax", "quantize_dynamic", "simquant", "rescale_u8", "pack_b"):
        assert callable(getattr(mod, name)) and callable(getattr(qnn, name))


@pytest.mark.parametrize("bad", [None, 3, np.zeros(4, np.float32), torch.zeros(4), torch.zeros(4, dtype=torch.float64)])
def test_tensors_of_the_wrong_kind_raise_type_errors(bad):
    with pytest.raises(TypeError):
        qnn.quantize(bad, 1.0, 0)
    with pytest.raises(TypeError):
        qnn.qgemm(bad, 0, bad, bad, bad, 0, 0, 255)


def test_pack_b_looks_at_the_tensor_before_it_allocates():
    with pytest.raises(TypeError):
        qnn.pack_b(torch.zeros(4, 4, dtype=torch.int8))


def test_nothing_that_throws_runs_without_the_interpreter_lock():
    # an exception between the two macros would leave the lock given up; and the library is C, the stream query is not
    src = open(os.path.join(os.path.dirname(binding.__file__), "csrc", "binding.cpp")).read()
    assert "Py_BEGIN_ALLOW_THREADS" not in src and "~Unlocked() { PyEval_RestoreThread" in src
    calls = re.findall(r'call\("qnn_\w+", \[&\](.*?)\}\);', src, re.S)
    assert len(calls) > 20 and all(c.startswith("(void *s)") and "stream()" not in c for c in calls)


@pytest.mark.gpu
def test_calls_follow_the_thread_s_own_stream():
    # several threads at once, each on a stream of its own
    x = torch.randn(1 << 16, device="cuda:0")
    want = oracle.quantize(x.cpu().numpy(), 0.03, 120)
    bad = []

    def work():
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.default_stream())
        with torch.cuda.stream(stream):
            outs = [qnn.quantize(x, 0.03, 120) for _ in range(50)]
        stream.synchronize()
        bad.extend(i for i, o in enumerate(outs) if not np.array_equal(o.cpu().numpy(), want))

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


@pytest.mark.gpu
def test_outputs_shapes_and_status_errors():
    x = torch.randn(5, 7, device="cuda:0")
    out = torch.empty(5, 7, dtype=torch.uint8, device="cuda:0")
    assert qnn.quantize(x, 0.1, 3, out=out) is out
    assert_same(host(out), oracle.quantize(x.cpu().numpy(), 0.1, 3), "caller's output")
    with pytest.raises(ValueError, match="shape"):
        qnn.quantize(x, 0.1, 3, out=out[:4])
    with pytest.raises(qnn.QnnError, match="QNN_EINVAL"):
        qnn.quantize(x, 0.0, 3)
    with pytest.raises(TypeError):
        qnn.quantize(x, 0.1, 3.5)
    w = dev(np.zeros((4, 3, 3, 8), np.int8))
    one = dev(np.full(4, 1 << 30, np.int32))
    img = torch.zeros(1, 6, 6, 8, dtype=torch.uint8, device="cuda:0")
    assert tuple(qnn.qconv2d(img, 0, w, [2, 1], [1, 0], one, dev(np.ones(4, np.int32)), 0, 0, 255).shape) == (1, 3, 4, 4)
    with pytest.raises(qnn.QnnError):
        qnn.qconv2d(img, 0, dev(np.zeros((4, 9, 9, 8), np.int8)), (1, 1), (0, 0), one, one, 0, 0, 255)
    assert qnn.quantize(x[:0], 0.1, 3).shape == (0, 7)


@pytest.mark.gpu
def test_numbers_that_int_takes():
    # these four convert with int(): zero-points and ranges that come as floats, numpy scalars or tensors
    x = torch.randn(1000, device="cuda:0")
    g = torch.randn(1000, device="cuda:0")
    q = qnn.quantize(x, 0.02, 120).view(10, 100)
    mult, shift = oracle.quantize_multiplier(0.7)
    for conv in (float, np.float32, np.int64, torch.tensor):
        z, lo, hi = conv(120), conv(3), conv(250)
        assert torch.equal(qnn.simquant(x, 0.02, z, lo, hi), qnn.simquant(x, 0.02, 120, 3, 250))
        assert torch.equal(qnn.simquant_backward(x, g, 0.02, z, lo, hi), qnn.simquant_backward(x, g, 0.02, 120, 3, 250))
        assert torch.equal(qnn.rescale_u8(q, z, mult, conv(shift), conv(128), lo, hi), qnn.rescale_u8(q, 120, mult, shift, 128, 3, 250))
        assert torch.equal(qnn.minmax(x, qnn.new_range_state(), 0.0, conv(8)), qnn.minmax(x, qnn.new_range_state(), 0.0, 8))
    with pytest.raises((TypeError, ValueError)):
        qnn.simquant(x, 0.02, "no number")


@pytest.mark.gpu
def test_depthwise_weights_of_one_channel_without_a_channel_dimension():
    rng = np.random.default_rng(3)
    x = rng.integers(0, 256, (2, 9, 8, 1)).astype(np.uint8)
    w = rng.integers(-128, 128, (3, 3)).astype(np.int8)
    mult, shift = oracle.quantize_multipliers([0.002])
    z_w = np.array([5], np.int32)
    args = (dev(mult), dev(shift), 120, 0, 255)
    want = oracle.qdwconv2d(x, 7, w[:, :, None], (1, 1), (1, 1), mult, shift, 120, 0, 255)
    assert_same(host(qnn.qdwconv2d(dev(x), 7, dev(w), (1, 1), (1, 1), *args)), want, "symmetric")
    want = oracle.qdwconv2d(x, 7, w[:, :, None], (1, 1), (1, 1), mult, shift, 120, 0, 255, z_w=z_w)
    assert_same(host(qnn.qdwconv2d_asym(dev(x), 7, dev(w), dev(z_w), (1, 1), (1, 1), *args)), want, "weight zero-point")
    with pytest.raises(TypeError):
        qnn.qdwconv2d(dev(x), 7, dev(w[0]), (1, 1), (1, 1), *args)


@pytest.mark.gpu
def test_tensors_too_small_for_the_call_are_refused():
    # (raised before anything is launched)
    x = torch.randn(6, 50, device="cuda:0")
    q = qnn.quantize(x, 0.02, 120)
    small, small_codes = x[:5].contiguous(), q[:5].contiguous()
    p = qnn.qadd_params(0.02, 0.03, 0.05)
    for bad in (lambda: qnn.dequantize(q, 0.02, 120, out=small), lambda: qnn.simquant(x, 0.02, 120, out=small),
                lambda: qnn.simquant_backward(x, x, 0.02, 120, out=small), lambda: qnn.simquant_backward(x, small, 0.02, 120),
                lambda: qnn.qadd(q, 120, small_codes, 120, p, 120, 0, 255)):
        with pytest.raises(ValueError, match="shape"):
            bad()
    # any tensor that holds the elements still does
    flat = torch.empty(300, device="cuda:0")
    assert qnn.dequantize(q, 0.02, 120, out=flat) is flat and torch.equal(flat.view(6, 50), qnn.dequantize(q, 0.02, 120))
    assert torch.equal(qnn.simquant_backward(x, x.view(-1), 0.02, 120), qnn.simquant_backward(x, x, 0.02, 120))
    assert torch.equal(qnn.qadd(q, 120, q.view(-1), 120, p, 120, 0, 255), qnn.qadd(q, 120, q, 120, p, 120, 0, 255))


@pytest.mark.gpu
def test_products_run_where_their_scratch_does_not_fit():
    rng = np.random.default_rng(5)
    M, N, K = 3000, 1500, 4099
    A, B = dev(rng.integers(0, 256, (M, K)).astype(np.uint8)), dev(rng.integers(-128, 128, (N, K)).astype(np.int8))
    mult, shift = (dev(v) for v in oracle.quantize_multipliers(rng.uniform(40.0, 120.0, N) / (K * 255.0 * 128)))
    assert qnn.qgemm_workspace_bytes(M, N, K) > (M + N) * K
    want = qnn.qgemm(A, 9, B, mult, shift, 120, 0, 255)
    out, z_w = torch.zeros_like(want), torch.zeros(N, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    filler = []
    try:
        torch.cuda.set_per_process_memory_fraction(1e-6)  # no new memory from here on ...
        with pytest.raises(torch.cuda.OutOfMemoryError):
            while True:  # ... nor what the allocator still holds
                filler.append(torch.empty(4 << 20, dtype=torch.uint8, device="cuda:0"))
        qnn.qgemm(A, 9, B, mult, shift, 120, 0, 255, out=out)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert_same(host(out), host(want), "without scratch")
    assert_same(host(qnn.qgemm_asym(A, 9, B, z_w, mult, shift, 120, 0, 255)), host(want), "afterwards")
