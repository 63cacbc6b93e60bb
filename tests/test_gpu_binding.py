"""The binding's native fast path against its Python path: the same results and the same objects on plain calls, the same exceptions
on the others."""
import sys
import threading
import time

import numpy as np
import pytest
import torch

from paper_2506_04985_amd import binding as fptq

pytestmark = pytest.mark.gpu


@pytest.fixture
def both(monkeypatch):
    """run(f) -> f's results on the native path and on the Python path."""
    fptq.lib()
    assert fptq._native is not None

    def run(f):
        native = f()
        with monkeypatch.context() as m:
            m.setattr(fptq, "_native", None)
            python = f()
        return native, python
    return run


def data(M=40, N=72, K=1024):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    x = (torch.randn((M, K), device="cuda", generator=g) * 1.3).to(torch.bfloat16)
    w = torch.randint(-8, 8, (N, K), dtype=torch.int8, device="cuda", generator=g)
    return x, w, torch.rand(N, device="cuda", generator=g) * 0.015 + 0.005, torch.rand(M, device="cuda", generator=g) + 0.5


def same(a, b):
    if isinstance(a, tuple):
        assert isinstance(b, tuple) and len(a) == len(b)
        for p, q in zip(a, b):
            same(p, q)
    elif a is None:
        assert b is None
    else:
        assert a.dtype == b.dtype and a.shape == b.shape and a.device == b.device
        assert torch.equal(a.contiguous().view(-1).view(torch.uint8), b.contiguous().view(-1).view(torch.uint8))


@pytest.mark.parametrize("M", [1, 40, 300])
def test_every_call_gives_the_same(both, M):
    N, K = 72, 1024
    x, w, s, r = data(M, N, K)
    wq, sums, xq = fptq.fptq_pack_weights(w), fptq.fptq_weight_row_sums(w), fptq.fptq_quantize_act(x, 0.4, 2, 0.0, r)[0]
    calls = [lambda: fptq.fptq_pack_weights(w), lambda: fptq.fptq_weight_row_sums(w),
             lambda: fptq.fptq_quantize_act(x, 0.4, fptq.SCALE_RMS, 1e-5), lambda: fptq.fptq_quantize_act(x, 1, 2, 0, r, want_row_scale=False),
             lambda: fptq.fptq_quantize_act(x, np.float32(0.4), 0), lambda: fptq.fptq_quantize_act_hadamard(x, 0.4, 512, 2, 0.0, r),
             lambda: fptq.fptq_quantize_act_asym(x, 0.4, -3), lambda: fptq.fptq_quantize_act_dynamic(x),
             lambda: fptq.fptq_residual_norm_quantize(x, x, 0.4, r, 1e-5), lambda: fptq.fptq_residual_norm_quantize(x, x, 0.4),
             lambda: fptq.fptq_w4a4_linear(xq, wq, M, N, K, 0.4, s), lambda: fptq.fptq_w4a4_linear(xq, wq, M, N, K, 0.4, s, r, want_acc=True),
             lambda: fptq.fptq_w4a4_linear_zp(xq, wq, M, N, K, 0.4, s, 5, sums, r, want_acc=True),
             lambda: fptq.fptq_w4a4_linear_noalloc(xq, wq, M, N, K, 0.4, s, want_acc=True),
             lambda: fptq.fptq_w4a4_linear_ws(xq, wq, M, N, K, 0.4, s, None), lambda: fptq.fptq_w4a4_linear(xq, wq, np.int64(M), N, K, 0.4, s)]
    for f in calls:
        same(*both(f))


def test_split_k_workspace_shapes(both):
    M, N, K = 256, 512, 6272
    x, w, s, r = data(M, N, K)
    wq, xq = fptq.fptq_pack_weights(w), fptq.fptq_quantize_act(x, 0.4, 2, 0.0, r)[0]
    need = fptq.fptq_linear_workspace_bytes(M, N, K)
    assert need > 0
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
    same(*both(lambda: fptq.fptq_w4a4_linear_ws(xq, wq, M, N, K, 0.4, s, ws, r)))
    same(*both(lambda: fptq.fptq_w4a4_linear(xq, wq, M, N, K, 0.4, s, r)))


@pytest.mark.parametrize("M,N,K", [(2048, 22016, 4096), (1000, 5120, 13824)])
def test_scratch_shapes(both, M, N, K):
    """Calls that bring scratch along, on either path, give what the call without any gives; captured, they go without."""
    assert fptq.fptq_linear_scratch_bytes(M, N, K) > 0 and fptq.fptq_linear_workspace_bytes(M, N, K) == 0
    x, w, s, r = data(M, N, K)
    wq, sums = fptq.fptq_pack_weights(w), fptq.fptq_weight_row_sums(w)
    xq, xz = fptq.fptq_quantize_act(x, 0.4, 2, 0.0, r)[0], fptq.fptq_quantize_act_asym(x, 0.4, 3, 2, 0.0, r)[0]
    ws = torch.zeros(256, dtype=torch.uint8, device="cuda")
    want = fptq.fptq_w4a4_linear_noalloc(xq, wq, M, N, K, 0.4, s, r)
    for f in (lambda: fptq.fptq_w4a4_linear(xq, wq, M, N, K, 0.4, s, r), lambda: fptq.fptq_w4a4_linear_ws(xq, wq, M, N, K, 0.4, s, ws, r),
              lambda: fptq.fptq_w4a4_linear_ws(xq, wq, M, N, K, 0.4, s, None, r), lambda: fptq.fptq_w4a4_linear_zp(xq, wq, M, N, K, 0.4, s, 0, sums, r)):
        native, python = both(f)
        same(native, want), same(python, want)
    fptq.fptq_set_linear_prefill(2)
    want_z = fptq.fptq_w4a4_linear_zp(xz, wq, M, N, K, 0.4, s, 3, sums, r, want_acc=True)
    fptq.fptq_set_linear_prefill(0)
    native, python = both(lambda: fptq.fptq_w4a4_linear_zp(xz, wq, M, N, K, 0.4, s, 3, sums, r, want_acc=True))
    same(native, want_z), same(python, want_z)
    y, yz = torch.zeros_like(want), torch.zeros_like(want)
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        fptq.fptq_w4a4_linear(xq, wq, M, N, K, 0.4, s, r, out=y)
        fptq.fptq_w4a4_linear_zp(xz, wq, M, N, K, 0.4, s, 3, sums, r, out=yz)
    for _ in range(3):
        y.zero_(), yz.zero_()
        graph.replay()
        torch.cuda.synchronize()
        same(y, want), same(yz, want_z[0])


def test_without_memory_for_scratch_the_call_goes_without(both):
    M, N, K = 8192, 8192, 8192
    assert fptq.fptq_linear_scratch_bytes(M, N, K) > 32 << 20                 # more than what the segments in use can have left
    xq, wq = (torch.randint(0, 256, (fptq.fptq_packed_bytes(n, K),), dtype=torch.uint8, device="cuda") for n in (M, N))
    s = torch.rand(N, device="cuda") * 0.015 + 0.005
    want = fptq.fptq_w4a4_linear_noalloc(xq, wq, M, N, K, 0.4, s)
    outputs = [torch.zeros_like(want) for _ in range(2)]
    left = iter(outputs)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    failed = lambda: torch.cuda.memory_stats()["num_ooms"]
    before = failed()
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (8 << 20)) / torch.cuda.get_device_properties(0).total_memory)
    try:
        both(lambda: fptq.fptq_w4a4_linear(xq, wq, M, N, K, 0.4, s, out=next(left)))
        assert failed() == before + 2
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert all(torch.equal(y, want) for y in outputs)


def test_given_outputs_are_filled_and_returned():
    M, N, K = 40, 72, 1024
    x, w, s, r = data(M, N, K)
    out, ro = torch.empty(fptq.fptq_packed_bytes(M, K), dtype=torch.uint8, device="cuda"), torch.empty(M, device="cuda")
    a, b = fptq.fptq_quantize_act(x, 0.4, 2, 0.0, r, out=out, row_scale_out=ro, want_row_scale=False)
    assert a is out and b is ro and torch.equal(ro, r)
    wo = torch.empty(fptq.fptq_packed_bytes(N, K), dtype=torch.uint8, device="cuda")
    assert fptq.fptq_pack_weights(w, out=wo) is wo
    y, acc = torch.empty((M, N), dtype=torch.bfloat16, device="cuda"), torch.empty((M, N), dtype=torch.int32, device="cuda")
    assert fptq.fptq_w4a4_linear(out, wo, M, N, K, 0.4, s, out=y) is y
    a, b = fptq.fptq_w4a4_linear(out, wo, M, N, K, 0.4, s, out=y, acc=acc)
    assert a is y and b is acc
    xn, sn = torch.empty_like(x), torch.empty(M, device="cuda")
    t = fptq.fptq_residual_norm_quantize(x, x, 0.4, None, 1e-5, xn, sn, out)
    assert t[0] is xn and t[1] is sn and t[2] is out


def test_what_was_refused_is_refused(both):
    M, N, K = 40, 72, 1024
    x, w, s, r = data(M, N, K)
    wq, xq = fptq.fptq_pack_weights(w), fptq.fptq_quantize_act(x, 0.4, 2, 0.0, r)[0]
    small = torch.empty(64, dtype=torch.uint8, device="cuda")
    calls = [lambda: fptq.fptq_quantize_act(x.float(), 0.4), lambda: fptq.fptq_quantize_act(x.t(), 0.4), lambda: fptq.fptq_quantize_act(x.cpu(), 0.4),
             lambda: fptq.fptq_quantize_act(x, -0.4), lambda: fptq.fptq_quantize_act(x, 0.4, 7), lambda: fptq.fptq_quantize_act(x, 0.4, 2),
             lambda: fptq.fptq_quantize_act(x, 0.4, out=small), lambda: fptq.fptq_quantize_act(x[0], 0.4), lambda: fptq.fptq_quantize_act(x, 0.4, 2, 0.0, r.double()),
             lambda: fptq.fptq_quantize_act_hadamard(x, 0.4, 128), lambda: fptq.fptq_quantize_act_asym(x, 0.4, 8),
             lambda: fptq.fptq_w4a4_linear(xq, wq, M, N, K, 0.4, s.double()), lambda: fptq.fptq_w4a4_linear(xq, wq, M + 1, N, K, 0.4, s),
             lambda: fptq.fptq_w4a4_linear(xq, wq, 0, N, K, 0.4, s), lambda: fptq.fptq_w4a4_linear(xq, wq, M, N, K, float("nan"), s),
             lambda: fptq.fptq_w4a4_linear(xq, wq, M, N, K, 0.4, s[:N - 1]), lambda: fptq.fptq_w4a4_linear_zp(xq, wq, M, N, K, 0.4, s, 0, None),
             lambda: fptq.fptq_w4a4_linear_zp(xq, wq, M, N, K, 0.4, s, 9, torch.zeros(N, dtype=torch.int32, device="cuda")),
             lambda: fptq.fptq_pack_weights(w.short()), lambda: fptq.fptq_pack_weights(w, out=small), lambda: fptq.fptq_weight_row_sums(w[:, ::2]),
             lambda: fptq.fptq_w4a4_linear_ws(xq, wq, M, N, K, 0.4, s, torch.zeros(512, dtype=torch.uint8, device="cuda")[64:])]

    def raised(f):
        try:
            f()
        except Exception as e:
            return type(e), str(e)
        return None
    for i, f in enumerate(calls):
        a, b = both(lambda: raised(f))
        assert a is not None and a == b, i


def test_none_is_no_value_for_a_block_or_a_zero_point(both):
    """None is not "no transform" or "symmetric grid": the calls that need a number refuse it on either path."""
    M, N, K = 40, 72, 1024
    x, w, s, r = data(M, N, K)
    wq, sums, xq = fptq.fptq_pack_weights(w), fptq.fptq_weight_row_sums(w), fptq.fptq_quantize_act(x, 0.4, 2, 0.0, r)[0]
    for f in (lambda: fptq.fptq_quantize_act_hadamard(x, 0.4, hadamard_block=None, row_scale_in=r), lambda: fptq.fptq_quantize_act_asym(x, 0.4, None),
              lambda: fptq.fptq_w4a4_linear_zp(xq, wq, M, N, K, 0.4, s, None, sums)):
        def refused():
            with pytest.raises(TypeError):
                f()
            return True
        assert both(refused) == (True, True)


@pytest.mark.parametrize("call", ["fptq_w4a4_linear", "fptq_w4a4_linear_zp", "fptq_w4a4_linear_ws", "fptq_w4a4_linear_noalloc"])
def test_a_refusal_names_the_call_that_was_made(both, call):
    """Whatever memory the wrapper would have brought along, the message is that of the entry point of the wrapper's name."""
    M, N, K = 2048, 22016, 4096
    assert fptq.fptq_linear_scratch_bytes(M, N, K) > 0
    xq, wq = (torch.empty(fptq.fptq_packed_bytes(rows, K), dtype=torch.uint8, device="cuda") for rows in (M, N))
    s, sums = torch.ones(N, device="cuda"), torch.zeros(N, dtype=torch.int32, device="cuda")
    more = {"fptq_w4a4_linear_zp": (3, sums), "fptq_w4a4_linear_ws": (None,)}.get(call, ())

    def message():
        with pytest.raises(fptq.FptqError) as e:
            getattr(fptq, call)(xq, wq, M, N, K, -1.0, s, *more)
        return str(e.value)
    assert both(message) == 2 * (f"FPTQ_ERR_VALUE: {call}: s_a must be finite and > 0",)


def test_other_threads_run_during_a_call():
    """The interpreter lock is free while the library launches.  With a switch interval of minutes a thread that wants it gets in only
    where a call lets go of it, at the latest where the queue is full and a launch waits for room."""
    x, _, _, r = data(2048, 8, 11008)
    out = fptq.fptq_quantize_act(x, 0.4, 2, 0.0, r, want_row_scale=False)[0]
    turns, stop, interval = [0], threading.Event(), sys.getswitchinterval()

    def other():
        while not stop.is_set():
            turns[0] += 1
            time.sleep(0)
    thread = threading.Thread(target=other)
    sys.setswitchinterval(600)
    try:
        thread.start()
        before, calls = turns[0], 0
        while turns[0] == before and calls < 40000:
            fptq.fptq_quantize_act(x, 0.4, 2, 0.0, r, out=out, want_row_scale=False)
            calls += 1
        seen = turns[0] > before
    finally:
        sys.setswitchinterval(interval)
        stop.set()
        thread.join()
        torch.cuda.synchronize()
    assert seen, calls


def test_runs_on_the_current_stream():
    """A call inside a side stream's context waits for what that stream did before."""
    M, N, K = 40, 72, 1024
    x, w, s, r = data(M, N, K)
    wq, want = fptq.fptq_pack_weights(w), fptq.fptq_quantize_act(x, 0.4, 2, 0.0, r)[0]
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        big = torch.randn((4096, 4096), device="cuda")
        for _ in range(20):
            big = big @ big * 1e-3
        late = x.clone()
        got = fptq.fptq_quantize_act(late, 0.4, 2, 0.0, r)[0]
    side.synchronize()
    assert torch.equal(got, want)
