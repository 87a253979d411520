"""Victims beside work the library does not start itself: the time they
report, the work-groups that fit beside them, and what they wait for."""
import ctypes as C

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(dev):
    from paper_2501_16909_amd import coloc
    c = coloc.Context(0)
    yield c
    c.close()


def _triad(ctx, dev, n):
    import torch
    b, c = torch.rand(n, device=dev), torch.rand(n, device=dev)
    return ctx.triad_desc(b, c, torch.empty_like(b))


# A stressor handle of intensity 0 launches nothing, so a run beside it is the
# same run: its time and its window [t_begin, t_end] come from the same events
# and stamps, alone and beside sweeps queued on another stream.  Medians of 400
# runs in turn; a run alone spreads by 4 % (p10 to p90), one beside sweeps
# depends by a factor of two on where in a sweep it starts, which is drawn
# here from two sweeps' time (its median then by 5 %).
@pytest.mark.parametrize("beside,tol", [(False, 0.05), (True, 0.25)])
def test_victim_time_is_one_quantity(ctx, dev, monkeypatch, beside, tol):
    import random
    import time

    import torch
    rng = random.Random(5)
    d, sweep = _triad(ctx, dev, 1 << 20), _triad(ctx, dev, 1 << 24)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device=dev)
    side = torch.cuda.Stream(device=dev)
    times, windows = ([], []), ([], [])
    torch.cuda.synchronize()
    monkeypatch.setattr(ctx, "_sync_torch", lambda: None)    # skipped beside a handle: the same calls in both
    for i in range(800):
        held = i % 2
        if held:
            h = ctx.stressor("hbm", 0.0, ws=ws)
        if beside:
            ctx.victim_enqueue(sweep, side, 14)
            until = time.perf_counter() + rng.random() * 60e-6
            while time.perf_counter() < until:
                pass
        r = ctx.victim_run(d)
        if held:
            h.stop()
        side.synchronize()
        times[held].append(r.time_ns)
        windows[held].append(r.t_end - r.t_begin)
    (t0, t1), (w0, w1) = map(np.median, times), map(np.median, windows)
    assert abs(t0 / t1 - 1) < tol, (t0, t1)
    assert abs(w0 / w1 - 1) < 2 * tol, (w0, w1)


def test_victim_window_is_stamped(ctx, dev):
    """Both ends of the window are device clock readings in the victim's own
    stream: later than a stamp that finished before the call, apart by at
    least the victim's time."""
    import torch
    d = _triad(ctx, dev, 1 << 24)
    ticks = torch.zeros(2, dtype=torch.int64, device=dev)
    side = torch.cuda.Stream(device=dev)
    for _ in range(50):
        ctx.stamp(ticks[0:1], side)
        side.synchronize()
        r = ctx.victim_run(d)
        ctx.stamp(ticks[1:2], side)
        side.synchronize()
        before, after = ticks.cpu().tolist()
        assert before <= r.t_begin <= r.t_end <= after
        assert (r.t_end - r.t_begin) * 1e6 / ctx.info.wall_clock_khz >= r.time_ns


# GEMMs of fewer than 256 tiles of 256 x 256 leave room on their CUs for a
# work-group that holds 64 KiB of LDS, and the largest of them for the cache
# stressor's waves: the slowdown beside such a work-group on every CU is that
# of sharing the CU (2 to 5), not the stressor's lifetime (100 ms, a hundred
# times the longest of these kernels).
@pytest.mark.parametrize("dtype,n", [("bf16", 2048), ("bf16", 2888), ("bf16", 3328), ("bf16", 3840), ("fp8", 3328),
                                     ("fp8", 3712), ("f32", 3072), ("f32", 3584)])
def test_gemm_shares_cus_with_lds_holders(ctx, dev, dtype, n):
    import torch
    x = torch.randn((n, n), device=dev)
    a = {"f32": lambda: x, "bf16": lambda: x.to(torch.bfloat16).view(torch.int16),
         "fp8": lambda: x.to(torch.float8_e4m3fn).view(torch.uint8)}[dtype]()
    d = ctx.gemm_desc(a, a.clone(), torch.empty((n, n), device=dev), dtype, n, n, n, 1.0, 1.0)
    win = torch.from_numpy(synth.u32(7, 8192).view(np.int32)).to(dev)
    l1 = torch.zeros(4096, dtype=torch.int32, device=dev)
    for res, opts in (("lds", dict(src0=win)), ("occupancy", dict(knob=64)), ("vl1d", dict(src0=l1, n=4096))):
        cell, = ctx.measure_sensitivity(d, [res], [opts], [1.0], reps=3, warmups=1, deadline_ms=100)
        assert cell["slowdown"] < 15, (res, cell["slowdown"])


# ------------------------------------------------ the caller's stream
def _calls(ctx, dev):
    """One call of each way into the library that takes a stream: name -> function
    of the stream, giving its output."""
    import torch
    d = _triad(ctx, dev, 1 << 20)
    w = torch.from_numpy(oracle.f32_to_bf16(synth.uniform_f32(1, 64 * 512)).view(np.int16)).to(dev).view(64, 512)
    v = w[:2].contiguous()
    q = torch.rand((1, 4, 128), device=dev)
    kv = w.reshape(1, 2, 128, 128)
    out = torch.empty((1, 512), dtype=torch.int16, device=dev)

    def on(s, f):
        old, ctx.stream = ctx.stream, s
        try:
            return f()
        finally:
            ctx.stream = old

    return {"victim": lambda s: ctx.victim_run(d, stream=s).checksum_bits,
            "gemv_rows": lambda s: on(s, lambda: ctx.gemv_bf16_rows(w, v).clone()),
            "attention": lambda s: on(s, lambda: ctx.attention_decode_noalloc(q, kv, kv, [100], 4, 2, 128, 128, out).clone())}


@pytest.mark.parametrize("name", ["victim", "gemv_rows", "attention"])
def test_captured_streams_are_refused(ctx, dev, monkeypatch, name):
    """A call that waits for its work cannot be part of a capture: on the
    capturing stream it is refused, and the capture and later calls go on.
    Beside a relaxed capture, calls on other streams work."""
    import torch
    from paper_2501_16909_amd import coloc
    call = _calls(ctx, dev)[name]
    hip = coloc.load_library()       # its dependencies' symbols too
    begin, end = hip.hipStreamBeginCapture, hip.hipStreamEndCapture
    begin.argtypes, end.argtypes = [C.c_void_p, C.c_int], [C.c_void_p, C.POINTER(C.c_void_p)]
    other = torch.cuda.Stream(device=dev)
    want = call(other)
    torch.cuda.synchronize()
    monkeypatch.setattr(ctx, "_sync_torch", lambda: None)    # waits, which a capture forbids
    for mode, same in ((1, True), (2, True), (2, False)):    # thread-local, relaxed
        side, graph = torch.cuda.Stream(device=dev), C.c_void_p()
        assert begin(side.cuda_stream, mode) == 0
        try:
            if same:
                with pytest.raises(coloc.CiError):
                    call(side)
            else:
                call(other)
        finally:
            ended = end(side.cuda_stream, C.byref(graph))
        got = call(side if same else other)
        assert ended == 0 and hip.hipGraphDestroy(graph) == 0
        assert torch.equal(got, want) if torch.is_tensor(want) else got == want


@pytest.mark.parametrize("name", ["victim", "gemv_rows"])
def test_calls_wait_for_the_callers_stream(ctx, dev, name):
    """Operands that a busy stream is still to write: the call given that
    stream reads them written."""
    import torch
    n = 1 << 20
    sweep = _triad(ctx, dev, 1 << 26)
    side = torch.cuda.Stream(device=dev)
    new = torch.rand(n, device=dev)
    old = torch.zeros_like(new)
    if name == "victim":
        c, out = torch.rand(n, device=dev), torch.empty(n, device=dev)
        d = ctx.triad_desc(old, c, out)
        ctx.victim_run(d)
    else:
        w = torch.ones((64, 512), device=dev).to(torch.bfloat16).view(torch.int16)
        v, new = old[:512].to(torch.bfloat16).view(1, 512), new[:512].to(torch.bfloat16).view(1, 512)
        out = torch.empty((1, 64), device=dev)
        ctx.gemv_bf16_rows(w, v.view(torch.int16), out=out)
    assert not torch.equal(new, old if name == "victim" else v)
    torch.cuda.synchronize()
    ctx.victim_enqueue(sweep, side, 200)              # about 30 ms
    with torch.cuda.stream(side):
        (old if name == "victim" else v).copy_(new)
    assert not side.query()
    if name == "victim":
        ctx.victim_run(d, stream=side)
        want = oracle.triad_f32(new.cpu().numpy(), c.cpu().numpy())
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32))
    else:
        keep, ctx.stream = ctx.stream, side
        try:
            ctx.gemv_bf16_rows(w, v.view(torch.int16), out=out)
        finally:
            ctx.stream = keep
        total = float(new.double().sum())             # 512 products in FP32
        assert np.all(np.abs(out.cpu().numpy() - total) <= 512 * 2.0 ** -24 * total)


def test_stream_of_another_device_is_refused(ctx, dev):
    import torch
    from paper_2501_16909_amd import coloc
    if torch.cuda.device_count() < 2:
        pytest.skip("needs two GPUs")
    with pytest.raises(coloc.CiError):
        ctx.victim_run(_triad(ctx, dev, 1 << 20), stream=torch.cuda.Stream(device=1))
