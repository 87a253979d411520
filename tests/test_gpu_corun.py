"""Victims beside work the library does not start itself: the time they
report, the work-groups that fit beside them, and what they wait for."""
import numpy as np
import pytest

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
# and stamps, alone and beside sweeps queued on another stream.  Medians of 200
# runs in turn; a run alone spreads by 4 % (p10 to p90), one beside sweeps
# depends on where in a sweep it starts (a factor of two, 0.2 of its median
# over 200 runs at the most).
@pytest.mark.parametrize("beside,tol", [(False, 0.05), (True, 0.25)])
def test_victim_time_is_one_quantity(ctx, dev, beside, tol):
    import torch
    d, sweep = _triad(ctx, dev, 1 << 20), _triad(ctx, dev, 1 << 24)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device=dev)
    side = torch.cuda.Stream(device=dev)
    times, windows = ([], []), ([], [])
    for i in range(400):
        held = i % 2
        if held:
            h = ctx.stressor("hbm", 0.0, ws=ws)
        if beside:
            ctx.victim_enqueue(sweep, side, 12)
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
    import synth
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
