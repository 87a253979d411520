"""Kernels at the sizes where their work division changes: remainders, the
smallest and the largest of a range, unaligned pointers."""
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


# one work-group, its last group of four, the second work-group, the last
# one that adds work-groups (1024 x 4096 words), longer ranges with a tail
@pytest.mark.parametrize("n", [0, 1, 3, 4, 1023, 4096, 4097, 8195, 1024 * 4096, 1024 * 4096 + 1, 9_000_003])
@pytest.mark.parametrize("skip", [0, 1, 3])
def test_checksum_edges(ctx, dev, n, skip):
    import torch
    h = synth.normal_f32(4242, n + skip)
    x = torch.from_numpy(h).to(dev)[skip:]
    bits, total = ctx.checksum(x)
    v = h[skip:].astype(np.float64)
    assert bits == oracle.bitsum_u32(h[skip:])
    # FP64 additions: fewer than n roundings of partial sums below sum |x|
    assert abs(total - float(np.sum(v))) <= 2 * n * 2.0 ** -53 * float(np.sum(np.abs(v)))


# less than a group of four, a tile's edge (4096), a second tile for each of
# the 1024 work-groups with a partial one behind
@pytest.mark.parametrize("n", [1, 3, 4, 4095, 4096, 4097, 12_289, 2048 * 4096 + 5])
@pytest.mark.parametrize("skip", [0, 1])
def test_quantize_edges(ctx, dev, n, skip):
    import torch
    h = (synth.normal_f32(4343, n + skip) * np.float32(37.0)).astype(np.float32)
    x = torch.from_numpy(h).to(dev)[skip:]
    codes, _ = ctx.quantize(x, "bf16")
    assert np.array_equal(codes.cpu().numpy().view(np.uint16), oracle.f32_to_bf16(h[skip:]))
    codes, s = ctx.quantize(x, "fp8")
    want, ws = oracle.quantize_fp8(h[skip:])
    assert s == ws
    assert np.array_equal(codes.cpu().numpy(), want)


def test_quantize_nan_and_inf_lanes(ctx, dev):
    """NaN in each lane of a group of four, infinities of both signs, beside
    ordinary values: the group's other elements keep their codes."""
    import torch
    h = synth.normal_f32(4444, 64)
    for i in range(4):
        h[8 * i + i] = np.float32(np.nan) if i % 2 else -np.float32(np.nan)
    x = torch.from_numpy(h).to(dev)
    nan = np.isnan(h)
    b = ctx.quantize(x, "bf16")[0].cpu().numpy().view(np.uint16)
    assert np.array_equal(b[~nan], oracle.f32_to_bf16(h)[~nan])
    assert np.array_equal(b[nan], (np.signbit(h[nan]) * np.uint16(0x8000)) | np.uint16(0x7FC0))
    codes, s = ctx.quantize(x, "fp8")
    clean = np.where(nan, np.float32(0), h)
    want, ws = oracle.quantize_fp8(clean)
    got = codes.cpu().numpy()
    assert s == ws and np.array_equal(got[~nan], want[~nan])
    assert np.array_equal(got[nan], (np.signbit(h[nan]) * np.uint8(0x80)) | np.uint8(0x7F))
    h = synth.normal_f32(4445, 64)
    h[5], h[6] = np.inf, -np.inf       # the maximum is infinite: no scaling, saturated codes
    codes, s = ctx.quantize(torch.from_numpy(h).to(dev), "fp8")
    got = codes.cpu().numpy()
    assert s == 1.0 and got[5] == 0x7E and got[6] == 0xFE
    t = oracle.e4m3_table()
    ok = np.ones(64, bool)
    ok[5:7] = False
    assert np.all(np.abs(t[got[ok]] - h[ok]) <= 2.0 ** -4 * np.abs(h[ok]) + 2.0 ** -10)


# One shape (or more) for every tiling: 64 x 64, 128 x 64, 128 x 128 and 256 x
# 256 in one round of CUs and in several, with ragged edges; K from a single
# 16-byte chunk through every remainder of a 128-byte stage to several stages.
GEMM_EDGES = ([(m, n, kb) for m, n in ((1, 1), (70, 65), (513, 300)) for kb in (16, 48, 64, 80, 112, 128, 144, 400)] +
              [(2000, 2047, kb) for kb in (32, 176, 384)] + [(2500, 2561, kb) for kb in (16, 96, 320)] +
              [(4001, 3900, kb) for kb in (64, 128, 192, 576, 1088)] +
              [(5001, 5100, kb) for kb in (64, 192, 320, 832)] + [(256, 66000, 192), (4001, 3900, 272)])


@pytest.mark.parametrize("dtype", ["f32", "bf16", "fp8"])
@pytest.mark.parametrize("m,n,kb", GEMM_EDGES)
def test_gemm_tilings(ctx, dev, dtype, m, n, kb):
    """Every entry of small products and 4096 fixed-seed entries (with the
    last row and column) of large ones, within the accumulation bound of the
    input type; nothing outside the output is written."""
    import torch
    elem = {"f32": 4, "bf16": 2, "fp8": 1}[dtype]
    k = kb // elem
    a = synth.normal_f32(5000 + m + kb, m * k).reshape(m, k)
    b = synth.normal_f32(6000 + n + kb, n * k).reshape(n, k)
    if dtype == "f32":
        qa, qb, fa, fb, s = a, b, a.astype(np.float64), b.astype(np.float64), 1.0
    elif dtype == "bf16":
        qa, qb = (oracle.f32_to_bf16(x).view(np.int16) for x in (a, b))
        fa, fb, s = oracle.bf16_to_f64(qa.view(np.uint16)), oracle.bf16_to_f64(qb.view(np.uint16)), 1.0
    else:
        (qa, sa), (qb, sb) = oracle.quantize_fp8(a), oracle.quantize_fp8(b)
        fa, fb, s = oracle.e4m3_to_f64(qa), oracle.e4m3_to_f64(qb), float(sa) * float(sb)
    fa, fb = fa.reshape(m, k), fb.reshape(n, k)
    qa, qb = qa.reshape(m, k), qb.reshape(n, k)
    guard = 64
    buf = torch.full((m * n + 2 * guard,), float("nan"), dtype=torch.float32, device=dev)
    out = buf[guard:guard + m * n]
    ctx.victim_run(ctx.gemm_desc(torch.from_numpy(np.ascontiguousarray(qa)).to(dev),
                                 torch.from_numpy(np.ascontiguousarray(qb)).to(dev), out, dtype, m, n, k,
                                 s if dtype == "fp8" else 1.0, 1.0))
    assert torch.isnan(buf[:guard]).all() and torch.isnan(buf[-guard:]).all()
    assert not torch.isnan(out).any()
    got = out.view(m, n)
    if m * n <= 1 << 18:
        rows, cols = np.repeat(np.arange(m), n), np.tile(np.arange(n), m)
    else:
        idx = synth.words(7000 + kb, 4096)
        rows, cols = (idx % np.uint64(m)).astype(np.int64), ((idx >> np.uint64(32)) % np.uint64(n)).astype(np.int64)
        rows[:64], cols[64:128] = m - 1, n - 1
    want = s * np.einsum("ij,ij->i", fa[rows], fb[cols])
    if dtype == "fp8":
        bound = np.concatenate([oracle.mfma_fp8_error_bound(qa[rows[i:i + 4096]], qb[cols[i:i + 4096]], s)
                                for i in range(0, len(rows), 4096)])
    else:
        absw = np.einsum("ij,ij->i", np.abs(fa[rows]), np.abs(fb[cols]))
        bound = oracle.accumulation_bound(k + 1, absw, 2.0 ** -23)
    g = got[torch.from_numpy(rows).to(dev), torch.from_numpy(cols).to(dev)].cpu().numpy().astype(np.float64)
    assert np.all(np.abs(g - want) <= bound + 1e-300)


# Both sides of the length from which loads are non-temporal, whole chunks of
# 256 and not, and (compared on the device) more elements than one launch has
# work-items.
@pytest.mark.parametrize("n", [255, 256, 257, (1 << 25) - 1, 1 << 25, (1 << 25) + 257, (1 << 32) + 333])
def test_triad_victim_lengths(ctx, dev, n):
    import torch
    b = torch.empty(n, dtype=torch.float32, device=dev)
    c, out = torch.empty_like(b), torch.full((n + 1,), -1.0, device=dev)
    for i, t in enumerate((b, c)):
        synth.device_fill_uniform_f32(t.data_ptr(), n, 700 + i)
    torch.cuda.synchronize()
    ctx.victim_triad(b, c, out[:n], passes=1)
    assert out[n].item() == -1.0
    for i in range(0, n, 1 << 28):
        x, y, z = (t[i:min(n, i + (1 << 28))] for t in (b, c, out))
        assert torch.equal(z, x + y * 3.0)     # two roundings in both


# Rows that end within a round of 256 chunks; the whole matrix is beyond the
# length from which weights are loaded non-temporally, its pieces are not.
@pytest.mark.parametrize("n,k", [(16391, 8200), (66000, 2056), (1 << 20, 136)])
def test_gemv_forms_agree(ctx, dev, n, k):
    import torch
    w = torch.from_numpy(oracle.f32_to_bf16(synth.uniform_f32(31, 1 << 22)).view(np.int16)).to(dev)
    w = w.repeat(-(-n * k // w.numel()))[: n * k].reshape(n, k)
    x = torch.from_numpy(oracle.f32_to_bf16(synth.uniform_f32(32, k)).view(np.int16)).to(dev)
    y, z = (torch.full((n,), float("nan"), device=dev) for _ in range(2))
    ctx.victim_run(ctx.gemv_desc(w, x, y, n, k))
    for i in range(0, n, n // 4 + 1):
        p = w[i:min(n, i + n // 4 + 1)]
        ctx.victim_run(ctx.gemv_desc(p, x, z[i:i + len(p)], len(p), k))
    assert torch.equal(y, z)


# One, two and four heads per wave, with heads left over; chunks of one, some
# and all positions.  What the caches hold past a sequence's end is not used.
@pytest.mark.parametrize("d,nq,nkv,max_ctx,pos", [
    (128, 3, 1, 130, [0, 62, 63, 64, 127, 129]), (128, 4, 4, 65, [64, 63]), (128, 10, 2, 200, [195, 30]),
    (128, 13, 1, 200, [199, 128]), (128, 12, 4, 2048, [2047, 1030, 64, 1984, 5, 700, 2000, 1]),
    (256, 3, 3, 100, [0, 95]), (256, 12, 2, 130, [128, 66]), (256, 15, 1, 200, [199, 15, 16]),
    (256, 8, 4, 2100, [2099, 1030, 64, 1983, 15, 700, 2046, 2047])])
def test_attention_edges(ctx, dev, d, nq, nkv, max_ctx, pos):
    import torch
    from oracle import decode as od
    batch = len(pos)
    q = synth.uniform_affine_f32(51, batch * nq * d, 3.0).reshape(batch, nq, d)
    codes = [oracle.f32_to_bf16(synth.uniform_f32(52 + i, batch * nkv * max_ctx * d)).reshape(batch, nkv, max_ctx, d)
             for i in range(2)]
    for c in codes:
        for b, p in enumerate(pos):
            c[b, :, p + 1:] = 0x7FC0
    k, v = (torch.from_numpy(c.view(np.int16)).to(dev) for c in codes)
    out = ctx.attention_decode(torch.from_numpy(q).to(dev), k, v, pos, nq, nkv, d, max_ctx)
    got = oracle.bf16_to_f64(out.cpu().numpy().view(np.uint16)).reshape(batch, nq, d)
    for b, p in enumerate(pos):
        kv, vv = (oracle.bf16_to_f64(c[b, :, :p + 1]) for c in codes)
        want = od.attention_decode(q[b].astype(np.float64), kv, vv)
        # FP32: sums of 64 terms per chunk, merged over the chunks; then one rounding to BF16
        eps = (64 + (p // 64 + 1) + 8) * 2.0 ** -23 * np.max(np.abs(vv))
        assert np.all(got[b] >= od.q_bf16(want - eps)) and np.all(got[b] <= od.q_bf16(want + eps))


# One tile of the vectors, one chunk more, halves filled in turn with a short
# last one; all vectors of a work-group present and some missing; normalised
# vectors kept in registers (up to 4096 elements) and read twice.
@pytest.mark.parametrize("batch", [1, 2, 3, 6, 8])
@pytest.mark.parametrize("k", [8, 504, 4096, 4104, 8192, 8200, 16384, 16392, 20488])
def test_gemv_rows_edges(ctx, dev, batch, k):
    import torch
    rows = 41
    w = oracle.f32_to_bf16(synth.uniform_affine_f32(61, rows * k, k ** -0.5)).reshape(rows, k)
    v = oracle.f32_to_bf16(synth.uniform_f32(62, batch * k)).reshape(batch, k)
    tw, tv = (torch.from_numpy(a.view(np.int16)).to(dev) for a in (w, v))
    out = ctx.gemv_bf16_rows(tw, tv)
    fw, fv = oracle.bf16_to_f64(w), oracle.bf16_to_f64(v)
    bound = oracle.accumulation_bound(k + 1, np.abs(fv) @ np.abs(fw).T, 2.0 ** -24)
    assert np.all(np.abs(out.cpu().numpy() - fv @ fw.T) <= bound)
    for b in range(batch):                 # whatever the batch, the same sums
        assert torch.equal(out[b], ctx.gemv_bf16_rows(tw, tv[b:b + 1])[0])
    x = torch.from_numpy(synth.uniform_affine_f32(63, batch * k, 2.0).reshape(batch, k)).to(dev)
    g = torch.from_numpy(oracle.f32_to_bf16(synth.uniform_affine_f32(64, k, 0.25, 1.0)).view(np.int16)).to(dev)
    fused = torch.empty_like(out)
    ctx.fused_gemv(tw, "plain", x=x, g=g, eps=1e-5, out=fused)
    assert torch.equal(fused, ctx.gemv_bf16_rows(tw, ctx.rmsnorm_bf16(x, g, 1e-5)))


# Rows beyond the length from which weights are loaded non-temporally, a row
# more than whole work-groups.
@pytest.mark.parametrize("batch", [1, 2, 4, 8])
@pytest.mark.parametrize("rows,k", [(33001, 4104), (8193, 16392)])
def test_gemv_rows_forms_agree(ctx, dev, batch, rows, k):
    import torch
    w = torch.from_numpy(oracle.f32_to_bf16(synth.uniform_f32(31, 1 << 22)).view(np.int16)).to(dev)
    w = w.repeat(-(-rows * k // w.numel()))[: rows * k].reshape(rows, k)
    v = torch.from_numpy(oracle.f32_to_bf16(synth.uniform_f32(32, batch * k)).view(np.int16).reshape(batch, k)).to(dev)
    whole = ctx.gemv_bf16_rows(w, v)
    for i in range(0, rows, rows // 3 + 1):
        assert torch.equal(whole[:, i:i + rows // 3 + 1], ctx.gemv_bf16_rows(w[i:i + rows // 3 + 1], v))


# The serving arena kept between runs: reused, replaced by a larger one, taken
# by one of two threads; given back with the context and beyond its bound.
def test_serve_arena(dev):
    import threading
    import torch
    from paper_2501_16909_amd import coloc
    c = coloc.Context(0)
    reqs = [dict(kind="triad", n=(1 << 20) + 7 * i, arrival_s=0.0, seed=800 + i) for i in range(3)]

    def run(budget):
        return [r["checksum_bits"] for r in c.serve(reqs, hbm_budget=budget, slots=2)]

    free0 = torch.cuda.mem_get_info()[0]
    want = run(64 << 20)
    total = torch.cuda.mem_get_info()[1]
    for budget in (32 << 20, 1 << 30, 64 << 20):
        assert run(budget) == want
    assert free0 - torch.cuda.mem_get_info()[0] <= 2 << 30
    got = [None, None]
    threads = [threading.Thread(target=lambda i=i: got.__setitem__(i, run((i + 1) << 30))) for i in range(2)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert got == [want, want]
    held = torch.cuda.mem_get_info()[0]
    assert run(total // 16 + (1 << 30)) == want       # replaces the kept one and is not kept itself
    assert torch.cuda.mem_get_info()[0] >= held
    c.close()
    assert free0 - torch.cuda.mem_get_info()[0] <= 256 << 20


# Inputs of served requests whose element counts are not whole groups of four.
def test_serve_input_remainders(ctx, dev):
    import torch
    reqs = [dict(kind="triad", n=n, arrival_s=0.0, seed=900 + 10 * n, out_copy=torch.empty(n, device=dev))
            for n in (1, 2, 3, 4, 5, 1023, 4098)]
    ctx.serve(reqs, hbm_budget=1 << 20, slots=3)
    for q in reqs:
        b, c = synth.uniform_f32(q["seed"], q["n"]), synth.uniform_f32(q["seed"] + 1, q["n"])
        assert np.array_equal(q["out_copy"].cpu().numpy().view(np.uint32), oracle.triad_f32(b, c).view(np.uint32))


# Rows of 8 and 16 MiB and a bit: the lane offsets of the largest tiles, their
# early touches (more tiles than CUs) and the ragged last stage.  The first and
# last rows against the small tiles, which add in the same order.
@pytest.mark.parametrize("dtype,m,kb", [("f32", 3900, (1 << 23) + 16), ("bf16", 4100, (1 << 24) + 144)])
def test_gemm_long_rows(ctx, dev, dtype, m, kb):
    import torch
    k = kb // {"f32": 4, "bf16": 2}[dtype]
    if torch.cuda.mem_get_info()[0] < m * kb + (4 << 30):
        pytest.skip("not enough free device memory")
    x = torch.empty((m, k), dtype={"f32": torch.float32, "bf16": torch.bfloat16}[dtype], device=dev).normal_()
    a = x if dtype == "f32" else x.view(torch.int16)
    out, part = torch.empty((m, m), device=dev), torch.empty((200, m), device=dev)
    ctx.victim_run(ctx.gemm_desc(a, a, out, dtype, m, m, k, 1.0, 1.0))
    for rows in (slice(0, 200), slice(m - 200, m)):
        ctx.victim_run(ctx.gemm_desc(a[rows], a, part, dtype, 200, m, k, 1.0, 1.0))
        assert torch.equal(out[rows], part)
    del x, a
    torch.cuda.empty_cache()
