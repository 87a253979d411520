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
