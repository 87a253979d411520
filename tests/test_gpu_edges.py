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
