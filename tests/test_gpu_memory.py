"""The device memory that a context keeps between serving runs: given back on
request and for a much smaller budget."""
import pytest

pytestmark = pytest.mark.gpu

GIB = 1 << 30
REQS = [dict(kind="triad", n=(1 << 20) + 7 * i, arrival_s=0.0, seed=800 + i) for i in range(3)]


def _run(c, budget):
    return [r["checksum_bits"] for r in c.serve(REQS, hbm_budget=budget, slots=2)]


def _free():
    import torch
    return torch.cuda.mem_get_info()[0]


def test_kept_arena_is_given_back_on_request(dev):
    from paper_2501_16909_amd import coloc
    with coloc.Context(0) as c:
        c.release_memory()                        # nothing kept: nothing to do
        want = _run(c, GIB // 4)
        free0 = _free()
        assert _run(c, 8 * GIB) == want
        assert free0 - _free() >= 7 * GIB         # kept for the next run
        c.release_memory()
        assert free0 - _free() <= GIB // 4
        assert _run(c, 8 * GIB) == want


def test_small_budget_does_not_hold_a_large_arena(dev):
    from paper_2501_16909_amd import coloc
    with coloc.Context(0) as c:
        want = _run(c, GIB // 4)
        free0 = _free()
        assert _run(c, 8 * GIB) == want
        assert _run(c, 3 * GIB) == want           # more than a quarter: reused
        assert free0 - _free() >= 7 * GIB
        assert _run(c, GIB) == want
        assert free0 - _free() <= GIB


@pytest.mark.skip(reason="a device allocation that finds no memory ended the process (segmentation fault) late in a "
                         "run of the whole suite; the cause is not known, so the library does not try again after one")
def test_kept_arena_yields_to_the_library_s_own_allocations(dev):
    """Another context's run finds no memory while the first one keeps its
    arena: it gets that memory instead of an error."""
    import torch
    from paper_2501_16909_amd import coloc
    with coloc.Context(0) as a, coloc.Context(0) as b:
        want = _run(a, 12 * GIB)
        hold = torch.empty(_free() - 6 * GIB, dtype=torch.uint8, device=dev)
        try:
            assert _run(b, 10 * GIB) == want
        finally:
            del hold
            torch.cuda.empty_cache()
        assert _run(a, 12 * GIB) == want
