"""GPU: the order of sorted launches, by its windows' size and by who draws the bins.

Photons keep their ids and random numbers however a launch is split: one
launch must give, bit for bit, what launches of its parts give.  Sizes at the
edges of a window of each shape, at the limits between the shapes, and where
the trace's blocks are no multiple of the eight XCDs.
"""

import pytest

from paper_2309_12496_amd import inputs as I

pytestmark = pytest.mark.gpu

SMALL, SMALL_PREFILTERED = 1 << 18, 1 << 22     # photons from which windows are larger


@pytest.mark.parametrize("prefilter", [False, True])
@pytest.mark.parametrize("length", [0.0, 1000.0])
@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 2049, 20011, 65537, SMALL - 1, SMALL, SMALL + 1, SMALL + 32769,
                               SMALL_PREFILTERED - 1, SMALL_PREFILTERED, SMALL_PREFILTERED + 8193])
def test_one_launch_equals_its_parts(n, length, prefilter):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2309_12496_amd import rich as R
    gs = R.Scene(I.scene_g2(sphere_quads=(34, 29), box_quads=3))
    src = I.point_source(direction=(0.02, -0.01, 1.0), length=length)
    if prefilter:
        src = I.with_prefilter(src)
    first = 11
    whole = R.propagate(gs, src, n, 3, first_id=first)
    total = torch.zeros_like(whole["fate_counts"])
    step = 900 if n < 100_000 else 100_003
    for lo in range(0, n, step):
        m = min(step, n - lo)
        part = R.propagate(gs, src, m, 3, first_id=first + lo)
        total += part["fate_counts"]
        for k in ("fate", "pixel", "hit_xyz", "hit_uv", "hit_time"):
            a, b = whole[k][lo:lo + m], part[k]
            same = (a == b) | (a.isnan() & b.isnan()) if a.is_floating_point() else a == b
            assert bool(same.all()), (k, lo)
    assert torch.equal(whole["fate_counts"], total) and int(total.sum()) == n
    assert gs.status() == 0
