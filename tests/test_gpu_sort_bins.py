"""GPU: sorted launches draw their bins in a launch of their own between a quarter window and a window per CU.

Photons keep their ids and random numbers however a launch is split: one
launch must give, bit for bit, what launches of its parts give that are too
small for it.  Sizes at the rule's lower end, at a window's edges, and where
the trace's blocks are no multiple of the eight XCDs.
"""

import pytest

from paper_2309_12496_amd import inputs as I

pytestmark = pytest.mark.gpu

PART = {False: 8191, True: 2047}      # the most photons whose bins the sort draws itself


@pytest.mark.parametrize("prefilter", [False, True])
@pytest.mark.parametrize("length", [0.0, 1000.0])
@pytest.mark.parametrize("n", [2047, 2048, 2049, 8191, 8192, 8193, 20011, 32767, 32769, 65537])
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
    for lo in range(0, n, PART[prefilter]):
        m = min(PART[prefilter], n - lo)
        part = R.propagate(gs, src, m, 3, first_id=first + lo)
        total += part["fate_counts"]
        for k in ("fate", "pixel", "hit_xyz", "hit_uv", "hit_time"):
            a, b = whole[k][lo:lo + m], part[k]
            same = (a == b) | (a.isnan() & b.isnan()) if a.is_floating_point() else a == b
            assert bool(same.all()), (k, lo)
    assert torch.equal(whole["fate_counts"], total) and int(total.sum()) == n
    assert gs.status() == 0
