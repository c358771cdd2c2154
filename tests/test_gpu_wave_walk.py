"""GPU: large launches from one source walk the tree a wave at a time; smaller ones each lane on its own.

Photons keep their ids and random numbers however a launch is split, so one
launch large enough for the wave phase must give, bit for bit, what launches
of its parts, too small for it, give: at the least such size and one photon
beyond it (a last wave of one lane), from a point along the axis (rays of
every sign), aslant (all of one sign), and from a long track.
"""

import numpy as np
import pytest

from paper_2309_12496_amd import inputs as I

pytestmark = pytest.mark.gpu

POINT_MIN, TRACK_MIN = 1 << 18, 1 << 20     # photons from which the wave phase is used


@pytest.fixture(scope="module")
def R():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2309_12496_amd import rich
    return rich


@pytest.fixture(scope="module")
def scenes(R):
    meshed = R.Scene(I.scene_g2())
    sd = I.scene_g5(seg_quads=(34, 57))
    segments = R.Scene(sd)
    segments.set_params(I.perturbed_params(5, sd))
    return {"meshed": meshed, "segments": segments}


@pytest.mark.parametrize("scene", ["meshed", "segments"])
@pytest.mark.parametrize("direction,length,n", [
    ((0.0, 0.0, 1.0), 0.0, POINT_MIN),
    ((0.12, 0.11, 0.9), 0.0, POINT_MIN + 1),
    ((-0.03, 0.02, 1.0), 1000.0, TRACK_MIN),
])
def test_one_launch_equals_its_parts(R, scenes, scene, direction, length, n):
    import torch
    gs = scenes[scene]
    src = I.point_source(direction=direction, length=length)
    whole = R.propagate(gs, src, n, 99)
    step = POINT_MIN - 1
    for first in range(0, n, step):
        m = min(step, n - first)
        part = R.propagate(gs, src, m, 99, first_id=first)
        for k in ("fate", "pixel", "hit_xyz", "hit_uv", "hit_time"):
            a, b = whole[k][first:first + m], part[k]
            same = (a == b) | (a.isnan() & b.isnan()) if a.is_floating_point() else a == b
            assert bool(same.all()), (k, first)
    torch.cuda.synchronize()
    assert gs.status() == 0
    counts = whole["fate_counts"].cpu().numpy()
    assert counts.sum() == n and np.count_nonzero(counts) >= 2   # (the aslant beam misses the detector)
