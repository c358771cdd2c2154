"""GPU: large launches of photon arrays on meshes claim their ids; smaller ones stride over them.

One launch at and around the limit must give, bit for bit, what launches of
its parts give.
"""

import numpy as np
import pytest

from paper_2309_12496_amd import inputs as I

pytestmark = pytest.mark.gpu

LIMIT = 5 << 18


@pytest.mark.parametrize("n", [LIMIT - 1, LIMIT, LIMIT + 65])
def test_one_launch_equals_its_parts(n):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2309_12496_amd import rich as R
    gs = R.Scene(I.scene_g2(sphere_quads=(34, 29), box_quads=3))
    rng = np.random.default_rng(6)
    d = rng.normal(size=(n, 3)) * (0.1, 0.1, 0.02) + (0.0, 0.0, 1.0)
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    o = rng.uniform(-5.0, 5.0, (n, 3))
    lam = rng.uniform(200.0, 600.0, n)
    whole = R.propagate(gs, I.explicit_source(o, d, lam), n, 3)
    step = 400_000
    for lo in range(0, n, step):
        k = slice(lo, min(n, lo + step))
        part = R.propagate(gs, I.explicit_source(o[k], d[k], lam[k]), k.stop - lo, 3, first_id=lo)
        for key in ("fate", "pixel", "hit_xyz", "hit_uv", "hit_time"):
            a, b = whole[key][k], part[key]
            same = (a == b) | (a.isnan() & b.isnan()) if a.is_floating_point() else a == b
            assert bool(same.all()), (key, lo)
    assert int(whole["fate_counts"].sum()) == n and gs.status() == 0
