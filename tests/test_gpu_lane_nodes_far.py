"""GPU: a facet that reaches beyond FP32 hides none of its mesh's others.

A plate of a segment's mesh has a triangle beside it with a vertex at 1e39,
whose boxes end nowhere along one or two axes.  Photons aimed at the plate end
on it, as they do without the triangle.
"""

import copy

import numpy as np
import pytest

from paper_2309_12496_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("far", [(1e39, 0.0, 0.0), (0.0, -1e39, 0.0), (0.0, 0.0, 1e39), (0.0, 1e39, -1e39)])
@pytest.mark.parametrize("n", [20_000, 600_000])
def test_far_vertex(far, n):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2309_12496_amd import rich as R
    sc = copy.deepcopy(I.scene_g5(seg_quads=(2, 2)))
    sg = sc["segments"]
    pivot = np.asarray(sg["pivot"][0], float)
    e1, e2 = np.array((1.0, 0.0, 0.0)), np.array((0.0, 1.0, 0.0))
    u0 = np.array((0.0, 0.0, 1.0))
    plate = I.rect_mesh(pivot, -u0, e1, e2, 100.0, 100.0, 40, 40)
    sc["box"] = None
    outs = []
    rng = np.random.default_rng(5)
    at = pivot + rng.uniform(-90.0, 90.0, (n, 1)) * e1 + rng.uniform(-90.0, 90.0, (n, 1)) * e2
    o = at - rng.uniform(10.0, 500.0, (n, 1)) * u0
    d = at + rng.uniform(-5.0, 5.0, (n, 1)) * e1 - o
    src = I.explicit_source(o, d / np.linalg.norm(d, axis=1, keepdims=True), np.full(n, 400.0))
    for with_far in (False, True):
        verts = plate
        if with_far:
            tri = np.array([pivot + 300.0 * e1, pivot + 300.0 * e1 + 5.0 * e2, pivot + np.array(far)])[None]
            verts = np.concatenate([plate[:1600], tri, plate[1600:]])
        # (another mesh beside it: with one alone there is no level above it)
        sc["meshes"] = [{"vertices": verts, "material": I.ABSORBER, "segment": 0},
                        {"vertices": plate + 9000.0 * e1, "material": I.ABSORBER, "segment": -1}]
        gs = R.Scene(sc)
        out = R.propagate(gs, src, n, 3)
        torch.cuda.synchronize()
        assert gs.status() == 0
        outs.append(out["fate"].cpu().numpy())
    assert (outs[0] == R.ABSORBED).all()
    assert np.array_equal(outs[0], outs[1]), np.unique(outs[1], return_counts=True)
