"""GPU: leaving a mirror sheet out of the query after a reflection by it changes no photon.

A mirror mesh whose facets lie on one sphere or one plane is a sheet, and the
builder refuses a curved mesh or a segment that holds a triangle without area.
The same scene with such a triangle added to each mirror (two equal vertices:
nothing can hit it) is therefore traced with every query over the bowl, and
over both moving segments, and must give the same outputs bit for bit.
"""

import copy

import numpy as np
import pytest

from paper_2309_12496_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2309_12496_amd import rich
    return rich


def scene(moving, refuse):
    """A 300 x 300 mm patch of the 8 m sphere in 2 mm facets, and a flat mirror facing it 400 mm above."""
    sc = copy.deepcopy(I.scene_g5(seg_quads=(2, 2)) if moving else I.scene_g2((2, 2), 2))
    sc["materials"] = I._materials(unit_reflectivity=True)
    centre, u0, e1, e2 = I.mirror_frame()
    bowl = I.sphere_mesh(-150.0, 150.0, -150.0, 150.0, 150, 150)
    flat = I.rect_mesh(I.PIVOT + 400.0 * u0, -u0, e1, e2, 150.0, 150.0, 40, 40)
    extra = np.zeros((1, 3, 3))
    meshes = []
    for k, verts in enumerate((bowl, flat)):
        if refuse:
            extra[0] = verts[0][[0, 0, 1]]
            verts = np.concatenate([verts, extra])
        meshes.append({"vertices": verts, "material": I.MIRROR, "segment": k if moving else -1})
    sc["meshes"] = meshes + [sc["meshes"][-1]]
    sc["max_bounces"] = 4
    return sc


def photons(n=20000, seed=41):
    """From just above the patch: along it (met again and again), near its normal (to the flat mirror and
    back), and at every angle between."""
    rng = np.random.default_rng(seed)
    centre, _, e1, e2 = I.mirror_frame()
    ab = rng.uniform(-140.0, 140.0, size=(n, 2))
    p = I.sphere_point(ab[:, 0], ab[:, 1])
    nrm = (centre - p) / np.linalg.norm(centre - p, axis=1, keepdims=True)
    o = p + rng.uniform(0.01, 0.05, size=(n, 1)) * nrm
    elevation = np.where(np.arange(n) % 3 == 0, np.exp(rng.uniform(np.log(3e-4), np.log(2e-2), n)),
                         np.where(np.arange(n) % 3 == 1, np.pi / 2 - rng.uniform(0.0, 0.1, n),
                                  rng.uniform(0.0, np.pi / 2, n)))
    elevation *= rng.choice([-1.0, 1.0], n)
    az = rng.uniform(0.0, 2.0 * np.pi, n)
    t = np.cos(az)[:, None] * e1 + np.sin(az)[:, None] * e2
    t -= (t * nrm).sum(axis=1, keepdims=True) * nrm
    d = np.cos(elevation)[:, None] * t / np.linalg.norm(t, axis=1, keepdims=True) + np.sin(elevation)[:, None] * nrm
    return I.explicit_source(o, d / np.linalg.norm(d, axis=1, keepdims=True), np.full(n, 400.0))


@pytest.mark.parametrize("moving", [False, True], ids=["fixed", "segments"])
def test_sheets_left_out_change_nothing(R, moving):
    import torch
    src = photons()
    n = len(src["lambda"])
    outs = []
    for refuse in (False, True):
        sc = scene(moving, refuse)
        gs = R.Scene(sc)
        if moving:
            p = np.array(sc["params"], np.float32)
            p[0, :3] += (0.3e-3, -0.2e-3, 3.0)
            p[1, :2] += (-0.4e-3, 0.1e-3)
            gs.set_params(p)
        out = R.propagate(gs, src, n, 3)
        torch.cuda.synchronize()
        assert gs.status() == 0
        outs.append({k: v.cpu().numpy() for k, v in out.items() if torch.is_tensor(v)})
    for k, v in outs[0].items():
        assert np.array_equal(v, outs[1][k], equal_nan=v.dtype.kind == "f"), k
    # photons that meet a mirror four times and photons that leave before are both there: a hit
    # wrongly left out would turn one of the first into one of the second
    many = int((outs[0]["fate"] == R.MAX_BOUNCES).sum())
    assert many > n // 20 and n - many > n // 20, many
