"""GPU: a moving mirror's sheet is left out of no query when its segment is scaled or shifted far.

The rule of a sheet is proved for the mesh as it was built.  Two plates, one
half over the other at a third of t_min, are a sheet; scaled, a photon between
them is stopped by the back of the upper one.  A plate a kilometre away has
reflection points that are rounded to beyond t_min behind it, and is met again
from there.  Either way the photons must end as they do in the same scene with
a triangle without area added to the mesh, which makes it no sheet.
"""

import copy

import numpy as np
import pytest

from paper_2309_12496_amd import inputs as I

pytestmark = pytest.mark.gpu

KEYS = ("fate", "pixel", "hit_xyz", "hit_uv", "hit_time")


@pytest.fixture(scope="module")
def R():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2309_12496_amd import rich
    return rich


def scene(plates, t_min, refuse):
    """plates: (offset along e1, height) of 200 x 200 mm plates of segment 0, facing its centre."""
    sc = copy.deepcopy(I.scene_g5(seg_quads=(2, 2)))
    sc["materials"] = I._materials(unit_reflectivity=True)
    sg = sc["segments"]
    pivot, u0, e1, e2 = (np.asarray(sg[k][0], float) for k in ("pivot", "u0", "e1", "e2"))
    verts = np.concatenate([I.rect_mesh(pivot + x * e1 + h * u0, u0, e1, e2, 100.0, 100.0, 8, 8) for x, h in plates])
    if refuse:
        verts = np.concatenate([verts, verts[0][[0, 0, 1]][None]])
    sc["meshes"] = [{"vertices": verts, "material": I.MIRROR, "segment": 0}]
    sc["t_min"] = t_min
    sc["max_bounces"] = 4
    sc["box"] = None
    return sc, (pivot, u0, e1, e2)


def traced(R, sc, params, src, initial):
    import torch
    sc = copy.deepcopy(sc)
    if initial:
        sc["params"] = params
    gs = R.Scene(sc)
    if not initial:
        gs.set_params(params)
    out = R.propagate(gs, src, len(src["lambda"]), 3)
    torch.cuda.synchronize()
    assert gs.status() == 0
    return {k: out[k].cpu().numpy() for k in KEYS}


def photons(origin, u0, e1, e2, slope, n=4000):
    rng = np.random.default_rng(12)
    ab = rng.uniform(-slope, slope, (n, 2))
    d = -u0 + ab[:, :1] * e1 + ab[:, 1:] * e2
    return I.explicit_source(origin, d / np.linalg.norm(d, axis=1, keepdims=True), np.full(n, 400.0))


@pytest.mark.parametrize("initial", [True, False], ids=["built", "set"])
@pytest.mark.parametrize("scale", [4.0, 30.0])
def test_scaled(R, scale, initial):
    rng = np.random.default_rng(13)
    outs = []
    for refuse in (False, True):
        sc, (pivot, u0, e1, e2) = scene([(0.0, 0.0), (100.0, 0.3)], 1.0, refuse)
        params = np.array(sc["params"], np.float32)
        params[0, 2] = scale * sc["segments"]["radius0"][0]
        ab = rng.uniform(30.0, 60.0, (4000, 1)) * e1 + rng.uniform(-20.0, 20.0, (4000, 1)) * e2 if not outs else ab
        src = photons(pivot + ab + 1.15 * u0, u0, e1, e2, 0.05)
        outs.append(traced(R, sc, params, src, initial))
    assert (outs[1]["fate"] == R.ABSORBED).all()          # by the upper plate's back
    for k in KEYS:
        assert np.array_equal(outs[0][k], outs[1][k], equal_nan=outs[0][k].dtype.kind == "f"), k


@pytest.mark.parametrize("initial", [True, False], ids=["built", "set"])
def test_shifted(R, initial):
    rng = np.random.default_rng(13)
    outs = []
    for refuse in (False, True):
        sc, (pivot, u0, e1, e2) = scene([(0.0, 0.0)], 0.02, refuse)
        params = np.array(sc["params"], np.float32)
        # 1e6 along z, which is nearly the normal: FP32 steps of 1/16 there, so a reflection point lies
        # up to 1/32 behind the plate and about 0.18 of them further than t_min
        params[0, 3:] = (0.4e6, -0.7e6, 1.0e6)
        off = rng.uniform(-50.0, 50.0, (4000, 1)) * e1 + rng.uniform(-50.0, 50.0, (4000, 1)) * e2 \
            + rng.uniform(20.0, 50.0, (4000, 1)) * u0 if not outs else off
        src = photons(pivot + params[0, 3:] + off, u0, e1, e2, 0.3)
        outs.append(traced(R, sc, params, src, initial))
    again = outs[1]["fate"] == R.ABSORBED                  # by the plate they have just left
    assert 0.05 < again.mean() < 0.5
    for k in KEYS:
        assert np.array_equal(outs[0][k], outs[1][k], equal_nan=outs[0][k].dtype.kind == "f"), k
