"""GPU: the boxes a lane walks by are rounded outwards, so no ray slips past a surface it meets.

A plate of 2 mm facets is seen from a hundredth of a millimetre to a kilometre
away, in the rays' and the plate's own large coordinates, along the axes and
aslant; its mesh is watertight, so every photon aimed well inside its outline
must end on it.
"""

import copy

import numpy as np
import pytest

from paper_2309_12496_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("normal", [(0.0, 0.0, 1.0), (0.0, -1.0, 0.0), (1.0, 0.0, 0.0), (0.48, -0.6, 0.64)])
@pytest.mark.parametrize("centre", [(0.0, 0.0, 0.0), (3.0e4, -7.0e4, 1.0e5)])
def test_no_photon_passes_a_plate(normal, centre):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2309_12496_amd import rich as R
    n, c = np.array(normal), np.array(centre)
    u = np.cross(n, (0.0, 0.0, 1.0) if abs(n[2]) < 0.9 else (1.0, 0.0, 0.0))
    u /= np.linalg.norm(u)
    v = np.cross(n, u)
    sc = copy.deepcopy(I.scene_g2((2, 2), 2))
    sc["box"] = None
    sc["meshes"] = [{"vertices": I.rect_mesh(c, n, u, v, 100.0, 100.0, 100, 100), "material": I.ABSORBER,
                     "segment": -1}]
    sc["detector"]["center"] = c + 5e6 * u                 # nothing else near
    gs = R.Scene(sc)
    rng = np.random.default_rng(23)
    m = 40000
    ab = rng.uniform(-80.0, 80.0, (m, 2))
    ab[::4] = np.round(ab[::4] / 2.0) * 2.0                # on the facets' edges and corners
    p = c + ab[:, :1] * u + ab[:, 1:] * v
    far = 10.0 ** rng.uniform(-2.0, 6.0, m)
    slope = np.where(np.arange(m) % 3 == 0, 0.0, rng.uniform(0.0, 1.0, m))
    az = rng.uniform(0.0, 2.0 * np.pi, m)
    d = -n + slope[:, None] * (np.cos(az)[:, None] * u + np.sin(az)[:, None] * v)
    d *= rng.choice([-1.0, 1.0], m)[:, None]
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    # a start rounded to FP32 may lie on the plate, or beyond it: then it is not this photon's to meet
    o = (p - far[:, None] * d).astype(np.float32)
    ahead = ((c - o.astype(np.float64)) @ n) / (d @ n) > sc["t_min"] + 2e-3 + 2.0 ** -20 * np.abs(o).max(axis=1)
    assert ahead.mean() > 0.5
    o, d = o[ahead], d[ahead]
    out = R.propagate(gs, I.explicit_source(o, d, np.full(len(o), 400.0)), len(o), 3)
    fate = out["fate"].cpu().numpy()
    assert (fate == R.ABSORBED).all(), (np.flatnonzero(fate != R.ABSORBED)[:8], np.unique(fate))
    assert gs.status() == 0
