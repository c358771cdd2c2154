"""GPU: which interval of a refractive index table a wavelength falls in, from one node to the most.

Photons sent straight at the detector arrive after L (n - lambda dn/dlambda) / c,
and the slopes of neighbouring intervals differ, so a wavelength looked up in
the wrong one is late or early by 1e-4 of the flight and more.  Wavelengths on
the nodes, next to them, between them and beyond both ends.
"""

import numpy as np
import pytest

from paper_2309_12496_amd import inputs as I

pytestmark = pytest.mark.gpu

C_MM_NS = 299.792458


@pytest.mark.parametrize("nodes, lo, hi", [(1, 400.0, 400.0), (2, 250.0, 500.0), (3, 200.0, 600.0), (17, 200.0, 600.0),
                                           (31, 210.0, 590.0), (32, 100.0, 450.0)])
def test_interval_of_a_wavelength(nodes, lo, hi):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2309_12496_amd import rich as R
    f32 = np.float32
    x = np.linspace(lo, hi, nodes).astype(f32)
    m = (1.4e-3 * (1.0 + 40.0 / x.astype(float) + 0.02 * (np.arange(nodes) % 2))).astype(f32)
    lam = np.concatenate([x, np.nextafter(x, f32(0)), np.nextafter(x, f32(1e9)), 0.5 * (x[1:] + x[:-1]),
                          np.array([50.0, 99.0, 201.0, 399.0, 601.0, 900.0], f32)]).astype(f32)
    scene = I.scene_g1()
    det = scene["detector"]
    length = 400.0
    o = np.asarray(det["center"]) + length * np.asarray(det["normal"]) + 3.0 * np.asarray(det["axis_u"])
    src = I.explicit_source(np.tile(o, (len(lam), 1)), np.tile(-np.asarray(det["normal"]), (len(lam), 1)), lam)
    src["dispersion"] = {"lambda": x.astype(float), "index": 1.0 + m.astype(float)}
    out = R.propagate(R.Scene(scene), src, len(lam), 3)
    t = out["hit_time"].cpu().numpy().astype(float)
    assert np.isfinite(t).all()
    # [x_j, x_{j+1}) takes the line from m_j; outside the table the end's index without slope
    xd, md, ld = x.astype(float), m.astype(float), lam.astype(float)
    j = np.searchsorted(xd, ld, side="right") - 1
    inside = (j >= 0) & (j < nodes - 1)
    j0 = np.clip(j, 0, nodes - 1)
    j1 = np.minimum(j0 + 1, nodes - 1)
    slope = np.where(inside, (md[j1] - md[j0]) / np.where(j1 > j0, xd[j1] - xd[j0], 1.0), 0.0)
    group = 1.0 + md[j0] + slope * (ld - xd[j0]) - slope * ld
    ref = length * group / C_MM_NS
    # the path (an FP32 start 2,800 mm out: 2^-13 mm and its length's rounding) and the
    # products: 2^-12 mm of light path and eight roundings of the time
    tol = 2.0 ** -12 / C_MM_NS + 8 * 2.0 ** -24 * ref
    if nodes > 2:
        assert np.abs(np.diff((md[1:] - md[:-1]) / (xd[1:] - xd[:-1]))).min() * 200.0 * length / C_MM_NS > 10 * tol.max()
    assert (np.abs(t - ref) <= tol).all(), (np.abs(t - ref).max(), tol.max(), lam[np.abs(t - ref) > tol])
