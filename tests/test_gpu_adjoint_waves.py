"""GPU: a photon's gradient is the same whichever wave, lane and launch sweep it back.

With an upstream gradient at one photon only, every other addend of the sums
over lanes, waves and blocks is zero, so the launch must give, bit for bit,
the gradient of that photon traced alone: at sizes around a wave, a block and
several blocks, for the first and the last photon that is detected, with and
without a mask.
"""

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


@pytest.fixture(scope="module")
def scenes(R):
    tiles = I.scene_g5(seg_quads=(8, 13))
    return {"caps": R.Scene(I.scene_g4()), "tiles": R.Scene(tiles)}


@pytest.mark.parametrize("scene", ["caps", "tiles"])
@pytest.mark.parametrize("n", [64, 65, 256, 257, 1025, 5000])
@pytest.mark.parametrize("masked", [False, True])
def test_one_photons_gradient(R, scenes, scene, n, masked):
    import torch
    gs = scenes[scene]
    src = I.point_source(direction=(0.01, -0.02, 1.0), length=500.0)
    out = R.propagate(gs, src, n, 7)
    on = np.flatnonzero(out["fate"].cpu().numpy() == R.DETECTED)
    assert len(on) >= 2
    for p in (int(on[0]), int(on[-1])):
        up = torch.zeros((n, 2), device="cuda")
        up[p, 0], up[p, 1] = 0.75, -1.25
        mask = None
        if masked:
            mask = (torch.arange(n, device="cuda") % 3 == p % 3).to(torch.uint8)
        grad, _ = R.adjoint(gs, src, 7, n=n, grad_uv=up, mask=mask)
        alone, _ = R.adjoint(gs, src, 7, n=1, first_id=p, grad_uv=up[p:p + 1])
        assert torch.isfinite(grad).all() and grad.abs().max() > 0
        assert torch.equal(grad, alone), (p, grad - alone)
    assert gs.status() == 0
