"""Many photons are read out through strips of the film in LDS, few straight onto it: the same image."""

import numpy as np
import pytest
import torch

from paper_2309_12496_amd import inputs as I

pytestmark = pytest.mark.gpu

FEW = (1 << 15) - 1        # the longest read-out that adds straight onto the image


@pytest.mark.parametrize("n, width, height, sigma", [
    (FEW + 1, 1320, 620, 0.5),        # 23 strips, the last of 26 rows
    (3 * FEW + 11, 1320, 620, 0.5),
    (FEW + 2, 36000, 9, 0.5),         # strips of one row
    (FEW + 7, 36001, 9, 0.5),         # a row does not fit: straight
    (FEW + 3, 1125, 1025, 0.5),       # 33 strips: straight
    (FEW + 5, 1125, 1024, 4.0),       # 32 strips, windows over three of them
    (FEW + 5, 7, 5, 0.5),             # one strip
])
def test_strips_against_photons_straight_onto_the_image(n, width, height, sigma):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2309_12496_amd import rich as R
    film = I.film_paper(width=width, height=height, sigma=sigma)
    scale = width / (2 * film["distance"] * np.tan(film["fov"] / 2))      # pixels per mm
    rng = np.random.default_rng(n)
    # a fifth outside, some far outside, some not a number
    px = rng.uniform(-0.1 * width, 1.1 * width, n).astype(np.float32)
    py = rng.uniform(-0.1 * height, 1.1 * height, n).astype(np.float32)
    uv = np.stack([(px - width / 2) / scale, (py - height / 2) / scale], 1).astype(np.float32)
    uv[::97] = np.nan
    uv[5::101] *= 1e30
    fate = (rng.random(n) < 0.5).astype(np.uint8) * 3
    fate, uv = torch.as_tensor(fate, device="cuda"), torch.as_tensor(uv, device="cuda")
    img, hits = R.film_readout(film, fate, uv)
    few = None
    for lo in range(0, n, FEW):
        few, few_hits = R.film_readout(film, fate[lo:lo + FEW].contiguous(), uv[lo:lo + FEW].contiguous(), image=few)
    # the addends are the same: two orders of summing K positive ones differ by
    # at most 2 (K - 1) roundings of the sum; K is at most the photons within
    # the window's reach of the pixel, rounded up to whole pixels
    reach = int(np.ceil(4 * sigma)) + 1
    inside = np.isfinite(uv.cpu().numpy()).all(1) & (fate.cpu().numpy() == 0)
    x, y = px[inside] + reach + 1, py[inside] + reach + 1
    count, _, _ = np.histogram2d(y, x, bins=[height + 2 * reach + 2, width + 2 * reach + 2],
                                 range=[[0, height + 2 * reach + 2], [0, width + 2 * reach + 2]])
    box = torch.nn.functional.avg_pool2d(torch.as_tensor(count)[None, None], 2 * reach + 3, 1, divisor_override=1)[0, 0]
    assert box.shape == (height, width)
    a, b = img.double().cpu(), few.double().cpu()
    assert b.max() > 0
    assert ((a - b).abs() <= 2 * box * 2.0 ** -24 * b).all()
    edge = (torch.clamp(b, max=255.0) - film["threshold"]).abs() <= 2 * box * 2.0 ** -24 * b
    assert torch.equal(hits.cpu()[~edge], few_hits.cpu()[~edge])
