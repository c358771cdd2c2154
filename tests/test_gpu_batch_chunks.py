"""GPU: the batch kernel on meshes at every kind of chunk, in id order and in the processing order.

Chunks are multiples of 64; only those made of whole 256-photon slices are
regrouped.  Every photon is traced once and alike, whatever the chunk; the
batches' tracks are too short for the sorted launches that longer ones take.
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
def batches(R):
    """Scene, and by order (tracks, mean) the batch and its outputs in chunks of 256."""
    sd = I.scene_g2((86, 72), 29)
    gs = R.Scene(sd)
    made = {}
    for ordered, (tracks, mean) in {False: (700, 700), True: (3600, 600)}.items():
        rng = np.random.default_rng(tracks)
        src = I.batch_source(I.sample_tracks(rng, tracks), rng.integers(mean - 100, mean + 101, tracks))
        made[ordered] = (R.make_batch(src), R.propagate_batch(gs, src, 5, tune=R.tuning(256, 256, 2)))
        n = made[ordered][0][2]
        assert (n >= 1 << 21) == ordered and n < (768 if ordered else 2048) * tracks
        # against the photons of one track by themselves
        k = tracks // 2
        first, count = int(src["offsets"][k]), int(src["offsets"][k + 1] - src["offsets"][k])
        row = src["tracks"][k]
        one = R.propagate(gs, I.point_source(row[:3], row[3:6], beta=row[7], length=row[6]), count, 5, first_id=first)
        for key in ("fate", "pixel"):
            agree = (one[key] == made[ordered][1][key][first:first + count]).float().mean()
            assert float(agree) >= 0.99, (key, float(agree))      # (the cone's constants are rounded elsewhere)
    return gs, made


@pytest.mark.parametrize("ordered", [False, True])
@pytest.mark.parametrize("block, chunk", [(128, 64), (128, 320), (128, 768), (64, 448), (512, 192), (256, 1024)])
def test_chunks(R, batches, ordered, block, chunk):
    import torch
    gs, made = batches
    (b, keep, n), ref = made[ordered]
    t, o = R.alloc_outputs(gs, n)
    t["fate"].fill_(99)
    t["pixel"].fill_(-9)
    R.rich_propagate_batch(gs.handle, b, n, 5, o, R.tuning(block, chunk, 2))
    torch.cuda.synchronize()
    for k in ("fate", "pixel", "hit_xyz", "hit_uv", "hit_time", "histogram", "fate_counts"):
        x, y = t[k], ref[k]
        same = (x == y) | (x.isnan() & y.isnan()) if x.is_floating_point() else x == y
        assert bool(same.all()), k
    assert int(t["fate_counts"].sum()) == n and gs.status() == 0
