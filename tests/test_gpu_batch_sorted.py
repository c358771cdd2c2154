"""GPU: large batches of long tracks are sorted and traced in waves; the batch kernel gives the same.

A batch is taken for one of long tracks by its mean, so the same tracks
followed by many that have no photons go to the batch kernel: both must agree
bit for bit, in id order and in the processing order, with tracks of no, few
and many photons mixed, at windows cut by tracks and by the end.
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
    sd = I.scene_g5(seg_quads=(34, 57))
    segments = R.Scene(sd)
    segments.set_params(I.perturbed_params(5, sd))
    return {"meshed": R.Scene(I.scene_g2()), "segments": segments}


@pytest.mark.parametrize("scene", ["meshed", "segments"])
@pytest.mark.parametrize("n_tracks, mean", [(1, 524288), (60, 9000), (2700, 800)])
@pytest.mark.parametrize("short", [0, 5])
def test_sorted_against_batch_kernel(R, scenes, scene, n_tracks, mean, short):
    import torch
    gs = scenes[scene]
    rng = np.random.default_rng(n_tracks)
    counts = rng.integers(mean // 2, mean + mean // 2 + 1, n_tracks) if n_tracks > 1 else np.array([mean])
    if n_tracks > 1:
        counts[3::7] = rng.integers(0, 3, len(counts[3::7]))
        counts[::5] += mean
    tracks = I.sample_tracks(rng, n_tracks)
    src = I.batch_source(tracks, counts)
    if short:
        src = I.with_dispersion(src)
    padded = dict(src)
    padded["tracks"] = np.concatenate([tracks, np.repeat(tracks[:1], 20000, 0)])
    padded["offsets"] = np.concatenate([src["offsets"], np.full(20000, src["offsets"][-1], np.uint64)])
    outs = []
    for s in (src, padded):
        b, keep, total = R.make_batch(s, "cuda")
        n = total - short
        t, o = R.alloc_outputs(gs, n, "cuda")
        for _ in range(2):
            R.rich_propagate_batch(gs.handle, b, n, 13, o, R.tuning(256, 256, 2))
        torch.cuda.synchronize()
        assert gs.status() == (R.FLAG_BATCH_SIZE if short else 0)
        outs.append(t)
    assert total >= 1 << 19 and int(outs[0]["fate_counts"].sum()) == 2 * n
    for k in ("fate", "pixel", "hit_xyz", "hit_uv", "hit_time", "histogram", "fate_counts"):
        x, y = outs[0][k], outs[1][k]
        same = (x == y) | (x.isnan() & y.isnan()) if x.is_floating_point() else x == y
        assert bool(same.all()), k
