"""GPU: batches without a tuning: none is timed for those that are sorted, and the others are tuned before they are ordered."""

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


def same(a, b):
    return bool(((a == b) | (a.isnan() & b.isnan()) if a.is_floating_point() else a == b).all())


def batch(tracks, mean):
    return I.batch_source(I.sample_tracks(np.random.default_rng(6), tracks), np.full(tracks, mean))


def test_sorted_batch_is_not_tuned(R, tmp_path, monkeypatch):
    """Nothing synchronises the stream: the first call of all can be captured, and no shape is stored."""
    import torch
    path = tmp_path / "tune.json"
    monkeypatch.setenv("RICH_TUNE_CACHE", str(path))
    src = batch(260, 2100)
    ref = R.propagate_batch(R.Scene(I.scene_g2((20, 33), 20)), src, 3, tune=R.tuning(256, 256, 2))
    gs = R.Scene(I.scene_g2((20, 33), 20))
    b, keep, n = R.make_batch(src)
    t, o = R.alloc_outputs(gs, n)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        R.rich_propagate_batch(gs.handle, b, n, 3, o, None, stream)
    for rep in range(3):
        for k in KEYS:
            t[k].zero_()
        graph.replay()
        torch.cuda.synchronize()
        for k in KEYS:
            assert same(t[k], ref[k]), (rep, k)
        R.rich_propagate_batch(gs.handle, b, n, 3, o, None, stream)    # eager work between the replays
        torch.cuda.synchronize()
    assert int(t["fate_counts"].sum()) == 6 * n and gs.status() == 0
    assert not path.exists()


def test_ordered_batch_is_tuned(R, tmp_path, monkeypatch):
    path = tmp_path / "tune.json"
    monkeypatch.setenv("RICH_TUNE_CACHE", str(path))
    src = batch(3500, 620)
    ref = R.propagate_batch(R.Scene(I.scene_g2((20, 33), 20)), src, 3, tune=R.tuning(256, 256, 2))
    assert not path.exists()
    gs = R.Scene(I.scene_g2((20, 33), 20))
    for _ in range(2):
        out = R.propagate_batch(gs, src, 3)
        for k in KEYS + ("histogram", "fate_counts"):
            assert same(out[k], ref[k]), k
    assert path.exists() and gs.status() == 0
    bad = R.rich_tuning(256, 100, 2, 0)
    with pytest.raises(R.RichError) as e:
        R.propagate_batch(gs, batch(260, 2100), 3, tune=bad)           # refused, sorted or not
    assert e.value.code == R.RICH_EINVAL
