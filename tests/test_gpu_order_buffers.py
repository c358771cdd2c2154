"""GPU: order buffers: a captured launch keeps its own, and a scene's first stream has one from the start.

A captured launch replays to its outputs after larger launches of other kinds on
its stream.  The order buffer that a graph was captured with grows under launches of photon
arrays and batches too.  The graph's own has to stay: memory allocated after
the growth is not the graph's to write.
"""

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


def photon_arrays(n, seed=5):
    rng = np.random.default_rng(seed)
    d = np.array((0.0, 0.0, 1.0)) + 0.05 * rng.normal(size=(n, 3))
    return I.explicit_source(np.zeros((n, 3)), d / np.linalg.norm(d, axis=1, keepdims=True), np.full(n, 400.0))


def long_batch(tracks, mean, seed=6):
    rng = np.random.default_rng(seed)
    return I.batch_source(I.sample_tracks(rng, tracks), np.full(tracks, mean))


@pytest.mark.parametrize("captured", ["track", "batch"])
@pytest.mark.parametrize("larger", ["batch", "arrays", "track"])
def test_captured_launch_after_a_larger_one(R, captured, larger):
    import torch
    gs = R.Scene(I.scene_g2((20, 33), 20))
    R.propagate(gs, I.point_source(), 1000, 1)            # the scene's first stream: it is made with a buffer for that
    stream = torch.cuda.Stream()
    tune = R.tuning(256, 256, 2)
    if captured == "track":
        n = 300_001
        s, keep = R.make_source(I.point_source(length=1000.0))
        launch = lambda o: R.rich_propagate(gs.handle, s, n, 3, 0, o, stream)
    else:
        s, keep, n = R.make_batch(long_batch(260, 2100))
        launch = lambda o: R.rich_propagate_batch(gs.handle, s, n, 3, o, tune, stream)
    t, o = R.alloc_outputs(gs, n)
    torch.cuda.synchronize()
    launch(o)                                             # the stream's buffers, at this launch's size
    torch.cuda.synchronize()
    ref = {k: t[k].clone() for k in KEYS}
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        launch(o)
    if larger == "batch":
        b, keep_b, m = R.make_batch(long_batch(2200, 1000))
        big, ob = R.alloc_outputs(gs, m)
        torch.cuda.synchronize()
        R.rich_propagate_batch(gs.handle, b, m, 4, ob, tune, stream)
    else:
        m = 2_300_000
        e, keep_e = R.make_source(photon_arrays(m) if larger == "arrays" else I.point_source())
        big, ob = R.alloc_outputs(gs, m)
        torch.cuda.synchronize()
        R.rich_propagate(gs.handle, e, m, 4, 0, ob, stream)
    torch.cuda.synchronize()
    # what the allocator hands out now lies in no buffer of a captured launch
    marks = [torch.full((k,), 0x5A5A5A5A, dtype=torch.int32, device="cuda") for k in (300_001, 546_000, 600_002, 1 << 21)]
    for rep in range(3):
        for k in KEYS:
            t[k].zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for k in KEYS:
            assert same(t[k], ref[k]), (rep, k)
        assert all(bool((x == 0x5A5A5A5A).all()) for x in marks), rep
        other = R.propagate(gs, I.point_source(), 1000, rep)      # eager work between the replays
        assert int(other["fate_counts"].sum()) == 1000
    assert gs.status() == 0


@pytest.mark.parametrize("source", ["arrays", "track", "batch"])
def test_first_call_allocates_nothing(R, source):
    import torch
    if source == "batch":
        s, keep, n = R.make_batch(long_batch(600, 2500))
        launch = lambda gs, o: R.rich_propagate_batch(gs.handle, s, n, 3, o, R.tuning(256, 256, 2))
    else:
        n = 1_500_000
        s, keep = R.make_source(photon_arrays(n) if source == "arrays" else I.point_source(length=1000.0))
        launch = lambda gs, o: R.rich_propagate(gs.handle, s, n, 3, 0, o)
    outs = []
    for _ in range(2):                                    # the first loads the kernels
        gs = R.Scene(I.scene_g2((20, 33), 20))
        t, o = R.alloc_outputs(gs, n)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        launch(gs, o)
        torch.cuda.synchronize()
        outs.append((gs, t, before - torch.cuda.mem_get_info()[0]))
    assert outs[1][2] == 0, outs[1][2]
    assert int(outs[1][1]["fate_counts"].sum()) == n and outs[1][0].status() == 0
