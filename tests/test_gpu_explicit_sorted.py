"""GPU: large launches of photon arrays on meshes are sorted by direction; smaller ones are not.

One launch at and around the limit, and one of more photons than a chunk of
the order buffer, must give, bit for bit, what launches of its parts give; so
must one captured into a graph on a stream that has no order buffer yet.
"""

import numpy as np
import pytest

from paper_2309_12496_amd import inputs as I

pytestmark = pytest.mark.gpu

LIMIT, CHUNK = 1 << 19, 1 << 24
OUTPUTS = ("fate", "pixel", "hit_xyz", "hit_uv", "hit_time")


@pytest.fixture(scope="module")
def R():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2309_12496_amd import rich
    return rich


def photons(n, kind, seed=6):
    rng = np.random.default_rng(seed)
    spread = {"cone": (0.1, 0.1, 0.02), "all round": (1.0, 1.0, 1.0), "parallel": (0.0, 0.0, 0.0)}[kind]
    d = rng.normal(size=(n, 3)) * spread + (0.0, 0.0, 1.0 if kind != "all round" else 0.0)
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    return rng.uniform(-5.0, 5.0, (n, 3)).astype(np.float32), d.astype(np.float32), rng.uniform(200.0, 600.0, n)


def same(a, b):
    return bool(((a == b) | (a.isnan() & b.isnan()) if a.is_floating_point() else a == b).all())


@pytest.mark.parametrize("kind", ["cone", "all round", "parallel"])
@pytest.mark.parametrize("n", [LIMIT - 1, LIMIT, LIMIT + 4097])
@pytest.mark.parametrize("prefilter", [False, True])
def test_one_launch_equals_its_parts(R, n, kind, prefilter):
    gs = R.Scene(I.scene_g2(sphere_quads=(34, 29), box_quads=3))
    o, d, lam = photons(n, kind)
    wrap = I.with_prefilter if prefilter else (lambda s: s)
    whole = R.propagate(gs, wrap(I.explicit_source(o, d, lam)), n, 3)
    step = 200_000
    for lo in range(0, n, step):
        k = slice(lo, min(n, lo + step))
        part = R.propagate(gs, wrap(I.explicit_source(o[k], d[k], lam[k])), k.stop - lo, 3, first_id=lo)
        for key in OUTPUTS:
            assert same(whole[key][k], part[key]), (key, lo)
    assert int(whole["fate_counts"].sum()) == n and gs.status() == 0


@pytest.mark.parametrize("prefilter", [False, True])
def test_more_than_a_chunk(R, prefilter):
    gs = R.Scene(I.scene_g2(sphere_quads=(34, 29), box_quads=3))
    n, m = CHUNK + 5000, 100_000
    o, d, lam = (np.resize(x, (n,) + x.shape[1:]) for x in photons(m, "cone"))
    wrap = I.with_prefilter if prefilter else (lambda s: s)
    whole = R.propagate(gs, wrap(I.explicit_source(o, d, lam)), n, 3)
    k = slice(CHUNK - 5000, n)
    part = R.propagate(gs, wrap(I.explicit_source(o[k], d[k], lam[k])), 10_000, 3, first_id=CHUNK - 5000)
    for key in OUTPUTS:
        assert same(whole[key][k], part[key]), key
    assert int(whole["fate_counts"].sum()) == n and gs.status() == 0


def test_captured_without_an_order_buffer(R):
    import torch
    gs = R.Scene(I.scene_g2(sphere_quads=(34, 29), box_quads=3))
    n = LIMIT + 11
    s, keep = R.make_source(I.explicit_source(*photons(n, "cone")))
    ref, ro = R.alloc_outputs(gs, n, "cuda")
    t, to = R.alloc_outputs(gs, n, "cuda")
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        R.rich_propagate(gs.handle, s, n, 3, 0, to, stream.cuda_stream)
    R.rich_propagate(gs.handle, s, n, 3, 0, ro)
    for _ in range(3):
        t["fate"].fill_(99)
        graph.replay()
        torch.cuda.synchronize()
        for key in OUTPUTS:
            assert same(t[key], ref[key]), key
    assert gs.status() == 0
