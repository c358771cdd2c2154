"""GPU: the histogram and fate counts of alloc_outputs, which share a buffer, for even and odd pixel counts."""

import copy

import pytest

from paper_2309_12496_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx, ny", [(208, 208), (207, 205), (1, 1)])
@pytest.mark.parametrize("per_photon", [True, False])
def test_counters(nx, ny, per_photon):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2309_12496_amd import rich as R
    sc = copy.deepcopy(I.scene_g1())
    sc["detector"] |= {"nx": nx, "ny": ny}
    gs = R.Scene(sc)
    n = 3000
    s, keep = R.make_source(I.point_source())
    t, o = R.alloc_outputs(gs, n, "cuda", per_photon=per_photon)
    assert t["histogram"].shape == (nx * ny,) and t["histogram"].dtype == torch.int32
    assert t["fate_counts"].shape == (R.N_FATES,) and t["fate_counts"].dtype == torch.int64
    for k in ("histogram", "fate_counts"):
        assert t[k].is_contiguous() and not t[k].any() and t[k].data_ptr() % 64 == 0
    for calls in (1, 2):                                # they accumulate
        R.rich_propagate(gs.handle, s, n, 5, 0, o)
        assert int(t["fate_counts"].sum()) == calls * n
    full = R.propagate(gs, I.point_source(), n, 5)
    assert torch.equal(t["fate_counts"], 2 * full["fate_counts"])
    pixel = full["pixel"][full["fate"] == R.DETECTED].long()
    assert torch.equal(t["histogram"].long(), 2 * torch.bincount(pixel[pixel >= 0], minlength=nx * ny))
