"""CPU: the tensors of alloc_outputs own their memory, no more than their own.

Fate counts kept from many calls must not keep the calls' histograms alive, nor
be saved with them.
"""

import io
import types

import pytest
import torch

from paper_2309_12496_amd import rich as R


@pytest.mark.parametrize("nx, ny", [(208, 208), (207, 205), (1, 1)])
@pytest.mark.parametrize("per_photon", [True, False])
def test_each_its_own(nx, ny, per_photon):
    t, o = R.alloc_outputs(types.SimpleNamespace(nx=nx, ny=ny), 100, "cpu", per_photon=per_photon, hit_list_capacity=5)
    tensors = {k: v for k, v in t.items() if torch.is_tensor(v)}
    assert len({v.untyped_storage().data_ptr() for v in tensors.values()}) == len(tensors)
    for k, v in tensors.items():
        assert v.untyped_storage().nbytes() == v.numel() * v.element_size(), k
        assert v.storage_offset() == 0 and getattr(o, k) == v.data_ptr(), k
    assert t["histogram"].shape == (nx * ny,) and t["histogram"].dtype == torch.int32 and not t["histogram"].any()
    assert t["fate_counts"].shape == (R.N_FATES,) and t["fate_counts"].dtype == torch.int64
    assert not t["fate_counts"].any()
    f = io.BytesIO()
    torch.save(t["fate_counts"], f)
    assert f.getbuffer().nbytes < 4096
