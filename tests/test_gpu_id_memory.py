"""Creating tables from IDs given as device memory that is not this device's own:
such IDs are copied by the runtime, not read by a kernel.  Pinned host memory stands
in for another device's."""

import ctypes

import numpy as np
import pytest

from workloads import make_elt_pool, make_yet

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_trials,lam", [(1, 1), (500, 37)])
def test_ids_outside_the_device(n_trials, lam):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1606_04473_amd import ara
    C = 70_000
    yet = make_yet(n_trials, lam, C, seed=lam)
    pool = make_elt_pool(2, C, 9_000, seed=1)
    base = ara.create_tables(yet.offsets, yet.ids, pool.losses)
    offsets = torch.from_numpy(yet.offsets).cuda()
    ids = torch.empty(max(yet.ids.size, 1), dtype=torch.int32, pin_memory=True)
    ids[:yet.ids.size].copy_(torch.from_numpy(yet.ids.view(np.int32)))
    torch.cuda.synchronize()
    h = ctypes.c_void_p()
    ara._check(ara.lib().ara_create_yet(base.handle, offsets.data_ptr(), n_trials, ids.data_ptr(), yet.ids.size,
                                        ara.ARA_DEVICE_PTR, ara._stream(None), ctypes.byref(h)))
    other = ara.Tables(h, n_trials, yet.ids.size, C, 2)
    spec = ara.LayerSpec(np.arange(2, dtype=np.int32), np.zeros(2), np.full(2, 1e9), 0.0, 1e9, 0.0, 1e12, 0, n_trials)
    for variant in (0, 2):
        ara.set_tuning(base, pass_variant=variant)
        ara.set_tuning(other, pass_variant=variant)
        assert np.array_equal(ara.run_layers(other, [spec]), ara.run_layers(base, [spec]))
    other.close()
    base.close()
