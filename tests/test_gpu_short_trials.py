"""Counting tables of short trials, a thread per trial: averages on both sides of 16
events, trials at the edges of a workgroup and of the 64 events a thread counts, one
trial of most of the events among empty ones, one part to 64, and bad offsets and IDs
refused as for others.  The 16-bit copy equals NumPy's; the 32-bit copy's passes agree
with the oracle within 1e-12 relative (both round a sum once)."""

import numpy as np
import pytest

import oracle
from test_gpu_indexing import _check_stream
from workloads import Layer, make_elt_pool
from workloads.generators import YET

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ara():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    from paper_1606_04473_amd import ara as mod
    mod.lib()
    return mod


_R = np.random.default_rng(8)
CASES = {
    "one_trial": ([5], 70_000),
    "a_workgroup": (_R.integers(0, 9, 256), 300_000),
    "one_more": (_R.integers(0, 9, 257), 300_000),
    "at_64": (np.tile([64, 65, 0, 0, 0, 0, 0, 0, 0, 63, 0, 0, 0, 0, 0, 0, 0], 40), 64 << 16),
    "below_16": (np.append(np.full(999, 16), 15), 131_073),
    "at_16": (np.full(1_000, 16), 131_073),
    "one_long_trial": (np.insert(np.zeros(20_000, np.int64), 7_001, 200_000), 40 << 16),
    "no_16_bit_copy": (_R.integers(0, 20, 2_000), (64 << 16) + 1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_counts_of_short_trials(ara, name):
    import torch
    lengths, C = CASES[name]
    rng = np.random.default_rng(C % 1000)
    offsets = np.zeros(len(lengths) + 1, dtype=np.int64)
    offsets[1:] = np.cumsum(lengths)
    yet = YET(offsets, rng.integers(0, C, int(offsets[-1])).astype(np.uint32), C)
    pool = make_elt_pool(2, C, min(C, 30_000), seed=9)
    layer = Layer(np.array([1, 0], dtype=np.int32), 1.0e3, 4.0e5, 1.0e4, 9.0e7, 0, yet.n_trials)
    ref, S = oracle.run_layer(yet, pool, layer)
    spec = ara.LayerSpec.from_layer(layer, pool, yet.n_trials)
    base = ara.create_tables(yet.offsets, yet.ids, pool.losses)
    off, ids = torch.from_numpy(yet.offsets).cuda(), torch.from_numpy(yet.ids.view(np.int32)).cuda()
    for t in (ara.create_yet(base, off, ids), base):
        if t.layout()["stream_parts"] > 0:
            _check_stream(ara, t, yet)
        for variant in (0, 2):
            ara.set_tuning(t, pass_variant=variant)
            assert np.all(np.abs(ara.run_layers(t, [spec]) - ref) <= 1e-12 * S), variant
        if t is not base:
            t.close()
    if yet.n_trials > 2 and yet.ids.size:
        down, bad = yet.offsets.copy(), yet.ids.copy()
        down[1] = down[-1] + 1
        bad[-1] = C
        for o, i, status in ((down, yet.ids, ara.ARA_ERR_INVALID_ARG), (yet.offsets, bad, ara.ARA_ERR_OUT_OF_RANGE),
                             (down, bad, ara.ARA_ERR_OUT_OF_RANGE)):
            with pytest.raises(ara.AraError) as e:
                ara.create_yet(base, torch.from_numpy(o).cuda(), torch.from_numpy(i.view(np.int32)).cuda())
            assert e.value.status == status
    base.close()
