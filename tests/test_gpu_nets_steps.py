"""Per-event nets where a step's events with a loss exceed the per-wave queue
(dense layers), where they are few, and where the coarse map's bits cover whole
probe words, against the oracle.  Nets are differences of totals that are each
rounded once, so they agree within 2^-52 of the trial's running total."""

import numpy as np
import pytest

import oracle
from workloads import Layer, make_elt_pool, make_yet

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


@pytest.mark.parametrize("n_trials,lam,C,J,nnz", [
    (300, 700, 9_001, 3, 8_000),            # nearly every event
    (2_000, 90, 50_021, 4, 20_000),         # most events, a start every 90 positions
    (900, 400, 1_200_007, 5, 30_000),       # a coarse bit per two events
    (700, 500, 34_000_000, 1, 30_000),      # a coarse bit per 64 events
    (1, 1_000, 4_096, 2, 1_000),
    (26_500, 520, 9_001, 3, 8_000),         # nearly every event of 9 million: many steps per wave
])
def test_event_nets_queue_and_coarse_map(ara, n_trials, lam, C, J, nnz):
    yet = make_yet(n_trials, lam, C, seed=3 * n_trials + lam)
    pool = make_elt_pool(J, C, nnz, seed=C + 1)
    idx = np.arange(J, dtype=np.int32)[::-1].copy()
    layer = Layer(idx, 2.0e3, 5.0e5, 1.0e5, 4.0e7, n_trials // 5, max(1, n_trials - n_trials // 3))
    ref = oracle.event_nets(yet, pool, layer)
    tables = ara.create_tables(yet.offsets, yet.ids, pool.losses)
    got = ara.event_nets(tables, ara.LayerSpec.from_layer(layer, pool, n_trials))
    tables.close()
    assert got.shape == ref.shape
    b, n = layer.trial_begin, layer.trial_count
    first = int(yet.offsets[b])
    _, o = oracle.occurrence_catalogue(pool, layer)
    lengths = np.diff(yet.offsets[b:b + n + 1])
    S = np.add.reduceat(np.append(o[yet.ids[first:first + ref.shape[0]]], 0.0),
                        np.minimum(yet.offsets[b:b + n] - first, ref.shape[0]))
    S[lengths == 0] = 0.0
    bound = np.repeat(S, lengths) * 2.0 ** -51
    assert np.all(np.abs(got - ref) <= bound)
    assert np.all(got[o[yet.ids[first:first + ref.shape[0]]] == 0.0] == 0.0)
