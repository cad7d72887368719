"""Building the copy of the events with a loss: each way of telling which events those
are at the edges of its catalogue sizes (their words whole in LDS, a bit per event, per
two), scans of trials at the edges of a round, tables whose copy turns out not to be
usable.  Losses are whole numbers, so every order of a sum gives the same."""

import numpy as np
import pytest

import oracle
from workloads import Layer, make_yet
from workloads.generators import YET, ELTPool

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


def _check(ara, yet, pool, copy):
    n = yet.n_trials
    tables = ara.create_tables(yet.offsets, yet.ids, pool.losses)
    info = tables.loss_copy()
    assert (info["columns"] > 0) == copy
    assert info["events"] == (np.count_nonzero(pool.losses.any(axis=0)) if copy else 0)
    for idx in ([0, 1], [1]):
        layer = Layer(np.array(idx, np.int32), 0.0, 3_500.0, 1_000.0, np.inf, 0, n)
        spec = ara.LayerSpec.from_layer(layer, pool, n)
        ref, S = oracle.run_layer(yet, pool, layer)
        assert np.array_equal(ara.run_layers(tables, [spec], flags=ara.ARA_CHECKPOINT_S), ref)
        g = oracle.gradients(yet, pool, layer, 0.9, ylt=ref, S=S)
        gm, gt = ara.backward(tables, spec, 0.9)
        assert np.array_equal(gm, g["grad_mean"]) and np.array_equal(gt, g["grad_tvar"])
    tables.close()


# catalogues whose probe words fit in LDS whole (to 638,976) and with a bit per event
# (to 1,277,952); one part of events with a loss, and several; long and short trials
@pytest.mark.parametrize("C", [638_976, 638_977, 1_277_952, 1_277_953])
@pytest.mark.parametrize("every,n_trials,lam", [(100, 300, 900), (9, 2_000, 60)])
def test_filters(ara, C, every, n_trials, lam):
    rng = np.random.default_rng(C + every)
    losses = np.zeros((2, C))
    at = np.unique(np.concatenate([np.arange(0, C, every), [C - 1]]))
    losses[rng.integers(0, 2, at.size), at] = rng.integers(1, 6, at.size) * 1_000.0
    pool = ELTPool(losses, np.array([0.0, 500.0]), np.array([2_500.0, 9_000.0]))
    yet = make_yet(n_trials, lam, C, seed=every)
    yet.ids[::7] = C - 1                            # the last event, in the last word
    _check(ara, yet, pool, True)


@pytest.mark.parametrize("n_trials", [15, 16, 17, 1_024, 16_383, 16_384, 16_385, 32_769])
def test_scans_of_trials(ara, n_trials):
    C = 5_000
    rng = np.random.default_rng(n_trials)
    pool = ELTPool(rng.integers(0, 4, (2, C)) * 1_000.0, np.zeros(2), np.full(2, 9_000.0))
    _check(ara, make_yet(n_trials, 20, C, seed=n_trials), pool, True)


def test_a_copy_past_its_positions(ara):
    """One trial with 150,000 events of a part of the copy, past its 16-bit positions,
    and at most 65,535 of each part of the whole copy."""
    C = 200_000
    rng = np.random.default_rng(1)
    losses = np.zeros((2, C))
    losses[:, ::10] = rng.integers(1, 6, (2, C // 10)) * 1_000.0
    ids = (rng.integers(0, C // 10, 150_000) * 10).astype(np.uint32)
    yet = YET(np.array([0, 150_000, 150_000], np.int64), ids, C)
    assert np.bincount(ids >> 16).max() < 65_536
    _check(ara, yet, ELTPool(losses, np.zeros(2), np.full(2, 9_000.0)), False)
