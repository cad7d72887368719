"""The streaming pass where a trial has many losses in one catalogue part: the
queue fills before its group of trials ends and several lanes share a trial.
Year losses against the oracle within 1e-12 relative (both round an exact or
double-double sum once), gradients equal (ratios of integers)."""

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


# trials, mean events, catalogue, tables, losses per table: one part almost
# full of losses (past the LDS copy), one part half full, a second part of
# three events, seven parts with a trial or two per full queue, one trial
@pytest.mark.parametrize("n_trials,lam,C,J,nnz", [
    (331, 900, 60_000, 6, 20_000),
    (64, 1400, 20_011, 3, 6_000),
    (1_000, 300, (1 << 16) + 3, 5, 20_000),
    (97, 3_000, 420_000, 9, 30_000),
    (1, 5_000, 40_000, 4, 12_000),
    (200, 1_500, 30_000, 4, 9_000),
])
def test_long_dense_trials(ara, n_trials, lam, C, J, nnz):
    yet = make_yet(n_trials, lam, C, seed=n_trials + lam)
    pool = make_elt_pool(J, C, nnz, seed=C)
    idx = np.arange(J, dtype=np.int32)
    plain = Layer(idx, 3.0e3, 4.0e5, 0.0, np.inf, 0, n_trials)
    _, S = oracle.run_layer(yet, pool, plain)
    low = float(np.median(S)) * 0.9
    layer = Layer(idx, 3.0e3, 4.0e5, low, float(np.max(S)) * 0.97 - low, 0, n_trials)
    ref, S = oracle.run_layer(yet, pool, layer)
    spec = ara.LayerSpec.from_layer(layer, pool, n_trials)
    tables = ara.create_tables(yet.offsets, yet.ids, pool.losses)
    assert tables.layout()["stream_parts"] > 0
    ylt = ara.run_layers(tables, [spec], flags=ara.ARA_CHECKPOINT_S)
    assert np.all(np.abs(ara.read_checkpoints(tables, 0) - S) <= 1e-12 * S)
    assert np.all(np.abs(ylt - ref) <= 1e-12 * S)
    gm, gt = ara.backward(tables, spec, 0.9)
    g = oracle.gradients(yet, pool, layer, 0.9, ylt=ref, S=S)
    assert np.array_equal(gm, g["grad_mean"]) and np.array_equal(gt, g["grad_tvar"])
    # a range of trials that starts and ends inside groups
    lo, n = n_trials // 3, max(1, n_trials // 2)
    part = ara.LayerSpec(spec.elt_index, spec.elt_retention, spec.elt_limit, spec.occ_retention, spec.occ_limit,
                         spec.agg_retention, spec.agg_limit, lo, n)
    assert np.array_equal(ara.run_layers(tables, [part]), ylt[lo:lo + n])
    tables.close()


# dense parts (past the backward's 32-bit counters) where one event makes up four
# fifths of the table: a workgroup's 16-bit counter of it passes 2^15; long
# trials (lanes share a trial) and short ones
@pytest.mark.parametrize("n_trials,lam", [(12_000, 2_000), (800_000, 28)])
def test_one_event_past_a_counter(ara, n_trials, lam):
    import torch
    C = 60_000
    yet = make_yet(n_trials, lam, C, seed=lam)
    rng = np.random.default_rng(lam)
    yet.ids[rng.random(yet.ids.size) < 0.8] = 77
    pool = make_elt_pool(3, C, 25_000, seed=5)
    pool.losses[0, 77] = 12_345.0
    idx = np.arange(3, dtype=np.int32)
    layer = Layer(idx, 0.0, 4.0e6, 1.0, np.inf, 0, n_trials)
    spec = ara.LayerSpec.from_layer(layer, pool, n_trials)
    both = ara.create_tables(yet.offsets, yet.ids, pool.losses)
    # tables without the copy of the events with a loss
    whole = ara.create_yet(both, torch.from_numpy(yet.offsets).cuda(), torch.from_numpy(yet.ids.view(np.int32)).cuda())
    ref, S = oracle.run_layer(yet, pool, layer)
    g = oracle.gradients(yet, pool, layer, 0.9, ylt=ref, S=S)
    for tables in (whole, both):
        assert tables.layout()["stream_parts"] == 1
        ara.run_layers(tables, [spec], flags=ara.ARA_CHECKPOINT_S)
        gm, gt = ara.backward(tables, spec, 0.9)
        assert np.array_equal(gm, g["grad_mean"]) and np.array_equal(gt, g["grad_tvar"])
        tables.close()
