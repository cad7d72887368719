"""Which 16-bit copy the passes stream, as ara_loss_copy_get reports it: the copy of
the events with a loss in each of its forms (groups of 64, groups of 128 with every
kind of last group, trials cut into columns, both together), and the whole copy's
queue and shared lanes on tables that hold no other.  Losses are whole numbers
where copies are compared, so every order of a sum gives the same."""

import numpy as np
import pytest

import oracle
from workloads import Layer, make_elt_pool, make_yet
from workloads.generators import ELTPool

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


def _layer_and_results(ara, yet, pool, idx, occ_limit, begin, count, p):
    idx = np.array(idx, np.int32)
    _, S = oracle.run_layer(yet, pool, Layer(idx, 0.0, occ_limit, 0.0, np.inf, begin, count))
    layer = Layer(idx, 0.0, occ_limit, float(np.median(S)) * 0.5, float(S.max()) * 0.9 + 1.0, begin, count)
    ref, S = oracle.run_layer(yet, pool, layer)
    g = oracle.gradients(yet, pool, layer, p, ylt=ref, S=S)
    return ara.LayerSpec.from_layer(layer, pool, yet.n_trials), ref, g


# every event of the catalogue has a loss; trials in a last group of 128 trials (1,
# its first half, one more, all but one), with two columns per part, with several
# parts; and groups of 64, the copy's smaller form, with and without columns
@pytest.mark.parametrize("n_trials,lam,C,group,columns", [
    (1_048_577, 4, 9_000, 128, 1),
    (1_048_640, 4, 9_000, 128, 1),
    (1_048_641, 4, 9_000, 128, 1),
    (1_048_703, 4, 9_000, 128, 1),
    (600_001, 50, 9_000, 128, 2),
    (300_001, 30, 90_000, 128, 6),
    (5_000, 300, 20_000, 64, 5),
    (65, 60, 9_000, 64, 2),
])
def test_forms_of_the_loss_copy(ara, n_trials, lam, C, group, columns):
    rng = np.random.default_rng(n_trials + lam)
    losses = rng.integers(0, 3, (2, C)) * 1_000.0
    losses[0, losses.sum(axis=0) == 0] = 3_000.0
    pool = ELTPool(losses, np.array([0.0, 500.0]), np.array([2_500.0, 9_000.0]))
    yet = make_yet(n_trials, lam, C, seed=C)
    tables = ara.create_tables(yet.offsets, yet.ids, losses)
    for idx, begin, count in (([1, 0], 0, n_trials), ([0], n_trials // 3, n_trials - n_trials // 3)):
        spec, ref, g = _layer_and_results(ara, yet, pool, idx, 3_500.0, begin, count, 0.9)
        info = tables.loss_copy([spec])
        assert info["streamed"] == 1 and info["events"] == C
        assert (info["group_trials"], info["columns"], info["groups"]) == (group, columns, -(-n_trials // group))
        assert tables.loss_copy([spec], ara.ARA_LITERAL)["streamed"] == 0
        assert np.array_equal(ara.run_layers(tables, [spec], flags=ara.ARA_CHECKPOINT_S), ref)
        gm, gt = ara.backward(tables, spec, 0.9)
        assert np.array_equal(gm, g["grad_mean"]) and np.array_equal(gt, g["grad_tvar"])
    tables.close()


# one part almost full of losses (past the LDS copy), one part half full, a second
# part of three events, seven parts with a trial or two per full queue, one trial
@pytest.mark.parametrize("n_trials,lam,C,J,nnz", [
    (331, 900, 60_000, 6, 20_000),
    (64, 1400, 20_011, 3, 6_000),
    (1_000, 300, (1 << 16) + 3, 5, 20_000),
    (97, 3_000, 420_000, 9, 30_000),
    (1, 5_000, 40_000, 4, 12_000),
    (200, 1_500, 30_000, 4, 9_000),
])
def test_long_dense_trials_over_the_whole_copy(ara, n_trials, lam, C, J, nnz):
    import torch
    yet = make_yet(n_trials, lam, C, seed=n_trials + lam)
    pool = make_elt_pool(J, C, nnz, seed=C)
    plain = Layer(np.arange(J, dtype=np.int32), 3.0e3, 4.0e5, 0.0, np.inf, 0, n_trials)
    _, S = oracle.run_layer(yet, pool, plain)
    low = float(np.median(S)) * 0.9
    layer = Layer(plain.elt_index, 3.0e3, 4.0e5, low, float(np.max(S)) * 0.97 - low, 0, n_trials)
    ref, S = oracle.run_layer(yet, pool, layer)
    g = oracle.gradients(yet, pool, layer, 0.9, ylt=ref, S=S)
    spec = ara.LayerSpec.from_layer(layer, pool, n_trials)
    base = ara.create_tables(yet.offsets[:1], yet.ids[:0], pool.losses)
    whole = ara.create_yet(base, torch.from_numpy(yet.offsets).cuda(), torch.from_numpy(yet.ids.view(np.int32)).cuda())
    assert whole.layout()["stream_parts"] > 0 and whole.loss_copy([spec])["columns"] == 0
    ylt = ara.run_layers(whole, [spec], flags=ara.ARA_CHECKPOINT_S)
    # both round an exact or double-double sum once
    assert np.all(np.abs(ara.read_checkpoints(whole, 0) - S) <= 1e-12 * S)
    assert np.all(np.abs(ylt - ref) <= 1e-12 * S)
    gm, gt = ara.backward(whole, spec, 0.9)
    assert np.array_equal(gm, g["grad_mean"]) and np.array_equal(gt, g["grad_tvar"])
    lo, n = n_trials // 3, max(1, n_trials // 2)
    part = ara.LayerSpec(spec.elt_index, spec.elt_retention, spec.elt_limit, spec.occ_retention, spec.occ_limit,
                         spec.agg_retention, spec.agg_limit, lo, n)
    assert np.array_equal(ara.run_layers(whole, [part]), ylt[lo:lo + n])
    whole.close()
    base.close()
