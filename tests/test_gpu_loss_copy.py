"""The copy of the events with a loss in some table: its parts' boundary (20479
events), its groups of 64 trials and of 128 in pairs, trials split into columns,
unions of one event and of none, each way of finding an event's slot at creation,
empty trials.  Year losses and gradients equal the oracle's and those of tables without that copy
(losses are whole numbers, so every order of a sum gives the same)."""

import numpy as np
import pytest

import oracle
from workloads import Layer, make_yet
from workloads.generators import ELTPool

pytestmark = pytest.mark.gpu


# union: events of each superblock of 4096 with a loss, the last entry repeated
@pytest.mark.parametrize("n_trials,lam,C,union", [
    (300, 900, 20_480, [4096, 4096, 4096, 4096, 4095]),     # one full part
    (300, 900, 20_480, [4096]),                             # one event more: two
    (1_000, 700, 66_000, [4096]),                           # five parts
    (63, 60, 9_000, [900]),
    (64, 60, 9_000, [900]),
    (65, 60, 9_000, [900]),
    (5_000, 300, 20_000, [4096]),                           # five columns
    (1, 50_000, 9_000, [4096]),
    (500, 400, 4_097, [0, 1]),                              # one event
    (500, 400, 9_000, [0]),                                 # none
    (3_000, 4, 9_000, [700]),                               # empty trials
    (400, 3_000, 1_300_000, [50]),                          # a bit per two events
    (400, 3_000, 3_000_000, [25]),                          # per four
    (200, 4_000, 5_200_000, [13]),                          # no map
    (1_048_576, 4, 9_000, [4096]),                          # pairs: whole groups, short
    (1_048_703, 8, 9_000, [3000, 0]),                       # a group of 127
    (300_001, 30, 90_000, [4096]),                          # several parts, a group of 97
    (1_100_001, 5, 9_000, [3500, 1]),                       # a group of 97, empty trials
])
def test_against_the_whole_copy(n_trials, lam, C, union):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1606_04473_amd import ara
    rng = np.random.default_rng(n_trials + lam + C)
    J = 3
    losses = np.zeros((J, C))
    for k, sb in enumerate(range(0, C, 4096)):
        size = min(4096, C - sb)
        pos = sb + rng.choice(size, size=min(union[min(k, len(union) - 1)], size), replace=False)
        losses[rng.integers(0, J, pos.size), pos] = rng.integers(1, 9, pos.size) * 1_000.0
    pool = ELTPool(losses, np.array([0.0, 1_000.0, 0.0]), np.array([8_000.0, 6_000.0, 5_000.0]))
    yet = make_yet(n_trials, lam, C, seed=C)
    tables = ara.create_tables(yet.offsets, yet.ids, losses)
    whole = ara.create_yet(tables, torch.from_numpy(yet.offsets).cuda(), torch.from_numpy(yet.ids.view(np.int32)).cuda())
    layers = []
    for idx, lo, n in (([2, 0, 1], 0, n_trials), ([1], 0, n_trials),
                       ([0, 1, 2], n_trials // 3, n_trials - n_trials // 3), ([0, 2], n_trials // 2, 1)):
        idx = np.array(idx, np.int32)
        _, S = oracle.run_layer(yet, pool, Layer(idx, 0.0, 7_000.0, 0.0, np.inf, lo, n))
        layers.append(Layer(idx, 0.0, 7_000.0, float(np.median(S)) * 0.5, float(S.max()) * 0.9 + 1.0, lo, n))
    specs = [ara.LayerSpec.from_layer(l, pool, n_trials) for l in layers]
    refs = [oracle.run_layer(yet, pool, l) for l in layers]
    for t in (tables, whole):
        assert np.array_equal(ara.run_layers(t, specs), np.concatenate([r for r, _ in refs]))
        for layer, spec, (ref, S) in zip(layers, specs, refs):
            assert np.array_equal(ara.run_layers(t, [spec], flags=ara.ARA_CHECKPOINT_S), ref)
            g = oracle.gradients(yet, pool, layer, 0.9, ylt=ref, S=S)
            gm, gt = ara.backward(t, spec, 0.9)
            assert np.array_equal(gm, g["grad_mean"])
            assert np.array_equal(gt, g["grad_tvar"])
    whole.close()
    tables.close()
