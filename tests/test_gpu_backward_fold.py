"""The backward's fold and its pass over the tables' entries: tables with none, a
few and more entries than a wave takes at once in a chunk of 4096 events, more
tables than waves, chunks past the catalogue's end, events at the kinks of the
occurrence terms, with the copies of the YET and without.  Gradients equal the
oracle's (ratios of integers)."""

import numpy as np
import pytest

import oracle
from workloads import Layer, make_yet
from workloads.generators import ELTPool

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,counts,n_trials,lam", [
    (4_096, [0], 300, 40),
    (4_097, [1, 0, 64], 300, 40),
    (9_000, [63, 64, 65, 0, 128, 700, 0, 0, 1, 2], 2_000, 30),
    (300_007, [40] * 31, 1_111, 900),
    (70_000, [2_500, 0, 129], 700, 300),
    (66_000, [17] * 64, 5, 2_000),
])
def test_gradients_of_tables(C, counts, n_trials, lam):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1606_04473_amd import ara
    rng = np.random.default_rng(C + lam)
    J = len(counts)
    losses = np.zeros((J, C))
    for j, n in enumerate(counts):
        for sb in range(0, C, 4096):
            size = min(4096, C - sb)
            pos = sb + rng.choice(size, size=min(n, size), replace=False)
            # whole numbers, so sums hit the occurrence terms exactly
            losses[j, pos] = rng.integers(1, 9, size=pos.size) * 1_000.0
    pool = ELTPool(losses, rng.integers(0, 3, J) * 1_000.0, rng.integers(2, 6, J) * 1_000.0)
    yet = make_yet(n_trials, lam, C, seed=J)
    idx = rng.permutation(J).astype(np.int32)
    free = Layer(idx, 1_000.0, 3_000.0, 0.0, np.inf, 0, n_trials)
    _, S = oracle.run_layer(yet, pool, free)
    layer = Layer(idx, 1_000.0, 3_000.0, float(np.median(S)) * 0.5, float(S.max()) * 0.9 + 1.0, 0, n_trials)
    ref, S = oracle.run_layer(yet, pool, layer)
    g = oracle.gradients(yet, pool, layer, 0.9, ylt=ref, S=S)
    spec = ara.LayerSpec.from_layer(layer, pool, n_trials)
    for flags in (0, ara.ARA_PLAIN_LAYOUT):
        tables = ara.create_tables(yet.offsets, yet.ids, losses, flags=flags)
        for variant in (0, 2):
            ara.set_tuning(tables, pass_variant=variant)
            ylt = ara.run_layers(tables, [spec], flags=ara.ARA_CHECKPOINT_S)
            assert np.array_equal(ylt, ref)
            gm, gt = ara.backward(tables, spec, 0.9)
            assert np.array_equal(gm, g["grad_mean"]), (flags, variant)
            assert np.array_equal(gt, g["grad_tvar"]), (flags, variant)
        tables.close()
