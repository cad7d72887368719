"""Portfolios in many more splits than trials, up to the largest count the call
takes, and in splits whose layers need more scratch than one batch: the same
year losses as unsplit, bit for bit (trials are independent)."""

import numpy as np
import pytest

import oracle
from workloads import Layer, make_elt_pool, make_yet

pytestmark = pytest.mark.gpu


# 600,000 trials over 64 parts: 12 bytes of partial sums each, past a batch's 384 MB
@pytest.mark.parametrize("n_trials,lam,C,splits", [
    (1_000, 60, 90_000, [999, 1_000, 1_001, 2 ** 31 - 1]),
    (600_000, 3, 64 << 16, [2, 7_001, 2 ** 31 - 1]),
])
def test_portfolio_in_many_splits(n_trials, lam, C, splits):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1606_04473_amd import ara
    yet = make_yet(n_trials, lam, C, seed=lam)
    pool = make_elt_pool(3, C, C // 8, seed=5)
    layers = [Layer(np.array(idx, np.int32), 2.0e3, 4.0e5, 1.0e4, 3.0e7, 0, n_trials) for idx in ([0, 1, 2], [1], [2, 0])]
    specs = [ara.LayerSpec.from_layer(l, pool, n_trials) for l in layers]
    both = ara.create_tables(yet.offsets, yet.ids, pool.losses)
    whole = ara.create_yet(both, torch.from_numpy(yet.offsets).cuda(), torch.from_numpy(yet.ids.view(np.int32)).cuda())
    for tables in (whole, both):
        want = ara.run_portfolio(tables, [specs[:2], specs[2:]])
        for layer, row in zip(layers, want["layer"]):
            ref, S = oracle.run_layer(yet, pool, layer)
            assert np.all(np.abs(row - ref) <= 1e-12 * S)
        for n in splits:
            got = ara.run_portfolio(tables, [specs[:2], specs[2:]], n_splits=n)
            assert all(np.array_equal(got[k], want[k]) for k in want), n
        tables.close()
