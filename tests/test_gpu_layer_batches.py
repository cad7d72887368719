"""Several layers, ranges and splits through shared launches of the streaming
pass: every year loss bit-identical to the layer run by itself (the same
exact sums, rounded once), eager, replayed from a graph and as a portfolio."""

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


# trials, mean events, catalogue, losses per table, layers: two layers; more
# layers than a batch takes units; folds of 48 layers past the scratch of a
# batch (four parts of 2^18 events, 9 MB each); a dense catalogue whose passes
# share lanes; one trial; few long trials
@pytest.mark.parametrize("n_trials,lam,C,nnz,n_layers", [
    (700, 60, 1_000_003, 9_000, 2),
    (333, 40, 70_001, 5_000, 70),
    (515, 50, 1_000_003, 2_000, 48),
    (400, 500, 20_011, 9_000, 7),
    (1, 900, 300_000, 9_000, 33),
    (37, 2_500, 140_000, 12_000, 5),
])
def test_layers_and_splits_share_launches(ara, n_trials, lam, C, nnz, n_layers):
    import torch
    rng = np.random.default_rng(C + n_layers)
    yet = make_yet(n_trials, lam, C, seed=n_trials)
    pool = make_elt_pool(8, C, nnz, seed=C)
    layers = []
    for i in range(n_layers):
        lo = int(rng.integers(0, n_trials))
        n = 0 if i % 9 == 4 else int(rng.integers(1, n_trials - lo + 1))
        if i % 5 == 0:
            lo, n = 0, n_trials
        idx = rng.permutation(8)[:1 + i % 8].astype(np.int32)
        layers.append(Layer(idx, 500.0 * (i % 4), 4.0e5, 1.0e4 * (i % 3), 3.0e6 + i, lo, n))
    specs = [ara.LayerSpec.from_layer(l, pool, n_trials) for l in layers]
    both = ara.create_tables(yet.offsets, yet.ids, pool.losses)
    # tables without the copy of the events with a loss
    whole = ara.create_yet(both, torch.from_numpy(yet.offsets).cuda(), torch.from_numpy(yet.ids.view(np.int32)).cuda())
    for tables in (whole, both):
        assert tables.layout()["stream_parts"] > 0
        single = [ara.run_layers(tables, [s]) for s in specs]
        want = np.concatenate(single)
        for l, y in list(zip(layers, single))[:3]:
            ref, S = oracle.run_layer(yet, pool, l)
            assert np.all(np.abs(y - ref) <= 1e-12 * S)
        assert np.array_equal(ara.run_layers(tables, specs), want)
        bytes_ = ara.footprint(tables, specs)
        assert bytes_ >= max(ara.footprint(tables, [s]) for s in specs)

        out = torch.empty(want.size, dtype=torch.float64, device="cuda")
        stream = torch.cuda.Stream()
        for _ in range(3):
            out.fill_(-1.0)
            torch.cuda.synchronize()
            ara.run_layers(tables, specs, out=out, flags=ara.ARA_GRAPH, stream=stream)
            stream.synchronize()
            assert np.array_equal(out.cpu().numpy(), want)

        # every layer over one range of trials, as programs in uneven splits
        lo, n = n_trials // 4, n_trials - n_trials // 4
        over = [ara.LayerSpec(s.elt_index, s.elt_retention, s.elt_limit, s.occ_retention, s.occ_limit, s.agg_retention,
                              s.agg_limit, lo, n) for s in specs]
        alone = np.stack([ara.run_layers(tables, [s]) for s in over])
        half = (n_layers + 1) // 2
        for n_splits in (1, 3, 7):
            res = ara.run_portfolio(tables, [over[:half], over[half:]], n_splits=n_splits)
            assert np.array_equal(res["layer"], alone)
        tables.close()
