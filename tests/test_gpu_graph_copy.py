"""Graph replays whose ELT choices change which 16-bit copy is the faster to stream:
each replay equals the eager call bit for bit.  Trial 0 holds losses 1, 2^-53 and
2^-100 in one part of the whole copy and two parts of the copy of the events with a
loss: a part's partial sum keeps 24 bits of its low half, so the year loss is 1 over
the first copy and 1 + 2^-52 over the second, which tells them apart."""

import numpy as np
import pytest

from workloads import make_elt_pool, make_yet

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first", [0, 1])
def test_replays_follow_the_choice(first):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1606_04473_amd import ara
    n, C, J = 10_000, 400_000, 60
    yet = make_yet(n, 400, C, seed=11)
    pool = make_elt_pool(J, C, 20_000, seed=12)
    marks = [0, 1, 65_000]
    pool.losses[:, marks] = 0.0
    pool.losses[0, marks] = [1.0, 2.0 ** -53, 2.0 ** -100]
    yet.ids[:yet.offsets[1]] = 2                    # trial 0: the three events and one without a loss
    pool.losses[:, 2] = 0.0
    yet.ids[:3] = marks
    tables = ara.create_tables(yet.offsets, yet.ids, pool.losses)
    specs = []
    for k in (1, J):
        idx = np.arange(k, dtype=np.int32)
        specs.append(ara.LayerSpec(idx, np.zeros(k), np.full(k, np.inf), 0.0, np.inf, 0.0, np.inf, 0, n))
    assert [tables.loss_copy([s])["streamed"] for s in specs] == [0, 1]
    want = [ara.run_layers(tables, [s]) for s in specs]
    assert [w[0] for w in want] == [1.0, 1.0 + 2.0 ** -52]
    probs = [0.9]
    metrics = [ara.analyze(tables, s, probs)[1] for s in specs]
    ylt = torch.empty(n, dtype=torch.float64, device="cuda")
    two = torch.empty(2 * n, dtype=torch.float64, device="cuda")
    out = torch.empty(3, dtype=torch.float64, device="cuda")
    stream = torch.cuda.Stream()
    for k in (first, 1 - first, first, first, 1 - first):
        ylt.fill_(-1.0)
        torch.cuda.synchronize()
        ara.run_layers(tables, [specs[k]], out=ylt, flags=ara.ARA_GRAPH, stream=stream)
        stream.synchronize()
        assert np.array_equal(ylt.cpu().numpy(), want[k])
        ylt.fill_(-1.0)
        out.fill_(-1.0)
        torch.cuda.synchronize()
        ara.analyze(tables, specs[k], probs, ylt=ylt, metrics=out, flags=ara.ARA_GRAPH, stream=stream)
        stream.synchronize()
        assert np.array_equal(ylt.cpu().numpy(), want[k]) and np.array_equal(out.cpu().numpy(), metrics[k])
        pair = [specs[k], specs[k]]
        two.fill_(-1.0)
        torch.cuda.synchronize()
        ara.run_layers(tables, pair, out=two, flags=ara.ARA_GRAPH, stream=stream)
        stream.synchronize()
        assert np.array_equal(two.cpu().numpy(), np.concatenate([want[k], want[k]]))
    tables.close()
