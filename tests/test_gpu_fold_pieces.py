"""The fold of a layer's tables where a table's entries in a superblock of 4096
events end at, before and after a piece of 512, are none, or are all of it:
per-event occurrence losses, packed values and bitmaps equal the oracle's (the
same sums in the same order)."""

import numpy as np
import pytest

import oracle
from workloads import Layer, make_yet
from workloads.generators import ELTPool

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,counts", [
    (4_096, [511, 512, 513]),
    (4_097, [0, 1, 0, 1024]),
    (70_000, [1025, 0, 0, 4_096, 64, 0]),
    (300_007, [2_048, 3, 1, 0, 513] * 12),
    (9_000, [0]),
    (8_192, [63] * 64),
])
def test_pieces_of_tables(C, counts):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1606_04473_amd import ara
    rng = np.random.default_rng(C)
    J = len(counts)
    losses = np.zeros((J, C))
    for j, n in enumerate(counts):
        for sb in range(0, C, 4096):
            size = min(4096, C - sb)
            pos = sb + rng.choice(size, size=min(n, size), replace=False)
            losses[j, pos] = rng.lognormal(10.0, 2.0, size=pos.size)
    pool = ELTPool(losses, rng.uniform(0.0, 2.0e4, J), rng.uniform(1.0e4, 1.0e6, J))
    yet = make_yet(50, 20, C, seed=J)
    tables = ara.create_tables(yet.offsets, yet.ids, losses)
    for idx in (np.arange(J), np.arange(J)[::-1].copy()):
        layer = Layer(idx.astype(np.int32), 1.0e4, 5.0e5, 0.0, np.inf, 0, 50)
        spec = ara.LayerSpec.from_layer(layer, pool, 50)
        _, o = oracle.occurrence_catalogue(pool, layer)
        assert np.array_equal(ara.debug_read(tables, ara.DEBUG_OCCURRENCE, spec), o)
        assert np.array_equal(ara.debug_read(tables, ara.DEBUG_COMPACT, spec), o[o != 0.0])
    tables.close()
