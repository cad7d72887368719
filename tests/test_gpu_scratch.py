"""Device memory that calls keep: what their passes use, and no dense array of the
catalogue's occurrence losses (8 bytes an event) that nothing reads."""

import numpy as np
import pytest

from workloads import make_elt_pool, make_yet

pytestmark = pytest.mark.gpu

MB = 1 << 20


@pytest.mark.parametrize("whole", [False, True])
def test_kept_scratch(whole):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1606_04473_amd import ara
    n, C = 2_000, 4_000_000                         # 32 MB of occurrence losses, part images 34 MB
    yet = make_yet(n, 50, C, seed=1)
    pool = make_elt_pool(2, C, 5_000, seed=2)
    base = ara.create_tables(yet.offsets, yet.ids, pool.losses)
    tables = ara.create_yet(base, yet.offsets, yet.ids) if whole else base
    idx = np.arange(2, dtype=np.int32)
    spec = ara.LayerSpec(idx, np.zeros(2), np.full(2, 1e9), 0.0, 1e9, 0.0, 1e12, 0, n)
    assert tables.loss_copy([spec])["streamed"] == (0 if whole else 1)
    fold = 35 * MB if whole else MB                 # the images and packed losses, or the table by slot
    want = ara.run_layers(tables, [spec])
    ylt = torch.empty(n, dtype=torch.float64, device="cuda")
    metrics = torch.empty(3, dtype=torch.float64, device="cuda")
    nets = torch.empty(yet.ids.size, dtype=torch.float64, device="cuda")
    stream = torch.cuda.Stream()
    # a graph captured once holds its scratch until the tables go; the first one also
    # brings the runtime's own memory
    for first, count in ((True, n), (False, n - 1)):
        part = ara.LayerSpec(idx, np.zeros(2), np.full(2, 1e9), 0.0, 1e9, 0.0, 1e12, 0, count)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        ara.analyze(tables, part, [0.9], ylt=ylt[:count], metrics=metrics, flags=ara.ARA_GRAPH, stream=stream)
        stream.synchronize()
        assert np.array_equal(ylt[:count].cpu().numpy(), want[:count])
        if not first:
            assert free - torch.cuda.mem_get_info()[0] <= fold + 8 * MB
    torch.cuda.synchronize()
    ara.release_cached_memory()
    held = ara.cached_memory()[0]
    ara.event_nets(tables, spec, out=nets)          # images and packed losses, a probe word per 32 events
    torch.cuda.synchronize()
    assert ara.cached_memory()[0] - held <= 1.25 * (35 + 2) * MB
    if whole:
        tables.close()
    base.close()
