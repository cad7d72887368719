"""Tables of more trials than one launch can hold workgroups for while the copies
are built: 5.4e8 trials of one event (2^32 threads at a workgroup of 512 per 63 or
64 trials).  Each year loss is its event's loss."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_half_a_billion_trials():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1606_04473_amd import ara
    n, C = 540_000_000, 60_000
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 80 GB of device memory")
    losses = torch.zeros(1, C, dtype=torch.float64, device="cuda")
    losses[0, ::3] = torch.rand(C // 3, dtype=torch.float64, device="cuda") + 0.5
    ids = torch.randint(0, C, (n,), dtype=torch.int32, device="cuda")
    tables = ara.create_tables(torch.arange(n + 1, dtype=torch.int64, device="cuda"), ids, losses)
    layout = tables.layout()
    assert layout["stream_parts"] == 1 and layout["image_parts"] == 1
    spec = ara.LayerSpec(np.zeros(1, np.int32), np.zeros(1), np.full(1, np.inf), 0.0, np.inf, 0.0, np.inf, 0, n)
    ylt = torch.empty(n, dtype=torch.float64, device="cuda")
    for variant in (0, 2):
        ylt.fill_(-1.0)
        ara.set_tuning(tables, pass_variant=variant)
        ara.run_layers(tables, [spec], out=ylt)
        for at in range(0, n, 60_000_000):
            part = slice(at, at + 60_000_000)
            assert torch.equal(ylt[part], losses[0][ids[part].long()]), (variant, at)
    tables.close()
    ara.release_cached_memory()
    torch.cuda.empty_cache()
