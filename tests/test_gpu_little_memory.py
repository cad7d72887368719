"""Creating tables where the device has memory for the 32-bit copy's counts and not
for the 16-bit copy's, four times as many: the 32-bit copy is built all the same."""

import numpy as np
import pytest

from workloads import make_elt_pool

pytestmark = pytest.mark.gpu


# no room for the finer counts; room for them but not beside the 32-bit copy's starts
@pytest.mark.parametrize("left_mb", [900, 1_200])
def test_counts_of_one_copy_fit(left_mb):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1606_04473_amd import ara
    n, C = 4_000_000, 64 << 16                      # counts: 1024 MB in 64 parts, 256 MB in 16
    rng = np.random.default_rng(3)
    offsets = np.zeros(n + 1, dtype=np.int64)
    offsets[1:] = np.cumsum(rng.integers(0, 3, n))
    ids = rng.integers(0, C, int(offsets[-1])).astype(np.uint32)
    pool = make_elt_pool(2, C, 60_000, seed=2)
    base = ara.create_tables(np.zeros(2, np.int64), ids[:0], pool.losses)
    spec = ara.LayerSpec(np.arange(2, dtype=np.int32), np.zeros(2), np.full(2, 1e9), 0.0, 1e9, 0.0, 1e12, 0, 5_000)
    everything = ara.create_yet(base, offsets, ids)
    assert everything.layout()["stream_parts"] == 64
    want = ara.run_layers(everything, [spec])
    everything.close()
    torch.cuda.synchronize()
    ara.release_cached_memory()
    torch.cuda.empty_cache()
    # offsets and IDs 50 MB, the copy's starts 268, its counts 268 or the copy 75; the
    # finer counts 1074
    first = torch.empty(torch.cuda.mem_get_info()[0] - (4 << 30), dtype=torch.uint8, device="cuda")
    hog = torch.empty(torch.cuda.mem_get_info()[0] - (left_mb << 20), dtype=torch.uint8, device="cuda")
    try:
        little = ara.create_yet(base, offsets, ids)
    finally:
        del first, hog
        torch.cuda.empty_cache()
    assert little.layout()["image_parts"] == 16 and little.layout()["stream_parts"] == 0
    assert np.array_equal(ara.run_layers(little, [spec]), want)
    little.close()
    base.close()
    ara.release_cached_memory()
