"""The metrics' selection over ranges of magnitude past its fine bins (32 octaves
below the largest finite loss): thresholds in the bins of one octave and at their
edge, infinities, subnormals, and a call's time over such losses against ordinary
ones.  PML is one of the losses, so it is exact; mean and TVaR are a sum rounded once
and a quotient rounded once on both sides: 4 x 2^-53 relative."""

import numpy as np
import pytest

import oracle

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


def _losses(kind, n, rng):
    y = rng.lognormal(12.0, 2.0, n)
    if kind == "edge":                          # keys on both sides of 32 octaves below the largest
        y = np.ldexp(1.0 + rng.integers(0, 64, n) / 64.0, rng.choice([0, -31, -32, -33], n, p=[0.01, 0.33, 0.33, 0.33]))
    elif kind == "outlier":
        y[n // 2] = 1.0e300
    elif kind == "infinity":
        y[n // 2] = np.inf
    elif kind == "infinities":
        y[rng.random(n) < 0.02] = np.inf
    elif kind == "zeros and infinities":
        y = np.where(rng.random(n) < 0.3, np.inf, 0.0)
    elif kind == "subnormal":
        y = rng.integers(0, 1 << 20, n) * 5e-324
    elif kind == "wide":
        y = np.ldexp(1.0 + rng.random(n), rng.integers(-1000, 1000, n))
    return y


@pytest.mark.parametrize("n", [2, 5_000, 16_385, 70_001])
@pytest.mark.parametrize("kind", ["edge", "outlier", "infinity", "infinities", "zeros and infinities", "subnormal"])
def test_ranges_past_the_fine_bins(ara, n, kind):
    import torch
    y = _losses(kind, n, np.random.default_rng(n + len(kind)))
    d = torch.from_numpy(y).cuda()
    for probs in ([0.99], [0.999, 0.5, 0.05, 0.3]):
        out = torch.empty(1 + 2 * len(probs), dtype=torch.float64, device="cuda")
        ara.risk_metrics(d, probs, outputs=out)
        got = out.cpu().numpy()
        ordered = np.sort(y)[::-1]
        k = len(probs)
        assert got[1:1 + k].tolist() == [ordered[ara.tail_count(n, p) - 1] for p in probs]
        if np.isfinite(y).all():
            mean, _, tvar = oracle.risk_metrics(y, probs)
            want = np.array([mean, *tvar])
            assert np.all(np.abs(got[[0, *range(1 + k, 1 + 2 * k)]] - want) <= 4 * 2.0 ** -53 * want)


@pytest.mark.parametrize("kind", ["infinity", "wide"])
def test_time_over_wide_ranges(ara, kind):
    """One bin for all losses far below the largest took 40 times as long as ordinary
    ones; a bin per octave is within 4."""
    import torch
    probs, stream, best = [0.95, 0.99, 0.996], torch.cuda.Stream(), {}
    for k in ("ordinary", kind):
        d = torch.from_numpy(_losses(k, 1_000_000, np.random.default_rng(1))).cuda()
        out = torch.empty(7, dtype=torch.float64, device="cuda")
        times = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(stream)
            for _ in range(10):
                ara.risk_metrics(d, probs, outputs=out, stream=stream)
            b.record(stream)
            b.synchronize()
            times.append(a.elapsed_time(b))
        best[k] = min(times)
    assert best[kind] < 4.0 * best["ordinary"]
