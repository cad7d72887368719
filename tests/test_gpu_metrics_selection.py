"""The metrics' selection at the edges of its launches (one workgroup up to
16,384 losses, several beyond) and of its bins: losses that share a bin by the
thousand, all equal, zeros below everything else, a range of magnitudes wider
than the bins, thresholds in the lowest bin.  PML is one of the losses, so it is
exact; mean and TVaR are a sum rounded once and a quotient rounded once on both
sides: 4 x 2^-53 relative."""

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
    if kind == "spread":
        return rng.lognormal(12.0, 2.0, n)
    if kind == "one bin":                       # thousands of candidates, all distinct
        return 1.0e6 * (1.0 + 1e-3 * rng.random(n))
    if kind == "equal":
        return np.full(n, 12345.678)
    if kind == "zeros":
        return np.where(rng.random(n) < 0.7, 0.0, rng.lognormal(10.0, 1.0, n))
    if kind == "cap":                           # a tie of a third of the losses at the top
        return np.minimum(rng.lognormal(12.0, 1.0, n), 2.5e5)
    # 2^-1000 .. 2^1000, so most losses fall below the lowest bin's edge
    return np.ldexp(1.0 + rng.random(n), rng.integers(-1000, 1000, n))


@pytest.mark.parametrize("n", [1, 3, 4_096, 4_097, 16_384, 16_385, 70_001])
@pytest.mark.parametrize("kind", ["spread", "one bin", "equal", "zeros", "cap", "wide"])
def test_metrics_selection_edges(ara, n, kind):
    import torch
    y = _losses(kind, n, np.random.default_rng(n + len(kind)))
    d = torch.from_numpy(y).cuda()
    for probs in ([], [0.99], [0.999, 0.5, 0.05, 0.3]):
        out = torch.empty(1 + 2 * len(probs), dtype=torch.float64, device="cuda")
        ara.risk_metrics(d, probs, outputs=out)
        got = out.cpu().numpy()
        mean, pml, tvar = oracle.risk_metrics(y, probs)
        k = len(probs)
        assert np.array_equal(got[1:1 + k], np.asarray(pml)), probs
        want = np.array([mean, *tvar])
        assert np.all(np.abs(got[[0, *range(1 + k, 1 + 2 * k)]] - want) <= 4 * 2.0 ** -53 * want), probs
