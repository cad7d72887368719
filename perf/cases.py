"""The work this library is measured on: calls of its public entry points over
the sizes that its configurations, tests and benchmark use.

A case is a dict of plain values.  `n_trials` x Poisson(`lam`) events over a
catalogue of `C` events; a pool of `pool` event loss tables with `nnz`
lognormal(10, 2) losses each; `layers` layers of `elts` tables each (with
several layers between 1 and `elts`); the trial range of each layer is a
share `span` of the trials (1.0: all of them).  `kind` says which entry points
a pass goes through.  Event IDs are uniform over the catalogue, per-table
terms are the 20th and 95th percentiles of the table's losses, and layer terms
come from quantiles of the combined losses and moments of the year's total, as
in the repository's workload generators.
"""

import math
from fractions import Fraction

import numpy as np
import torch

from paper_1606_04473_amd import ara
from paper_1606_04473_amd.autograd import mean_and_tvar

_PROBS = {1: [0.99], 2: [0.99, 0.996], 3: [0.95, 0.99, 0.996], 4: [0.9, 0.99, 0.996, 0.999]}
_CHUNK = 100_000_000                    # events evaluated at a time by exact()
_SCALE = float(2 ** 20)
_stream_of_program = []


def listed():
    return [
        # the small configuration, one analysis replayed as a graph: latency
        dict(name="analyze_small", kind="analyze", n_trials=10_000, lam=100, C=100_000, pool=4, nnz=10_000,
             layers=1, elts=4, span=1.0, probs=1),
        # the paper-scale share of one GPU, the benchmark's step
        dict(name="analyze_paper_scale", kind="analyze", n_trials=1_000_000, lam=1000, C=2_000_000, pool=16,
             nnz=20_000, layers=1, elts=16, span=1.0, probs=2),
        # a layer of 30 tables over a small catalogue: most events have a loss
        dict(name="analyze_dense", kind="analyze", n_trials=100_003, lam=500, C=500_009, pool=30, nnz=30_000,
             layers=1, elts=30, span=1.0, probs=2),
        # a tenant's request on resident tables: a few layers over a slice of
        # the trials, metrics of each, eager calls
        dict(name="request_resident", kind="request", n_trials=200_000, lam=1000, C=2_000_000, pool=48, nnz=20_000,
             layers=3, elts=32, span=0.309, probs=2),
        # a tenant's request that ships its own trials: tables built for them,
        # layers, metrics, tables destroyed
        dict(name="request_shipped", kind="shipped", n_trials=150_001, lam=1000, C=2_000_000, pool=48, nnz=20_000,
             layers=2, elts=32, span=1.0, probs=1),
        # many layers of uneven table and trial counts in one graph call
        dict(name="layers_library", kind="layers", n_trials=250_000, lam=1000, C=2_000_000, pool=64, nnz=20_000,
             layers=12, elts=32, span=0.0, probs=1),
        # programs of layers with per-program and portfolio sums, the trials split in two
        dict(name="portfolio", kind="portfolio", n_trials=50_021, lam=800, C=1_000_003, pool=40, nnz=20_000,
             layers=9, elts=24, span=1.0, probs=1),
        # the gradients of mean and TVaR through autograd on the small configuration
        dict(name="gradient_small", kind="autograd", n_trials=10_000, lam=100, C=100_000, pool=4, nnz=10_000,
             layers=1, elts=4, span=1.0, probs=1),
        # a checkpointed forward and the adjoint at the paper's trial length
        dict(name="gradient_large", kind="gradient", n_trials=500_000, lam=1000, C=2_000_000, pool=16, nnz=20_000,
             layers=1, elts=16, span=1.0, probs=1),
        # per-event net losses of a few short trials, ragged sizes
        dict(name="nets_ragged", kind="nets", n_trials=7_001, lam=137, C=300_007, pool=5, nnz=12_345, layers=1,
             elts=3, span=1.0, probs=1),
        # per-event net losses at the paper's trial length
        dict(name="nets_large", kind="nets", n_trials=250_000, lam=1000, C=2_000_000, pool=16, nnz=20_000, layers=1,
             elts=16, span=1.0, probs=1),
        # risk metrics alone over a million year losses
        dict(name="metrics_1m", kind="metrics", n_trials=1_000_000, lam=1000, C=2_000_000, pool=16, nnz=20_000,
             layers=1, elts=16, span=1.0, probs=3),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["analyze", "analyze", "request", "shipped", "layers", "portfolio", "autograd", "gradient",
                       "nets", "nets", "metrics"])
    lam = log_int(20, 1500)
    most = {"nets": 250_000_000, "shipped": 200_000_000, "layers": 250_000_000, "portfolio": 60_000_000,
            "request": 250_000_000, "autograd": 100_000_000}.get(kind, 500_000_000)
    n_trials = log_int(200, min(1_000_000, most // lam))
    C = log_int(20_000, 2_000_000)
    layers = {"request": rng.randint(1, 6), "shipped": rng.randint(1, 4), "layers": rng.randint(2, 16),
              "portfolio": rng.randint(2, 12)}.get(kind, 1)
    elts = rng.randint(1, 32)
    span = round(rng.uniform(0.1, 1.0), 3) if kind in ("request", "analyze") and rng.random() < 0.5 else 1.0
    return dict(kind=kind, n_trials=n_trials, lam=lam, C=C, pool=elts + rng.randint(0, 12),
                nnz=min(log_int(5_000, 30_000), C // 4), layers=layers, elts=elts,
                span=0.0 if kind == "layers" else span, probs=rng.randint(1, 4))


def _stream():
    # the stream a program runs its analyses on (the null stream takes no graph)
    if not _stream_of_program:
        _stream_of_program.append(torch.cuda.Stream())
    return _stream_of_program[0]


def _yet(case, gen):
    lengths = torch.poisson(torch.full((case["n_trials"],), float(case["lam"]), device="cuda"), generator=gen)
    lengths = lengths.to(torch.int64)
    # the expected number of events in all, so that outputs per event have one size
    surplus = int(lengths.sum()) - case["n_trials"] * case["lam"]
    while surplus:
        some = torch.nonzero(lengths > 0)[:abs(surplus), 0] if surplus > 0 else \
            torch.arange(min(-surplus, case["n_trials"]), device="cuda")
        lengths[some] -= 1 if surplus > 0 else -1
        surplus -= int(some.numel()) * (1 if surplus > 0 else -1)
    offsets = torch.zeros(case["n_trials"] + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lengths, 0, out=offsets[1:])
    ids = torch.randint(0, case["C"], (case["n_trials"] * case["lam"],), dtype=torch.int32, device="cuda", generator=gen)
    return offsets, ids


def _pool(case, gen):
    losses = torch.zeros(case["pool"], case["C"], dtype=torch.float64, device="cuda")
    terms = np.empty((2, case["pool"]))
    n = case["nnz"]
    for j in range(case["pool"]):
        values = torch.exp(10.0 + 2.0 * torch.randn(n, dtype=torch.float64, device="cuda", generator=gen))
        losses[j, torch.randperm(case["C"], device="cuda", generator=gen)[:n]] = values
        ordered = torch.sort(values).values
        for i, q in enumerate((0.20, 0.95)):
            k = min(max(math.ceil(q * n), 1), n - 1)
            terms[i, j] = float((ordered[k - 1] + ordered[k]) * 0.5)
    return losses, terms


def _clamp(v, retention, limit):
    return torch.clamp(torch.clamp(v - retention, min=0.0), max=limit)


def _occurrence(losses, spec_elts, retention, limit):
    y = torch.zeros(losses.shape[1], dtype=torch.float64, device="cuda")
    for k, j in enumerate(spec_elts):
        y = y + _clamp(losses[int(j)], float(retention[k]), float(limit[k]))
    return y


def _layers(case, losses, terms, host):
    n, out = case["n_trials"], []
    sizes = np.random.RandomState(n)                # trial counts go with the case, so that outputs have one size
    for _ in range(case["layers"]):
        J = case["elts"] if case["layers"] == 1 else int(host.randint(1, case["elts"] + 1))
        idx = host.permutation(case["pool"])[:J].astype(np.int32)
        count = n if case["span"] == 1.0 else max(1, int(round(n * (case["span"] or sizes.uniform(0.04, 1.0)))))
        begin = int(host.randint(0, n - count + 1))
        R, Lim = terms[0, idx].copy(), terms[1, idx].copy()
        y = _occurrence(losses, idx, R, Lim)
        positive = torch.sort(y[y > 0.0]).values
        lo, hi = (float(positive[int(q * (positive.numel() - 1))]) * 1.0000001 for q in (0.10, 0.99))
        o = _clamp(y, lo, hi - lo)
        mean, square = case["lam"] * float(o.mean()), case["lam"] * float((o * o).mean())
        out.append(ara.LayerSpec(idx, R, Lim, lo, hi - lo, mean, 3.1 * math.sqrt(square), begin, count))
    return out


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    host = np.random.RandomState(seed % (2 ** 32))
    if case["kind"] == "metrics":
        # year losses of a layer: zeros below the aggregate retention, ties at the limit
        S = 1e7 * torch.exp(0.6 * torch.randn(case["n_trials"], dtype=torch.float64, device="cuda", generator=gen))
        return _clamp(S, 1.0e7, 9.0e7)
    losses, terms = _pool(case, gen)
    layers = _layers(case, losses, terms, host)
    offsets, ids = _yet(case, gen)
    return losses, layers, offsets, ids


def _programs(case, layers):
    k = max(1, case["layers"] // 3)
    return [layers[i:i + k] for i in range(0, len(layers), k)]


def prepare(case, seed):
    kind, probs = case["kind"], _PROBS[case["probs"]]
    state = dict(kind=kind, probs=probs, stream=_stream(), case=case)
    f64 = dict(dtype=torch.float64, device="cuda")
    if kind == "metrics":
        state.update(ylt=_inputs(case, seed), metrics=torch.empty(1 + 2 * len(probs), **f64))
        return state
    losses, layers, offsets, ids = _inputs(case, seed)
    if kind == "shipped":
        # the resident pool, and this request's trials as they arrived on the device
        base = ara.create_tables(torch.zeros(2, dtype=torch.int64, device="cuda"), ids[:0], losses)
        state.update(base=base, offsets=offsets, ids=ids)
    else:
        state["tables"] = ara.create_tables(offsets, ids, losses)
    state["layers"] = layers
    total = sum(l.trial_count for l in layers)
    if kind == "nets":
        state["nets"] = torch.empty(max(int(ids.numel()), 1), **f64)
    elif kind == "portfolio":
        programs = _programs(case, layers)
        n = case["n_trials"]
        state.update(programs=programs, outs={"layer": torch.empty(len(layers), n, **f64),
                                              "program": torch.empty(len(programs), n, **f64),
                                              "portfolio": torch.empty(n, **f64)})
    else:
        state["ylt"] = torch.empty(total, **f64)
    if kind in ("analyze", "request", "shipped"):
        state["metrics"] = [torch.empty(1 + 2 * len(probs), **f64) for _ in layers]
    if kind == "gradient":
        P = 2 * layers[0].n_elts + 4
        state.update(grad_mean=torch.empty(P, **f64), grad_tvar=torch.empty(P, **f64))
    if kind == "autograd":
        state["theta"] = torch.tensor(layers[0].theta(), **f64)
    torch.cuda.synchronize()
    return state


def _request(state, tables):
    at = 0
    for spec, metrics in zip(state["layers"], state["metrics"]):
        ylt = state["ylt"][at:at + spec.trial_count]
        at += spec.trial_count
        ara.run_layers(tables, [spec], out=ylt, stream=state["stream"])
        ara.risk_metrics(ylt, state["probs"], outputs=metrics, stream=state["stream"])


def run(state):
    kind, stream = state["kind"], state["stream"]
    if kind == "analyze":
        ara.analyze(state["tables"], state["layers"][0], state["probs"], ylt=state["ylt"],
                    metrics=state["metrics"][0], flags=ara.ARA_GRAPH, stream=stream)
        return [state["ylt"], state["metrics"][0]]
    if kind == "request":
        _request(state, state["tables"])
        return [state["ylt"], *state["metrics"]]
    if kind == "shipped":
        tables = ara.create_yet(state["base"], state["offsets"], state["ids"], stream=stream)
        _request(state, tables)
        tables.close()
        return [state["ylt"], *state["metrics"]]
    if kind == "layers":
        ara.run_layers(state["tables"], state["layers"], out=state["ylt"], flags=ara.ARA_GRAPH, stream=stream)
        return [state["ylt"]]
    if kind == "portfolio":
        ara.run_portfolio(state["tables"], state["programs"], 2, outs=state["outs"], stream=stream)
        return [state["outs"][k] for k in ("layer", "program", "portfolio")]
    if kind == "gradient":
        ara.run_layers(state["tables"], state["layers"], out=state["ylt"], flags=ara.ARA_CHECKPOINT_S, stream=stream)
        ara.backward(state["tables"], state["layers"][0], state["probs"][-1], grad_mean=state["grad_mean"],
                     grad_tvar=state["grad_tvar"], stream=stream)
        return [state["ylt"], state["grad_mean"], state["grad_tvar"]]
    if kind == "autograd":
        with torch.cuda.stream(stream):
            theta = state["theta"].clone().requires_grad_(True)
            mean, tvar, ylt = mean_and_tvar(theta, state["tables"], state["layers"][0], state["probs"][-1])
            (grad,) = torch.autograd.grad(0.5 * mean + tvar, theta)
            return [mean.detach(), tvar.detach(), ylt, grad]
    if kind == "nets":
        ara.event_nets(state["tables"], state["layers"][0], out=state["nets"], stream=stream)
        return [state["nets"]]
    ara.risk_metrics(state["ylt"], state["probs"], outputs=state["metrics"], stream=stream)
    return [state["metrics"]]


def work(case):
    """An event ID cannot take fewer than two bytes in any order kept for the
    passes; the calls that read the trials in time order or as they are
    shipped read four.  The pool's nonzero losses take ten bytes each.  One
    addition per event and layer."""
    n, events, layers = case["n_trials"], case["n_trials"] * case["lam"], case["layers"]
    kind = case["kind"]
    if kind == "metrics":
        return {"bytes": 8 * n, "flops": 2 * n}
    share = case["span"] if case["span"] else 0.52
    elts = case["elts"] if layers == 1 else layers * (case["elts"] + 1) / 2
    pool = 10 * case["nnz"] * min(elts, case["pool"])
    out = 8 * n * share * layers
    read = {"nets": 4, "shipped": 4, "gradient": 4, "autograd": 4}.get(kind, 2) * events
    if kind == "nets":
        out = 8 * events
    if kind == "portfolio":
        out += 8 * n * (len(_programs(case, list(range(layers)))) + 1)
    if kind in ("request", "analyze"):
        read *= share
    flops = events * share * layers * (2 if kind in ("gradient", "autograd") else 1)
    return {"bytes": int(read + pool + out), "flops": int(flops)}


# ---------------------------------------------------------------------------
# the same results in plain torch, 64 bits
# ---------------------------------------------------------------------------

def _running(values):
    """Running totals of float64 values as (multiples of 2^-20 in int64, the
    rest in float64): differences of the first are exact, the rest is tiny."""
    units = torch.floor(values * _SCALE)
    rest = values - units / _SCALE
    return torch.cumsum(units.to(torch.int64), 0), torch.cumsum(rest, 0)


def _blocks(offsets, first, last):
    """Trial ranges of at most about _CHUNK events."""
    at = first
    while at < last:
        target = int(offsets[at]) + _CHUNK
        end = int(np.searchsorted(offsets, target, side="right")) - 1
        end = min(max(end, at + 1), last)
        yield at, end
        at = end


def _combine(units, rest):
    return units.to(torch.float64) / _SCALE + rest if int(units.abs().max()) < 2 ** 53 else \
        (units >> 20).to(torch.float64) + ((units & (2 ** 20 - 1)).to(torch.float64) / _SCALE + rest)


def _totals(layer, o, offsets, ids):
    host = offsets.cpu().numpy()
    out = []
    for a, b in _blocks(host, layer.trial_begin, layer.trial_begin + layer.trial_count):
        lo, hi = int(host[a]), int(host[b])
        if hi == lo:
            out.append(torch.zeros(b - a, dtype=torch.float64, device="cuda"))
            continue
        units, rest = _running(o[ids[lo:hi].long()])
        zero = torch.zeros(1, device="cuda")
        units = torch.cat([zero.to(units.dtype), units])
        rest = torch.cat([zero.to(rest.dtype), rest])
        at = offsets[a:b + 1] - lo
        out.append(_combine(units[at[1:]] - units[at[:-1]], rest[at[1:]] - rest[at[:-1]]))
    return torch.cat(out)


def _fold(layer, losses):
    y = _occurrence(losses, layer.elt_index, layer.elt_retention, layer.elt_limit)
    return y, _clamp(y, layer.occ_retention, layer.occ_limit)


def _year(layer, losses, offsets, ids):
    S = _totals(layer, _fold(layer, losses)[1], offsets, ids)
    return S, _clamp(S, layer.agg_retention, layer.agg_limit)


def _tail(n, p):
    return min(max(math.ceil(n * (1 - Fraction(repr(p)))), 1), n)


def _metrics(ylt, probs):
    ordered = torch.sort(ylt, descending=True).values.cpu().tolist()
    n = len(ordered)
    ms = [_tail(n, p) for p in probs]
    return torch.tensor([math.fsum(ordered) / n] + [ordered[m - 1] for m in ms] +
                        [math.fsum(ordered[:m]) / m for m in ms], dtype=torch.float64)


def _gradients(layer, losses, offsets, ids, p):
    S, ylt = _year(layer, losses, offsets, ids)
    n = layer.trial_count
    m = _tail(n, p)
    t = S - layer.agg_retention
    band, above = (t > 0) & (t < layer.agg_limit), t > layer.agg_limit
    v = torch.sort(ylt, descending=True).values[m - 1]
    c_gt, c_eq = int((ylt > v).sum()), int((ylt == v).sum())
    weight = torch.where(ylt > v, c_eq, torch.where(ylt == v, m - c_gt, 0)).to(torch.int64)
    C = losses.shape[1]
    W = [torch.zeros(C, dtype=torch.int64, device="cuda") for _ in range(2)]
    host = offsets.cpu().numpy()
    first = layer.trial_begin
    for a, b in _blocks(host, first, first + n):
        lo, hi = int(host[a]), int(host[b])
        lengths = offsets[a + 1:b + 1] - offsets[a:b]
        for k, w in enumerate((torch.ones_like(weight), weight)):
            w = torch.where(band, w, torch.zeros_like(w))[a - first:b - first]
            per_event = torch.repeat_interleave(w, lengths)
            used = per_event != 0
            W[k].index_add_(0, ids[lo:hi][used].long(), per_event[used])
    y, _ = _fold(layer, losses)
    to = y - layer.occ_retention
    inside, over = (to > 0) & (to < layer.occ_limit), to > layer.occ_limit
    grads = []
    for w, trial, divisor in ((W[0], torch.ones_like(weight), n), (W[1], weight, m * c_eq)):
        down, up = [], []
        for k, j in enumerate(layer.elt_index):
            tj = losses[int(j)] - float(layer.elt_retention[k])
            L = float(layer.elt_limit[k])
            down.append(-int(w[inside & (tj > 0) & (tj < L)].sum()))
            up.append(int(w[inside & (tj > L)].sum()))
        counts = down + up + [-int(w[inside].sum()), int(w[over].sum()), -int(trial[band].sum()),
                              int(trial[above].sum())]
        grads.append(torch.tensor([c / divisor for c in counts], dtype=torch.float64))
    return ylt, grads[0], grads[1]


def _nets(layer, losses, offsets, ids):
    host = offsets.cpu().numpy()
    o = _fold(layer, losses)[1]
    out = []
    floor = min(max(0.0 - layer.agg_retention, 0.0), layer.agg_limit)
    for a, b in _blocks(host, layer.trial_begin, layer.trial_begin + layer.trial_count):
        lo, hi = int(host[a]), int(host[b])
        if hi == lo:
            continue
        units, rest = _running(o[ids[lo:hi].long()])
        lengths = offsets[a + 1:b + 1] - offsets[a:b]
        starts = (offsets[a:b] - lo)[lengths > 0]
        lengths = lengths[lengths > 0]
        at = starts - 1
        base = [torch.where(at >= 0, x[at.clamp(min=0)], torch.zeros_like(x[:1])) for x in (units, rest)]
        units -= torch.repeat_interleave(base[0], lengths)
        rest -= torch.repeat_interleave(base[1], lengths)
        A = _clamp(_combine(units, rest), layer.agg_retention, layer.agg_limit)
        before = torch.empty_like(A)
        before[1:] = A[:-1]
        before[starts] = floor
        out.append(A - before)
    return torch.cat(out) if out else torch.zeros(1, dtype=torch.float64)


def exact(case, seed):
    kind, probs = case["kind"], _PROBS[case["probs"]]
    if kind == "metrics":
        return [_metrics(_inputs(case, seed), probs)]
    losses, layers, offsets, ids = _inputs(case, seed)
    if kind == "nets":
        return [_nets(layers[0], losses, offsets, ids)]
    if kind in ("gradient", "autograd"):
        ylt, grad_mean, grad_tvar = _gradients(layers[0], losses, offsets, ids, probs[-1])
        if kind == "gradient":
            return [ylt, grad_mean, grad_tvar]
        metrics = _metrics(ylt, probs[-1:])
        return [metrics[0], metrics[2], ylt, 0.5 * grad_mean + grad_tvar]
    years = [_year(l, losses, offsets, ids)[1] for l in layers]
    if kind == "portfolio":
        groups = _programs(case, years)
        # exact sums of a few values: multiples of 2^-20 and the rest apart
        def total(rows):
            units = [torch.floor(r * _SCALE) for r in rows]
            rest = sum(r - u / _SCALE for r, u in zip(rows, units))
            return _combine(sum(u.to(torch.int64) for u in units), rest)
        return [torch.stack(years), torch.stack([total(g) for g in groups]), total(years)]
    if kind == "layers":
        return [torch.cat(years)]
    return [torch.cat(years), *[_metrics(y, probs) for y in years]]
