"""Performance cases of the averaged-RQA library: the calls that programs make
of it, over the sizes, embeddings, norms, line classes and target sets of its
configurations, harnesses and tests.

A case is a dict of plain values:
  kind     "run"        one series through Context.run (thresholds, RR, DET)
           "batch"      many series through one Context.batch call
           "curve"      Context.det_curve at given thresholds (the grid variant)
           "histogram"  Context.batch_hist: DET and the whole line histogram
           "gradients"  the bracket network's forward and backward pass
  systems  comma-separated signal generators, dealt out to the series in turn
  series   number of series; n, n_low: lengths log-uniform in [n_low, n]
           (n_low = n: all n samples)
  snr_hi, snr_lo  signal-to-noise ratio in dB, falling linearly over the series
  embed    "own": m = 3, tau = 5 for Lorenz and m = 1 otherwise, as in the
           workload configurations; "same": m and tau for every series
  norm     0 maximum, 1 squared Euclidean; theiler, lmin as in rqa_params
  K        targets 0.01, 0.02, ..., K / 100 (curve: thresholds 1/400 .. K/400)
  select   "auto", or "learned": the key window of the committed network
  batch    rows of a gradients call

Series are float32, generated from the seed alone; nothing is tuned, so calls
take the library's default launch shapes.
"""
import math
import os

import numpy as np
import torch

import paper_2208_09136_amd
from paper_2208_09136_amd import bracket, rqa

OWN_EMBEDDING = {"sine": (1, 1), "logistic": (1, 1), "lorenz": (3, 5)}
NETWORK = os.path.join(os.path.dirname(os.path.abspath(paper_2208_09136_amd.__file__)), "bracket_params.npz")


def _case(name, kind, systems="logistic", series=1, n=1000, n_low=0, snr_hi=10.0, snr_lo=10.0, embed="same", m=1,
          tau=1, norm=1, theiler=1, lmin=2, K=20, select="auto"):
    c = {"kind": kind, "systems": systems, "series": series, "n": n, "n_low": n_low or n, "snr_hi": snr_hi,
         "snr_lo": snr_lo, "embed": embed, "m": m, "tau": tau, "norm": norm, "theiler": theiler, "lmin": lmin,
         "K": K, "select": select}
    return {"name": name, **c} if name else c


def listed():
    return [
        # one short series, the smallest configured call: latency and launches
        _case("one_1e3", "run", n=1000, norm=0),
        # one ordinary series with the Lorenz embedding, as an interactive analysis makes it
        _case("one_1e4_lorenz", "run", "lorenz", n=10_000, snr_hi=0.0, embed="own"),
        # an embedding no kernel is compiled for (m = 4, tau = 7), a Theiler window and a ragged length
        _case("one_20011_m4", "run", "lorenz", n=20_011, snr_hi=5.0, m=4, tau=7, theiler=21),
        # lines of at least five points, maximum norm, m = 2: the general line class
        _case("one_5003_lmin5", "run", "lorenz", n=5003, snr_hi=5.0, m=2, tau=3, norm=0, theiler=6, lmin=5),
        # the medium configuration: three systems at five noise levels in one call
        _case("medium_15x1e4", "batch", "sine,logistic,lorenz", 15, 10_000, 0, 20.0, -20.0, "own"),
        # the large configuration (bench step): two long series
        _case("large_2x1e5", "batch", "lorenz,logistic", 2, 100_000, 0, 0.0, -10.0, m=3, tau=5),
        # the uneven ensemble: 600 series of 100 to 20,000 samples
        _case("ensemble_600", "batch", "sine,logistic,lorenz", 600, 20_000, 100, 20.0, -25.0, "own"),
        # one cell of the sorting-rate ensemble: 100 series, the whole RR set 1..99 %
        _case("sorting_100x1e4_k99", "batch", "lorenz", 100, 10_000, 0, 10.0, 0.0, m=3, tau=3, norm=0, K=99),
        # held-out series inside the trained network's key window
        _case("learned_8x5e4", "batch", "sine,logistic,lorenz", 8, 50_000, 0, 20.0, -25.0, m=3, tau=5,
              select="learned"),
        # the grid variant: RR and DET at a hundred fixed thresholds of a [0, 1]-scaled series
        _case("grid_1e4_100", "curve", "logistic", 1, 10_000, 0, 10.0, 10.0, norm=0, K=100),
        # average and longest line lengths: the whole line-length histogram with the path
        _case("histogram_4x2e4", "histogram", "lorenz,sine", 4, 20_000, 0, 10.0, -10.0, m=3, tau=5),
        # one training batch of the bracket network, forward and backward
        {"name": "gradients_256", "kind": "gradients", "batch": 256},
    ]


def _span(rng, lo, hi):
    """An integer log-uniform in [lo, hi]."""
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))


def draw(rng):
    kind = rng.choice(["run", "run", "run", "batch", "batch", "curve", "histogram", "gradients"])
    if kind == "gradients":
        return {"kind": kind, "batch": _span(rng, 16, 1024)}
    system = rng.choice(["sine", "logistic", "lorenz"])
    snr = round(rng.uniform(-20.0, 20.0), 1)
    m, tau = rng.choice([(1, 1), (1, 1), (3, 3), (3, 5), (3, 5), (2, 1), (2, 3), (3, 10), (4, 7), (5, 2)])
    common = {"m": m, "tau": tau, "norm": rng.choice([0, 1]), "theiler": rng.choice([1, 1, 5, 21]),
              "lmin": rng.choice([2, 2, 2, 2, 1, 3, 5, 10])}
    if kind == "run":
        return _case("", kind, system, n=_span(rng, 120, 30_000), snr_hi=snr, K=rng.choice([1, 5, 20, 20, 20, 50, 99]),
                     **common)
    if kind == "curve":
        return _case("", kind, system, n=_span(rng, 200, 20_000), snr_hi=snr, K=rng.choice([1, 10, 50, 100]), **common)
    if kind == "histogram":
        return _case("", kind, system, _span(rng, 1, 4), _span(rng, 200, 20_000), snr_hi=snr, snr_lo=snr - 10.0,
                     K=rng.choice([5, 20, 20, 40]), **{**common, "lmin": 2})
    n = _span(rng, 300, 10_000)
    return _case("", kind, "sine,logistic,lorenz", _span(rng, 2, 60), n, rng.choice([100, n]), 20.0, -20.0,
                 **{**common, "lmin": 2}, embed=rng.choice(["own", "same"]), K=rng.choice([20, 20, 20, 99]))


# ------------------------------------------------------------------ inputs

def _signals(system, lengths, rng):
    """Noise-free float64 series of one system, iterated together: a sine of
    37.3 samples, the logistic map r = 4, or the z-normalised x-component of
    the Lorenz system (Runge-Kutta, step 0.01)."""
    count, longest = len(lengths), max(lengths)
    out = np.empty((longest, count))
    if system == "sine":
        out[:] = np.sin(2.0 * math.pi / 37.3 * np.arange(longest)[:, None] + rng.uniform(0, 2 * math.pi, count))
    elif system == "logistic":
        x = rng.uniform(0.1, 0.9, count)
        for t in range(-200, longest):
            if t >= 0:
                out[t] = x
            x = 4.0 * x * (1.0 - x)
    else:
        def rate(x, y, z):
            return 10.0 * (y - x), x * (28.0 - z) - y, x * y - 8.0 / 3.0 * z
        state = 1.0 + rng.normal(0.0, 0.5, (3, count))
        x, y, z = (float(v[0]) for v in state) if count == 1 else state  # plain floats step faster than arrays of one
        h = 0.01
        for t in range(-1000, longest):
            if t >= 0:
                out[t] = x
            a1, b1, c1 = rate(x, y, z)
            a2, b2, c2 = rate(x + 0.5 * h * a1, y + 0.5 * h * b1, z + 0.5 * h * c1)
            a3, b3, c3 = rate(x + 0.5 * h * a2, y + 0.5 * h * b2, z + 0.5 * h * c2)
            a4, b4, c4 = rate(x + h * a3, y + h * b3, z + h * c3)
            x = x + h / 6.0 * (a1 + 2.0 * (a2 + a3) + a4)
            y = y + h / 6.0 * (b1 + 2.0 * (b2 + b3) + b4)
            z = z + h / 6.0 * (c1 + 2.0 * (c2 + c3) + c4)
    columns = [out[:n, i] for i, n in enumerate(lengths)]
    return [(v - v.mean()) / v.std() for v in columns] if system == "lorenz" else columns


def _series(case, seed):
    """float32 series of a case: clean signals plus Gaussian noise."""
    rng = np.random.default_rng([int(seed), 2208])
    names = case["systems"].split(",")
    count = case["series"]
    u = rng.uniform(math.log(case["n_low"]), math.log(case["n"]), count)
    lengths = [int(round(math.exp(v))) for v in u]
    own = [names[i % len(names)] for i in range(count)]
    steps = max(1, -(-count // len(names)) - 1)
    out = [None] * count
    for name in names:
        mine = [i for i in range(count) if own[i] == name]
        if not mine:
            continue
        for i, clean in zip(mine, _signals(name, [lengths[i] for i in mine], rng)):
            snr = case["snr_hi"] + (case["snr_lo"] - case["snr_hi"]) * min(1.0, (i // len(names)) / steps)
            noise = math.sqrt(clean.var() / 10.0 ** (snr / 10.0))
            out[i] = (clean + noise * rng.standard_normal(len(clean))).astype(np.float32)
    if case["kind"] == "curve":  # the grid variant rescales every series into [0, 1]
        out = [((y - y.min()) / (y.max() - y.min())).astype(np.float32) for y in out]
    return out, own


def _params(case, own):
    rest = (case["norm"], case["theiler"], case["lmin"])
    if case["embed"] == "own":
        return [OWN_EMBEDDING[name] + rest for name in own]
    return [(case["m"], case["tau"]) + rest] * len(own)


def _targets(case):
    return np.arange(1, case["K"] + 1) / 100.0


def _grid(case):
    e = np.arange(1, case["K"] + 1) / 400.0
    return (e if case["norm"] == 0 else e * e).astype(np.float32)


def _rows(case, seed):
    """Network weights, inputs and targets of a training batch: standardised
    columns, as the training loop feeds them."""
    rng = np.random.default_rng([int(seed), 1286])
    shapes = ((66, 128), (128,), (128, 128), (128,), (128, 20), (20,))
    theta = [rng.uniform(-1, 1, s) * (math.sqrt(6.0 / s[0]) if len(s) == 2 else 0.1) for s in shapes]
    x, t = rng.standard_normal((case["batch"], 66)), rng.standard_normal((case["batch"], 20))
    return [w.astype(np.float32) for w in theta], x.astype(np.float32), t.astype(np.float32)


def prepare(case, seed):
    ctx = rqa.Context(0, torch.cuda.current_stream())
    if case["kind"] == "gradients":
        theta, x, t = _rows(case, seed)
        ctx.mlp_set_params(np.concatenate([w.ravel() for w in theta]))
        return {"kind": case["kind"], "ctx": ctx, "x": torch.from_numpy(x).cuda(), "t": torch.from_numpy(t).cuda()}
    ys, own = _series(case, seed)
    state = {"kind": case["kind"], "ctx": ctx, "params": _params(case, own), "flags": rqa.RQA_SEL_AUTO,
             "series": torch.from_numpy(np.concatenate(ys)).cuda(),
             "offsets": np.concatenate([[0], np.cumsum([len(y) for y in ys])]).astype(np.uint64),
             "rr": np.tile(_targets(case), (len(ys), 1)), "longest": max(len(y) for y in ys)}
    if case["kind"] == "curve":
        state["eps"] = _grid(case)
    if case["select"] == "learned":
        bracket.load(ctx, NETWORK)
        state["flags"] = rqa.RQA_SEL_LEARNED
    return state


def run(state):
    ctx, kind = state["ctx"], state["kind"]
    if kind == "gradients":
        gradient, loss = ctx.mlp_gradients(state["x"], state["t"])
        return {"gradient": gradient, "loss": loss}
    if kind == "run":
        return ctx.run(state["series"], state["params"][0], state["rr"][0], state["flags"])
    if kind == "curve":
        return ctx.det_curve(state["series"], state["params"][0], state["eps"])
    if kind == "histogram":
        return ctx.batch_hist(state["series"], state["offsets"], state["params"], state["rr"], state["longest"] + 1,
                              state["flags"])
    return ctx.batch(state["series"], state["offsets"], state["params"], state["rr"], state["flags"])


# ------------------------------------------------------------------ work and exact values

def _mean_pairs(case):
    """Pairs of a case; for lengths log-uniform in [n_low, n] their expected number."""
    n, low = case["n"], case["n_low"]
    square = n * n if n == low else (n * n - low * low) / (2.0 * math.log(n / low))
    return case["series"] * square / 2.0


def work(case):
    if case["kind"] == "gradients":
        weights, rows = 66 * 128 + 128 + 128 * 128 + 128 + 128 * 20 + 20, case["batch"]
        return {"bytes": 4 * (2 * weights + rows * 86), "flops": 6 * rows * (66 * 128 + 128 * 128 + 128 * 20)}
    # per pair: one new component difference (squared), m - 1 folds, the rank
    # of the key and the minimum and maximum of the line rule
    embeddings = [OWN_EMBEDDING[s] for s in case["systems"].split(",")] if case["embed"] == "own" else [(case["m"], 0)]
    m = sum(e[0] for e in embeddings) / len(embeddings)
    flops = _mean_pairs(case) * (1 + (case["norm"] == 1) + (m - 1) + 3)
    n, low, rows = case["n"], case["n_low"], case["series"] * case["K"]
    mean = n if n == low else (n - low) / math.log(n / low)
    out = rows * (28 + (8 * (n + 1) if case["kind"] == "histogram" else 0))
    return {"bytes": int(4 * case["series"] * mean + out), "flops": int(flops)}


def _exact_series(y, params, rr, eps):
    """Thresholds, RR and DET of one series in 64 bits over the whole matrix of
    (diagonal, position) cells; eps given, or selected at the targets rr."""
    m, tau, norm, w, lmin = params
    y = torch.from_numpy(y).to("cuda", torch.float64)
    nv = len(y) - (m - 1) * tau
    diagonals = nv - w
    t = torch.arange(diagonals, device=y.device)
    cell = t[None, :] < (diagonals - t)[:, None]  # row d - w, column the earlier index
    j = torch.where(cell, t[None, :] + w + t[:, None], t[None, :])
    key = torch.zeros((diagonals, diagonals), dtype=torch.float64, device=y.device)
    for k in range(m):
        d = (y[(m - 1 - k) * tau:][t][None, :] - y[(m - 1 - k) * tau:][j]).abs()
        key = torch.maximum(key, d) if norm == 0 else key + d * d
    key[~cell] = math.inf
    pairs = diagonals * (diagonals + 1) // 2
    if eps is None:
        ranks = [min(max(-(-round(r * 1e9) * pairs // 10 ** 9), 1), pairs) for r in rr]
        ordered = torch.sort(key[cell])[0]
        eps = ordered[torch.tensor(ranks, device=y.device) - 1]
        del ordered
    else:
        eps = torch.from_numpy(eps).to(y.device, torch.float64)
    # a cell's line value: the least, over runs of lmin cells that hold it, of the run's largest key
    pad = torch.nn.functional.pad(key, (lmin - 1, lmin - 1), value=math.inf)
    top = pad
    for i in range(1, lmin):
        top = torch.maximum(top[:, :-1], pad[:, i:])
    line = top[:, :diagonals]
    for i in range(1, lmin):
        line = torch.minimum(line, top[:, i:i + diagonals])
    counts = torch.stack([(key <= e).sum() for e in eps]).double()
    lines = torch.stack([(line <= e).sum() for e in eps]).double()
    det = lines / counts
    return eps.cpu().numpy(), (counts / pairs).cpu().numpy(), det.cpu().numpy(), float(det.mean())


def exact(case, seed):
    if case["kind"] == "gradients":
        theta, x, t = _rows(case, seed)
        w = [torch.from_numpy(v).double().requires_grad_() for v in theta]
        gelu = torch.nn.functional.gelu
        y = gelu(gelu(torch.from_numpy(x).double() @ w[0] + w[1]) @ w[2] + w[3]) @ w[4] + w[5]
        loss = ((y - torch.from_numpy(t).double()) ** 2).mean()
        loss.backward()
        return {"gradient": np.concatenate([v.grad.numpy().ravel() for v in w]), "loss": float(loss)}
    if case["n"] > 12_000 or _mean_pairs(case) * case["K"] > 2e10:
        return None
    ys, own = _series(case, seed)
    given = _grid(case) if case["kind"] == "curve" else None
    found = [_exact_series(y, p, _targets(case), given) for y, p in zip(ys, _params(case, own))]
    eps, rr, det = (np.stack([f[i] for f in found]) for i in range(3))
    mean = np.array([f[3] for f in found])
    if case["kind"] == "curve":
        return {"count": None, "rr": rr[0], "det": det[0], "det_mean": float(mean[0]), "hist": None}
    if case["kind"] == "run":
        return {"eps": eps[0], "k": None, "count": None, "rr": rr[0], "det": det[0], "det_mean": float(mean[0])}
    out = {"eps": eps, "rr": rr, "det": det, "det_mean": mean, "count": None}
    return {**out, "hist": None} if case["kind"] == "histogram" else out
