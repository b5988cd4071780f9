"""Performance cases of the integrator, through its public entry points.

Each case is one thing that a program built on this package does over and over:

  integrate   a whole integration with new parameters: restart the grid, adapt
              it, accumulate, read the combined result and the adapted grid
              (a parameter scan over one context)
  stream      the same with iterations larger than one call, in chunks
  user        an integration of the caller's own device source
  grad        a training step: the estimate as a differentiable function of the
              Gaussian's centre and width, forward and backward
  batch       many independent integrations as one planned run

A case is a dict of plain values; `listed` gives the fixed ones, `draw` more of
the same ranges, `prepare` what the program holds before the call, `run` one
pass, `work` what a pass cannot do without and `exact` the pass's outputs in
plain 64-bit torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2002_12921_amd as va
from paper_2002_12921_amd.autograd import vegas_integral
from paper_2002_12921_amd.batch import VegasBatch
from paper_2002_12921_amd.user_integrands import GAUSSIAN, OSCILLATORY

ALPHA = 1.5


def _case(name, op, kind, dim, bins, prec, events, adapt, accumulate, **more):
    return {"name": name, "op": op, "kind": kind, "dim": dim, "bins": bins, "prec": prec, "events": events,
            "adapt": adapt, "accumulate": accumulate, **more}


def listed():
    return [
        # a two-dimensional integral inside another program's loop: launches and latency
        _case("gauss_d2_fp64_3x2e3", "integrate", "gauss", 2, 50, "fp64", 2000, 3, 0),
        # the small FP64 schedule of the benchmark: ten refined iterations, all combined
        _case("gauss_d4_fp64_10x1e5", "integrate", "gauss", 4, 50, "fp64", 100_000, 10, 0),
        # the headline workload, five adaptation and five accumulation iterations, in both precisions
        _case("gauss_d8_mixed_5+5x1e7", "integrate", "gauss", 8, 50, "fp32_mixed", 10_000_000, 5, 5),
        _case("gauss_d8_fp64_5+5x1e7", "integrate", "gauss", 8, 50, "fp64", 10_000_000, 5, 5),
        # the paper's Genz integrands at d = 16
        _case("disc_d16_fp64_3+2x1e7", "integrate", "genz_disc", 16, 50, "fp64", 10_000_000, 3, 2),
        _case("peak_d16_mixed_3+2x1e7", "integrate", "genz_peak", 16, 50, "fp32_mixed", 10_000_000, 3, 2),
        # odd dimensions, odd bin counts and ragged event counts
        _case("peak_d5_fp64_5+5x1234567", "integrate", "genz_peak", 5, 100, "fp64", 1_234_567, 5, 5),
        _case("gauss_d13_mixed_4+4x3000017", "integrate", "gauss", 13, 37, "fp32_mixed", 3_000_017, 4, 4),
        # 1e8 events per iteration, streamed in chunks of 1e7
        _case("bimodal_d20_mixed_stream", "stream", "bimodal", 20, 100, "fp32_mixed", 100_000_000, 1, 1,
              chunk=10_000_000),
        # the caller's own integrand, compiled at run time
        _case("user_d8_fp64_3+2x1e7", "user", "gauss", 8, 50, "fp64", 10_000_000, 3, 2),
        # a training step on a frozen grid, FP32 parameters
        _case("grad_d8_mixed_1e7", "grad", "gauss", 8, 50, "fp32_mixed", 10_000_000, 0, 1, fused=True),
        # 256 independent Gaussians, d = 2..16, 1e4..1e7 events each
        _case("batch256_mixed_5+5", "batch", "gauss", 16, 50, "fp32_mixed", 10_000_000, 5, 5, problems=256),
    ]


def draw(rng):
    """One more case: every dimension and precision, sizes spread over their logarithms."""
    op = rng.choice(["integrate"] * 6 + ["stream", "user", "grad", "grad", "batch"])
    prec = rng.choice(["fp64", "fp32_mixed"])
    events = int(round(10 ** rng.uniform(3, 7)))
    bins = int(round(math.exp(rng.uniform(math.log(10), math.log(128)))))
    if rng.random() < 0.4:
        bins = 50
    dim = rng.randint(1, 20)
    kind = rng.choice(["gauss", "bimodal", "genz_disc", "genz_peak"])
    adapt, accumulate = rng.choice([(5, 5), (3, 2), (10, 0), (4, 1)])
    if op == "integrate":
        return _case("", op, kind, dim, bins, prec, events, adapt, accumulate)
    if op == "stream":
        return _case("", op, kind, rng.randint(4, 20), bins, prec, 3 * events, 1, 1, chunk=events)
    if op == "user":
        return _case("", op, rng.choice(["gauss", "oscillatory"]), rng.randint(2, 13), bins, prec, events, 3, 2)
    if op == "grad":
        return _case("", op, "gauss", rng.randint(2, 16), bins, prec, events, 0, 1, fused=rng.random() < 0.75)
    return _case("", op, kind, rng.randint(6, 16), bins, prec, min(events, 1_000_000), 3, 2,
                 problems=rng.randint(8, 64))


# ---------------------------------------------------------------------------
# Inputs: parameters of the benchmark's ranges, from the seed alone.

def _params(kind, d, rng):
    """The integrand's parameter vector (layouts of the package)."""
    if kind == "gauss":
        return [rng.uniform(0.09, 0.13)] + list(rng.uniform(0.3, 0.7, d))
    if kind == "bimodal":
        return [rng.uniform(0.05, 0.08)] + list(rng.uniform(0.3, 0.36, d)) + list(rng.uniform(0.64, 0.7, d))
    if kind == "genz_disc":
        return list(rng.uniform(0.5, 1.5, d)) + list(rng.uniform(0.05, 0.3, d))
    if kind == "genz_peak":
        return list(rng.uniform(2.0, 4.0, d)) + list(rng.uniform(0.3, 0.7, d))
    return [rng.uniform(0.1, 0.7)] + list(rng.uniform(0.2, 3.0, d))  # oscillatory: u, c


def _inputs(case, seed):
    """What the seed gives: Philox seed, parameters and, for batches, the problems."""
    rng = np.random.default_rng([2002, 12921, seed])
    out = {"key": int(rng.integers(1 << 40))}
    d = case["dim"]
    if case["op"] == "batch":
        # the sizes are the case's own, so that every seed asks for the same work
        n, probs = case["problems"], []
        sizes = np.random.default_rng([n, case["events"]])
        top = math.log10(case["events"])
        for p in range(n):
            dp, m = int(sizes.integers(2, d + 1)), int(round(10.0 ** sizes.uniform(max(top - 3, 1), top)))
            q = _params(case["kind"], dp, rng)
            if case["kind"] == "gauss":
                q[0] = rng.uniform(0.05, 0.3)
            probs.append({"dim": dp, "n_bins": case["bins"], "integrand": case["kind"],
                          "params": [float(v) for v in q], "n_events": m, "precision": case["prec"],
                          "seed": out["key"], "alpha": ALPHA, "problem": p})
        out["problems"] = probs
        return out
    q = np.array(_params(case["kind"], d, rng))
    if case["op"] == "grad" and case["prec"] == "fp32_mixed":
        q = q.astype(np.float32).astype(np.float64)
    out["params"] = q
    return out


def _uniform(case):
    return np.tile(np.arange(case["bins"] + 1) / case["bins"], (case["dim"], 1))


def prepare(case, seed):
    x = _inputs(case, seed)
    op, d, N, prec = case["op"], case["dim"], case["bins"], case["prec"]
    if op == "batch":
        b = VegasBatch(x["problems"], n_iter=case["adapt"] + case["accumulate"], n_adapt=case["adapt"])
        return {"case": case, "batch": b}
    q = [float(v) for v in x["params"]]
    if op == "user":
        source = GAUSSIAN if case["kind"] == "gauss" else OSCILLATORY
        v = va.Vegas(d, N, params=q, precision=prec, seed=x["key"], alpha=ALPHA, source=source)
    else:
        v = va.Vegas(d, N, case["kind"], q, prec, seed=x["key"], alpha=ALPHA)
    state = {"case": case, "vegas": v, "params": torch.tensor(q, dtype=torch.float64, device="cuda"),
             "uniform": _uniform(case)}
    if op == "grad":
        # the frozen grid of a training run: adapted once, in FP64
        g = va.Vegas(d, N, "gauss", q, "fp64", seed=x["key"] + 1, alpha=ALPHA)
        for _ in range(5):
            g.iterate(200_000, refine=True, record=False)
        v.set_edges(g.edges())
        g.close()
        dt = torch.float32 if prec == "fp32_mixed" else torch.float64
        state["a"] = torch.tensor(q[0], dtype=dt, device="cuda", requires_grad=True)
        state["mu"] = torch.tensor(q[1:], dtype=dt, device="cuda", requires_grad=True)
    return state


def _result(r):
    return {k: np.float64(r[k]) for k in ("integral", "sigma", "chi2_dof", "last_integral", "last_sigma")} | {
        k: int(r[k]) for k in ("n_iter", "n_combined", "n_events")}


def run(state):
    case = state["case"]
    op = case["op"]
    if op == "batch":
        b = state["batch"]
        b.run()
        rs = [_result(r) for r in b.results()]
        return {k: np.array([r[k] for r in rs]) for k in rs[0]}
    v, M = state["vegas"], case["events"]
    if op == "grad":
        mu, a = state["mu"], state["a"]
        mu.grad = a.grad = None
        est = vegas_integral(mu, a, v, M, case["fused"])
        est.backward()
        return {"estimate": est.detach(), "mu_grad": mu.grad, "a_grad": a.grad}
    v.set_params_device(state["params"])
    v.set_edges(state["uniform"])
    v.reset_results()
    # without accumulation iterations every iteration counts, with them only those on the final grid
    all_count = case["accumulate"] == 0
    for refine in [True] * case["adapt"] + [False] * case["accumulate"]:
        if op == "stream":
            chunk = case["chunk"]
            for e0 in range(0, M, chunk):
                at = "begin" if e0 == 0 else "end" if e0 + chunk >= M else "mid"
                last = at == "end"
                v.iterate(min(chunk, M - e0), refine=refine and last, combine=all_count or not refine, chunk=at,
                          hist=refine)
        else:
            v.iterate(M, refine=refine, combine=all_count or not refine, hist=refine)
    return _result(v.result()) | {"edges": v.edges()}


# ---------------------------------------------------------------------------
# What a pass cannot do without: the point, map, integrand and sums of every
# event in operations (ten Philox rounds of two products and two three-way XORs
# per four dimensions; binning, map, exponent or denominator, Jacobian and
# table address per dimension; the histogram's add and address in an adaptation
# iteration; the gradient's product and add per component), the parameters and
# results in bytes.

def _ops(kind, d, hist, grad=False):
    per = 9 * d + 17 + (2 * d if kind == "bimodal" else 0)
    return 40 * math.ceil(d / 4) + per + (2 * d if hist else 0) + (2 * (d + 1) if grad else 0)


def work(case):
    d, N = case["dim"], case["bins"]
    if case["op"] == "batch":
        ops, size = 0.0, 0
        for q in _inputs(case, 0)["problems"]:
            for hist, n in ((True, case["adapt"]), (False, case["accumulate"])):
                ops += n * q["n_events"] * _ops(case["kind"], q["dim"], hist)
            size += 8 * len(q["params"]) + 64
        return {"bytes": size, "flops": ops}
    ops = case["events"] * (case["adapt"] * _ops(case["kind"], d, True) +
                            case["accumulate"] * _ops(case["kind"], d, False, case["op"] == "grad"))
    return {"bytes": 8 * (2 * d + 2) + 2 * 8 * d * (N + 1), "flops": float(ops)}


# ---------------------------------------------------------------------------
# The same pass in plain 64-bit torch.

_MASK = 0xFFFFFFFF


def _philox(e, t, c3, key):
    """Words of Philox4x32-10 at counters (e lo, e hi, t, c3), as int64."""
    c0, c1 = e & _MASK, (e >> 32) & _MASK
    c2, c3 = torch.full_like(e, t), torch.full_like(e, c3)
    k0, k1 = key & _MASK, (key >> 32) & _MASK
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((p1 >> 32) & _MASK) ^ (c1 ^ k0), p1 & _MASK, ((p0 >> 32) & _MASK) ^ (c3 ^ k1), p0 & _MASK
        k0, k1 = (k0 + 0x9E3779B9) & _MASK, (k1 + 0xBB67AE85) & _MASK
    return c0, c1, c2, c3


def _density(kind, q, x):
    """f at the points x[d] (a list of tensors)."""
    d = len(x)
    if kind in ("gauss", "bimodal"):
        a = q[0]
        nu = (a * math.sqrt(math.pi)) ** -d
        s = sum((x[i] - q[1 + i]) ** 2 for i in range(d))
        if kind == "gauss":
            return nu * torch.exp(-s / (a * a))
        s2 = sum((x[i] - q[1 + d + i]) ** 2 for i in range(d))
        return 0.5 * nu * (torch.exp(-s / (a * a)) + torch.exp(-s2 / (a * a)))
    if kind == "genz_disc":
        nu = math.prod(q[i] / (math.exp(q[i]) - math.exp(q[i] * q[d + i])) for i in range(d))
        f = nu * torch.exp(sum(q[i] * x[i] for i in range(d)))
        for i in range(d):
            f = torch.where(x[i] > q[d + i], f, 0.0)
        return f
    if kind == "genz_peak":
        f = torch.ones_like(x[0])
        for i in range(d):
            c, a = q[i], q[d + i]
            f = f / (c * (math.atan(c * (1 - a)) + math.atan(c * a))) / (c ** -2 + (x[i] - a) ** 2)
        return f
    return torch.cos(2 * math.pi * q[0] + sum(q[1 + i] * x[i] for i in range(d)))


def _iteration(kind, q, E, M, t, key, hist, problem=0, grad=False):
    """S1, S2, H[d][N] (or None) and the gradient sums of M events on the edges E."""
    d, N = E.shape[0], E.shape[1] - 1
    dev = torch.device("cuda")
    lo = torch.tensor(E[:, :-1], device=dev)
    wid = torch.tensor(E[:, 1:] - E[:, :-1], device=dev)
    s1 = s2 = 0.0
    H = torch.zeros(d, N, dtype=torch.float64, device=dev) if hist else None
    G = np.zeros(d + 1)
    step = 1 << 22
    for e0 in range(0, M, step):
        e = torch.arange(e0, min(M, e0 + step), device=dev, dtype=torch.int64)
        x, bins, w = [], [], torch.ones(len(e), dtype=torch.float64, device=dev)
        for i in range(d):
            if i % 4 == 0:
                words = _philox(e, t, problem * 256 + i // 4, key)
            p = (2 * words[i % 4] + 1) * N  # y N = p / 2^33
            b = p >> 33
            wb = wid[i][b]
            x.append(lo[i][b] + ((p & (2 ** 33 - 1)).double() * 2.0 ** -33) * wb)
            w = w * (N * wb)
            bins.append(b)
        v = _density(kind, q, x) * w
        s1 += float(v.sum())
        s2 += float((v * v).sum())
        if hist:
            for i in range(d):
                H[i] += torch.bincount(bins[i], weights=v * v, minlength=N)
        if grad:
            a = q[0]
            r2 = sum((x[i] - q[1 + i]) ** 2 for i in range(d))
            for i in range(d):
                G[i] += float((v * (2 * (x[i] - q[1 + i]) / (a * a))).sum())
            G[d] += float((v * ((2 * r2 / (a * a) - d) / a)).sum())
    return s1, s2, None if H is None else H.cpu().numpy(), G


def _refine(H, E):
    """Smooth, normalise, damp and rebin each dimension."""
    d, N = H.shape
    out = E.copy()
    for i in range(d):
        h = H[i]
        if not (0.0 < h.sum() < np.inf):
            continue
        s = np.empty(N)
        s[0], s[-1] = (h[0] + h[1]) / 2, (h[-2] + h[-1]) / 2
        s[1:-1] = (h[:-2] + h[1:-1] + h[2:]) / 3
        s = s / s.sum()
        r = np.zeros(N)
        at = (s > 0) & (s != 1)
        r[at] = ((s[at] - 1) / np.log(s[at])) ** ALPHA
        r[s == 1] = 1.0
        c = np.cumsum(r)
        level = np.arange(1, N) * c[-1] / N
        b = np.minimum(np.searchsorted(c, level, side="left"), N - 1)
        below = np.where(b > 0, c[b - 1], 0.0)
        out[i, 1:N] = E[i][b] + (level - below) / (c[b] - below) * (E[i][b + 1] - E[i][b])
    return out


def _integrate(kind, q, E, M, adapt, accumulate, key, problem=0):
    records, used = [], []
    for t in range(adapt + accumulate):
        s1, s2, H, _ = _iteration(kind, q, E, M, t, key, t < adapt, problem)
        mean = s1 / M
        records.append((mean, (s2 / M - mean * mean) / (M - 1)))
        if t >= adapt or accumulate == 0:
            used.append(records[-1])
        if H is not None:
            E = _refine(H, E)
    val, var = np.array(used).T
    sw = (1 / var).sum()
    mean = (val / var).sum() / sw
    chi2 = ((val - mean) ** 2 / var).sum()
    chi2 = chi2 / (len(used) - 1) if len(used) > 1 else math.nan
    return {"integral": mean, "sigma": sw ** -0.5, "chi2_dof": np.float64(chi2), "last_integral": np.float64(records[-1][0]),
            "last_sigma": np.sqrt(np.float64(records[-1][1])), "n_iter": len(records),
            "n_combined": len(used), "n_events": M * len(records)}, E


def exact(case, seed):
    x = _inputs(case, seed)
    key = x["key"]
    if case["op"] == "batch":
        cost = sum(q["n_events"] * math.ceil(q["dim"] / 4) for q in x["problems"]) * (case["adapt"] + case["accumulate"])
        if cost > 1.5e9:
            return None  # more than about 20 seconds
        rs = [_integrate(case["kind"], q["params"], np.tile(np.arange(q["n_bins"] + 1) / q["n_bins"], (q["dim"], 1)),
                         q["n_events"], case["adapt"], case["accumulate"], key, q["problem"])[0] for q in x["problems"]]
        return {k: np.array([r[k] for r in rs]) for k in rs[0]}
    q = [float(v) for v in x["params"]]
    E, M, d = _uniform(case), case["events"], case["dim"]
    if case["op"] == "grad":
        for t in range(5):
            E = _refine(_iteration("gauss", q, E, 200_000, t, key + 1, True)[2], E)
        s1, _, _, G = _iteration("gauss", q, E, M, 0, key, False, grad=True)
        return {"estimate": torch.tensor(s1 / M, dtype=torch.float64),
                "mu_grad": torch.tensor(G[:d] / M, dtype=torch.float64),
                "a_grad": torch.tensor(G[d] / M, dtype=torch.float64)}
    r, E = _integrate(case["kind"], q, E, M, case["adapt"], case["accumulate"], key)
    return r | {"edges": E}
