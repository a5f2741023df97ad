"""The work that this library is used for, as cases that can be timed.

A case is a dict of plain values. ``listed()`` names the fixed ones, ``draw``
gives more of the same ranges, ``prepare`` makes what a user's program holds
before the call, ``run`` is one pass through the public entry points, ``work``
is what a pass cannot do without and ``exact`` is the answer in float64.

Kinds of work:
  greedy   a ground set is made resident and summarised (Dataset + greedy)
  sets     f of many CSR sets over a resident ground set (eval_sets)
  gains    marginal gains of a candidate list for the caller's running minima
  sieve    a streaming summary of a resident ground set
  batch    many resident instances of uneven size advanced together
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2105_12026_amd import ebc

F64 = torch.float64


# ---- cases -----------------------------------------------------------------

def listed():
    return [
        # the smallest call: a summary of 5 out of 1000 short rows; latency and launches count
        {"name": "greedy_f32_n1000_d16_k5", "kind": "greedy", "data": "normal", "n": 1000, "d": 16, "k": 5,
         "dtype": "f32", "dist": "sqeuclidean"},
        # an offline summary of a large ground set in full precision (the benchmark's default size)
        {"name": "greedy_f32_n100000_d100_k50", "kind": "greedy", "data": "mixture", "n": 100000, "d": 100, "k": 50,
         "dtype": "f32", "dist": "sqeuclidean"},
        # the largest ground set and summary, with outliers, in the default reduced precision
        {"name": "greedy_bf16_n200000_d64_k100", "kind": "greedy", "data": "outliers", "n": 200000, "d": 64, "k": 100,
         "dtype": "bf16", "dist": "sqeuclidean"},
        # an ordinary request of ragged size in the narrowest type
        {"name": "greedy_fp8_n30011_d33_k20", "kind": "greedy", "data": "curves", "n": 30011, "d": 33, "k": 20,
         "dtype": "fp8", "dist": "sqeuclidean"},
        # few very long series: one machine's process curves
        {"name": "greedy_f32_n1000_d3524_k50", "kind": "greedy", "data": "curves", "n": 1000, "d": 3524, "k": 50,
         "dtype": "f32", "dist": "sqeuclidean"},
        # the Manhattan distance, ragged
        {"name": "greedy_l1_n10007_d50_k10", "kind": "greedy", "data": "mixture", "n": 10007, "d": 50, "k": 10,
         "dtype": "f32", "dist": "l1"},
        # many small sets over a large ground set, full precision
        {"name": "sets_f32_n50000_d100_l5000_s10", "kind": "sets", "data": "normal", "n": 50000, "d": 100, "l": 5000,
         "size": 10, "ragged": False, "dtype": "f32"},
        # the same scored in the data set's own reduced precision
        {"name": "sets_bf16_n50000_d100_l5000_s10", "kind": "sets", "data": "normal", "n": 50000, "d": 100, "l": 5000,
         "size": 10, "ragged": False, "dtype": "bf16"},
        # sets of 1 to 150 members, no size a multiple of a tile
        {"name": "sets_f32_n29501_d77_l701_s75", "kind": "sets", "data": "mixture", "n": 29501, "d": 77, "l": 701,
         "size": 75, "ragged": True, "dtype": "f32"},
        # one step of a stochastic optimiser that lives in the caller: gains of (n/k) ln(1/eps) sampled candidates
        {"name": "gains_f32_n50000_d100_c2303", "kind": "gains", "data": "mixture", "n": 50000, "d": 100, "c": 2303,
         "dtype": "f32"},
        # a streaming summary of the long series
        {"name": "sieve_f32_n1000_d3524_k50", "kind": "sieve", "data": "curves", "n": 1000, "d": 3524, "k": 50,
         "dtype": "f32", "algo": "sieve_streaming"},
        # instances of uneven size summarised together
        {"name": "batch_bf16_i16_n2000_50000_k20", "kind": "batch", "count": 16, "n_lo": 2000, "n_hi": 50000, "k": 20,
         "dtype": "bf16"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["greedy", "greedy", "greedy", "greedy", "sets", "sets", "gains", "sieve", "batch"])
    if kind == "greedy":
        form = rng.choice(["f32", "bf16", "f16", "fp8", "long", "l1"])
        c = {"kind": kind, "data": rng.choice(["mixture", "outliers", "curves"]), "dtype": form, "dist": "sqeuclidean"}
        if form == "f32":
            c.update(n=_log_int(rng, 500, 100000), d=_log_int(rng, 3, 100), k=_log_int(rng, 3, 50))
        elif form == "long":
            c.update(dtype=rng.choice(["f32", "bf16", "f16", "fp8"]), n=_log_int(rng, 300, 4000),
                     d=_log_int(rng, 129, 3524), k=_log_int(rng, 3, 50))
        elif form == "l1":
            c.update(dtype="f32", dist="l1", n=_log_int(rng, 500, 12000), d=_log_int(rng, 3, 64),
                     k=_log_int(rng, 3, 12))
        else:
            c.update(n=_log_int(rng, 500, 200000), d=_log_int(rng, 3, 64), k=_log_int(rng, 3, 100))
        return c
    if kind == "sets":
        dtype = rng.choice(["f32", "f32", "bf16", "f16", "fp8"])
        n, size = _log_int(rng, 1000, 50000), _log_int(rng, 2, 150)
        return {"kind": kind, "data": rng.choice(["normal", "mixture"]), "n": n, "d": _log_int(rng, 5, 100),
                "l": _log_int(rng, 20, max(21, 50000 // size)), "size": size, "ragged": rng.random() < 0.5,
                "dtype": dtype}
    if kind == "gains":
        n = _log_int(rng, 1000, 100000)
        return {"kind": kind, "data": "mixture", "n": n, "d": _log_int(rng, 5, 100),
                "c": min(n, _log_int(rng, 1, 10000)), "dtype": rng.choice(["f32", "bf16", "f16", "fp8"])}
    if kind == "sieve":
        return {"kind": kind, "data": "curves", "n": _log_int(rng, 300, 3000), "d": _log_int(rng, 16, 1000),
                "k": _log_int(rng, 5, 50), "dtype": rng.choice(["f32", "bf16"]),
                "algo": rng.choice(["sieve_streaming", "three_sieves"])}
    return {"kind": kind, "count": rng.randint(2, 16), "n_lo": 2000, "n_hi": _log_int(rng, 4000, 50000),
            "k": _log_int(rng, 3, 20), "dtype": rng.choice(["bf16", "f16", "fp8"])}


# ---- inputs ----------------------------------------------------------------

def _device():
    return torch.device("cuda:0" if torch.cuda.is_available() else "cpu")


def _points(data, n, d, seed):
    """float32 [n, d] on the GPU: i.i.d. normal points, a mixture of 20 Gaussians (means N(0, 4 I)), the mixture
    with 1% uniform outliers in [-20, 20]^d, or process curves (three jittered bumps, noise, 5% drifted)."""
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=g, device=dev, dtype=F64)

    def uniform(*shape):
        return torch.rand(*shape, generator=g, device=dev, dtype=F64)

    if data == "normal":
        return normal(n, d).float()
    if data == "curves":
        t = torch.linspace(0.0, 1.0, d, device=dev, dtype=F64)
        x = normal(n, d) * math.sqrt(0.05)
        for _ in range(3):
            centre, width, height = 0.1 + 0.8 * uniform(1), 0.03 + 0.12 * uniform(1), 0.5 + 1.5 * uniform(1)
            c = centre + 0.02 * normal(n, 1)
            w = width * (1.0 + 0.1 * normal(n, 1))
            h = height * (1.0 + 0.1 * normal(n, 1))
            x += h * torch.exp(-0.5 * ((t - c) / w) ** 2)
        drift = (uniform(n, 1) < 0.05) * (0.2 + 0.4 * uniform(n, 1))
        return (x + drift * t).float()
    comps = 20
    weights = -torch.log(uniform(comps).clamp_min(1e-12))
    means = 2.0 * normal(comps, d)
    which = torch.searchsorted(torch.cumsum(weights / weights.sum(), 0), uniform(n)).clamp_max(comps - 1)
    x = means[which] + normal(n, d)
    if data == "outliers":
        out = uniform(n) < 0.01
        x[out] = uniform(int(out.sum()), d) * 40.0 - 20.0
    return x.float()


def _sets(case, seed):
    """CSR sets of random members: all of one size, or sizes uniform in 1 .. 2 size - 1."""
    rng = np.random.default_rng([seed, 1])
    sizes = rng.integers(1, 2 * case["size"], case["l"]) if case["ragged"] else np.full(case["l"], case["size"])
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    idx = rng.integers(0, case["n"], int(offsets[-1])).astype(np.int32)
    return torch.from_numpy(offsets).to(_device()), torch.from_numpy(idx).to(_device())


def _candidates(case, seed):
    """The caller's running minima for a summary of 5 random points, and a sample of distinct candidates."""
    rng = np.random.default_rng([seed, 2])
    x = _points(case["data"], case["n"], case["d"], seed).to(F64)
    m = (x * x).sum(1)
    for i in rng.integers(0, case["n"], 5):
        m = torch.minimum(m, ((x - x[int(i)]) ** 2).sum(1))
    cand = rng.choice(case["n"], case["c"], replace=False).astype(np.int32)
    return m, torch.from_numpy(cand).to(_device())


def _instances(case, seed):
    """(points, k) of every instance of a batch: n uniform, d one of five row lengths."""
    rng = np.random.default_rng([seed, 3])
    out = []
    for i in range(case["count"]):
        n = int(rng.integers(case["n_lo"], case["n_hi"] + 1))
        d = int(rng.choice(np.asarray([8, 16, 32, 64, 128])))
        out.append((_points("mixture", n, d, int(rng.integers(1 << 30))), case["k"]))
    return out


def prepare(case, seed):
    kind = case["kind"]
    state = {"case": case}
    if kind == "batch":
        inst = _instances(case, seed)
        state["ks"] = [k for _, k in inst]
        state["batch"] = ebc.Batch([ebc.Dataset(x, dtype=case["dtype"]) for x, _ in inst])
        return state
    x = _points(case["data"], case["n"], case["d"], seed)
    if kind == "greedy":
        # the ground set is new in every pass: making it resident belongs to the pass
        state["x"] = x
        return state
    state["ds"] = ebc.Dataset(x, dtype=case["dtype"])
    if kind == "sets":
        state["offsets"], state["idx"] = _sets(case, seed)
    elif kind == "gains":
        state["m"], state["cand"] = _candidates(case, seed)
    return state


# ---- one pass --------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "greedy":
        ds = ebc.Dataset(state["x"], dtype=case["dtype"], dist=case["dist"])
        return ds.greedy(case["k"])
    if kind == "sets":
        return state["ds"].eval_sets(state["offsets"], state["idx"], in_dtype=case["dtype"] != "f32")
    if kind == "gains":
        return state["ds"].marginal_gains(m=state["m"], cand=state["cand"])
    if kind == "sieve":
        if case["algo"] == "three_sieves":
            return state["ds"].three_sieves(case["k"], 0.1, 5)
        return state["ds"].sieve_streaming(case["k"], 0.1)
    return state["batch"].greedy(state["ks"])


# ---- what a pass cannot do without -----------------------------------------

def _greedy_work(n, d, k):
    # every pair once (all gains at the empty set), then per step the distances of all points to the new member;
    # two operations per dimension of a pair under either distance
    return {"bytes": 4 * n * d + 20 * k, "flops": 2 * d * n * n + 2 * d * n * k}


def work(case):
    kind = case["kind"]
    if kind == "greedy":
        return _greedy_work(case["n"], case["d"], case["k"])
    if kind == "batch":
        # instances are drawn from the seed: mean of n and n^2 over the uniform range, mean row length 49.6
        lo, hi, c = case["n_lo"], case["n_hi"], case["count"]
        n1 = (lo + hi) / 2
        n2 = (lo * lo + lo * hi + hi * hi) / 3
        return {"bytes": int(c * 4 * n1 * 49.6), "flops": int(c * 2 * 49.6 * (n2 + n1 * case["k"]))}
    n, d = case["n"], case["d"]
    if kind == "sets":
        members = case["l"] * case["size"]
        return {"bytes": 4 * n * d + 8 * (case["l"] + 1) + 4 * members + 8 * case["l"], "flops": 2 * d * n * members}
    if kind == "gains":
        return {"bytes": 4 * n * d + 8 * n + 12 * case["c"], "flops": 2 * d * n * case["c"]}
    # sieves: float64 distances (subtract, multiply-add) of the examined points, at least k of them
    seen = n if case["algo"] == "sieve_streaming" else case["k"]
    return {"bytes": 4 * n * d + 12 * case["k"], "flops": 3 * d * n * seen}


# ---- the answer in float64 -------------------------------------------------

def _dist(a, b, dist="sqeuclidean"):
    """float64 distances [rows of a, rows of b]."""
    if dist == "l1":
        out = torch.zeros(a.shape[0], b.shape[0], dtype=F64, device=a.device)
        for k in range(a.shape[1]):
            out += (a[:, k, None] - b[None, :, k]).abs_()
        return out
    return ((a * a).sum(1)[:, None] + (b * b).sum(1)[None, :] - 2.0 * (a @ b.T)).clamp_min_(0.0)


def _gains(x, m, rows, dist, cells=1 << 28):
    step = max(1, cells // x.shape[0])
    out = [(m[None, :] - _dist(x[r], x, dist)).clamp_min_(0.0).sum(1) for r in torch.split(rows, step)]
    return torch.cat(out)


def _greedy(x, k, dist):
    """Greedy by stale upper bounds (the gains only shrink): the same picks as scoring every point at every step."""
    x = x.to(F64)
    n = x.shape[0]
    m = x.abs().sum(1) if dist == "l1" else (x * x).sum(1)
    l0 = m.mean()
    bound = _gains(x, m, torch.arange(n, device=x.device), dist)
    sel, f, gain = [], [], []
    for t in range(k):
        fresh = torch.zeros(n, dtype=torch.bool, device=x.device)
        if t == 0:
            fresh[:] = True
        while True:
            top = torch.topk(bound, min(n, 256)).indices
            if bool(fresh[top[0]]):
                break
            todo = top[~fresh[top]]
            bound[todo] = _gains(x, m, todo, dist)
            fresh[todo] = True
        best = int(torch.nonzero(bound == bound.max())[0])
        gain.append(bound[best] / n)
        bound[best] = -math.inf
        new = (x - x[best]).abs().sum(1) if dist == "l1" else ((x - x[best]) ** 2).sum(1)
        m = torch.minimum(m, new)
        sel.append(best)
        f.append(l0 - m.mean())
    return torch.stack(f), torch.stack(gain)


def _sieve(x, k, eps, algo, T):
    """Three Sieves or Sieve Streaming over the points in index order (see paper_2105_12026_amd/ebc.py)."""
    x = x.to(F64)
    n = x.shape[0]
    D = _dist(x, x)
    m0 = (x * x).sum(1)
    top = float((m0[None, :] - D).clamp_min(0.0).sum(1).max()) / n
    lo, hi = math.ceil(math.log(top) / math.log1p(eps) - 1e-12), math.floor(math.log(k * top) / math.log1p(eps) + 1e-12)
    grid = [(1.0 + eps) ** i for i in range(hi, lo - 1, -1)]
    if algo == "three_sieves":
        M, f, hits, rej, g = m0.clone(), [], 0, 0, 0
        for e in range(n):
            if hits == k:
                break
            gain = float((M - D[e]).clamp_min(0.0).sum()) / n
            cur = f[-1] if f else 0.0
            if gain >= (grid[g] / 2 - cur) / (k - hits):
                M = torch.minimum(M, D[e])
                f.append(float((m0 - M).mean()))
                hits, rej = hits + 1, 0
            else:
                rej += 1
                if rej >= T and g + 1 < len(grid):
                    g, rej = g + 1, 0
        return torch.tensor(f, dtype=F64)
    v = torch.tensor(grid, dtype=F64, device=x.device)
    M = m0[None, :].repeat(len(grid), 1)
    cnt = torch.zeros(len(grid), dtype=F64, device=x.device)
    cur = torch.zeros_like(cnt)
    hist = torch.zeros(len(grid), k, dtype=F64, device=x.device)
    for e in range(n):
        gain = (M - D[e]).clamp_min(0.0).sum(1) / n
        take = (cnt < k) & (gain >= (v / 2 - cur) / (k - cnt).clamp_min(1.0))
        M = torch.where(take[:, None], torch.minimum(M, D[e]), M)
        cur = torch.where(take, (m0 - M).mean(1), cur)
        rows = torch.nonzero(take).flatten()
        hist[rows, cnt[rows].long()] = cur[rows]
        cnt += take
    best = int(torch.nonzero(cur == cur.max())[0])
    return hist[best, :int(cnt[best])]


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        out = []
        for x, k in _instances(case, seed):
            f, gain = _greedy(x, k, "sqeuclidean")
            out.append((None, f, gain))
        return out
    x = _points(case["data"], case["n"], case["d"], seed)
    if kind == "greedy":
        f, gain = _greedy(x, case["k"], case["dist"])
        return None, f, gain
    if kind == "sets":
        offsets, idx = _sets(case, seed)
        x = x.to(F64)
        m0 = (x * x).sum(1)
        per = max(1, (1 << 27) // case["n"])  # members scored at a time
        off = offsets.tolist()
        out = torch.empty(case["l"], dtype=F64, device=x.device)
        j = 0
        while j < case["l"]:
            e = j + 1
            while e < case["l"] and off[e + 1] - off[j] <= per:
                e += 1
            d = _dist(x[idx[off[j]:off[e]].long()], x)
            for q in range(j, e):
                near = torch.minimum(m0, d[off[q] - off[j]:off[q + 1] - off[j]].amin(0))
                out[q] = (m0 - near).mean()
            j = e
        return out
    if kind == "gains":
        m, cand = _candidates(case, seed)
        return _gains(x.to(F64), m, cand.long(), "sqeuclidean") / case["n"]
    f = _sieve(x, case["k"], 0.1, case["algo"], 5)
    return (None, f, None) if case["algo"] == "three_sieves" else (None, f, None, None)
