"""Performance cases of the library: the calls its users make, over their real range.

Each case names one public entry point and its sizes.  `prepare` makes what a
program holds before the call (a context with the shipped tuning table, a cell
list, a dataset), `run` is one pass, `work` what a pass cannot do without, and
`exact` the same results in plain FP64 torch/numpy, written from the paper's
equations and the sampling contract of include/zpl.h.
"""
from __future__ import annotations

import math
from pathlib import Path

import numpy as np
import torch

import paper_1305_6738_amd as zpl

ROOT = Path(__file__).resolve().parent.parent
GAMMAS = [0.25, 0.5, 0.75, 1.0, 1.25, 1.5, 1.75, 2.0, 2.5, 3.0, 3.5, 4.0]
QS = [(9, 10), (95, 100), (99, 100), (999, 1000)]
# Largest number of draws that exact() recomputes (about ten seconds on the GPU).
EXACT_DRAWS = 1_000_000_000


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # one critical value while a program runs: the smallest call, latency and launches
        {"name": "cell", "kind": "cells", "alpha_lo": 2.5, "alpha_hi": 2.5, "n_lo": 100,
         "n_hi": 100, "cells": 1, "R": 10000, "spread": "even", "full": True},
        # the benchmark's table slice: 9 exponents at n = 1000, R = 100,000
        {"name": "slice", "kind": "cells", "alpha_lo": 1.5, "alpha_hi": 3.5, "n_lo": 1000,
         "n_hi": 1000, "cells": 9, "R": 100000, "spread": "even", "full": False},
        # uneven batch: n log-uniform on [10, 1e5], alpha uniform on [1.5, 3.5] (the largest case)
        {"name": "uneven", "kind": "cells", "alpha_lo": 1.5, "alpha_hi": 3.5, "n_lo": 10,
         "n_hi": 100000, "cells": 256, "R": 10000, "spread": "random", "full": False},
        # heavy tails: alpha in {1.2, 1.3, 1.4, 1.5} at n = 10,000
        {"name": "heavy-tail", "kind": "cells", "alpha_lo": 1.2, "alpha_hi": 1.5, "n_lo": 10000,
         "n_hi": 10000, "cells": 4, "R": 20000, "spread": "even", "full": True},
        # columns of the paper's Table 2 (K = 20) and Table 6 (K = 1000), one run each
        {"name": "table-K20", "kind": "critical", "kmax": 20, "n_lo": 10, "n_hi": 1000, "rows": 3,
         "gammas": 12, "seeds": 1, "R": 50000},
        {"name": "table-K1000", "kind": "critical", "kmax": 1000, "n_lo": 100, "n_hi": 1000,
         "rows": 2, "gammas": 12, "seeds": 1, "R": 50000},
        # the law with a lower cutoff: alpha in {2, 2.5, 3} x xmin in {10, 100}
        {"name": "cutoff", "kind": "cutoff", "alpha_lo": 2.0, "alpha_hi": 3.0, "alphas": 3,
         "xmin_lo": 10, "xmin_hi": 100, "xmins": 2, "n": 1000, "R": 100000},
        # the KS-minimising cutoff among 1,000 candidates, data on the device
        {"name": "scan", "kind": "scan", "n": 100000, "candidates": 1000, "alpha": 2.5,
         "device": True},
        # one fit of a dataset a program holds in host memory: latency
        {"name": "fit", "kind": "fit", "n": 5000, "alpha": 2.3, "kmax": 0, "xmin": 1,
         "device": False},
        # one fit of a large dataset already on the device
        {"name": "fit-large", "kind": "fit", "n": 10000000, "alpha": 2.2, "kmax": 0, "xmin": 1,
         "device": True},
        # the bespoke cutoff of Sect. 4 as a p-value (README's example)
        {"name": "bootstrap", "kind": "bootstrap", "n": 5000, "alpha": 2.3, "B": 2500},
        # a burst of serving requests of mixed size, submitted together
        {"name": "serve", "kind": "serve", "requests": 16, "n_lo": 50, "n_hi": 20000,
         "alpha_lo": 1.6, "alpha_hi": 3.4, "B": 2500},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["cells", "cells", "heavy", "critical", "cutoff", "scan", "fit", "fit",
                       "bootstrap", "serve"])
    if kind == "cells":
        cells, n_hi = _logint(rng, 1, 64), _logint(rng, 20, 50000)
        most = int(min(100000, 4e9 / (cells * n_hi)))  # draws stay well below the uneven batch's
        lo = rng.uniform(1.5, 3.0)
        return {"kind": "cells", "alpha_lo": lo, "alpha_hi": rng.uniform(lo, 3.5), "n_lo": 10,
                "n_hi": n_hi, "cells": cells, "R": _logint(rng, min(500, most), most),
                "spread": "random", "full": rng.random() < 0.5}
    if kind == "heavy":
        n = _logint(rng, 500, 20000)
        return {"kind": "cells", "alpha_lo": 1.15, "alpha_hi": 1.5, "n_lo": n, "n_hi": n,
                "cells": rng.randint(1, 5), "R": _logint(rng, 500, min(20000, int(1.5e8 / n))),
                "spread": "random", "full": True}
    if kind == "critical":
        n_hi = _logint(rng, 50, 5000)
        return {"kind": "critical", "kmax": rng.choice([0, _logint(rng, 5, 4096)]), "n_lo": 10,
                "n_hi": n_hi, "rows": rng.randint(1, 4), "gammas": rng.randint(2, 12),
                "seeds": rng.randint(1, 3), "R": _logint(rng, 1000, min(50000, int(4e7 / n_hi)))}
    if kind == "cutoff":
        n = _logint(rng, 30, 5000)
        return {"kind": "cutoff", "alpha_lo": 1.8, "alpha_hi": rng.uniform(2.0, 3.5),
                "alphas": rng.randint(1, 4), "xmin_lo": _logint(rng, 2, 50),
                "xmin_hi": _logint(rng, 51, 3000), "xmins": rng.randint(1, 3), "n": n,
                "R": _logint(rng, 500, min(50000, int(1e8 / n)))}
    if kind == "scan":
        return {"kind": "scan", "n": _logint(rng, 500, 300000),
                "candidates": _logint(rng, 5, 2000), "alpha": rng.uniform(1.7, 3.3),
                "device": rng.random() < 0.5}
    if kind == "fit":
        device = rng.random() < 0.6
        law = rng.choice(["pure", "pure", "truncated", "cutoff"])
        return {"kind": "fit", "n": _logint(rng, 50, 10000000 if device else 300000),
                "alpha": rng.uniform(1.6, 3.4),
                "kmax": _logint(rng, 20, 4096) if law == "truncated" else 0,
                "xmin": _logint(rng, 2, 100) if law == "cutoff" else 1, "device": device}
    if kind == "bootstrap":
        return {"kind": "bootstrap", "n": _logint(rng, 50, 50000), "alpha": rng.uniform(1.6, 3.4),
                "B": _logint(rng, 500, 5000)}
    return {"kind": "serve", "requests": rng.randint(2, 24), "n_lo": 50,
            "n_hi": _logint(rng, 500, 30000), "alpha_lo": 1.6, "alpha_hi": rng.uniform(2.0, 3.4),
            "B": _logint(rng, 500, 2500)}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
_CTX = None


def _context():
    """The program's one context, with the shipped form-cost table."""
    global _CTX
    if _CTX is None:
        _CTX = zpl.Context(0)
        _CTX.set_tuning(zpl.load_tuning(ROOT / "paper_1305_6738_amd" / "tuning" / "mi355x.json"))
    return _CTX


_SERVING = False


def _serving():
    global _SERVING
    ctx = _context()
    if not _SERVING:
        ctx.serve_start()
        _SERVING = True
    return ctx


def _sizes(lo, hi, k):
    """k whole numbers from lo to hi, spread over the logarithm."""
    if k == 1:
        return [hi]
    return [int(round(math.exp(math.log(lo) + i * (math.log(hi) - math.log(lo)) / (k - 1))))
            for i in range(k)]


def _cell_list(case, seed):
    """The case's cells as (alpha, n, R, seed, stream, kmax, xmin)."""
    kind = case["kind"]
    if kind == "cells":
        c, lo, hi = case["cells"], case["alpha_lo"], case["alpha_hi"]
        if case["spread"] == "even":
            al = [lo + (hi - lo) * i / max(c - 1, 1) for i in range(c)]
            ns = [case["n_hi"]] * c
        else:
            g = np.random.Generator(np.random.PCG64(c * 1000003 + case["n_hi"]))
            al = [float(v) for v in g.uniform(lo, hi, c)]
            ns = [int(round(v)) for v in
                  np.exp(g.uniform(math.log(case["n_lo"]), math.log(case["n_hi"]), c))]
        return [(al[i], ns[i], case["R"], seed, i, 0, 0) for i in range(c)]
    if kind == "cutoff":
        xs, k = _sizes(case["xmin_lo"], case["xmin_hi"], case["xmins"]), case["alphas"]
        al = [case["alpha_lo"] + (case["alpha_hi"] - case["alpha_lo"]) * i / max(k - 1, 1)
              for i in range(k)]
        return [(a, case["n"], case["R"], seed, 100 * i + j, 0, x)
                for i, a in enumerate(al) for j, x in enumerate(xs)]
    gs, ns = _gammas(case), _sizes(case["n_lo"], case["n_hi"], case["rows"])
    return [(g, n, case["R"], seed + s, i * len(gs) + j, case["kmax"], 0)
            for i, n in enumerate(ns) for j, g in enumerate(gs) for s in range(case["seeds"])]


def _gammas(case):
    if case["kmax"] == 0:  # the pure law's exponents
        k = case["gammas"]
        return [1.5 + 2.0 * i / max(k - 1, 1) for i in range(k)]
    return GAMMAS[:case["gammas"]]


def _zipf(rng, alpha, n):
    return np.minimum(rng.zipf(alpha, size=n), 1 << 62).astype(np.int64)


def _data_device(case, seed, xmin=1):
    """n values that follow a power law from xmin on, made on the device: the
    rounded continuous Pareto, which is close to the discrete law."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    u = torch.rand(case["n"], generator=g, device="cuda", dtype=torch.float64)
    y = (xmin - 0.5) * (1.0 - u).pow(-1.0 / (case["alpha"] - 1.0)) + 0.5
    x = y.clamp_(max=float(1 << 52)).floor_().to(torch.int64)
    if case.get("kmax"):
        # the truncated law: fold what lies above K back onto 1..K
        x = torch.where(x > case["kmax"], x % case["kmax"] + 1, x)
    return x


def _dataset(case, seed):
    if case["kind"] == "scan":
        # a body below the cutoff 60 that is no power law, and a tail that is
        g = torch.Generator(device="cuda").manual_seed(seed)
        nb = (3 * case["n"]) // 10
        tail = _data_device({"n": case["n"] - nb, "alpha": case["alpha"]}, seed + 1, 60)
        body = torch.randint(1, 60, (nb,), generator=g, device="cuda", dtype=torch.int64)
        x = torch.cat([body, tail])
        x = x[torch.randperm(case["n"], generator=g, device="cuda")].contiguous()
        return x if case["device"] else x.cpu().numpy()
    if case["kind"] == "fit" and case["device"]:
        return _data_device(case, seed)
    x = _zipf(np.random.Generator(np.random.PCG64(seed)), case["alpha"], case["n"])
    if case.get("kmax"):
        x = np.where(x > case["kmax"], x % case["kmax"] + 1, x)
    return x


def _candidates(case):
    return list(range(1, case["candidates"] + 1))


def _requests(case, seed):
    g = np.random.Generator(np.random.PCG64(case["requests"] * 7919 + case["n_hi"]))
    ns = [int(round(v)) for v in
          np.exp(g.uniform(math.log(case["n_lo"]), math.log(case["n_hi"]), case["requests"]))]
    al = [float(v) for v in g.uniform(case["alpha_lo"], case["alpha_hi"], case["requests"])]
    rng = np.random.Generator(np.random.PCG64(seed))
    return [_zipf(rng, al[i], ns[i]) for i in range(case["requests"])]


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "seed": seed, "ctx": _serving() if kind == "serve" else _context()}
    if kind in ("cells", "cutoff"):
        cells = _cell_list(case, seed)
        s["cells"] = zpl.cell_array(cells)
        if kind == "cutoff" or case["full"]:
            total = sum(c[2] for c in cells)
            s["D"] = torch.zeros(total, dtype=torch.float64, device="cuda")
            s["alpha"] = torch.zeros(total, dtype=torch.float64, device="cuda")
            s["flags"] = torch.zeros(total, dtype=torch.int32, device="cuda")
    elif kind == "critical":
        s["gammas"] = _gammas(case)
        s["ns"] = _sizes(case["n_lo"], case["n_hi"], case["rows"])
    elif kind == "serve":
        s["x"] = _requests(case, seed)
    else:
        s["x"] = _dataset(case, seed)
    return s


def run(s):
    case, ctx, kind = s["case"], s["ctx"], s["case"]["kind"]
    if kind in ("cells", "cutoff"):
        if "D" in s:
            q = ctx.simulate_cells(s["cells"], quantiles=QS, d_out=s["D"],
                                   alpha_hat_out=s["alpha"], flags_out=s["flags"])
            return {"q": q, "D": s["D"], "alpha": s["alpha"], "flags": s["flags"]}
        return {"q": ctx.simulate_cells(s["cells"], quantiles=QS)}
    if kind == "critical":
        return {"table": ctx.critical_table(s["gammas"], s["ns"], kmax=case["kmax"],
                                            seeds=case["seeds"], seed0=s["seed"],
                                            replicates=case["R"], quantiles=QS)}
    if kind == "scan":
        r = ctx.fit_scan(s["x"], _candidates(case))
        return {k: r[k] for k in ("best", "alpha_hat", "D", "n_tail", "flags")}
    if kind == "fit":
        return ctx.fit(s["x"], kmax=case["kmax"], xmin=case["xmin"])
    if kind == "bootstrap":
        return ctx.bootstrap_pvalue(s["x"], case["B"], s["seed"])
    tickets = [ctx.serve_submit(x, case["B"], s["seed"], i) for i, x in enumerate(s["x"])]
    rs = []
    for t in tickets:
        r = None
        while r is None:
            r = ctx.serve_poll(t, 1000)
        rs.append(r)
    return {"alpha_hat": np.array([r["alpha_hat"] for r in rs]),
            "D": np.array([r["D"] for r in rs]), "p": np.array([r["p_value"] for r in rs]),
            "status": np.array([r["status"] for r in rs])}


def work(case):
    """Per draw 49 integer operations (Philox, the uniform, the table search,
    the count), per replicate 2,000 (the fit and the distance); the inputs are
    cell lists or datasets, the outputs a few bytes per replicate or fit."""
    kind = case["kind"]
    per = lambda n, reps: 49.0 * n * reps + 2000.0 * reps  # noqa: E731
    if kind in ("cells", "cutoff", "critical"):
        cells = _cell_list(case, 0)
        total = sum(c[2] for c in cells)
        out = 8 * len(QS) * len(cells)
        if kind == "cutoff" or case.get("full"):
            out += 20 * total
        return {"bytes": 56 * len(cells) + out, "flops": sum(per(c[1], c[2]) for c in cells)}
    if kind == "fit":
        return {"bytes": 8 * case["n"] + 24, "flops": 2 * case["n"] + 2000}
    if kind == "scan":
        k = case["candidates"]
        return {"bytes": 8 * case["n"] + 40 * k, "flops": 2 * case["n"] + 2000 * k}
    if kind == "bootstrap":
        return {"bytes": 8 * case["n"] + 32, "flops": per(case["n"], case["B"])}
    ns = [len(x) for x in _requests(case, 0)]
    return {"bytes": 8 * sum(ns) + 32 * len(ns), "flops": sum(per(n, case["B"]) for n in ns)}


# ---------------------------------------------------------------------------
# The same results in plain FP64: Philox4x32-10, inversion over F(1..4096),
# the rejection tail, the MLE by bisection and the KS distance over the sorted
# sample.
# ---------------------------------------------------------------------------
_B = [1 / 12, -1 / 720, 1 / 30240, -1 / 1209600, 1 / 47900160, -691 / 1307674368000,
      1 / 74724249600, -3617 / 10670622842880000]


def _dev():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _philox(c0, c1, c2, c3, seed):
    M = 0xffffffff
    k0, k1 = seed & M, (seed >> 32) & M
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        h0, h1 = (p0 >> 32) & M, (p1 >> 32) & M
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, p1 & M, h0 ^ c3 ^ k1, p0 & M
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    return c0, c1, c2, c3


def _u53(hi, lo):
    return ((hi << 21) | (lo >> 11) | 1).to(torch.float64) * 2.0 ** -53


def _em(s, q, lq):
    """Sum of k^-s over k >= q, times q^s exp(-s lq) (Euler-Maclaurin, large q)."""
    iq = 1.0 / q
    acc, P, e = torch.zeros_like(s * iq), s, iq
    for i, c in enumerate(_B):
        acc = acc + c * P * e
        P = P * (s + (2 * i + 1)) * (s + (2 * i + 2))
        e = e * iq * iq
    return torch.exp(-s * lq) * (q / (s - 1.0) + 0.5 + acc)


def _survival(s, t, x0):
    """Sum of k^-s over k > t, times x0^s (x0 the law's smallest value)."""
    q = t + 1.0
    z = torch.zeros_like(s * q)
    for j in range(16):
        z = z + torch.exp(-s * torch.log((q + j) / x0))
    return z + _em(s, q + 16.0, torch.log((q + 16.0) / x0))


def _mu(s, K, x0):
    """E[ln X] under exponent s, for a vector s (and x0 one value, or one for each s)."""
    x0 = torch.as_tensor(x0, dtype=torch.float64, device=s.device).reshape(-1, 1)
    k = x0 + torch.arange(K or 64, device=s.device, dtype=torch.float64)[None, :]
    w = torch.exp(-s[:, None] * torch.log(k / x0))
    z0, z1 = w.sum(1), (w * torch.log(k)).sum(1)
    if K:
        return z1 / z0
    # the tail from x0 + 64 on and minus its s-derivative
    x0 = x0[:, 0]
    q = x0 + 64.0
    L = torch.log(q)
    a0 = q / (s - 1.0) + 0.5
    a1 = -q / (s - 1.0) ** 2
    P, dP, e = s, torch.ones_like(s), 1.0 / q
    for i, c in enumerate(_B):
        a0, a1 = a0 + c * P * e, a1 + c * dP * e
        for j in (1, 2):
            f = s + (2 * i + j)
            dP, P = dP * f + P, P * f
        e = e / (q * q)
    qs = torch.exp(-s * torch.log(q / x0))
    return (z1 + qs * (L * a0 - a1)) / (z0 + qs * a0)


def _mle(m, K, x0):
    """Root of mu(a) = m by bisection, a vector; the bracket's end where there is none."""
    out = []
    step = max(1, (1 << 26) // (K or 64))
    x0 = torch.as_tensor(x0, dtype=torch.float64, device=m.device).expand(m.shape)
    for part, xp in zip(m.split(step), x0.split(step)):
        lo = torch.full_like(part, -64.0 if K else 1.0 + 2.0 ** -20)
        hi = torch.full_like(part, 64.0)
        for _ in range(58):
            mid = 0.5 * (lo + hi)
            up = _mu(mid, K, xp) > part
            lo, hi = torch.where(up, mid, lo), torch.where(up, hi, mid)
        out.append(0.5 * (lo + hi))
    return torch.cat(out)


def _F(a, t, K, x0):
    """The CDF at integers t >= x0 - 1 (a and t broadcast)."""
    if K:
        ks = torch.arange(1, K + 1, device=a.device, dtype=torch.float64)
        P = torch.exp(-a.reshape(-1, 1) * torch.log(ks)[None, :]).cumsum(1)
        P = torch.cat([torch.zeros_like(P[:, :1]), P], 1) / P[:, -1:]
        return P.gather(1, t.to(torch.int64).expand(P.shape[0], -1))
    z = _survival(a, torch.full_like(a, x0 - 1.0), float(x0))
    return 1.0 - _survival(a, t, float(x0)) / z


def _ks(x, a, K, x0):
    """D of each row of the sorted sample x [rows, n] under the rows' exponents a."""
    n = x.shape[1]
    i = torch.arange(n, device=x.device, dtype=torch.float64)[None, :]
    same = x[:, 1:] == x[:, :-1]
    edge = torch.zeros((x.shape[0], 1), dtype=torch.bool, device=x.device)
    first, last = ~torch.cat([edge, same], 1), ~torch.cat([same, edge], 1)
    t = x.to(torch.float64)
    a = a[:, None]
    up = torch.where(last, (_F(a, t, K, x0) - (i + 1.0) / n).abs(), 0.0)
    dn = torch.where(first, (_F(a, t - 1.0, K, x0) - i / n).abs(), 0.0)
    return torch.maximum(up.amax(1), dn.amax(1))


def _table(alpha, K, x0):
    d = _dev()
    a = torch.tensor([alpha], dtype=torch.float64, device=d)
    if K:
        t = torch.arange(1, K + 1, device=d, dtype=torch.float64)
        w = torch.exp(-alpha * torch.log(t))
        suf = w.flip(0).cumsum(0).flip(0)  # from the smallest terms up
        T = torch.ones(4096, device=d, dtype=torch.float64)
        T[: K - 1] = 1.0 - suf[1:] / suf[0]
        return T
    t = torch.arange(x0, x0 + 4096, device=d, dtype=torch.float64)
    return _F(a, t, 0, x0)


def _draws(alpha, n, seed, stream, r0, r1, K, x0, T):
    """The draws of replicates r0..r1-1, [r1 - r0, n]."""
    d = T.device
    rep = torch.arange(r0, r1, device=d, dtype=torch.int64)[:, None]
    j = torch.arange((n + 1) // 2, device=d, dtype=torch.int64)[None, :]
    z = torch.zeros_like(rep + j)
    w = _philox(z + j, z + rep, z + stream, z, seed)
    U = torch.stack([_u53(w[0], w[1]), _u53(w[2], w[3])], 2).reshape(len(rep), -1)[:, :n]
    x = torch.searchsorted(T, U.contiguous()) + x0
    todo = (U > T[-1]).nonzero()
    rr, ii = todo[:, 0], todo[:, 1]
    beta, m0 = alpha - 1.0, float(x0 + 4096)

    def g(k):
        return 1.0 / (-k * torch.expm1(-beta * torch.log1p(1.0 / k)))
    gm = float(g(torch.tensor(m0, dtype=torch.float64)))
    attempt = 0
    while len(rr):
        o = torch.zeros_like(ii)
        w = _philox(ii, rr + r0, o + stream, o + (0x80000000 | attempt), seed)
        y = m0 * torch.exp(-torch.log(_u53(w[0], w[1])) / beta)
        X = y.clamp(max=2.0 ** 62.99).floor()
        ok = (y < 2.0 ** 63) & (_u53(w[2], w[3]) * gm <= g(X))
        x[rr[ok], ii[ok]] = X[ok].to(torch.int64)
        rr, ii = rr[~ok], ii[~ok]
        attempt += 1
    return x


def _simulate(cell):
    """(D, alpha_hat) of every replicate of a cell."""
    alpha, n, R, seed, stream, K, xmin = cell
    x0 = max(xmin, 1)
    T = _table(alpha, K, x0)
    Ds, As = [], []
    step = max(1, (1 << 25) // n)
    if K:
        step = min(step, max(1, (1 << 25) // K))
    for r0 in range(0, R, step):
        x = _draws(alpha, n, seed, stream, r0, min(R, r0 + step), K, x0, T)
        a = _alpha(x, K, x0)
        Ds.append(_ks(x.sort(1).values, a, K, x0))
        As.append(a)
    return torch.cat(Ds), torch.cat(As)


def _alpha(x, K, x0):
    S = torch.log(x.to(torch.float64)).sum(1)
    n = x.shape[1]
    flat = (x == x0).all(1)  # every value at the smallest one: one counts as the next
    S = torch.where(flat, (n - 1) * math.log(x0) + math.log(x0 + 1.0), S)
    return _mle(S / n, K, x0)


def _fit(x, K, x0):
    """alpha_hat and D of one dataset, over its distinct values."""
    v, c = torch.unique(x, return_counts=True)
    n = int(c.sum())
    t, w = v.to(torch.float64), c.to(torch.float64)
    S = float((torch.log(t) * w).sum())
    if len(v) == 1 and int(v[0]) == x0:
        S = (n - 1) * math.log(x0) + math.log(x0 + 1.0)
    a = _mle(torch.tensor([S / n], dtype=torch.float64, device=x.device), K, x0)
    C = w.cumsum(0)
    up = (_F(a[:, None], t[None, :], K, x0) - C / n).abs().max()
    dn = (_F(a[:, None], t[None, :] - 1.0, K, x0) - (C - w) / n).abs().max()
    return float(a[0]), float(torch.maximum(up, dn)), n


def _quantiles(D):
    s = D.sort().values
    return [float(s[(len(s) * a) // b]) for a, b in QS]


def exact(case, seed):
    kind = case["kind"]
    dev = _dev()
    if kind in ("cells", "cutoff", "critical"):
        cells = _cell_list(case, seed)
        if sum(c[1] * c[2] for c in cells) > EXACT_DRAWS:
            return None
        got = [_simulate(c) for c in cells]
        q = np.array([_quantiles(D) for D, _ in got])
        if kind == "critical":
            ns, gs = case["rows"], case["gammas"]
            return {"table": q.reshape(ns, gs, case["seeds"], len(QS)).mean(2)}
        if kind == "cutoff" or case["full"]:
            return {"q": q, "D": torch.cat([D for D, _ in got]),
                    "alpha": torch.cat([a for _, a in got]), "flags": None}
        return {"q": q}
    if kind == "serve":
        xs = _requests(case, seed)
        if sum(len(x) for x in xs) * case["B"] > EXACT_DRAWS:
            return None
        rs = [_bootstrap(torch.from_numpy(x).to(dev), case["B"], seed, i)
              for i, x in enumerate(xs)]
        return {"alpha_hat": np.array([r[0] for r in rs]), "D": np.array([r[1] for r in rs]),
                "p": np.array([r[2] for r in rs]), "status": None}
    x = _dataset(case, seed)
    x = torch.from_numpy(x).to(dev) if isinstance(x, np.ndarray) else x.to(dev)
    if kind == "bootstrap":
        if case["n"] * case["B"] > EXACT_DRAWS:
            return None
        a, D, p = _bootstrap(x, case["B"], seed, 0)
        return {"alpha_hat": a, "D": D, "p_value": p, "flags": None}
    if kind == "fit":
        x0 = case["xmin"]
        a, D, n = _fit(x[x >= x0], case["kmax"], x0)
        r = {"alpha_hat": a, "D": D, "flags": None, "status": None}
        if x0 > 1:
            r["n_tail"] = n
        return r
    return _scan(x, _candidates(case))


def _scan(x, cand):
    """The fit at every candidate cutoff, over the distinct values above it."""
    v, c = torch.unique(x, return_counts=True)
    t, w = v.to(torch.float64), c.to(torch.float64)
    x0 = torch.tensor(cand, dtype=torch.float64, device=x.device)
    at = torch.searchsorted(t, x0)  # first distinct value of each candidate
    live = at < len(t)
    at = at.clamp(max=len(t) - 1)
    below = torch.cat([torch.zeros_like(w[:1]), w.cumsum(0)])
    lw = torch.cat([(torch.log(t) * w).flip(0).cumsum(0).flip(0), torch.zeros_like(w[:1])])
    n = below[-1] - below[at]
    S = lw[at]
    flat = (at == len(t) - 1) & (t[-1] == x0)
    S = torch.where(flat, (n - 1) * torch.log(x0) + torch.log(x0 + 1.0), S)
    a = _mle(S / n, 0, x0)
    D = []
    step = max(1, (1 << 25) // len(t))
    for i in range(0, len(cand), step):
        s, q, p, m = (y[i:i + step, None] for y in (a, x0, at, n))
        tt = torch.maximum(t[None, :], q)
        z = _survival(s, q - 1.0, q)
        Cn = (below[1:][None, :] - below[p]) / m
        up = (1.0 - _survival(s, tt, q) / z - Cn).abs()
        dn = (1.0 - _survival(s, tt - 1.0, q) / z - (Cn - w[None, :] / m)).abs()
        D.append(torch.where(t[None, :] >= q, torch.maximum(up, dn), 0.0).amax(1))
    D = torch.where(live, torch.cat(D), math.inf)
    return {"best": None, "alpha_hat": torch.where(live, a, 0.0).cpu().numpy(),
            "D": D.cpu().numpy(), "n_tail": None, "flags": None}


def _bootstrap(x, B, seed, stream):
    a, D, _ = _fit(x, 0, 1)
    Db, _ = _simulate((a, len(x), B, seed, stream, 0, 0))
    return a, D, float((Db >= D - 1e-13).to(torch.float64).mean())
