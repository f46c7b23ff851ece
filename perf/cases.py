"""Timed cases: the calls that a user of the library makes, over their real range.

A case is one pass through the public entry points on device-resident inputs:
top-N mining (the main path), thresholds with the users' lists, scores of new
items, the relaxed score and its gradient, and the two indexes.  Inputs follow
the synthetic workloads of this repository (log-normal norms, isotropic or
64-cluster directions), drawn on the GPU from the seed.
"""
import math
from statistics import NormalDist

import numpy as np
import torch

import paper_2504_13445_amd as rm

# the largest n * m * d of a drawn case: a quarter of the largest listed one,
# because item norms with a small spread let a scan reach four times as far
_DRAW_PAIRS = 1.0e13


def listed():
    return [
        # the smallest catalogue: a call is launches and one synchronisation
        dict(name="topn_tiny", kind="topn", n=2_000, m=1_000, d=16, k=10, N=10, prec="fp32",
             clusters=0, us=0.3, ps=0.3),
        # a matrix-factorisation sized catalogue at the default precision
        dict(name="topn_100k", kind="topn", n=100_000, m=20_000, d=50, k=10, N=10, prec="fp32",
             clusters=0, us=0.25, ps=0.6),
        # sizes that fill no tile, a long list per user, BF16 screening
        dict(name="topn_ragged_bf16", kind="topn", n=130_051, m=23_501, d=75, k=25, N=20,
             prec="bf16", clusters=64, us=0.25, ps=0.7),
        # a regional catalogue with BF16 screening
        dict(name="topn_500k_bf16", kind="topn", n=500_000, m=50_000, d=100, k=20, N=50,
             prec="bf16", clusters=64, us=0.25, ps=0.8),
        # the same catalogue with e4m3 screening
        dict(name="topn_500k_fp8", kind="topn", n=500_000, m=50_000, d=100, k=20, N=50,
             prec="fp8", clusters=64, us=0.25, ps=0.8),
        # the whole catalogue: 2M users, 100k items, 200 dimensions
        dict(name="topn_2m", kind="topn", n=2_000_000, m=100_000, d=200, k=10, N=100,
             prec="fp32", clusters=64, us=0.25, ps=0.8),
        # every user's exact list (k-MIPS itself), ragged sizes
        dict(name="lists_200k", kind="lists", n=200_003, m=30_011, d=128, k=20, N=0, prec="fp32",
             clusters=64, us=0.25, ps=0.6),
        # how many users a thousand new items would reach
        dict(name="scores_500k", kind="scores", n=500_000, m=10_000, d=100, k=10, N=0,
             prec="fp32", clusters=64, us=0.25, ps=0.8, q=1_000),
        # one ascent step of new-item design: forward and backward over all users
        dict(name="soft_1m", kind="soft", n=1_000_000, m=5_000, d=100, k=10, N=0, prec="fp32",
             clusters=64, us=0.25, ps=0.8, q=256),
        # the same on a small user sample and few queries, forward and backward apart
        dict(name="soft_30k", kind="soft2", n=30_011, m=2_000, d=61, k=10, N=0, prec="fp32",
             clusters=64, us=0.25, ps=0.6, q=40),
        # the k_max table: built once per catalogue, then asked for two (k, N)
        dict(name="index_100k", kind="index", n=100_000, m=20_000, d=50, k=25, N=20, prec="fp32",
             clusters=0, us=0.25, ps=0.6),
        # the budgeted index and one query
        dict(name="budget_50k", kind="budget", n=50_021, m=10_007, d=50, k=25, N=20, prec="bf16",
             clusters=0, us=0.25, ps=0.6),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["topn", "topn", "topn", "topn", "lists", "scores", "soft", "soft2",
                       "index", "budget"])
    prec = rng.choice(["fp32", "fp32", "bf16", "bf16", "fp8"]) if kind == "topn" \
        else rng.choice(["fp32", "bf16"])
    hi_n = {"topn": 2_000_000, "lists": 400_000, "scores": 1_000_000, "soft": 1_000_000,
            "soft2": 100_000, "index": 200_000, "budget": 100_000}[kind]
    hi_m = {"topn": 100_000, "lists": 50_000, "scores": 10_000, "soft": 5_000,
            "soft2": 5_000, "index": 30_000, "budget": 20_000}[kind]
    n, m = _log_int(rng, 2_000, hi_n), _log_int(rng, 1_000, hi_m)
    d = _log_int(rng, 16, 200)
    k = _log_int(rng, 1, 32)
    N = _log_int(rng, 10, 100)
    ps = round(rng.uniform(0.3, 0.8), 2)
    if prec == "fp8":  # its wide band is meant for rows and norms like the listed case's
        d, k, ps = min(d, 128), min(k, 20), max(ps, 0.6)
        n, m = min(n, 500_000), min(m, 50_000)
    if kind in ("index", "budget"):
        k = max(k, 10)
    if n * m * d > _DRAW_PAIRS:
        n = max(2_000, int(_DRAW_PAIRS / (m * d)))
    c = dict(kind=kind, n=n, m=m, d=d, k=k, N=N, prec=prec, clusters=rng.choice([0, 64]),
             us=0.25, ps=ps)
    if kind == "scores":
        c["q"] = _log_int(rng, 32, 2_000)
    if kind in ("soft", "soft2"):
        c["prec"] = "fp32"
        c["q"] = _log_int(rng, 16, 256)
    return c


def _rows(g, count, d, sigma, clusters):
    """Directions (isotropic, or a mixture of `clusters` normal centres with
    spread 0.5) with LogNormal(0, sigma) norms, FP32 on the GPU."""
    x = torch.randn((count, d), generator=g, device="cuda")
    if clusters:
        c = torch.randn((clusters, d), generator=g, device="cuda")
        z = torch.randint(0, clusters, (count,), generator=g, device="cuda")
        x.mul_(0.5).add_(c[z])
    r = torch.exp(sigma * torch.randn(count, generator=g, device="cuda"))
    return x.mul_((r / x.norm(dim=1)).unsqueeze(1))


def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(1_000_003 * seed + 17)
    n, m, d = case["n"], case["m"], case["d"]
    s = {"U": _rows(g, n, d, case["us"], case["clusters"]),
         "P": _rows(g, m, d, case["ps"], 0)}
    if "q" in case:
        s["Q"] = torch.randn((case["q"], d), generator=g, device="cuda") / math.sqrt(d)
        if case["kind"] == "scores":
            # new items worth asking about: norms from the upper part of the catalogue's
            s["Q"] *= torch.exp(case["ps"] * (1.0 + torch.randn(
                (case["q"], 1), generator=g, device="cuda").abs()))
        s["dS"] = torch.rand(case["q"], generator=g, device="cuda") + 0.5
    if case["kind"] in ("soft", "soft2"):
        # temperature: 0.05 of the standard deviation of u . p, from the moments
        U, P = s["U"].double(), s["P"].double()
        second = ((U.T @ U / n) * (P.T @ P / m)).sum()
        s["T"] = 0.05 * float(torch.sqrt(second - (U.mean(0) @ P.mean(0)) ** 2))
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    kind, n, m, d, k, N, prec = (case[x] for x in ("kind", "n", "m", "d", "k", "N", "prec"))
    s["case"] = case
    if kind == "topn":
        # a program that calls again keeps its workspace
        s["ws"] = rm.topn_workspace(n, m, d, k, N, prec, torch.device("cuda"))
    if kind in ("scores", "soft", "soft2"):
        # the users' thresholds against the present catalogue, found once
        tau, tid = rm.thresholds(s["U"], s["P"], k, "bf16")
        s["tau"], s["tid"] = (tau, tid) if kind == "scores" else (tau.float(), tid)
    if kind == "soft":
        s["Q"].requires_grad_(True)
    torch.cuda.synchronize()
    return s


def run(s):
    c = s["case"]
    kind, k, N, prec = c["kind"], c["k"], c["N"], c["prec"]
    U, P = s["U"], s["P"]
    if kind == "topn":
        ids, sc, _ = rm.topn(U, P, k, N, prec, ws=s["ws"])
        return ids, sc
    if kind == "lists":
        return rm.thresholds(U, P, k, prec, with_topk=True)
    if kind == "scores":
        return rm.scores(U, s["tau"], s["tid"], s["Q"], prec=prec)
    if kind == "soft":
        Q = s["Q"]
        S = rm.SoftScore.apply(Q, U, s["tau"], s["T"])
        (dQ,) = torch.autograd.grad(S, Q, s["dS"])
        return S.detach(), dQ
    if kind == "soft2":
        return (rm.soft_fwd(U, s["tau"], s["Q"], s["T"]),
                rm.soft_bwd(U, s["tau"], s["Q"], s["T"], s["dS"]))
    if kind == "index":
        ix = rm.Index(U, P, k, prec)
        tau, tid = ix.thresholds(10)
        ids1, sc1, _ = ix.topn(10, N)
        ids2, sc2, _ = ix.topn(k, 2 * N)
        return tau, tid, ids1, sc1, ids2, sc2
    ix = rm.BudgetIndex(U, P, k, 2 * k, 8 * k * c["n"], prec=prec)
    ids, sc, _ = ix.topn(10, N)
    return ids, sc


def _reach(c):
    """Share of the norm-ordered items that no scan can leave out: with
    isotropic items u . p / |u| = |p| x, x ~ N(0, 1/d); t is the value that k
    items reach, and the items with |p| >= t are open under Cauchy-Schwarz."""
    nd, s, m, d = NormalDist(), c["ps"], c["m"], c["d"]
    norms = [math.exp(s * nd.inv_cdf((i + 0.5) / 400)) for i in range(400)]
    lo, hi = 0.0, max(norms)
    for _ in range(40):
        t = 0.5 * (lo + hi)
        above = sum(1.0 - nd.cdf(t / r * math.sqrt(d)) for r in norms) * m / 400
        lo, hi = (t, hi) if above > c["k"] else (lo, t)
    return max(c["k"] / m, 1.0 - nd.cdf(math.log(max(lo, 1e-9)) / s))


def work(case):
    n, m, d, k, N = (case[x] for x in ("n", "m", "d", "k", "N"))
    kind = case["kind"]
    rows = 4.0 * d * (n + m)
    scan = 2.0 * d * n * m * _reach(case)
    if kind == "topn":
        return {"bytes": rows + 8.0 * N, "flops": scan}
    if kind == "lists":
        return {"bytes": rows + n * (12.0 + 4.0 * k), "flops": scan}
    if kind == "scores":
        return {"bytes": 4.0 * d * (n + case["q"]) + 12.0 * n + 4.0 * case["q"],
                "flops": 2.0 * d * n * case["q"]}
    if kind in ("soft", "soft2"):
        q = case["q"]
        once = 4.0 * d * (n + q) + 4.0 * n + 4.0 * q * (d + 2)
        # one pass gives both directions; apart, the backward forms the products again
        return {"bytes": once if kind == "soft" else 2.0 * once,
                "flops": (4.0 if kind == "soft" else 6.0) * d * n * q}
    if kind == "index":  # the table of k values, ids and bounds; thresholds of one k
        return {"bytes": rows + n * 12.0 * k + m * 4.0 * k + 12.0 * n, "flops": scan}
    return {"bytes": rows + n * 12.0 * k + m * 4.0 * k, "flops": scan}


def _lists64(U, P, k):
    """Values and ids of each user's k largest products, FP64."""
    P64 = P.double()
    step = max(1, int(4e8) // P.shape[0])
    vs, js = [], []
    for i in range(0, U.shape[0], step):
        v, j = torch.topk(U[i:i + step].double() @ P64.T, k, dim=1)
        vs.append(v)
        js.append(j)
    return torch.cat(vs), torch.cat(js)


def _top64(js, m, N):
    sc = torch.bincount(js.reshape(-1), minlength=m)
    key = sc * m + (m - 1 - torch.arange(m, device=sc.device))
    ids = torch.topk(key, N).indices
    return ids.cpu().numpy().astype(np.int32), sc[ids].cpu().numpy().astype(np.int32)


def exact(case, seed):
    n, m, d, k, N = (case[x] for x in ("n", "m", "d", "k", "N"))
    kind = case["kind"]
    if n * m > 3e10:
        return None
    s = _inputs(case, seed)
    U, P = s["U"], s["P"]
    v, j = _lists64(U, P, k)
    if kind == "topn":
        return _top64(j, m, N)
    if kind == "lists":
        return v[:, k - 1], j[:, k - 1].int(), j.int()
    if kind == "index":
        return (v[:, 9], j[:, 9].int()) + _top64(j[:, :10], m, N) + _top64(j, m, 2 * N)
    if kind == "budget":
        return _top64(j[:, :10], m, N)
    Q, tau = s["Q"].double(), v[:, k - 1]
    step = max(1, int(2e8) // Q.shape[0])
    if kind == "scores":
        return sum(((U[i:i + step].double() @ Q.T) > tau[i:i + step, None]).sum(0)
                   for i in range(0, n, step)).int()
    tau, T = tau.float().double(), s["T"]
    T = float(np.float32(T))  # the temperature is an FP32 argument
    S = torch.zeros(Q.shape[0], dtype=torch.float64, device="cuda")
    G = torch.zeros(Q.shape, dtype=torch.float64, device="cuda")
    for i in range(0, n, step):
        u = U[i:i + step].double()
        w = torch.sigmoid((u @ Q.T - tau[i:i + step, None]) / T)
        S += w.sum(0)
        G += (w * (1.0 - w) / T).T.contiguous() @ u
    return S, G * s["dS"].double()[:, None]
