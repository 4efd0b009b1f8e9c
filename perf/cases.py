"""Workloads of the library as its users run them, for timing and for checking.

Every case is a dict of plain values.  ``prepare`` makes what a program holds before the
call (instances drawn from the seed, a handle, a batch plan or a server, starts and
result buffers on the GPU); ``run`` is one pass through the public entry points of
``paper_2307_11248_amd.qap``; ``exact`` is the same answer from plain numpy.

Kinds:
  cost    Eq. (1) of many permutations (``Handle.cost_async``)
  table   the whole exchange neighbourhood of many permutations (``delta_table_async``)
  2opt    best-improvement local search to a local optimum from many starts
  tabu    tabu search from many starts; ``via`` "async" (device tensors), "noalloc" (the
          allocation-free entry point) or "host" (the blocking call on numpy arrays)
  freq    tabu search with the frequency memory, diversification and a tabu attribute
  batch   many instances of uneven n in one planned batch (``Batch.run_async``)
  serve   requests of uneven n and length through the continuous-batching ``Server``

Instances: "dense" (asymmetric, entries uniform in [0, 99], as QAPLIB's tai*a), "euclid"
(symmetric, 70 % zero flows, rounded Euclidean distances, as tai*b), "grid" (asymmetric
sparse flows on a Manhattan grid).
"""
import math

import numpy as np
import torch

from paper_2307_11248_amd import qap
from paper_2307_11248_amd import workloads as W


def listed():
    return [
        # the smallest call: 32 local searches at n = 12, bound by
        # launches and latency
        dict(name="2opt_n12", kind="2opt", n=12, k=32, inst="euclid"),
        # costs of a population of an odd size
        dict(name="cost_n101", kind="cost", n=101, k=1024, inst="dense"),
        # neighbourhoods of the starts of the n = 128 local searches
        dict(name="table_n128", kind="table", n=128, k=1024, inst="euclid"),
        # multistart local search, more starts than compute units
        dict(name="2opt_n128", kind="2opt", n=128, k=1024, inst="euclid"),
        # one tabu search on host arrays: what a caller without device tensors pays
        dict(name="tabu_host_n40", kind="tabu", n=40, k=1, iters=1000, inst="dense", via="host"),
        # the three sizes of the register-tile tabu kernels in use: fewer searches than
        # compute units, and one search a compute unit
        dict(name="tabu_n64", kind="tabu", n=64, k=128, iters=5000, inst="dense", via="async"),
        dict(name="tabu_n128", kind="tabu", n=128, k=256, iters=3000, inst="euclid", via="async"),
        # the sizes whose neighbourhood is large: the serving stream's largest requests, and
        # the largest n of the library
        dict(name="tabu_n256", kind="tabu", n=256, k=256, iters=1000, inst="dense", via="async"),
        dict(name="tabu_n512", kind="tabu", n=512, k=256, iters=400, inst="dense", via="async"),
        # the extensions: frequency memory, diversification, marked units; an odd size
        dict(name="freq_n81", kind="freq", n=81, k=64, iters=2000, inst="grid", div=200, attr=1),
        # the batched delivery: 512 instances of uneven n, 8 starts each (the largest case)
        dict(name="batch_512x8", kind="batch", m=512, k=8, nmin=20, nmax=150, iters=2000),
        # serving: 64 requests of uneven n and length, each with its own matrices
        dict(name="serve_64", kind="serve", count=64, nmin=30, nmax=256, itmin=2000, itmax=6000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["cost", "table", "2opt", "tabu", "tabu", "tabu", "tabu", "freq", "batch", "serve"])
    inst = rng.choice(["dense", "euclid", "grid"])
    if kind == "batch":
        nmin = rng.randint(8, 60)
        return dict(kind=kind, m=_log_int(rng, 4, 128), k=rng.randint(1, 8), nmin=nmin,
                    nmax=rng.randint(nmin, 200), iters=_log_int(rng, 200, 2000))
    if kind == "serve":
        nmin = rng.randint(10, 100)
        return dict(kind=kind, count=_log_int(rng, 4, 64), nmin=nmin, nmax=rng.randint(nmin, 256), itmin=500,
                    itmax=_log_int(rng, 1000, 5000))
    n = _log_int(rng, 8, 512)
    k = _log_int(rng, 1, 1024)
    if kind in ("cost", "table"):
        return dict(kind=kind, n=n, k=max(1, min(k, 2 ** 24 // (n * n))), inst=inst)
    if kind == "2opt":
        return dict(kind=kind, n=n, k=max(1, min(k, 2 ** 24 // (n * n))), inst=inst)
    # searches: at most as many entry-steps as the n = 256 case
    iters = _log_int(rng, 100, 5000)
    if n > 176:
        iters = min(iters, 1000)
    k = max(1, min(k, 2 ** 34 // (n * n * iters)))
    if kind == "freq":
        n = min(n, 256)
        return dict(kind=kind, n=n, k=min(k, 128), iters=min(iters, 1000), inst=inst,
                    div=rng.choice([0, 50, 300]), attr=rng.randint(0, 2))
    via = rng.choice(["async", "async", "noalloc", "host"])
    if via == "noalloc":   # its scratch is a fixed 64 MiB: tables and streamed tile state
        k = max(1, min(k, (48 << 20) // (8 * n * n)))
    return dict(kind=kind, n=n, k=k, iters=iters, inst=inst, via=via)


def _matrices(rng, n, inst):
    if inst == "dense":
        return W.uniform_matrix(rng, n, 0, 99), W.uniform_matrix(rng, n, 0, 99)
    if inst == "euclid":
        return W.symmetrise_upper(W.sparse_matrix(rng, n, 0.7)), W.euclid_points(rng, n)
    return W.sparse_matrix(rng, n, 0.8), W.grid_manhattan(n)


def _starts(rng, n, k):
    return rng.permuted(np.tile(np.arange(n, dtype=np.int32), (k, 1)), axis=1)


def _tenure(case, n):
    # unit marking takes Zhu et al.'s short tenure, every other search the usual range
    return (3, 3 + n // 10) if case["kind"] == "freq" and case["attr"] == 1 else W.tabu_tenure_range(n)


def _inputs(case, seed):
    """Matrices, starts and search seeds: made from the case and the seed alone."""
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    if kind in ("batch", "serve"):
        count = case["m"] if kind == "batch" else case["count"]
        k = case["k"] if kind == "batch" else 1
        sizes = np.random.default_rng([count, case["nmin"], case["nmax"]])   # the case's, for every seed
        out = []
        for i in range(count):
            n = int(sizes.integers(case["nmin"], case["nmax"] + 1))
            it = case["iters"] if kind == "batch" else int(sizes.integers(case["itmin"], case["itmax"] + 1))
            F, D = _matrices(rng, n, "dense" if i % 2 == 0 else "grid")
            out.append((F, D, _starts(rng, n, k), it, int(rng.integers(0, 2 ** 62))))
        return out
    F, D = _matrices(rng, case["n"], case["inst"])
    return F, D, _starts(rng, case["n"], case["k"]), int(rng.integers(0, 2 ** 62))


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "serve":
        s["requests"] = _inputs(case, seed)
        s["server"] = qap.Server(1 << 30, 256)
        return s
    if kind == "batch":
        reqs = _inputs(case, seed)
        ns = [len(r[0]) for r in reqs]
        handles = [qap.Handle(r[0], r[1]) for r in reqs]
        ten = [W.tabu_tenure_range(n) for n in ns]
        s["plan"] = qap.Batch(handles, [case["k"]] * len(ns), case["iters"], [t[0] for t in ten],
                              [t[1] for t in ten], [r[4] for r in reqs])
        s["starts"] = torch.from_numpy(np.concatenate([r[2].reshape(-1) for r in reqs])).cuda()
        k = s["plan"].starts
    else:
        F, D, starts, s["seed"] = _inputs(case, seed)
        k, n = case["k"], case["n"]
        s["handle"] = qap.Handle(F, D)
        if case.get("via") == "host":
            s["starts"] = starts
            return s
        s["starts"] = torch.from_numpy(starts).cuda()
        if kind == "table":
            s["table"] = torch.empty((k, n * (n - 1) // 2), dtype=torch.int32, device="cuda")
            return s
        if kind == "freq":
            s["freq"] = torch.empty((k, n * (n - 1) // 2), dtype=torch.int32, device="cuda")
    s["cost"] = torch.empty(k, dtype=torch.int64, device="cuda")
    s["moves"] = torch.empty(k, dtype=torch.int32, device="cuda")
    s["perms"] = torch.empty_like(s["starts"])
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "serve":
        srv = s["server"]
        tickets = []
        for F, D, start, iters, seed in s["requests"]:
            lo, hi = W.tabu_tenure_range(len(F))
            tickets.append(srv.submit(F, D, start[0], iters, lo, hi, seed))
        while True:
            _, active, pending = srv.step()
            if active == 0 and pending == 0:
                break
        res = [srv.result(t) for t in tickets]
        return (np.concatenate([r[0] for r in res]), np.array([r[1] for r in res]), np.array([r[2] for r in res]))
    if kind == "cost":
        s["handle"].cost_async(s["starts"], s["cost"])
        return s["cost"]
    if kind == "table":
        s["handle"].delta_table_async(s["starts"], s["table"])
        return s["table"]
    if case.get("via") == "host":
        lo, hi = _tenure(case, case["n"])
        return s["handle"].tabu(s["starts"], case["iters"], lo, hi, s["seed"])
    perms, cost, moves = s["perms"], s["cost"], s["moves"]
    perms.copy_(s["starts"])   # the searches work in place
    if kind == "batch":
        s["plan"].run_async(perms, cost, moves)
        return perms, cost, moves
    h = s["handle"]
    if kind == "2opt":
        h.two_opt_async(perms, cost, moves)
        return perms, cost, moves
    lo, hi = _tenure(case, case["n"])
    if kind == "freq":
        h.tabu_freq_async(perms, case["iters"], lo, hi, s["seed"], cost, s["freq"], moves, div=case["div"],
                          attr=case["attr"])
        return perms, cost, moves, s["freq"]
    call = h.tabu_noalloc_async if case["via"] == "noalloc" else h.tabu_async
    call(perms, case["iters"], lo, hi, s["seed"], cost, moves)
    return perms, cost, moves


def work(case):
    """Bytes: matrices (one byte an entry) and starts in, results out, once.  Operations:
    8 for each neighbourhood entry made current and considered in a step (two packed
    subtractions and a two-term product sum, the tabu and aspiration tests, the minimum;
    6 without the tabu list), 2 for each product of a contraction."""
    kind = case["kind"]
    if kind in ("batch", "serve"):
        b = f = 0
        for F, _, starts, it, _ in _inputs(case, 0):
            n, k = len(F), len(starts)
            b += 2 * n * n + k * (8 * n + 12)
            f += k * (4 * n ** 3 + 4 * n * (n - 1) * it)
        return {"bytes": b, "flops": f}
    n, k = case["n"], case["k"]
    m = n * (n - 1) // 2
    if kind == "cost":
        return {"bytes": 2 * n * n + k * (4 * n + 8), "flops": 2 * k * n * n}
    contraction = 2 * n ** 3 if case["inst"] == "euclid" else 4 * n ** 3
    if kind == "table":
        return {"bytes": 2 * n * n + k * (4 * n + 4 * m), "flops": k * contraction}
    b = 2 * n * n + k * (8 * n + 12)
    if kind == "2opt":   # a start at random makes about 1.5 n moves
        return {"bytes": b, "flops": k * (contraction + int(1.5 * n) * 6 * m)}
    return {"bytes": b + (4 * k * m if kind == "freq" else 0), "flops": k * (contraction + case["iters"] * 8 * m)}


# ---- the same answers from plain numpy, in 64 bits

def _cost(F, D, p):
    return int((F[np.ix_(p, p)] * D).sum())


def _deltas(F, D, p):
    """z(p with i, j exchanged) - z(p) for every pair, from Eq. (2) with its diagonal term:
    with G = F[p][p] and T = G D^T + G^T D, T_ij + T_ji - T_ii - T_jj plus the k = i, j
    terms.  The products are below 2^53, so float64 matrix products are exact."""
    G = F[np.ix_(p, p)]
    Gf, Df = G.astype(np.float64), D.astype(np.float64)
    T = (Gf @ Df.T + Gf.T @ Df).astype(np.int64)
    t, g, d = np.diag(T), np.diag(G), np.diag(D)
    gi, gj, di, dj = g[:, None], g[None, :], d[:, None], d[None, :]
    c = (-(D.T - di) * (gi - G.T) - (dj - D) * (G - gj) - (D - di) * (gi - G) - (dj - D.T) * (G.T - gj)
         + (D.T - D) * (G - G.T) + (dj - di) * (gi - gj))
    return T + T.T - t[:, None] - t[None, :] + c


def _tenures(seed, start, iters, lo, hi):
    """Tenure of moves 1 .. iters: the first word of Philox4x64-10 with key (seed, 0) and
    counter (it, start, 0, 0); numpy steps its counter before each block."""
    out = []
    for it in range(1, iters + 1):
        bg = np.random.Philox(key=[seed, 0], counter=[it - 1, start, 0, 0])
        x = int(bg.random_raw())
        out.append(lo + ((x >> 32) * (hi - lo + 1) >> 32))
    return out


def _search(F, D, start, tenures):
    """One search: 2opt when tenures is None, else tabu with these tenures."""
    n = len(F)
    p = start.copy()
    r_, s_ = np.triu_indices(n, 1)
    until = np.zeros(len(r_), dtype=np.int64)
    cur = best = _cost(F, D, p)
    bestp, it = p.copy(), 0
    while tenures is None or it < len(tenures):
        dl = _deltas(F, D, p)[r_, s_]
        it += 1
        if tenures is not None:
            dl = np.where((until <= it) | (cur + dl < best), dl, np.iinfo(np.int64).max)
        i = int(dl.argmin())
        if (dl[i] >= 0) if tenures is None else (dl[i] == np.iinfo(np.int64).max):
            it -= 1
            break
        r, s = r_[i], s_[i]
        p[r], p[s] = p[s], p[r]
        cur += int(dl[i])
        if cur < best:
            best, bestp = cur, p.copy()
        if tenures is not None:
            until[i] = it + tenures[it - 1]
    return (p, cur, it) if tenures is None else (bestp, best, it)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("batch", "serve", "freq"):
        return None   # whole searches of these sizes take numpy minutes
    F, D, starts, key = _inputs(case, seed)
    F, D = F.astype(np.int64), D.astype(np.int64)
    n, k = case["n"], case["k"]
    if kind == "cost":
        return np.array([_cost(F, D, p) for p in starts], dtype=np.int64)
    if kind == "table":
        iu = np.triu_indices(n, 1)
        return np.stack([_deltas(F, D, p)[iu] for p in starts]).astype(np.int32)
    steps = 2 * n if kind == "2opt" else case["iters"]
    if k * steps * (60e-6 + n * n * 120e-9 + n ** 3 * 1e-10) > 15:   # about the seconds it takes
        return None
    lo, hi = _tenure(case, n)
    res = [_search(F, D, starts[j], None if kind == "2opt" else _tenures(key, j, case["iters"], lo, hi))
           for j in range(k)]
    return (np.stack([r[0] for r in res]).astype(np.int32), np.array([r[1] for r in res], dtype=np.int64),
            np.array([r[2] for r in res], dtype=np.int32))
