"""The work that a program has this library do, as timed cases.

Each case is one call, or one short sequence of calls, that the repository's own programs make: the
whole path over one stream (build, count, reduction, estimators: bench.py's step), counts of a built
graph under new parameters (the replicas of an error study), windows of a stream, Algorithm 2's pair
counters, parallel MASCOT, a batch of jobs, a stream appended in chunks, and one served request that
arrives in host memory.  Sizes run from the 2,000-node stream of the smoke test to R-MAT scale 24.

Streams are drawn on the GPU from the seed alone, with the shapes of the repository's generators:
Erdos-Renyi, Chung-Lu power law (exponent 2.1) and R-MAT (0.57, 0.19, 0.19).
"""
from __future__ import annotations

import functools
import math
from fractions import Fraction

import numpy as np
import torch

from paper_1811_09136_amd import rept
from paper_1811_09136_amd.batch import Batch, Job
from paper_1811_09136_amd.serve import DeviceExecutor, Request, run_fifo_plain

DEV = "cuda"


def _case(name, kind, graph, n, edges, m, c, **more):
    return {"name": name, "kind": kind, "graph": graph, "n": n, "edges": edges, "m": m, "c": c, **more}


def listed():
    return [
        # the smallest whole path: the smoke test's stream, where launches and latency are all there is
        _case("step_er_20k", "step", "er", 2000, 20_000, 10, 10),
        # a whole path of an ordinary size (a served request's median), odd, with four hash groups
        _case("step_powerlaw_200k", "step", "powerlaw", 10_001, 200_003, 50, 200),
        # the 1M/20M power-law stream of the benchmark
        _case("step_powerlaw_20m", "step", "powerlaw", 1_000_000, 20_000_000, 10, 40),
        # the largest single-GPU workload of the benchmark
        _case("step_rmat_24", "step", "rmat", 1 << 24, 16 << 24, 100, 100),
        # one more hash seed on a built graph: a replica of an error study (the batched workload's stream)
        _case("count_powerlaw_5m", "count", "powerlaw", 250_000, 5_000_000, 20, 20),
        # the newest tenth of a stream, added to running counters
        _case("window_powerlaw_2m", "window", "powerlaw", 100_000, 2_000_000, 10, 30),
        # Algorithm 2 with its per-node pair counters, c mod m != 0
        _case("eta_powerlaw_2m", "eta", "powerlaw", 100_000, 2_000_000, 10, 35),
        # parallel MASCOT, eight independent samplers
        _case("mascot_powerlaw_2m", "mascot", "powerlaw", 100_000, 2_000_000, 10, 8),
        # many small streams and replicas of one of them in one launch
        _case("batch_32", "batch", "powerlaw", 25_000, 500_000, 20, 20, jobs=32, replicas=8),
        # a stream taken in ten large chunks, counters up to date after each
        _case("append_10_of_200k", "append", "powerlaw", 100_000, 2_000_000, 10, 40, head=0, chunk=200_000),
        # small chunks that arrive behind a long prefix
        _case("append_16_of_1k", "append", "powerlaw", 25_000, 516_000, 10, 10, head=500_000, chunk=1_000),
        # one request whose stream arrives in host memory, served alone
        _case("request_100k", "request", "powerlaw", 5_000, 100_000, 10, 40),
    ]


def draw(rng):
    """One more case: sizes log-uniform over each kind's range, odd ones among them."""
    kind = rng.choice(["step", "step", "step", "count", "count", "window", "eta", "mascot", "batch", "append", "append",
                       "request"])
    lo, hi = {"step": (1e3, 2e7), "count": (2e4, 1e7), "window": (2e4, 5e6), "eta": (1e4, 5e6), "mascot": (1e4, 5e6),
              "batch": (2e4, 1e6), "append": (5e4, 3e6), "request": (1e3, 2e6)}[kind]
    edges = int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    graph = rng.choice(["powerlaw", "powerlaw", "rmat", "er"])
    if graph == "rmat":
        n = 1 << max(6, round(math.log2(edges / 16)))
        edges = 16 * n  # draws; the repeated pairs fall out
    else:
        n = max(64, edges // rng.choice([10, 20, 20, 40]) + rng.randrange(7))
    m = rng.choice([7, 10, 20, 50, 100])
    c = {"eta": m + 1 + rng.randrange(2 * m), "mascot": rng.choice([3, 8])}.get(kind, rng.choice([m, m, 2 * m, 4 * m]))
    if kind == "eta" and c % m == 0:
        c += 1
    more = {}
    if kind == "count":
        more["per_proc"] = edges < 1_000_000 and rng.random() < 0.25
        if rng.random() < 0.25:
            c = max(1, m // 2)
    elif kind == "batch":
        more = {"jobs": rng.choice([5, 16, 31]), "replicas": rng.choice([0, 2, 5])}
    elif kind == "append":
        chunks = rng.choice([5, 9, 16])
        more["head"] = rng.choice([0, edges // 2, 9 * edges // 10])
        more["chunk"] = max(1, (edges - more["head"]) // chunks)
    return {"kind": kind, "graph": graph, "n": n, "edges": edges, "m": m, "c": c, **more}


# ------------------------------------------------------------------------------ streams

@functools.lru_cache(maxsize=16)
def _powerlaw_cum(n, edges):
    """Cumulative node weights (i + i0) ** (-1 / 1.1), the largest expected degree min(5e4, n / 2)."""
    idx = np.arange(n, dtype=np.float64)
    target = min(5.0e4, n / 2) / (2.0 * edges)
    lo, hi = 1e-9, float(n)
    for _ in range(40):
        mid = math.sqrt(lo * hi)
        w = (idx + mid) ** (-1 / 1.1)
        lo, hi = (mid, hi) if w[0] > target * w.sum() else (lo, mid)
    return np.cumsum((idx + hi) ** (-1 / 1.1))


def _pairs(graph, n, edges, count, gen):
    """`count` draws of an endpoint pair."""
    def uniform(k):
        return torch.rand(k, generator=gen, device=DEV, dtype=torch.float64)

    if graph == "er":
        return (torch.randint(n, (count,), generator=gen, device=DEV),
                torch.randint(n, (count,), generator=gen, device=DEV))
    if graph == "powerlaw":
        cum = torch.from_numpy(_powerlaw_cum(n, edges)).to(DEV)
        return tuple(torch.searchsorted(cum, uniform(count) * cum[-1], right=True).clamp_(max=n - 1) for _ in range(2))
    u = torch.zeros(count, dtype=torch.int64, device=DEV)
    v = torch.zeros(count, dtype=torch.int64, device=DEV)
    for _ in range(n.bit_length() - 1):
        r = torch.rand(count, generator=gen, device=DEV)
        u = 2 * u + (r >= 0.76)
        v = 2 * v + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    return u, v


def _stream(graph, n, edges, seed):
    """A simple stream as device int32[E, 2].  R-MAT: `edges` draws, the first of each pair kept, in
    the order of the draws; otherwise exactly `edges` pairs in a random order."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    if graph == "rmat":
        u, v = _pairs(graph, n, edges, edges, gen)
        key, at = torch.sort((torch.minimum(u, v) << 32) | torch.maximum(u, v), stable=True)
        first = torch.ones_like(key, dtype=torch.bool)
        first[1:] = key[1:] != key[:-1]
        at = torch.sort(at[first])[0]
        at = at[u[at] != v[at]]
        return torch.stack([u[at], v[at]], 1).to(torch.int32)
    edges = min(edges, n * (n - 1) // 4)
    keys = torch.empty(0, dtype=torch.int64, device=DEV)
    while keys.numel() < edges:
        u, v = _pairs(graph, n, edges, edges + edges // 4 + 64, gen)
        key = ((torch.minimum(u, v) << 32) | torch.maximum(u, v))[u != v]
        keys = torch.unique(torch.cat([keys, key]))
    keys = keys[torch.randperm(keys.numel(), generator=gen, device=DEV)[:edges]]
    a, b = keys >> 32, keys & 0xffffffff
    flip = torch.rand(edges, generator=gen, device=DEV) < 0.5
    return torch.stack([torch.where(flip, b, a), torch.where(flip, a, b)], 1).to(torch.int32)


# ------------------------------------------------------------------------------ cases

def _params(case, seed):
    return rept.Params(case["m"], case["c"], seed, per_proc=case.get("per_proc", False),
                       mascot=case["kind"] == "mascot")


def _hash_seed(seed):
    return (seed * 0x9E3779B97F4A7C15 + 20181122) % 2 ** 64


def prepare(case, seed):
    kind, n = case["kind"], case["n"]
    p = _params(case, _hash_seed(seed))
    if kind == "batch":
        # the jobs' sizes belong to the case, their streams to the seed
        sizes = np.random.default_rng(case["jobs"]).uniform(math.log(max(1e3, case["edges"] / 50)), math.log(case["edges"]),
                                                            case["jobs"] - case["replicas"])
        graphs = []
        for k, e in enumerate(np.exp(sizes).astype(int).tolist()):
            ns = 1 << max(6, round(math.log2(e / 16))) if case["graph"] == "rmat" else max(64, e // 20)
            graphs.append(rept.Graph(_stream(case["graph"], ns, e, 1000 * seed + k), ns))
        if case["replicas"]:
            graphs.append(rept.Graph(_stream(case["graph"], n, case["edges"], 1000 * seed + 999), n))
            graphs += [graphs[-1]] * (case["replicas"] - 1)
        jobs = [Job(g, rept.Params(p.m, p.c, _hash_seed(1000 * seed + k))) for k, g in enumerate(graphs)]
        return {"kind": kind, "jobs": jobs, "batch": Batch(jobs)}
    edges = _stream(case["graph"], n, case["edges"], seed)
    E = edges.shape[0]
    st = {"kind": kind, "n": n, "E": E, "params": p, "edges": edges}
    if kind == "step":
        pb, sb = rept.rept_query_sizes(n, E)
        st["persistent"] = torch.empty(pb, dtype=torch.uint8, device=DEV)
        st["scratch"] = torch.empty(sb, dtype=torch.uint8, device=DEV)
        st["glob"] = torch.empty(p.c, dtype=torch.int64, device=DEV)
        st["loc"] = torch.empty((p.rows, n), dtype=torch.int64, device=DEV)
        st["sums"] = torch.empty(n, dtype=torch.int64, device=DEV)
        st["h_glob"] = torch.empty(p.c, dtype=torch.int64, pin_memory=True)
        st["h_sums"] = torch.empty(n, dtype=torch.int64, pin_memory=True)
        st["tau_v"] = np.empty(n)
        # 16 bits per edge and group, the groups padded to 1, 2, 4 or 8
        st["ws"] = torch.empty(max(256, 2 * E * (1 << (p.groups - 1).bit_length()) + 256), dtype=torch.uint8, device=DEV)
    elif kind in ("count", "mascot", "window", "eta"):
        st["g"] = rept.Graph(edges, n)
        st["out"] = st["g"].outputs(p)
    elif kind == "append":
        # an R-MAT stream is shorter than its draws: the same shares of it
        st["head"] = case["head"] * E // case["edges"]
        st["chunk"] = max(1, case["chunk"] * E // case["edges"])
    elif kind == "request":
        st["executor"] = DeviceExecutor(DEV, arena_bytes=64 << 20 if E < 100_000 else 640 * E + 400 * n + (64 << 20))
        st["request"] = Request(0, 0.0, edges.cpu().numpy().view(np.uint32), n, p.m, p.c, p.seed)
    return st


def run(st):
    kind = st["kind"]
    if kind == "step":
        sp = torch.cuda.current_stream().cuda_stream
        n, p, loc = st["n"], st["params"], st["loc"]
        h = rept.rept_build(n, st["edges"].data_ptr(), st["E"], st["persistent"].data_ptr(), st["persistent"].numel(),
                            st["scratch"].data_ptr(), st["scratch"].numel(), sp)
        rept.rept_count(h, p, st["glob"].data_ptr(), loc.data_ptr(), st["ws"].data_ptr(), st["ws"].numel(), sp)
        rept.rept_reduce_local(loc.data_ptr(), p.rows, n, st["sums"].data_ptr(), sp)
        st["h_glob"].copy_(st["glob"], non_blocking=True)
        st["h_sums"].copy_(st["sums"], non_blocking=True)
        torch.cuda.current_stream().synchronize()
        tau_hat, tau_v = rept.rept_estimate_sums(n, p, st["h_glob"].numpy(), st["h_sums"].numpy(), st["tau_v"])
        rept.rept_destroy(h)
        return {"global": st["glob"], "local": loc, "tau_hat": tau_hat, "tau_v": tau_v}
    if kind in ("count", "mascot"):
        g, loc = st["g"].count(st["params"], out=st["out"])
        return {"global": g, "local": loc}
    if kind == "window":
        g, loc = st["out"]
        g.zero_()
        loc.zero_()
        st["g"].count_range(st["params"], st["E"] - st["E"] // 10, st["E"], (g, loc))
        return {"global": g, "local": loc}
    if kind == "eta":
        g, loc, eta, eta_v = st["g"].count_eta(st["params"])
        return {"global": g, "local": loc, "eta": eta, "eta_v": eta_v}
    if kind == "batch":
        st["batch"].launch()
        return [j.out for j in st["jobs"]]
    if kind == "append":
        E, head, chunk = st["E"], st["head"], st["chunk"]
        s = rept.IncrementalStream(st["n"], E, max(head, chunk), st["params"], DEV)
        if head:
            s.append(st["edges"][:head])
        for a in range(head, E, chunk):
            s.append(st["edges"][a:a + chunk])
        return {"global": s.counts[0], "local": s.counts[1]}
    res = run_fifo_plain(st["executor"], [st["request"]])[0]
    if res.status != "ok":
        raise RuntimeError(res.status)
    return {"global": res.glob, "local": res.loc, "tau_hat": res.tau_hat}


def work(case):
    """Each stream edge read once and each counter written once.  The operations are not counted:
    the path has no contraction, and how many probes it makes is the algorithm's choice."""
    p = _params(case, 0)
    n, E, jobs = case["n"], case["edges"], case.get("jobs", 1)
    if case["kind"] == "batch":  # sizes are log-uniform over [edges / 50, edges]
        own = case["jobs"] - case["replicas"]
        mean = E * (1 - 1 / 50) / math.log(50)
        return {"bytes": 8.0 * (own * mean * (1 + 1 / 20) + (E + n) * case["replicas"] + jobs * p.c), "flops": 0.0}
    out = 8.0 * (p.c + p.rows * n)
    if case["kind"] == "step":
        out += 8.0 * n
    elif case["kind"] == "eta":
        out += 16.0 * (p.c + n)
    return {"bytes": 8.0 * E + out, "flops": 0.0}


# ------------------------------------------------------------------------------ exact values

def _slots(edges, m, group, seed):
    """h_k of every edge: a cubic over GF(2^61 - 1) with SplitMix64 coefficients, scaled to [0, m)."""
    prime, mask = (1 << 61) - 1, (1 << 64) - 1
    coef = []
    for q in range(4 * group, 4 * group + 4):
        z = (seed + (q + 1) * 0x9E3779B97F4A7C15) & mask
        z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & mask
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & mask
        coef.append(((z ^ (z >> 31)) >> 3) % prime)
    out = []
    for u, v in edges:
        x = (min(u, v) << 32) | max(u, v)
        out.append(((((coef[3] * x + coef[2]) * x + coef[1]) * x + coef[0]) % prime * m) >> 61)
    return out


def exact(case, seed):
    """Algorithm 1's counters from a list of all triangles (each belongs to its last edge, and to the
    processor of each group that holds both earlier edges), and the estimators in exact arithmetic;
    streams of up to 30,000 edges."""
    if case["kind"] not in ("step", "count", "request") or case["edges"] > 30_000 or case.get("per_proc"):
        return None
    n, m, c = case["n"], case["m"], case["c"]
    p = _params(case, _hash_seed(seed))
    edges = _stream(case["graph"], n, case["edges"], seed).cpu().tolist()
    when = {}
    later = [[] for _ in range(n)]
    for t, (u, v) in enumerate(edges):
        when[(min(u, v), max(u, v))] = t
        later[min(u, v)].append(max(u, v))
    slots = [_slots(edges, m, k, p.seed) for k in range(p.groups)]
    glob, loc = np.zeros(c, np.int64), np.zeros((p.groups, n), np.int64)
    for x in range(n):
        after = sorted(later[x])
        for i, y in enumerate(after):
            for z in after[i + 1:]:
                t = when.get((y, z))
                if t is None:
                    continue
                e, f, _ = sorted((t, when[(x, y)], when[(x, z)]))
                for k in range(p.groups):
                    if slots[k][e] == slots[k][f] and k * m + slots[k][e] < c:
                        glob[k * m + slots[k][e]] += 1
                        for node in (x, y, z):
                            loc[k, node] += 1
    tau_hat = float(Fraction(int(glob.sum()) * m * m, c))
    if case["kind"] == "count":
        return {"global": glob, "local": loc}
    if case["kind"] == "request":
        return {"global": glob, "local": loc, "tau_hat": tau_hat}
    tau_v = np.array([float(Fraction(int(s) * m * m, c)) for s in loc.sum(0)])
    return {"global": glob, "local": loc, "tau_hat": tau_hat, "tau_v": tau_v}
