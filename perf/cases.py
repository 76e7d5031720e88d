"""The measured cases: what users of the library run, from the smallest request to the
largest graph, through the package's public entry points.

A case is a dict of plain values: `call` (lpa, louvain, leiden, batched, serve, sweep,
refine, modularity), a graph family with its sizes, and the parameters of the call.
Graphs are drawn on the GPU from the seed alone:

  rmat     2**scale vertices, ef * 2**scale edge samples, weights in [1, 8] (skewed: web
           and social graphs, and the requests a server gets);
  chunglu  n vertices, mean degree `deg`, power-law expected degrees (exponent 2.1, as
           the large web crawls), weights in [1, 4];
  planted  n vertices in communities of log-uniform sizes, 12 intra and 4 inter edges
           per vertex, unit weights (clear communities: the batched workload);
  chains   n vertices in chains of mean length 16 joined at their ends, unit weights
           (about two entries per vertex: k-mer graphs with random ids, road networks
           with ids that keep locality).
"""
import math

import numpy as np
import torch

import paper_2411_02268_amd as mg
from paper_2411_02268_amd import synth

ALGOS = {"lpa": mg.ALGO_LPA, "louvain": mg.ALGO_LOUVAIN, "leiden": mg.ALGO_LEIDEN}


def listed():
    return [
        # a small community query: launches and host round trips are all of it
        {"name": "lpa-planted-10k", "call": "lpa", "graph": "planted", "n": 10000, "cmin": 500, "cmax": 500,
         "mode": 1, "k": 8},
        # the smallest request of the serving stream, called on its own
        {"name": "louvain-rmat14", "call": "louvain", "graph": "rmat", "scale": 14, "ef": 8, "mode": 1, "k": 8},
        # the benchmark's graph and parameters
        {"name": "louvain-rmat20", "call": "louvain", "graph": "rmat", "scale": 20, "ef": 16, "mode": 1, "k": 8},
        # label propagation on the same kind of graph (ends in one giant label)
        {"name": "lpa-rmat20", "call": "lpa", "graph": "rmat", "scale": 20, "ef": 16, "mode": 1, "k": 8},
        # the exact table, the baseline that users check the sketch against
        {"name": "louvain-rmat19-exact", "call": "louvain", "graph": "rmat", "scale": 19, "ef": 16, "mode": 0, "k": 8},
        # the large graph: Leiden with its default sketch, storage copy by default
        {"name": "leiden-chunglu22", "call": "leiden", "graph": "chunglu", "n": 1 << 22, "deg": 32, "mode": 1, "k": 16},
        # the paper's slot count for Leiden
        {"name": "leiden-rmat18-k64", "call": "leiden", "graph": "rmat", "scale": 18, "ef": 16, "mode": 1, "k": 64},
        # the low-degree class (k-mer graphs): rows shorter than the sketch
        {"name": "louvain-chains", "call": "louvain", "graph": "chains", "n": 5000011, "local": False, "mode": 1, "k": 8},
        # many small graphs in one call
        {"name": "batched-louvain", "call": "batched", "algo": "louvain", "graph": "planted", "count": 192,
         "nmin": 1000, "nmax": 50000, "cmin": 20, "cmax": 2000, "mode": 1, "k": 8},
        # a server with a burst of requests queued
        {"name": "serve-louvain", "call": "serve", "algo": "louvain", "graph": "rmat", "count": 24, "smin": 14,
         "smax": 18, "ef": 8, "mode": 1, "k": 8},
        # one sweep from a given membership (callers with drivers of their own)
        {"name": "sweep-louvain-k16", "call": "sweep", "algo": "louvain", "graph": "chunglu", "n": 1200007, "deg": 24,
         "mode": 1, "k": 16, "groups": 60000, "direction": 1},
        # scoring a membership
        {"name": "modularity-rmat20", "call": "modularity", "graph": "rmat", "scale": 20, "ef": 16, "groups": 100000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, family, most):
    """Sizes of one graph of `family` with at most about `most` entries."""
    if family == "rmat":
        ef = rng.choice([5, 8, 11, 16])
        top = min(20, int(math.log2(most / (2 * ef))))
        return {"graph": "rmat", "scale": rng.randint(14, top), "ef": ef}
    if family == "chunglu":
        deg = rng.randint(6, 40)
        return {"graph": "chunglu", "n": _log_int(rng, 10000, most / deg), "deg": deg}
    if family == "planted":
        return {"graph": "planted", "n": _log_int(rng, 1000, most / 16), "cmin": 20, "cmax": rng.choice([200, 2000])}
    return {"graph": "chains", "n": _log_int(rng, 10000, min(most / 2, 6e6)), "local": rng.random() < 0.5}


def draw(rng):
    call = rng.choice(["lpa", "louvain", "louvain", "leiden", "leiden", "batched", "serve", "sweep", "refine",
                       "modularity"])
    if call in ("lpa", "louvain", "leiden"):
        mode, k = rng.choice([(1, 8), (1, 8), (1, 16), (1, 16), (1, 32), (1, 64), (0, 8), (2, 8), (3, 16)])
        most = 2e7 if mode == 0 or k > 16 else 1e8  # the exact table and the wide sketches cost more per entry
        family = rng.choice(["rmat", "chunglu", "chunglu", "planted", "chains"])
        return {"call": call, **_draw_graph(rng, family, most), "mode": mode, "k": k}
    if call == "batched":
        return {"call": "batched", "algo": rng.choice(["lpa", "louvain"]), "graph": "planted",
                "count": rng.randint(3, 192), "nmin": 1000, "nmax": rng.choice([5000, 20000, 50000]), "cmin": 20,
                "cmax": rng.choice([200, 2000]), "mode": 1, "k": rng.choice([8, 16, 32])}
    if call == "serve":
        return {"call": "serve", "algo": rng.choice(["lpa", "louvain", "leiden"]), "graph": "rmat",
                "count": rng.randint(5, 24), "smin": 14, "smax": rng.randint(15, 18), "ef": rng.choice([5, 8]),
                "mode": 1, "k": 8}
    g = _draw_graph(rng, rng.choice(["rmat", "chunglu", "planted", "chains"]), 6e7)
    n = g["n"] if "n" in g else 1 << g["scale"]
    g["groups"] = _log_int(rng, 20, n / 4)
    if call == "modularity":
        return {"call": call, **g}
    mode, k = rng.choice([(1, 4), (1, 8), (1, 16), (1, 32), (1, 64), (0, 8)])
    if call == "sweep":
        return {"call": call, "algo": rng.choice(["lpa", "louvain"]), **g, "mode": mode, "k": k,
                "direction": rng.choice([-1, 0, 1])}
    return {"call": call, **g, "mode": mode, "k": k}


# ---- graphs ------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed & 0x7FFFFFFF)
    return g


def _csr(n, u, v, wmax, seed):
    """Symmetric CSR of an undirected edge sample: self-loops dropped, duplicates
    collapsed, columns ascending, weights a hash of the pair in [1, wmax]."""
    keep = u != v
    lo, hi = torch.minimum(u, v)[keep], torch.maximum(u, v)[keep]
    pair = torch.unique(lo * n + hi)
    lo, hi = pair // n, pair % n
    mix = (pair + 0x632BE59BD9B4E019 + (seed << 20)) * 0x2545F4914F6CDD1D  # wraps in 64 bits
    w = ((mix >> 33) & 0x3FFFFFFF) % wmax + 1
    key, order = torch.sort(torch.cat([lo * n + hi, hi * n + lo]))
    rows = key // n
    off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    off[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return mg.DeviceGraph(off, (key % n).to(torch.int32), torch.cat([w, w])[order].to(torch.int32))


def _chunglu(n, deg, seed):
    g, a = _gen(seed), 1.0 / 1.1
    mean = lambda i0: math.sqrt(n * deg) * i0 ** a * ((n + i0) ** (1 - a) - i0 ** (1 - a)) / ((1 - a) * n)
    lo, hi = 1e-3, float(n)
    for _ in range(100):  # i0: the largest expected degree is sqrt(n deg), the mean deg
        mid = math.sqrt(lo * hi)
        lo, hi = (mid, hi) if mean(mid) < deg else (lo, mid)
    x0, x1 = lo ** (1 - a), (n + lo) ** (1 - a)
    perm = torch.randperm(n, generator=g, device="cuda")
    ends = []
    for _ in range(2):
        r = torch.rand(n * deg // 2, generator=g, device="cuda", dtype=torch.float64)
        ends.append(perm[((r * (x1 - x0) + x0) ** (1 / (1 - a)) - lo).long().clamp_(0, n - 1)])
    return _csr(n, ends[0], ends[1], 4, seed)


def _planted(n, cmin, cmax, seed):
    rng = np.random.default_rng(seed)
    sizes = np.exp(rng.uniform(math.log(cmin), math.log(cmax + 1), size=n // cmin + 2)).astype(np.int64)
    ends = np.minimum(np.cumsum(sizes), n)
    ends = ends[:int(np.searchsorted(ends, n)) + 1]
    ends[-1] = n
    g = _gen(seed)
    end = torch.from_numpy(ends).to("cuda")
    start = torch.cat([end.new_zeros(1), end[:-1]])
    i = torch.arange(n, device="cuda")
    c = torch.searchsorted(end, i, right=True)
    size, pos = (end - start)[c], i - start[c]
    u, v = [], []
    for _ in range(6):  # a random circulant inside each community
        hop = (torch.rand(len(ends), generator=g, device="cuda") * ((end - start) // 2)).long() + 1
        u.append(i)
        v.append(start[c] + (pos + hop[c]) % size)
    stubs = torch.randperm(4 * n, generator=g, device="cuda") // 4
    u.append(stubs[:2 * n])
    v.append(stubs[2 * n:])
    perm = torch.randperm(n, generator=g, device="cuda")
    return _csr(n, perm[torch.cat(u)], perm[torch.cat(v)], 1, seed)


def _chains(n, local, seed):
    g = _gen(seed)
    i = torch.arange(n, device="cuda")
    linked = torch.rand(n - 1, generator=g, device="cuda") >= 1 / 16
    ends = i[:-1][~linked]
    ends = torch.cat([ends, ends + 1])
    ends = ends[torch.rand(ends.shape[0], generator=g, device="cuda") < 0.9]
    if local:  # branches lead nearby, as streets do
        far = (ends + torch.randint(-2000, 2001, ends.shape, generator=g, device="cuda")).clamp_(0, n - 1)
    else:
        far = torch.randint(0, n, ends.shape, generator=g, device="cuda")
    u, v = torch.cat([i[:-1][linked], ends]), torch.cat([i[:-1][linked] + 1, far])
    if not local:
        perm = torch.randperm(n, generator=g, device="cuda")
        u, v = perm[u], perm[v]
    return _csr(n, u, v, 1, seed)


def _graph(case, seed):
    if case["graph"] == "rmat":
        return mg.DeviceGraph(*synth.rmat_torch(case["scale"], case["ef"], seed=seed & 0x7FFFFFFF))
    if case["graph"] == "chunglu":
        return _chunglu(case["n"], case["deg"], seed)
    if case["graph"] == "planted":
        return _planted(case["n"], case["cmin"], case["cmax"], seed)
    return _chains(case["n"], case["local"], seed)


def _membership(n, groups, seed):
    """Communities of skewed sizes; every id is one of its members' (as labels are)."""
    g = _gen(seed + 1)
    r = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    heads = torch.randperm(n, generator=g, device="cuda")[:groups]
    return heads[(r * r * groups).long().clamp_(0, groups - 1)].to(torch.int32)


def _counts(case):
    """Vertex counts (batched) or scales (serve) of a case's graphs, by the case alone."""
    rng = np.random.default_rng(case["count"])
    if case["call"] == "serve":
        return rng.integers(case["smin"], case["smax"] + 1, size=case["count"]).tolist()
    return np.exp(rng.uniform(math.log(case["nmin"]), math.log(case["nmax"]), size=case["count"])).astype(int).tolist()


# ---- one pass ----------------------------------------------------------------------

class _Serving:
    """A server as a program keeps it, closed with its owner."""

    def __init__(self, case):
        self.server = mg.Server(ALGOS[case["algo"]], 6 << 30, slots=32, stepped=True, mode=case["mode"], k=case["k"])

    def __del__(self):
        self.server.close()


def prepare(case, seed):
    call = case["call"]
    if call == "batched":
        graphs = [_planted(n, case["cmin"], case["cmax"], seed * 1000 + i) for i, n in enumerate(_counts(case))]
        need = mg.batched_workspace_bytes(ALGOS[case["algo"]], graphs, mode=case["mode"], k=case["k"])
        return {"case": case, "graphs": graphs, "workspace": torch.empty(need, dtype=torch.uint8, device="cuda")}
    if call == "serve":
        graphs = [mg.DeviceGraph(*synth.rmat_torch(s, case["ef"], seed=(seed * 1000 + i) & 0x7FFFFFFF))
                  for i, s in enumerate(_counts(case))]
        return {"case": case, "graphs": graphs, "serving": _Serving(case)}
    g = _graph(case, seed)
    state = {"case": case, "graph": g}
    if "groups" in case:
        state["labels"] = _membership(g.n, case["groups"], seed)
    return state


FIELDS = ("iterations", "passes", "communities", "edges_scanned", "moved_last")


def _result(labels, stats):
    return {"labels": labels, **{f: stats[f] for f in FIELDS}}


def _results(pairs):
    """The labels of many graphs, one after another, and a row of counts for each."""
    return {"labels": torch.cat([l for l, _ in pairs]), "counts": np.array([[s[f] for f in FIELDS] for _, s in pairs])}


def run(state):
    case = state["case"]
    call = case["call"]
    if call == "modularity":
        return mg.modularity(state["graph"], state["labels"])
    kw = {"mode": case["mode"], "k": case["k"]}
    if call in ("lpa", "louvain", "leiden"):
        return _result(*getattr(mg, call)(state["graph"], **kw))
    if call == "batched":
        labels, per_graph, _ = mg.run_batched(ALGOS[case["algo"]], state["graphs"], workspace=state["workspace"], **kw)
        return _results(list(zip(labels, per_graph)))
    if call == "serve":
        server = state["serving"].server
        tickets = [server.submit(g) for g in state["graphs"]]
        return _results([server.wait(t)[:2] for t in tickets])
    if call == "sweep":
        labels, gain, counters = mg.move_sweep(state["graph"], ALGOS[case["algo"]], state["labels"],
                                               direction=case["direction"], **kw)
        return {"labels": labels, "gain": gain, "counters": counters}
    return mg.refine(state["graph"], state["labels"], **kw)


def work(case):
    """Every entry (index and weight) and offset read once, every label written once (a
    given membership read once); one addition and one comparison per entry."""
    if case["call"] == "batched":
        n = sum(_counts(case))
        nnz = 16 * n
    elif case["call"] == "serve":
        n = sum(1 << s for s in _counts(case))
        nnz = 2 * case["ef"] * n
    elif case["graph"] == "rmat":
        n = 1 << case["scale"]
        nnz = 2 * case["ef"] * n
    else:
        n = case["n"]
        nnz = {"chunglu": case.get("deg", 0), "planted": 16, "chains": 2}[case["graph"]] * n
    out = {"modularity": 0, "sweep": 12}.get(case["call"], 4)
    return {"bytes": 8 * nnz + 8 * n + (4 * n if "groups" in case else 0) + out * n, "flops": 2 * nnz}


def exact(case, seed):
    """Only modularity computes a number that is not whole."""
    if case["call"] != "modularity":
        return None
    state = prepare(case, seed)
    g, c = state["graph"], state["labels"].long()
    w = g.weights.long()
    rows = torch.repeat_interleave(torch.arange(g.n, device="cuda"), g.offsets[1:] - g.offsets[:-1])
    total = int(w.sum())
    intra = int(w[c[rows] == c[g.indices.long()]].sum())
    sums = torch.zeros(g.n, dtype=torch.int64, device="cuda").index_add_(0, c[rows], w)
    sums = sums.cpu().numpy().astype(object)
    squares = int((sums * sums).sum())
    return float(np.float64(intra) / total - np.float64(squares) / (np.float64(total) * total))
