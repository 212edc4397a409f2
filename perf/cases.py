"""Timed workloads of the library: single queries, core numbers, batches,
on-the-fly updates, serving, community search and the build, through the
package's entry points.

A case names its work (``kind``), its graph and its thresholds.  Graphs are
drawn on the GPU: ``records`` endpoint pairs, each endpoint chosen with a
probability proportional to its power-law expected degree (exponent ``gamma``
of the degree distribution, degrees capped at 50,000; 0 = uniform), with ids
shuffled.  Repeated pairs stay in, as in an edge log; the build removes them
(about a tenth of 24 million records, so that graph keeps about 20 million
edges).
"""
import math

import torch

import paper_2606_07148_amd as ab

CAP = 50_000
CHUNK = 1 << 26

# index-free queries run on the CSR alone, as Algorithm 1 does
INDEX_FREE = 2


def listed():
    big = {"n_upper": 1_000_000, "n_lower": 500_000, "records": 24_000_000, "gamma": 2.1}
    wide = {"n_upper": 10_000_000, "n_lower": 5_000_000, "records": 220_000_000, "gamma": 2.1}
    return [
        # the smallest call: one query on a graph of a few thousand vertices,
        # where launches and the host path count
        {"name": "gcc_small", "kind": "gcc", "n_upper": 2_000, "n_lower": 1_500,
         "records": 20_000, "gamma": 0.0, "alpha": 3, "beta": 2, "index_free": False},
        # the ordinary query without preprocessing (bench.py's headline shape)
        {"name": "gcc_20m", "kind": "gcc", **big, "alpha": 10, "beta": 10, "index_free": True},
        # the same graph as a handle is used by default, unequal thresholds
        {"name": "gcc_default_20m", "kind": "gcc", **big, "alpha": 5, "beta": 20,
         "index_free": False},
        # a query too large for the caches; sizes that divide by nothing
        {"name": "gcc_450m", "kind": "gcc", "n_upper": 20_000_003, "n_lower": 9_999_991,
         "records": 450_000_000, "gamma": 2.15, "alpha": 16, "beta": 16, "index_free": True},
        # GCC+ between unequal thresholds, core numbers at hand
        {"name": "plus_20m", "kind": "plus", **big, "alpha": 40, "beta": 8},
        # core numbers (GCC+'s preprocessing, and a result of its own)
        {"name": "cores_20m", "kind": "cores", **big},
        {"name": "cores_200m", "kind": "cores", **wide},
        # many queries of one graph at once
        {"name": "batch_200m", "kind": "batch", **wide, "queries": 256, "top": 256},
        # on-the-fly queries one at a time: insertions and deletions
        {"name": "gfq_20m", "kind": "gfq", **big, "requests": 16, "top": 64},
        # the same through the serving engine, all requests admitted at once
        {"name": "serve_20m", "kind": "serve", **big, "requests": 48, "top": 64},
        # the connected part of a core around a vertex
        {"name": "community_20m", "kind": "community", **big, "alpha": 8, "beta": 8},
        # an edge list to a handle, and its sorted, deduplicated CSR back
        {"name": "build_20m", "kind": "build", **big},
    ]


def draw(rng):
    kind = rng.choice(["gcc", "gcc", "gcc", "plus", "cores", "batch", "gfq", "serve",
                       "community", "build"])
    most = {"gcc": 3e8, "plus": 1e8, "cores": 2e8, "batch": 5e7, "gfq": 5e7, "serve": 5e7,
            "community": 1e8, "build": 1e8}[kind]

    def log_uniform(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    records = int(log_uniform(2e4, most)) | 1
    n_upper = max(500, int(records / log_uniform(8, 40)))
    n_lower = max(400, int(n_upper * rng.uniform(0.3, 1.5)))
    gamma = rng.choice([0.0, round(rng.uniform(2.05, 2.6), 3), round(rng.uniform(2.05, 2.3), 3)])
    case = {"kind": kind, "n_upper": n_upper, "n_lower": n_lower, "records": records,
            "gamma": gamma}
    if kind in ("gcc", "plus", "community"):
        # thresholds that leave a part of the graph: near the mean degree of
        # a uniform graph, from 2 to past it on a skewed one
        for name, n in (("alpha", n_upper), ("beta", n_lower)):
            mean = records / n
            if gamma == 0.0:
                case[name] = max(2, int(mean * rng.uniform(0.55, 0.75)))
            else:
                case[name] = int(log_uniform(2.0, max(3.5, mean * (1.5 if gamma < 2.3 else 0.7))))
    if kind == "gcc":
        case["index_free"] = rng.random() < 0.5
    if kind == "batch":
        case["queries"] = rng.randint(3, 64)
        case["top"] = 64
    if kind in ("gfq", "serve"):
        case["requests"] = 2 * rng.randint(4, 12)
        case["top"] = max(4, min(64, int(records / max(n_upper, n_lower))))
    return case


# ------------------------------------------------------------------ inputs --

class _Layer:
    """Endpoints of one layer: rank r (from 0) has the expected degree
    min(cap, s * (r + 1)^-a), a = 1 / (gamma - 1), in its continuous form;
    ``ids`` maps a rank to its vertex."""

    def __init__(self, n, records, gamma, gen):
        self.n = n
        self.ids = torch.randperm(n, device="cuda", generator=gen).to(torch.int32)
        self.uniform = gamma == 0.0
        if self.uniform:
            return
        self.a = a = 1.0 / (gamma - 1.0)
        self.total = float(records)
        cap = max(float(min(CAP, records)), 2.0 * records / n)

        def h(x):  # integral of t^-a from 1 to x
            return (x ** (1.0 - a) - 1.0) / (1.0 - a)

        def weight(k):  # all weights when the first k ranks are capped
            return cap * (k + (k + 1.0) ** a * (h(n + 1.0) - h(k + 1.0)))

        lo, hi = 0.0, float(n)
        if weight(0.0) >= self.total:
            hi = 0.0
        for _ in range(80):
            mid = (lo + hi) / 2
            lo, hi = (mid, hi) if weight(mid) < self.total else (lo, mid)
        self.k, self.cap = hi, cap
        self.hk = h(hi + 1.0)
        self.scale = (self.total - hi * cap) / (h(n + 1.0) - self.hk)

    def sample(self, count, gen):
        u = torch.rand(count, dtype=torch.float64, device="cuda", generator=gen)
        if self.uniform:
            r = (u * self.n).to(torch.int64)
        else:
            u *= self.total
            flat = u / self.cap
            t = (self.hk + (u - self.k * self.cap).clamp_(min=0.0) / self.scale) * (1.0 - self.a)
            t = (t + 1.0).pow_(1.0 / (1.0 - self.a)) - 1.0
            r = torch.where(flat < self.k, flat, t).to(torch.int64)
        return self.ids[r.clamp_(0, self.n - 1)]


def _edges(case, gen):
    upper = _Layer(case["n_upper"], case["records"], case["gamma"], gen)
    lower = _Layer(case["n_lower"], case["records"], case["gamma"], gen)
    eu = torch.empty(case["records"], dtype=torch.int32, device="cuda")
    ev = torch.empty_like(eu)
    for i in range(0, case["records"], CHUNK):
        c = min(CHUNK, case["records"] - i)
        eu[i:i + c] = upper.sample(c, gen)
        ev[i:i + c] = lower.sample(c, gen)
    return upper, lower, eu, ev


def _thresholds(count, top, gen):
    t = torch.rand(2, count, generator=gen, dtype=torch.float64)
    lo = 1.0 if top > 64 else 2.0
    t = torch.exp(math.log(lo) + t * math.log((top + 0.99) / lo)).to(torch.int64)
    return t[0].tolist(), t[1].tolist()


def _absent_pairs(count, case, upper, lower, eu, ev, gen):
    """Distinct pairs, drawn like the edges, that are not edges."""
    cand_u = upper.sample(8 * count + 64, gen).to(torch.int64)
    cand_v = lower.sample(8 * count + 64, gen).to(torch.int64)
    cand = torch.unique(cand_u * case["n_lower"] + cand_v)
    present = torch.zeros(cand.numel(), dtype=torch.bool, device="cuda")
    for i in range(0, case["records"], CHUNK):
        key = eu[i:i + CHUNK].to(torch.int64) * case["n_lower"] + ev[i:i + CHUNK]
        at = torch.searchsorted(cand, key).clamp_(max=cand.numel() - 1)
        hit = cand[at] == key
        present[at[hit]] = True
    cand = cand[~present]
    pick = cand[torch.randperm(cand.numel(), device="cuda", generator=gen)[:count]].tolist()
    return [(k // case["n_lower"], k % case["n_lower"]) for k in pick]


class _State:
    pass


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    host = torch.Generator()
    host.manual_seed(seed)
    upper, lower, eu, ev = _edges(case, gen)
    s = _State()
    s.case = case
    s.n = case["n_upper"] + case["n_lower"]
    if case["kind"] == "build":
        s.eu, s.ev = eu, ev
        return s
    s.g = ab.abcore_build_csr(case["n_upper"], case["n_lower"], eu, ev)
    s.out = torch.zeros((s.n + 31) // 32, dtype=torch.int32, device="cuda")
    kind = case["kind"]
    if kind == "gcc" and case["index_free"]:
        ab.abcore_set_option(s.g, ab.ABCORE_OPT_RANK_ORDER, INDEX_FREE)
    elif kind == "plus":
        ab.abcore_core_numbers(s.g)
    elif kind == "batch":
        s.alphas, s.betas = _thresholds(case["queries"], case["top"], host)
        s.out = torch.zeros((case["queries"], (s.n + 31) // 32), dtype=torch.int32,
                            device="cuda")
    elif kind == "gfq":
        # half the requests insert new pairs, and the pass deletes them
        # again: a stream of updates that leaves the graph as it was
        ab.abcore_components(s.g)
        half = case["requests"] // 2
        pairs = _absent_pairs(half, case, upper, lower, eu, ev, gen)
        s.stream = [(u, v, 1) for u, v in pairs] + [(u, v, -1) for u, v in pairs]
        s.alphas, s.betas = _thresholds(len(s.stream), case["top"], host)
    elif kind == "serve":
        # a pool of new pairs, taken in turn: each pass inserts some and
        # deletes them again (the engine takes new storage for each)
        ab.abcore_components(s.g)
        s.pairs = _absent_pairs(2048, case, upper, lower, eu, ev, gen)
        s.next = 0
        s.alphas, s.betas = _thresholds(case["requests"], case["top"], host)
        ab.abcore_serve_start(s.g)
    elif kind == "community":
        ab.abcore_components(s.g)
        s.vertex = int(upper.ids[0])  # the vertex of the largest expected degree
    return s


# -------------------------------------------------------------------- runs --

def run(s):
    case = s.case
    kind = case["kind"]
    if kind == "gcc":
        return ab.abcore_compute(s.g, case["alpha"], case["beta"], ab.ABCORE_GCC, out=s.out)
    if kind == "plus":
        return ab.abcore_compute(s.g, case["alpha"], case["beta"], ab.ABCORE_GCC_PLUS,
                                 out=s.out)
    if kind == "cores":
        # the option drops the cached core numbers: they are computed anew
        ab.abcore_set_option(s.g, ab.ABCORE_OPT_KCORE_SWITCH, 0)
        return ab.abcore_core_numbers(s.g)
    if kind == "batch":
        return ab.abcore_compute_batch(s.g, s.alphas, s.betas, out=s.out)
    if kind == "gfq":
        got = [ab.abcore_query(s.g, u, v, op, a, b)
               for (u, v, op), a, b in zip(s.stream, s.alphas, s.betas)]
        return torch.tensor([int(answer) for answer, _ in got]), torch.tensor([b for _, b in got])
    if kind == "serve":
        half = case["requests"] // 2
        pairs = [s.pairs[(s.next + i) % len(s.pairs)] for i in range(half)]
        s.next += half
        stream = [(u, v, 1) for u, v in pairs] + [(u, v, -1) for u, v in pairs]
        tickets = [ab.abcore_submit(s.g, u, v, op, a, b)
                   for (u, v, op), a, b in zip(stream, s.alphas, s.betas)]
        bits = []
        for t in tickets:
            r = ab.abcore_poll(s.g, t)
            while r is None:
                r = ab.abcore_poll(s.g, t)
            bits.append(r["bits"])
        return torch.tensor(bits)
    if kind == "community":
        members, size = ab.abcore_community(s.g, s.vertex, case["alpha"], case["beta"],
                                            connected=True, out=s.out)
        return members, size
    g = ab.abcore_build_csr(case["n_upper"], case["n_lower"], s.eu, s.ev)
    off, cols = ab.abcore_export_csr(g)
    g.destroy()
    # into arrays of the log's size, whatever number of edges it holds
    return off, torch.nn.functional.pad(cols, (0, 2 * case["records"] - cols.numel()), value=-1)


def work(case):
    """Each input read once and each output written once: the CSR (8 bytes an
    offset, both directions of an edge at 4 bytes), bitmasks at n / 8."""
    n = case["n_upper"] + case["n_lower"]
    m = case["records"]
    csr, bits = 8 * (n + 1) + 8 * m, n // 8
    kind = case["kind"]
    if kind == "plus":
        moved = csr + bits + 4 * n
    elif kind == "cores":
        moved = csr + 4 * n
    elif kind == "batch":
        moved = csr + case["queries"] * bits
    elif kind in ("gfq", "serve"):
        # every request looks at the labels and degrees of its graph version
        moved = csr + case["requests"] * 8 * n
    elif kind == "build":
        moved = 8 * m + csr
    else:
        moved = csr + bits
    return {"bytes": moved, "flops": 0}


def exact(case, seed):
    """Every output is a whole number, the same for any order of the work."""
    return None
