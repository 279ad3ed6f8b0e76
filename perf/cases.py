"""The work that users of this framework have it do, as cases that can be timed.

A case is a dict of plain values.  Kinds, each through the public entry points of
paper_1509_08089_amd.moss:

  estimate   one estimate on a resident graph whose tables are built
  step       a graph is handed over, estimated once and dropped: creation with its
             checks, tables, sampling, finals, destruction (device or host CSR)
  ingest     a graph is handed over and every table set is built, nothing is drawn but a
             first small estimate
  batch      many requests over resident graphs in one call
  serve      a burst of requests submitted to a running server and waited for
  classes    the class of every sample of an index range, by the call that allocates
             nothing or the one that may
  precision  pilot, planned budget and final estimate for a relative error

Graphs are power-law (Chung-Lu with repeated pairs dropped) like those of graphgen, made
on the GPU from the seed alone.  A case without "seed"-dependent sizes costs the same for
every seed: budgets and graph sizes of batches are spread evenly over their logarithms.
"""
import math

import numpy as np
import torch

from paper_1509_08089_amd import moss

SAMPLERS = {"moss4": moss.MOSS_SAMPLER_MOSS4, "moss4min": moss.MOSS_SAMPLER_MOSS4MIN,
            "t5": moss.MOSS_SAMPLER_T5, "path5": moss.MOSS_SAMPLER_PATH5}
RESULT = np.dtype(moss.moss_result)


def listed():
    return [
        # a small graph asked for a quick answer: launches and latency (the C1 workload)
        dict(name="k4 small graph", kind="estimate", n=2_000, m=10_000, beta=2.5, dmax=200, k=4, samples=100_000,
             flags=0),
        # the same on 5 nodes, odd sizes, the paper's mix weights
        dict(name="k5 small graph", kind="estimate", n=12_347, m=98_765, beta=2.3, dmax=900, k=5, samples=300_001,
             flags=moss.MOSS_MIX_PAPER),
        # the ordinary 4-node estimate (C2): tables past the L2s, inside the MALL
        dict(name="k4 1e7 on m=1e6", kind="estimate", n=100_000, m=1_000_000, beta=2.2, dmax=3_000, k=4,
             samples=10_000_000, flags=0),
        # MOSS-4 mixed with MOSS-4Min on a graph between the two
        dict(name="k4+min 4e6 on m=3e6", kind="estimate", n=300_017, m=3_000_029, beta=2.2, dmax=6_000, k=4,
             samples=4_000_037, flags=moss.MOSS_K4_MIN),
        # the largest plain estimate (C3): tables past the MALL
        dict(name="k5 1e8 on m=1e7", kind="estimate", n=1_000_000, m=10_000_000, beta=2.1, dmax=20_000, k=5,
             samples=100_000_000, flags=0),
        # a new graph from host arrays, asked once
        dict(name="step k4 host CSR", kind="step", n=20_011, m=150_007, beta=2.4, dmax=1_500, k=4, samples=500_000,
             flags=0, host=True),
        # the whole path on a large graph: every table set, the first answer
        dict(name="ingest m=1e7", kind="ingest", n=1_000_000, m=10_000_000, beta=2.1, dmax=20_000),
        # an offline job: hundreds of requests over resident graphs of all sizes (C4)
        dict(name="batch 256 over 32", kind="batch", graphs=32, m_lo=1e3, m_hi=5e6, requests=256, budget_lo=1e4,
             budget_hi=1e7),
        # an interactive batch: a few small requests, where the call itself counts
        dict(name="batch 12 over 4 small", kind="batch", graphs=4, m_lo=2e3, m_hi=1e5, requests=12, budget_lo=5e3,
             budget_hi=2e5),
        # a burst at a server: most requests small, some long (C5's mix, bounded)
        dict(name="serve 48 over 8", kind="serve", graphs=8, m_lo=5e3, m_hi=2e6, requests=48, budget_lo=1e4,
             budget_hi=1e7),
        # per-sample classes into a caller's buffer, nothing allocated
        dict(name="classes path5 noalloc", kind="classes", n=200_003, m=2_000_003, beta=2.2, dmax=5_000,
             sampler="path5", samples=(1 << 22) - 5, first=12_345_678_901, alloc=False),
        # an estimate asked for by its error
        dict(name="k5 to precision", kind="precision", n=50_021, m=400_009, beta=2.3, dmax=2_500, k=5, eps=0.01,
             delta=0.05, mask=0b1011101, pilot=100_000, most=5_000_000, flags=0),
    ]


def _spread(rng, lo, hi):
    """Spread evenly over the logarithm, a whole number."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _drawn_graph(rng, m_lo, m_hi):
    m = _spread(rng, m_lo, m_hi)
    n = max(100, int(m / rng.uniform(4.0, 16.0)))
    return dict(n=n, m=min(m, n * (n - 1) // 8), beta=round(rng.uniform(2.05, 2.6), 3),
                dmax=max(8, min(20_000, int(n / rng.uniform(6.0, 60.0)))))


def draw(rng):
    """One more case of the same ranges: any kind, graphs of 1e3 to 1e7 edges."""
    kind = rng.choice(["estimate", "estimate", "estimate", "step", "ingest", "batch", "serve", "classes", "precision"])
    c = dict(kind=kind)
    if kind == "estimate":
        c.update(_drawn_graph(rng, 1e3, 1e7))
        k, flags = rng.choice([(4, 0), (4, moss.MOSS_K4_MIN), (4, moss.MOSS_K4_MIN | moss.MOSS_MIX_PAPER), (5, 0),
                               (5, moss.MOSS_MIX_PAPER)])
        c.update(k=k, flags=flags, samples=_spread(rng, 1e3, 8e7))
    elif kind == "step":
        c.update(_drawn_graph(rng, 1e3, 3e6))
        c.update(k=rng.choice([4, 5]), flags=0, samples=_spread(rng, 1e4, 2e7), host=rng.random() < 0.4)
    elif kind == "ingest":
        c.update(_drawn_graph(rng, 1e4, 1e7))
    elif kind in ("batch", "serve"):
        requests = _spread(rng, 1, 200)
        c.update(graphs=rng.randint(1, 16), m_lo=1e3, m_hi=float(_spread(rng, 1e4, 4e6)), requests=requests,
                 budget_lo=1e4, budget_hi=float(_spread(rng, 1e5, 1e7)))
    elif kind == "classes":
        c.update(_drawn_graph(rng, 1e3, 5e6))
        alloc = rng.random() < 0.5
        c.update(sampler=rng.choice(sorted(SAMPLERS)), alloc=alloc, first=rng.randrange(1 << 40),
                 samples=_spread(rng, 1e3, 2e7 if alloc else (1 << 22)))
    else:
        c.update(_drawn_graph(rng, 1e4, 2e6))
        c.update(k=rng.choice([4, 5]), eps=round(rng.uniform(0.005, 0.1), 4), delta=0.05, mask=0b1011101,
                 pilot=_spread(rng, 1e4, 1e6), most=_spread(rng, 1e6, 1e7), flags=0)
        if c["k"] == 4:
            c["mask"] = 0b001001
    return c


# ---- inputs ------------------------------------------------------------------------------
def _power_law(n, m, beta, dmax, seed):
    """(row_ptr, col) on the GPU: m distinct pairs drawn with probability proportional to
    w_i w_j, w_i ~ (i + i0)^(-1/(beta-1)) with the largest weight dmax, ids shuffled."""
    dev = "cuda"
    idx = torch.arange(n, device=dev, dtype=torch.float64)
    lo, hi = math.log(1e-6), math.log(1e13)
    for _ in range(40):  # the largest share falls as i0 grows
        mid = 0.5 * (lo + hi)
        w = (idx + math.exp(mid)).pow_(-1.0 / (beta - 1.0))
        if float(w[0] / w.sum()) > dmax / (2.0 * m):
            lo = mid
        else:
            hi = mid
    w = (idx + math.exp(0.5 * (lo + hi))).pow_(-1.0 / (beta - 1.0)).cpu().numpy()
    cdf = np.cumsum(w)
    cdf = torch.from_numpy(cdf / cdf[-1]).to(dev)
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    keys = torch.empty(0, dtype=torch.int64, device=dev)
    while keys.numel() < m:
        take = int(1.3 * (m - keys.numel())) + 64
        a, b = (torch.searchsorted(cdf, torch.rand(take, generator=gen, device=dev, dtype=torch.float64),
                                   right=True).clamp_(max=n - 1) for _ in range(2))
        new = (torch.minimum(a, b) * n + torch.maximum(a, b))[a != b]
        keys = torch.unique(torch.cat([keys, new]))
    keep = torch.randperm(keys.numel(), generator=gen, device=dev)[:m]
    keys = keys[keep]
    ids = torch.randperm(n, generator=gen, device=dev)
    a, b = ids[keys // n], ids[keys % n]
    both = torch.sort(torch.cat([a * n + b, b * n + a])).values
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=dev)
    row_ptr[1:] = torch.cumsum(torch.bincount(both // n, minlength=n), 0)
    return row_ptr.to(torch.int32), (both % n).to(torch.int32)


def _graph_of(case, seed):
    return _power_law(case["n"], case["m"], case["beta"], case["dmax"], seed)


class _HostCSR:
    def __init__(self, row_ptr, col):
        self.row_ptr, self.col = row_ptr.cpu().numpy(), col.cpu().numpy()
        self.n, self.nnz = len(self.row_ptr) - 1, len(self.col)


class _Server:
    """A server and the graphs registered with it, ended together."""

    def __init__(self, graphs):
        self.graphs = graphs
        self.h = moss.moss_server_create(mem_budget_bytes=4 << 30)
        self.ids = [moss.moss_server_add_graph(self.h, g.h) for g in graphs]

    def __del__(self):
        moss.moss_server_destroy(self.h)


def _tables(k, flags):
    if k == 5:
        return moss.MOSS_TABLES_K5
    return moss.MOSS_TABLES_K4 | (moss.MOSS_TABLES_K4MIN if flags & moss.MOSS_K4_MIN else 0)


def _even_log(rng, lo, hi, count):
    """count whole numbers, one in each of count equal steps of the logarithm, shuffled."""
    at = (rng.permutation(count) + rng.random(count)) / count
    return np.rint(np.exp(math.log(lo) + at * math.log(hi / lo))).astype(np.int64)


def _sample_seed(seed):
    return (seed * 0x9E3779B97F4A7C15 + 1) & ((1 << 63) - 1)


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case, seed=_sample_seed(seed))
    if kind in ("batch", "serve"):
        rng = np.random.Generator(np.random.PCG64(seed))
        graphs = []
        for i, m in enumerate(_even_log(rng, case["m_lo"], case["m_hi"], case["graphs"])):
            n = max(100, int(m) // 10)
            m = min(int(m), n * (n - 1) // 4)
            g = moss.Graph.from_device(*_power_law(n, m, 2.2, min(3_000, n // 4), seed * 1000 + i))
            g.build_tables(moss.MOSS_TABLES_K4 | moss.MOSS_TABLES_K5)
            graphs.append(g)
        count = case["requests"]
        budgets = _even_log(rng, case["budget_lo"], case["budget_hi"], count)
        where, ks = rng.integers(0, len(graphs), count), 4 + rng.permutation(count) % 2
        if kind == "batch":
            s["graphs"] = graphs
            s["requests"] = [(graphs[g].h, int(k), int(b), s["seed"] + i, 0)
                             for i, (g, k, b) in enumerate(zip(where, ks, budgets))]
        else:
            s["server"] = _Server(graphs)
            s["requests"] = [(s["server"].ids[g], int(k), int(b), s["seed"] + i)
                             for i, (g, k, b) in enumerate(zip(where, ks, budgets))]
        return s
    row_ptr, col = _graph_of(case, seed)
    if kind in ("step", "ingest"):
        s["csr"] = _HostCSR(row_ptr, col) if case.get("host") else (row_ptr, col)
        return s
    s["graph"] = g = moss.Graph.from_device(row_ptr, col)
    if kind == "classes":
        s["sampler"] = SAMPLERS[case["sampler"]]
        g.build_tables({"moss4": moss.MOSS_TABLES_K4, "moss4min": moss.MOSS_TABLES_K4MIN}.get(case["sampler"],
                                                                                             moss.MOSS_TABLES_K5))
        s["classes"] = torch.empty(case["samples"], dtype=torch.uint8, device="cuda")
    else:
        g.build_tables(_tables(case["k"], case["flags"]))
    return s


# ---- one pass ----------------------------------------------------------------------------
def _answer(results):
    """What a user reads of the results: hits, estimates, variances (a copy of each)."""
    r = np.concatenate([np.frombuffer(x, RESULT) for x in results])
    return dict(hits=r["hits"].astype(np.int64), budget=r["K"].astype(np.int64), estimate=r["estimate"].copy(),
                variance=r["variance"].copy())


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "estimate":
        return _answer([s["graph"].estimate(case["k"], case["samples"], s["seed"], case["flags"])])
    if kind == "batch":
        return _answer(moss.moss_estimate_batch(s["requests"]))
    if kind == "serve":
        h = s["server"].h
        tickets = [moss.moss_server_submit(h, *q) for q in s["requests"]]
        return _answer([moss.moss_server_wait(h, t) for t in tickets])
    if kind == "classes":
        call = moss.moss_sample_range if case["alloc"] else moss.moss_sample_range_noalloc
        hits = call(s["graph"].h, s["sampler"], s["seed"], case["first"], case["first"] + case["samples"],
                    s["classes"])
        return dict(hits=hits.astype(np.int64), classes=s["classes"])
    if kind == "precision":
        return _answer([s["graph"].estimate_to_precision(case["k"], case["eps"], case["delta"], case["mask"],
                                                         case["pilot"], s["seed"] + 1, case["most"], s["seed"],
                                                         case["flags"])])
    csr = s["csr"]
    g = moss.Graph(csr, device_tensors=False) if case.get("host") else moss.Graph.from_device(*csr)
    if kind == "step":
        out = _answer([g.estimate(case["k"], case["samples"], s["seed"], case["flags"])])
    else:
        g.build_tables(moss.MOSS_TABLES_K4 | moss.MOSS_TABLES_K5 | moss.MOSS_TABLES_K4MIN)
        i = g.info()
        out = _answer([g.estimate(4, 10_000, s["seed"], moss.MOSS_K4_MIN)])
        out["totals"] = np.array([i.gamma, i.gamma1, i.gamma2, i.gamma_min, i.lambda3, i.lambda4],
                                 np.uint64).view(np.int64)
    g.close()
    return out


# ---- what a pass cannot do without ----------------------------------------------------------
PHILOX_OPS = 160          # 80 32-bit multiply-adds of a Philox4x64-10 block
RESULT_BYTES = RESULT.itemsize


def _csr_bytes(n, m):
    return 4 * (n + 1) + 8 * m


def _sampling(n, m, k, samples):
    """Bytes: the CSR read once, or the few entries that the samples touch if those are
    fewer; operations: a sample's random words (one Philox block, two on 5 nodes)."""
    return (min(_csr_bytes(n, m), 4 * (2 * k + 2) * samples), PHILOX_OPS * samples * (1 if k == 4 else 2))


def work(case):
    kind = case["kind"]
    if kind in ("batch", "serve"):
        count = case["requests"]
        at = (np.arange(count) + 0.5) / count
        budgets = np.exp(math.log(case["budget_lo"]) + at * math.log(case["budget_hi"] / case["budget_lo"]))
        at = (np.arange(case["graphs"]) + 0.5) / case["graphs"]
        ms = np.exp(math.log(case["m_lo"]) + at * math.log(case["m_hi"] / case["m_lo"]))
        return dict(bytes=float(min((8.4 * ms).sum(), 36 * budgets.sum()) + RESULT_BYTES * count),
                    flops=float(1.5 * PHILOX_OPS * budgets.sum()))
    n, m = case["n"], case["m"]
    if kind == "ingest":  # the CSR in; prefixes, ranks and descending rows of every entry and node out
        return dict(bytes=_csr_bytes(n, m) + 2 * m * (4 + 8 + 8 + 8 + 4) + n * (16 + 4 * 8) + RESULT_BYTES,
                    flops=float(PHILOX_OPS * 10_000))
    if kind == "classes":
        b, f = _sampling(n, m, 4 if case["sampler"].startswith("moss4") else 5, case["samples"])
        return dict(bytes=b + case["samples"], flops=float(f))
    if kind == "precision":  # the pilot and a final run of at least its size, as a rule
        b, f = _sampling(n, m, case["k"], 2 * case["pilot"])
        return dict(bytes=b + RESULT_BYTES, flops=float(f))
    b, f = _sampling(n, m, case["k"], case["samples"])
    if kind == "step":  # the CSR in; the prefixes of the set out
        b = _csr_bytes(n, m) + 2 * m * (4 if case["k"] == 4 else 12) + n * (16 + 8 * (case["k"] - 3))
    return dict(bytes=b + RESULT_BYTES, flops=float(f))


# ---- plain 64-bit values -----------------------------------------------------------------
def _philox(counter, seed, tag):
    """The four words of Philox4x64-10 (Salmon et al., SC 2011), counter (k, 0, 0, 0)."""
    def wide(a, b):
        lo32 = np.uint64(0xFFFFFFFF)
        s = np.uint64(32)
        a0, a1, b0, b1 = a & lo32, a >> s, np.uint64(b & 0xFFFFFFFF), np.uint64(b >> 32)
        p, q, r = a0 * b0, a1 * b0, a0 * b1
        t = q + (p >> s)
        u = r + (t & lo32)
        return a1 * b1 + (t >> s) + (u >> s), a * np.uint64(b)

    x = [counter.astype(np.uint64)] + [np.zeros(len(counter), np.uint64) for _ in range(3)]
    k0, k1, mask = seed, tag, (1 << 64) - 1
    for _ in range(10):
        h0, l0 = wide(x[0], 0xD2E7470EE14C6C93)
        h1, l1 = wide(x[2], 0xCA5A826395121157)
        x = [h1 ^ x[1] ^ np.uint64(k0), l1, h0 ^ x[3] ^ np.uint64(k1), l0]
        k0, k1 = (k0 + 0x9E3779B97F4A7C15) & mask, (k1 + 0xBB67AE8584CAA73B) & mask
    return x, wide


def exact(case, seed):
    """MOSS-4 (Algorithm 1) drawn again in plain numpy with its estimates and variances
    (Theorems 2 and 3).  The other kinds have no plain form that ends in seconds: their
    floating outputs are functions of the hits, which are whole numbers."""
    if case["kind"] not in ("estimate", "step") or case["k"] != 4 or case["flags"] or case["samples"] > 1_500_000:
        return None
    if case["m"] > 2_000_000:
        return None
    rp, col = (x.cpu().numpy().astype(np.int64) for x in _graph_of(case, seed))
    n, K = case["n"], case["samples"]
    d = np.diff(rp)
    row = np.repeat(np.arange(n), d)
    sig = np.concatenate([[0], np.cumsum(d[col] - 1)])        # over all entries
    S = sig[rp[1:]] - sig[rp[:-1]]
    acc = np.cumsum((d - 1) * S)
    gamma = int(acc[-1])
    lam = float(sum(int(x) * (int(x) - 1) * (int(x) - 2) // 6 for x in d))
    W, wide = _philox(np.arange(K), _sample_seed(seed), 0x4)

    def below(word, bound):  # floor(word * bound / 2^64), bound < 2^63
        lo32, s = np.uint64(0xFFFFFFFF), np.uint64(32)
        b = np.broadcast_to(np.asarray(bound, np.uint64), word.shape)
        a0, a1, b0, b1 = word & lo32, word >> s, b & lo32, b >> s
        t = a1 * b0 + (a0 * b0 >> s)
        u = a0 * b1 + (t & lo32)
        return (a1 * b1 + (t >> s) + (u >> s)).astype(np.int64)

    v = np.searchsorted(acc, below(W[0], gamma), side="right")
    e = np.searchsorted(sig, sig[rp[v]] + below(W[1], S[v]), side="right") - 1
    u, iu = col[e], e - rp[v]
    iw = below(W[2], d[v] - 1)
    w = col[rp[v] + iw + (iw >= iu)]
    back = np.searchsorted(row * n + col, u * n + v) - rp[u]   # v's place in u's row
    ir = below(W[3], d[u] - 1)
    r = col[rp[u] + ir + (ir >= back)]
    keys = row * n + col

    def linked(a, b):
        at = np.minimum(np.searchsorted(keys, a * n + b), len(keys) - 1)
        return keys[at] == a * n + b

    uw, vr, wr = linked(u, w), linked(v, r), linked(w, r)
    extra = uw.astype(int) + vr + wr
    cls = np.where(extra == 3, 6, np.where(extra == 2, 5, np.where(extra == 0, 1, np.where(wr, 3, 4))))
    hits = np.bincount(np.where(r == w, 0, cls), minlength=22)
    est, var = np.zeros(21), np.zeros(21)
    p = {i: 2.0 * f / gamma for i, f in ((1, 1), (3, 4), (4, 2), (5, 6), (6, 12))}
    c = {i: hits[i] / (K * p[i]) for i in p}
    for i in p:
        est[i - 1], var[i - 1] = c[i], max(0.0, c[i] / K * (1.0 / p[i] - c[i]))
    s = c[4] + 2 * c[5] + 4 * c[6]
    est[1] = lam - s
    var[1] = max(0.0, (c[4] / p[4] + 4 * c[5] / p[5] + 16 * c[6] / p[6] - s * s) / K)
    return dict(hits=np.stack([hits, np.zeros(22, np.int64)])[None], budget=np.array([[K, 0]]), estimate=est[None],
                variance=var[None])
