"""Performance cases: what programs built on this library ask of it, through the Python binding.

A case names a kind of call and its sizes:

  step     transactions on the device -> index -> frequent pairs -> index destroyed (frequent pair mining)
  host     sets in host memory -> index -> frequent pairs in host memory (a one-off analysis)
  all      all pair supports of a resident index (slot_bits 8, or 0: chosen from the set sizes)
  dense    all pair supports of a resident index by the plain bitmap route
  subset   pair supports among k items of a resident index (one interactive query)
  server   a burst of subset queries through the continuous-batching server
  batch    all pairs of several uneven instances, replayed as one batch
  cross    |A_i cap B_j| of two resident set families (sparse boolean matrix product)
  triples  |S_a cap S_b cap S_c| for every triple among the `top` largest sets

Item probabilities are constant (alpha 0) or a capped Zipf law with mean `density`; incidences are
independent Bernoulli draws, made on the GPU from the seed.
"""
import functools
import math
import random

import numpy as np
import torch

import paper_1102_1003_amd as bm

DEV = "cuda:0"


def listed():
    return [
        # the smallest mining step a program repeats: launches and host round trips count
        dict(name="tiny-step", kind="step", m=10_000, n=200, alpha=0.0, density=0.02, sigma=8, prune=False),
        # the headline mining step: 10^6 transactions, 4e7 incidences, skewed popularity
        dict(name="zipf-step", kind="step", m=1_000_000, n=2_000, alpha=1.0, density=0.02, sigma=1_000, prune=False),
        # a script that holds its sets in numpy and wants the pairs back in numpy (odd sizes)
        dict(name="host-sets", kind="host", m=30_011, n=613, alpha=0.0, density=0.03, sigma=30, prune=True),
        # the paper's own instance (n = 4000, 10^7 incidences, 5 %) queried on its resident index
        dict(name="replica-all", kind="all", m=50_000, n=4_000, alpha=0.0, density=0.05, slot_bits=8),
        # a sparse wide universe, where the library picks the slot width from the sizes
        dict(name="sparse-all", kind="all", m=1_048_576, n=8_192, alpha=0.0, density=0.0005, slot_bits=0),
        # the dense comparator at its own sizes
        dict(name="dense-gram", kind="dense", m=1_048_576, n=4_096, alpha=0.0, density=0.05),
        # one small interactive query against resident maps: latency
        dict(name="subset-small", kind="subset", m=1_000_000, n=8_192, alpha=1.1, density=0.01, k=48),
        # one large query against resident maps
        dict(name="subset-large", kind="subset", m=1_000_000, n=8_192, alpha=1.1, density=0.01, k=2_048),
        # a burst of queries of mixed sizes through the server
        dict(name="server-mix", kind="server", m=1_000_000, n=8_192, alpha=1.1, density=0.01, queries=24, k_hi=1_024),
        # many uneven instances in one replayed batch
        dict(name="batch-uneven", kind="batch", count=8, m_lo=10_000, m_hi=400_000, n_lo=100, n_hi=3_000),
        # product of two set families over one universe
        dict(name="cross", kind="cross", m=500_000, n=2_000, nb=1_500, alpha=1.0, density=0.02),
        # itemsets of three among the most popular items
        dict(name="triples", kind="triples", m=1_000_000, n=500, alpha=1.0, density=0.02, top=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "host", "all", "all", "dense", "subset", "subset", "server", "batch", "cross",
                       "triples"])
    alpha = rng.choice([0.0, 1.0, 1.1])
    density = round(math.exp(rng.uniform(math.log(0.005), math.log(0.08))), 5)
    if kind in ("step", "host"):
        top = 1_000_000 if kind == "step" else 120_000
        m, n = _log(rng, 8_000, top), _log(rng, 60, 4_000)
        cap = 3e7 if kind == "step" else 2e6
        density = round(min(density, cap / (m * n)), 7)
        return dict(kind=kind, m=m, n=n, alpha=alpha, density=density,
                    sigma=max(1, int(m * density * density * rng.uniform(0.3, 1.5))), prune=rng.random() < 0.5)
    if kind == "all":
        if rng.random() < 0.4:
            m, n = _log(rng, 100_000, 1_048_576), _log(rng, 500, 8_192)
            density = round(math.exp(rng.uniform(math.log(0.0001), math.log(0.001))), 6)
            return dict(kind=kind, m=m, n=n, alpha=0.0, density=density, slot_bits=0)
        m, n = _log(rng, 8_000, 500_000), _log(rng, 100, 4_000)
        return dict(kind=kind, m=m, n=n, alpha=alpha, density=round(min(density, 3e7 / (m * n)), 7), slot_bits=8)
    if kind == "dense":
        return dict(kind=kind, m=_log(rng, 10_000, 1_048_576), n=_log(rng, 100, 4_096), alpha=alpha, density=density)
    if kind == "subset":
        n = _log(rng, 1_000, 8_192)
        return dict(kind=kind, m=_log(rng, 50_000, 1_000_000), n=n, alpha=rng.choice([0.0, 1.1]), density=0.01,
                    k=min(n, _log(rng, 16, 2_048)))
    if kind == "server":
        return dict(kind=kind, m=_log(rng, 100_000, 1_000_000), n=_log(rng, 1_500, 8_192), alpha=1.1, density=0.01,
                    queries=rng.randint(8, 32), k_hi=_log(rng, 200, 1_024))
    if kind == "batch":
        return dict(kind=kind, count=rng.randint(3, 8), m_lo=10_000, m_hi=_log(rng, 50_000, 400_000), n_lo=100,
                    n_hi=_log(rng, 500, 3_000))
    if kind == "cross":
        return dict(kind=kind, m=_log(rng, 10_000, 500_000), n=_log(rng, 100, 2_000), nb=_log(rng, 100, 2_000),
                    alpha=alpha, density=min(density, 0.03))
    return dict(kind=kind, m=_log(rng, 20_000, 1_000_000), n=_log(rng, 64, 600), alpha=1.0,
                density=round(rng.uniform(0.01, 0.03), 4), top=rng.randint(12, 64))


# ---------------------------------------------------------------- inputs

@functools.lru_cache(maxsize=64)
def _probs(n, alpha, density):
    """Item probabilities by rank: min(1, c rank^-alpha) with mean `density` (c by bisection)."""
    if alpha == 0.0:
        return np.full(n, density)
    base = np.arange(1, n + 1, dtype=np.float64) ** -alpha
    lo, hi = 0.0, 1e9
    for _ in range(200):
        c = 0.5 * (lo + hi)
        lo, hi = (c, hi) if np.minimum(1.0, c * base).mean() < density else (lo, c)
    return np.minimum(1.0, 0.5 * (lo + hi) * base)


def _item_probs(c, n, seed):
    """Probabilities by item id: ranks shuffled by the seed."""
    p = _probs(n, c["alpha"], c["density"])
    return p[np.random.default_rng(seed).permutation(n)]


def _masks(rows, cols, probs, seed, probs_by_row):
    """0/1 blocks (first row, bool tensor) of a rows x cols Bernoulli matrix on the GPU."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    p = torch.tensor(probs, dtype=torch.float32, device=DEV)
    step = max(1, (1 << 29) // cols)
    for r0 in range(0, rows, step):
        r1 = min(rows, r0 + step)
        u = torch.rand((r1 - r0, cols), generator=g, device=DEV)
        yield r0, u < (p[r0:r1, None] if probs_by_row else p[None, :])


def _csr(rows, cols, probs, seed, probs_by_row):
    sizes, parts = [], []
    for _, hit in _masks(rows, cols, probs, seed, probs_by_row):
        sizes.append(hit.sum(dim=1))
        parts.append(hit.nonzero()[:, 1].to(torch.int32))
    off = torch.zeros(rows + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(torch.cat(sizes), 0)
    tids = torch.cat(parts)
    torch.cuda.synchronize()                # the library reads them on the context's own stream
    return off, tids


def _sets(c, seed, n=None):
    """Tidlists (offsets, tids): each set sorted, n sets over m transactions."""
    n = n or c["n"]
    return _csr(n, c["m"], _item_probs(c, n, seed), seed, True)


def _transactions(c, seed):
    return _csr(c["m"], c["n"], _item_probs(c, c["n"], seed), seed, False)


def _instances(c, seed):
    """Uneven Bernoulli instances: m log-uniform, n uniform, density uniform 1-10 %.  The sizes come from
    the case alone, so that every seed is the same amount of work."""
    r = random.Random(c["count"] * 1_000_003 + c["m_hi"] * 31 + c["n_hi"])
    return [dict(m=_log(r, c["m_lo"], c["m_hi"]), n=r.randint(c["n_lo"], c["n_hi"]), alpha=0.0,
                 density=r.uniform(0.01, 0.10)) for _ in range(c["count"])]


def _queries(c, seed):
    r = random.Random(c["queries"] * 7919 + c["k_hi"])      # the sizes: the same for every seed
    ks = [max(2, min(_log(r, 16, c["k_hi"]), c["n"])) for _ in range(c["queries"])]
    rng = np.random.default_rng(seed)
    return [rng.choice(c["n"], size=k, replace=False).astype(np.uint32) for k in ks]


def _subset(c, seed):
    return np.random.default_rng(seed + 1).choice(c["n"], size=c["k"], replace=False).astype(np.uint32)


def _triples(c, off):
    """Every triple among the `top` largest sets."""
    sizes = (off[1:] - off[:-1])
    top = torch.sort(torch.topk(sizes, c["top"]).indices).values
    return top[torch.combinations(torch.arange(c["top"], device=DEV), 3)].to(torch.int32).contiguous()


@functools.lru_cache(maxsize=1)
def _context():
    """The program's one context, on a stream of its own."""
    return bm.Context(0, torch.cuda.Stream())


def _out(count):
    out = torch.zeros(max(count, 1), dtype=torch.int32, device=DEV)
    torch.cuda.synchronize()
    return out


def prepare(case, seed):
    c, ctx, kind = case, _context(), case["kind"]
    s = dict(case=c, ctx=ctx)
    if kind == "step":
        s["off"], s["items"] = _transactions(c, seed)
        s["out"] = _out(3 * bm.n_pairs(c["n"]))
    elif kind == "host":
        off, tids = _sets(c, seed)
        s["off"] = off.cpu().numpy().astype(np.uint64)
        s["tids"] = tids.cpu().numpy().astype(np.uint32)
        s["out"] = np.zeros(3 * bm.n_pairs(c["n"]), dtype=np.uint32)
    elif kind == "batch":
        insts = _instances(c, seed)
        s["idx"] = [bm.Index.from_sets(ctx, i["m"], *_sets(i, seed * 64 + q)) for q, i in enumerate(insts)]
        s["outs"] = [_out(bm.n_pairs(i["n"])) for i in insts]
        s["batch"] = bm.Batch(ctx, s["idx"], s["outs"])
    elif kind == "cross":
        s["a"] = bm.Index.from_sets(ctx, c["m"], *_sets(c, seed))
        s["b"] = bm.Index.from_sets(ctx, c["m"], *_sets(c, seed + 500_009, c["nb"]))
        s["out"] = _out(c["n"] * c["nb"])
    elif kind == "triples":
        off, tids = _sets(c, seed)
        s["triples"] = _triples(c, off)
        s["idx"] = bm.Index.from_sets(ctx, c["m"], off, tids, order=3)
        s["out"] = _out(s["triples"].shape[0])
    else:
        s["idx"] = bm.Index.from_sets(ctx, c["m"], *_sets(c, seed), slot_bits=c.get("slot_bits", 8))
        if kind == "subset":
            s["query"] = _subset(c, seed)
            s["out"] = _out(bm.n_pairs(c["k"]))
        elif kind == "server":
            s["queries"] = _queries(c, seed)
            s["server"] = bm.Server(s["idx"])
        else:
            s["out"] = _out(bm.n_pairs(c["n"]))
    return s


def run(s):
    c, ctx = s["case"], s["ctx"]
    kind = c["kind"]
    if kind == "step":
        idx = bm.Index.from_transactions(ctx, c["n"], s["off"], s["items"],
                                         min_support=c["sigma"] if c["prune"] else 0)
        found = idx.frequent_pairs_into(c["sigma"], s["out"])
        idx.close()
        return [s["out"], found]
    if kind == "host":
        idx = bm.Index.from_sets(ctx, c["m"], s["off"], s["tids"], min_support=c["sigma"] if c["prune"] else 0)
        found = idx.frequent_pairs_into(c["sigma"], s["out"])
        idx.close()
        return [s["out"], found]
    if kind == "all":
        return s["idx"].all_pair_supports(s["out"])
    if kind == "dense":
        return s["idx"].all_pair_supports_dense(s["out"])
    if kind == "subset":
        return s["idx"].subset_pair_supports(s["query"], s["out"])
    if kind == "server":
        ids = [s["server"].submit(q) for q in s["queries"]]
        return [s["server"].wait(i)[0] for i in ids]
    if kind == "batch":
        s["batch"].run()
        return s["outs"]
    if kind == "cross":
        return bm.cross_pair_supports(s["a"], s["b"], s["out"])
    return s["idx"].triple_supports(s["triples"], s["out"])


# ---------------------------------------------------------------- exact results

def _gram(c, seed, rows=None, transactions=False, other=None):
    """|S_i cap S_j| in 64 bits: the product of the 0/1 matrix with its transpose (or with the other family's)."""
    if transactions:
        n = c["n"]
        g = torch.zeros((n, n), dtype=torch.float64, device=DEV)
        for _, hit in _masks(c["m"], n, _item_probs(c, n, seed), seed, False):
            a = hit.to(torch.float64)
            g += a.T.contiguous() @ a
        return g

    def bits(n, sd):
        return torch.cat([hit for _, hit in _masks(n, c["m"], _item_probs(c, n, sd), sd, True)])

    a = bits(c["n"], seed)
    if rows is not None:
        a = a[rows]
    b = a if other is None else bits(*other)
    g = torch.zeros((a.shape[0], b.shape[0]), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 28) // max(a.shape[0], b.shape[0]))
    for t0 in range(0, c["m"], step):
        x = a[:, t0:t0 + step].to(torch.float64)
        y = x if other is None else b[:, t0:t0 + step].to(torch.float64)
        g += x @ y.T.contiguous()
    return g


def _packed(g):
    i, j = torch.triu_indices(g.shape[0], g.shape[0], 1, device=DEV)
    return g[i, j].to(torch.int64)


def _rows(g, sigma):
    """(i, j, support) rows with support >= sigma, by (i, j), in a buffer for every pair, and their number."""
    i, j = torch.triu_indices(g.shape[0], g.shape[0], 1, device=DEV)
    v = g[i, j].to(torch.int64)
    k = v >= sigma
    found = int(k.sum())
    out = torch.zeros(3 * v.numel(), dtype=torch.int64, device=DEV)
    out[:3 * found] = torch.stack([i[k], j[k], v[k]], 1).reshape(-1)
    return [out, found]


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "step":
        return _rows(_gram(c, seed, transactions=True), c["sigma"])
    if kind == "host":
        return _rows(_gram(c, seed), c["sigma"])
    if kind in ("all", "dense"):
        return _packed(_gram(c, seed))
    if kind == "subset":
        return _packed(_gram(c, seed, rows=torch.from_numpy(_subset(c, seed).astype(np.int64)).to(DEV)))
    if kind == "server":
        qs = [torch.from_numpy(q.astype(np.int64)).to(DEV) for q in _queries(c, seed)]
        every, at = torch.unique(torch.cat(qs), return_inverse=True)
        g = _gram(c, seed, rows=every)
        parts = torch.split(at, [q.numel() for q in qs])
        return [_packed(g[p][:, p]) for p in parts]
    if kind == "batch":
        return [_packed(_gram(i, seed * 64 + q)) for q, i in enumerate(_instances(c, seed))]
    if kind == "cross":
        return _gram(c, seed, other=(c["nb"], seed + 500_009)).to(torch.int64).reshape(-1)
    off, _ = _sets(c, seed)
    t = _triples(c, off).to(torch.int64)
    every, at = torch.unique(t, return_inverse=True)
    bits = torch.cat([hit for _, hit in _masks(c["n"], c["m"], _item_probs(c, c["n"], seed), seed, True)])[every]
    k = every.numel()
    g3 = torch.zeros((k, k, k), dtype=torch.float64, device=DEV)
    for t0 in range(0, c["m"], 1 << 20):
        a = bits[:, t0:t0 + (1 << 20)].to(torch.float64)
        at_ = a.T.contiguous()
        for x in range(k):
            g3[x] += (a * a[x]) @ at_
    return g3[at[:, 0], at[:, 1], at[:, 2]].to(torch.int64)


# ---------------------------------------------------------------- work of one pass

def _shared(m, p, q=None):
    """Expected sum over the pairs of |S_i cap S_j|: the additions a count of the pairs cannot do without."""
    p = np.asarray(p)
    if q is None:
        return m * (p.sum() ** 2 - (p * p).sum()) / 2
    return m * p.sum() * np.asarray(q).sum()


def work(case):
    """Inputs read once and outputs written once (tidlists 4 bytes an incidence, 4 bytes a support), and one
    multiply and add per shared incidence; for the bitmap route, the product of the 0/1 matrix it is."""
    c, kind = case, case["kind"]
    if kind == "batch":
        each = [(i["m"], _probs(i["n"], 0.0, i["density"])) for i in _instances(c, 0)]
        return {"bytes": float(sum(4 * m * p.sum() + 4 * bm.n_pairs(len(p)) for m, p in each)),
                "flops": float(sum(2 * _shared(m, p) for m, p in each))}
    m, n = c["m"], c["n"]
    p = _probs(n, c["alpha"], c["density"])
    nnz = m * p.sum()
    if kind in ("step", "host"):
        inputs = 4 * nnz + 8 * ((m if kind == "step" else n) + 1)
        # pairs kept: by the normal law around each pair's expected support
        e = m * np.outer(p, p)
        keep = 0.5 * (1 + np.vectorize(math.erf)((e - c["sigma"] + 0.5) / np.sqrt(2 * np.maximum(e, 1e-9)))) \
            if n <= 300 else (e >= c["sigma"])
        kept = (keep.sum() - np.trace(keep)) / 2
        return {"bytes": float(inputs + 12 * kept), "flops": float(2 * _shared(m, p))}
    if kind == "all":
        return {"bytes": float(4 * nnz + 4 * bm.n_pairs(n)), "flops": float(2 * _shared(m, p))}
    if kind == "dense":
        return {"bytes": float(4 * nnz + 4 * bm.n_pairs(n)), "flops": 2.0 * m * bm.n_pairs(n)}
    if kind in ("subset", "server"):
        # k items drawn among all: expected incidences and shared incidences of the drawn ones
        ks = [c["k"]] if kind == "subset" else [q.size for q in _queries(c, 0)]
        return {"bytes": float(sum(4 * nnz * k / n + 4 * k + 4 * bm.n_pairs(k) for k in ks)),
                "flops": float(sum(2 * _shared(m, p) * bm.n_pairs(k) / bm.n_pairs(n) for k in ks))}
    if kind == "cross":
        q = _probs(c["nb"], c["alpha"], c["density"])
        return {"bytes": float(4 * nnz + 4 * m * q.sum() + 4 * n * c["nb"]), "flops": float(2 * _shared(m, p, q))}
    t = np.sort(p)[::-1][:c["top"]]
    s1, s2, s3 = t.sum(), (t ** 2).sum(), (t ** 3).sum()
    count = math.comb(c["top"], 3)
    return {"bytes": float(4 * m * s1 + 16 * count), "flops": float(2 * m * (s1 ** 3 - 3 * s1 * s2 + 2 * s3) / 6)}
