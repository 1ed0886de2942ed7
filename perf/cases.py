"""Performance cases of the threshold-aware IVF search.

A case is one call of a public entry point (``Index.search``, ``search_fixed``,
``search_calibrated``, ``search_multi``) on an index that the caller has loaded, with the
queries on the GPU.  The inputs are deduplication self-joins: a mixture corpus on the unit
sphere with planted near-duplicate groups, an IVF built by a few k-means rounds with
nearest-centroid assignment, and queries that are rows of the corpus and exclude themselves.

Every case is a dict of plain values:
  call      "search" | "fixed" | "calibrated" | "multi"
  n, d, dtype, nlist     corpus rows, dimension, "f32" | "f16", partitions (per shard in "multi")
  nq, k, tau, W, nprobe  queries, results per query, threshold, window, probe cap (fixed: probes)
  mode      "lookahead" | "speculative" | "basic" (search and multi only)
  shards    indexes ("multi" only, else 1)
  sigma, dup_sigma, dup_frac, zipf   spread of a mixture component, of a near-duplicate group,
                                     share of grouped rows, group sizes (Zipf, else geometric)
"""
import math

import torch

import paper_2608_03199_amd as ps

#: sampled share and loss target of the calibrated calls
SAMPLE_RATE, EPS, W_FALLBACK = 0.02, 0.005, 8


def _case(name, call, n, d, dtype, nlist, nq, *, k=10, tau=0.92, W=8, nprobe=128,
          mode="lookahead", shards=1, sigma=0.25, dup_sigma=0.015, dup_frac=0.15, zipf=False):
    c = dict(call=call, n=n, d=d, dtype=dtype, nlist=nlist, nq=nq, k=k, tau=tau, W=W,
             nprobe=nprobe, mode=mode, shards=shards, sigma=sigma, dup_sigma=dup_sigma,
             dup_frac=dup_frac, zipf=zipf)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # one new row checked against the corpus at ingest: latency, launches and host round trips
        _case("one_query_1m_d128_f32", "search", 1_000_000, 128, "f32", 1024, 1),
        # a small ingest batch against a corpus of long rows: few queries per partition, row reads
        _case("batch_100_1m_d768_f16", "search", 1_000_000, 768, "f16", 512, 100, tau=0.95,
              nprobe=64, sigma=0.2, dup_sigma=0.008),
        # the tiny self-join: a corpus that fits a cache
        _case("join_20k_d64_f32", "search", 20_000, 64, "f32", 64, 1_000, tau=0.90, nprobe=32,
              sigma=0.3, dup_sigma=0.02, dup_frac=0.10),
        # the mid-size self-join in fp32
        _case("join_1m_d128_f32", "search", 1_000_000, 128, "f32", 1024, 10_000),
        # loose threshold and many results: every probe finds neighbours, many rounds, the whole
        # candidate and merge machinery
        _case("loose_1m_d128_f32_k50", "search", 1_000_000, 128, "f32", 1024, 4_000, k=50,
              tau=0.30),
        # the window chosen inside the call from a fully probed sample
        _case("calibrated_1m_d128_f32", "calibrated", 1_000_000, 128, "f32", 1024, 10_000),
        # dimensions of public embedding sets that have no kernel of their own: 96 and 512
        _case("join_4m_d96_f16", "search", 4_000_000, 96, "f16", 2048, 50_000, tau=0.90,
              nprobe=256, dup_sigma=0.02),
        _case("join_2m_d512_f16", "search", 2_000_037, 512, "f16", 1500, 20_001, tau=0.93,
              nprobe=90, sigma=0.2, dup_sigma=0.01),
        # the fixed-probe baseline on fp16 rows: long rankings, one dense round
        _case("fixed_8m_d128_f16", "fixed", 8_000_000, 128, "f16", 4096, 20_000, tau=0.90,
              nprobe=256, dup_sigma=0.02),
        # coarse shards, each with its own index and stop rule
        _case("multi_8x1m_d128_f16", "multi", 1_000_000, 128, "f16", 512, 50_000, tau=0.90,
              nprobe=64, shards=8, dup_sigma=0.02, dup_frac=0.10, zipf=True),
        # the large self-joins: long rows, and the largest corpus
        _case("join_10m_d768_f16", "search", 10_000_000, 768, "f16", 4096, 100_000, tau=0.95,
              nprobe=256, sigma=0.2, dup_sigma=0.008, dup_frac=0.20, zipf=True),
        _case("join_48m_d128_f16", "search", 48_000_000, 128, "f16", 8192, 480_000, tau=0.90,
              nprobe=512, dup_sigma=0.02, dup_frac=0.10, zipf=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["search", "search", "search", "search", "fixed", "calibrated", "multi"])
    dtype = rng.choice(["f16", "f16", "f32"])
    # the dimensions with kernels of their own, and others (whole 16-byte segments)
    d = rng.choice([64, 96, 128, 128, 256, 384, 512, 768, 8 * rng.randint(4, 120)])
    if dtype == "f32":
        d = min(d, 512)
    row_bytes = d * (2 if dtype == "f16" else 4)
    shards = rng.randint(2, 8) if call == "multi" else 1
    n = _log(rng, 20_000, min(20_000_000, 8_000_000_000 // row_bytes) // shards)
    nlist = max(16, min(8192, n // _log(rng, 300, 5000)))
    mode = "lookahead"
    if call in ("search", "multi"):
        mode = rng.choice(["lookahead", "lookahead", "lookahead", "speculative", "basic"])
    tau = rng.choice([0.85, 0.90, 0.92, 0.95, 0.95, 0.30])
    nprobe = min(nlist, _log(rng, 24, 256))
    W = rng.choice([2, 4, 8, 8, 8, 16])
    # queries: from one to a tenth of the corpus, bounded by the row products of the call
    per_query = (n / nlist) * 2 * d * (nprobe if call == "fixed" or tau < 0.5 else W + 1)
    if call == "calibrated":
        per_query *= 1 + SAMPLE_RATE * nprobe / W
    cap = int(min(n // 10, 200_000, (4e12 if dtype == "f16" else 4e11) / (per_query * shards)))
    nq = _log(rng, 1, max(2, cap))
    return _case(None, call, n, d, dtype, nlist, nq, k=rng.choice([1, 5, 10, 10, 10, 50]),
                 tau=tau, W=W, nprobe=nprobe, mode=mode, shards=shards,
                 sigma=0.2 if d >= 512 else 0.25, dup_sigma=round(math.sqrt(0.045 / d), 4),
                 dup_frac=rng.choice([0.10, 0.15, 0.20]), zipf=rng.random() < 0.5)


# ---- inputs ----

def _unit(x):
    return x / x.norm(dim=1, keepdim=True).clamp_min(1e-30)


def _nearest(x, cent, rows):
    """Highest-inner-product centroid of every row, in blocks of `rows` rows."""
    ct = cent.t().contiguous()
    return torch.cat([(b @ ct).argmax(dim=1).to(torch.int32) for b in x.split(rows)])


def _corpus(case, seed):
    """The stored rows in id order and the rows that are queries (and the generator)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1_000_003 + 17)
    n, d = case["n"] * case["shards"], case["d"]
    dt = torch.float16 if case["dtype"] == "f16" else torch.float32
    dev = "cuda"
    ncomp = max(8, 6 * case["nlist"])
    centres = _unit(torch.randn(ncomp, d, generator=g, device=dev))
    x = torch.empty(n, d, dtype=dt, device=dev)
    step = max(1, (1 << 28) // d)
    for a in range(0, n, step):
        m = min(step, n - a)
        z = torch.randn(m, d, generator=g, device=dev).mul_(case["sigma"])
        z += centres[torch.randint(ncomp, (m,), generator=g, device=dev)]
        x[a:a + m] = _unit(z)
        del z
    # near-duplicate groups over a random permutation; a group's first row stays
    target = int(case["dup_frac"] * n)
    perm = torch.randperm(n, generator=g, device=dev)
    if target >= 2:
        u = torch.rand(target // 2 + 1, generator=g, device=dev, dtype=torch.float64)
        if case["zipf"]:   # P(size > s) = s^-0.5, capped at 500
            sizes = (1 + torch.floor((1 - u).clamp_min(1e-12) ** -2.0)).clamp_max(500)
        else:              # 1 + geometric(1/3)
            sizes = 2 + torch.floor(torch.log((1 - u).clamp_min(1e-12)) / math.log(2 / 3))
        starts = torch.cumsum(sizes.to(torch.int64), 0)
        at = torch.arange(target, device=dev)
        group = torch.searchsorted(starts, at, right=True)
        first = torch.cat([starts.new_zeros(1), starts])[group]
        member = (at != first).nonzero().flatten()
        rows, seeds = perm[member], perm[first[member]]
        for a in range(0, rows.numel(), step):
            r, s = rows[a:a + step], seeds[a:a + step]
            z = torch.randn(r.numel(), d, generator=g, device=dev).mul_(case["dup_sigma"])
            x[r] = _unit(x[s].float() + z).to(dt)
            del z
        del u, sizes, starts, at, group, first, member, rows, seeds
    # the query sample: distinct rows, grouped ones in their share of the corpus (at least one)
    nq = case["nq"]
    grouped = min(nq, target, math.ceil(case["dup_frac"] * nq))
    at = torch.randperm(target, generator=g, device=dev)[:grouped]
    qrows = torch.cat([perm[at], perm[target:target + nq - grouped]])
    return x, qrows[torch.randperm(nq, generator=g, device=dev)], g


def _ivf(x, ids, nlist, g):
    """(vectors, offsets, ids, centroids), partition-major: k-means on a sample, then the
    nearest centroid of every row.  Cluster sums are differences of fp64 prefix sums, so a seed
    gives the same bits each time."""
    n, d = x.shape
    block = max(1, (1 << 31) // nlist)
    samp = x[torch.randperm(n, generator=g, device=x.device)[:min(n, 24 * nlist)]]
    cent = samp[:nlist].clone()
    for _ in range(4):
        a = _nearest(samp, cent, block).to(torch.int64)
        order = torch.sort(a, stable=True).indices
        cnt = torch.bincount(a, minlength=nlist)
        ends = torch.cumsum(cnt, 0)
        pre = torch.zeros(samp.shape[0] + 1, d, dtype=torch.float64, device=x.device)
        pre[1:] = torch.cumsum(samp[order].double(), 0)
        sums = (pre[ends] - pre[ends - cnt]).float()
        cent = torch.where((cnt == 0)[:, None], cent, _unit(sums).to(x.dtype))
        del pre, sums
    a = _nearest(x, cent, block)
    order = torch.sort(a, stable=True).indices
    offsets = torch.zeros(nlist + 1, dtype=torch.int64, device=x.device)
    offsets[1:] = torch.cumsum(torch.bincount(a, minlength=nlist), 0)
    return x[order], offsets, ids[order], cent.contiguous()


def _data(case, seed):
    """What a caller holds: the indexes' arrays, the queries and their own ids, the sample."""
    x, qrows, g = _corpus(case, seed)
    queries = x[qrows].contiguous()
    ids = torch.arange(x.shape[0], device="cuda")
    parts = []
    if case["shards"] == 1:
        parts.append(_ivf(x, ids, case["nlist"], g))
    else:  # coarse shards: the nearest of a few coarse centres
        coarse = _unit(torch.randn(case["shards"], case["d"], generator=g, device="cuda"))
        a = _nearest(x, coarse.to(x.dtype), 1 << 24)
        for s in range(case["shards"]):
            rows = (a == s).nonzero().flatten()
            parts.append(_ivf(x[rows], rows, case["nlist"], g))
    ns = max(1, int(SAMPLE_RATE * case["nq"]))
    sample = torch.randperm(case["nq"], generator=g, device="cuda")[:ns].to(torch.int32)
    del x
    return parts, queries, qrows, sample


def prepare(case, seed):
    """The loaded index (or the shards' indexes) and the query batch."""
    parts, queries, exclude, sample = _data(case, seed)
    indexes = []
    while parts:
        vectors, offsets, ids, cent = parts.pop(0)
        indexes.append(ps.Index(vectors, offsets, ids, cent))
        del vectors, offsets, ids, cent
    torch.cuda.empty_cache()
    return {"case": case, "indexes": indexes, "queries": queries, "exclude": exclude,
            "sample": sample}


def run(state):
    """One call: (ids, scores, probes), and the chosen window of a calibrated call."""
    c, q, ex = state["case"], state["queries"], state["exclude"]
    ix = state["indexes"][0]
    look = dict(lookahead=c["mode"] != "basic", speculative=c["mode"] == "speculative")
    if c["call"] == "search":
        return ix.search(q, ex, c["k"], c["tau"], c["W"], c["nprobe"], **look)
    if c["call"] == "fixed":
        return ix.search_fixed(q, ex, c["k"], c["tau"], c["nprobe"])
    if c["call"] == "calibrated":
        return ix.search_calibrated(q, ex, c["k"], c["tau"], c["nprobe"], state["sample"], EPS,
                                    W_FALLBACK)
    return ps.search_multi(state["indexes"], q, ex, c["k"], c["tau"], c["W"], c["nprobe"], **look)


def work(case):
    """Every touched partition read once, queries and centroids read, results written; the
    centroid products of the ranking and the row products of the probes the rule makes (the
    window and a little more under a near-duplicate threshold, the cap under a loose one)."""
    e = 2 if case["dtype"] == "f16" else 4
    d, nq, nlist, sh = case["d"], case["nq"], case["nlist"], case["shards"]
    per_list = case["n"] / nlist
    n = min(case["nprobe"], nlist)
    probes = n if case["call"] == "fixed" or case["tau"] < 0.5 else min(n, case["W"] + 0.3)
    if case["call"] == "calibrated":
        probes += SAMPLE_RATE * n
    touched = nlist * (1 - (1 - 1 / nlist) ** (nq * probes))
    nbytes = sh * (touched * per_list * d * e + nlist * d * e) + nq * (d * e + 12 * case["k"] + 12)
    flops = 2.0 * d * nq * sh * (nlist + probes * per_list)
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    """Scores are sums in 32 bits of products of the stored values; results within rounding of
    each other may swap places, and a row within rounding of the threshold may change sides."""
    return {"rel": 1e-6, "max": 1e-5, "differ": 2e-3}


# ---- the same results in 64 bits ----

def _exact_ranks(q, cent, n):
    c64 = cent.double().t().contiguous()
    step = max(1, (1 << 28) // cent.shape[0])
    return torch.cat([torch.sort(b.double() @ c64, dim=1, descending=True, stable=True)
                      .indices[:, :n] for b in q.split(step)])


class _Exact:
    """Threshold search of one index in fp64, list by list; qs: the query rows searched."""

    def __init__(self, case, part, q, ex):
        self.vec, off, self.ids, cent = part
        self.off = off.tolist()
        self.q, self.ex, self.k, self.tau = q, ex, case["k"], float(torch.tensor(case["tau"]))
        self.n = min(case["nprobe"], case["nlist"])
        self.P = _exact_ranks(q, cent, self.n)
        nq = q.shape[0]
        self.sc = torch.full((nq, self.k), -math.inf, dtype=torch.float64, device=q.device)
        self.id = torch.full((nq, self.k), -1, dtype=torch.int64, device=q.device)
        self.rk = torch.full((nq, self.k), -1, dtype=torch.int64, device=q.device)

    def scan(self, qi, rank):
        """Search items (query, rank); returns whether each found a neighbour."""
        lists = self.P[qi, rank]
        order = torch.sort(lists, stable=True).indices
        cnt = torch.bincount(lists, minlength=len(self.off) - 1).tolist()
        hit = torch.zeros(qi.numel(), dtype=torch.bool, device=qi.device)
        at = 0
        for l, m in enumerate(cnt):
            a, b = self.off[l], self.off[l + 1]
            o = order[at:at + m]
            at += m
            if m == 0 or a == b:
                continue
            v = self.vec[a:b].double().t().contiguous()
            step = max(1, (1 << 27) // (b - a))
            for oo in o.split(step):
                i = qi[oo]
                s = self.q[i].double() @ v
                s.masked_fill_((s < self.tau) | (self.ids[a:b][None, :] == self.ex[i][:, None]),
                               -math.inf)
                top, pos = s.topk(min(self.k, b - a), dim=1)
                hit[oo] = top[:, 0] > -math.inf
                sc = torch.cat([self.sc[i], top], 1)
                idn = torch.cat([self.id[i], self.ids[a:b][pos]], 1)
                rk = torch.cat([self.rk[i], rank[oo][:, None].expand(-1, top.shape[1])], 1)
                best, at2 = sc.topk(self.k, dim=1)
                self.sc[i] = best
                self.id[i] = torch.where(best > -math.inf, idn.gather(1, at2), -1)
                self.rk[i] = torch.where(best > -math.inf, rk.gather(1, at2), -1)
        return hit

    def search(self, W, rows):
        """The stop rule over query rows `rows`; returns their probe counts."""
        stop = torch.full_like(rows, min(W, self.n))
        done = torch.zeros_like(rows)
        while bool((done < stop).any()):
            todo = stop - done
            own = torch.repeat_interleave(torch.arange(rows.numel(), device=rows.device), todo)
            rank = torch.arange(own.numel(), device=rows.device) - (todo.cumsum(0) - todo)[own] \
                + done[own]
            hit = self.scan(rows[own], rank)
            last = torch.zeros_like(rows).scatter_reduce_(
                0, own, torch.where(hit, rank + 1, 0), "amax")
            done = stop
            stop = torch.where(last > 0, torch.maximum(stop, (last + W).clamp_max(self.n)), stop)
        return stop

    def window(self, sample):
        """The calibrated window of a fully probed sample (Appendix A)."""
        own = torch.repeat_interleave(sample, self.n)
        rank = torch.arange(self.n, device=sample.device).repeat(sample.numel())
        hit = self.scan(own, rank).reshape(sample.numel(), self.n).cpu()
        need = []
        for h, fr in zip(hit.tolist(), self.rk[sample].tolist()):
            longest, run, upto = 0, 0, []
            for x in h:
                upto.append(longest)
                run = 0 if x else run + 1
                longest = max(longest, run)
            need += [1 + upto[f] for f in fr if f >= 0]
        if not need:
            return W_FALLBACK
        eps = float(torch.tensor(EPS))
        for w in range(1, self.n):
            if 1.0 - sum(x <= w for x in need) / len(need) < eps:
                return w
        return self.n


def exact(case, seed):
    if case["n"] * case["d"] > 1.2e9 or case["nq"] * case["nprobe"] > 3e7:
        return None  # minutes of list-by-list products in 64 bits
    parts, q, ex, sample = _data(case, seed)
    every = torch.arange(q.shape[0], device=q.device)
    found, w = [], None
    for part in parts:
        e = _Exact(case, part, q, ex)
        if case["call"] == "fixed":
            probes = e.search(e.n, every)
        elif case["call"] == "calibrated":
            smp = sample.to(torch.int64)
            w = e.window(smp)
            rest = torch.ones(q.shape[0], dtype=torch.bool, device=q.device)
            rest[smp] = False
            probes = torch.full_like(every, e.n)
            probes[rest] = e.search(w, every[rest])
        else:
            probes = e.search(case["W"], every)
        found.append((e.id, e.sc, probes))
    sc, at = torch.cat([f[1] for f in found], 1).topk(case["k"], dim=1)
    ids = torch.cat([f[0] for f in found], 1).gather(1, at)
    probes = sum(f[2] for f in found).to(torch.int32)
    return (ids, sc, probes) if w is None else (ids, sc, probes, w)
