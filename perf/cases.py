"""The searches that this library's speed is measured on.

Learned-sparse retrieval as a program uses it: an index resident on the GPU, queries arriving one at a
time, a few at a time or in batches, exact top-k per query. Collections and queries are synthetic, of the
shape of SPLADE passages: 30,522 terms, Zipf (s = 1.1) term frequencies, about 120 terms per document and
30 per query (or long-tailed), weights log1p(lognormal(0, 0.8)) capped at 3. Everything is drawn on the GPU
from the seed; the index is built from host arrays, as gs_build_index takes them.
"""
import functools
import math
import types

import numpy as np
import torch

VOCAB = 30522
DOC_TERMS = 120.0
MAX_QUERY_TERMS = 250


def listed():
    return [
        # one query against a small collection, results for a page: all latency and launches
        {"name": "point-10k-u8", "entry": "search", "precision": "u8", "docs": 10_000, "queries": 1, "law": "plain",
         "k": 10, "kernel": "auto"},
        # a handful of queries on a small collection
        {"name": "tiny-10k-fp32", "entry": "search", "precision": "fp32", "docs": 10_000, "queries": 8, "law": "plain",
         "k": 100, "kernel": "auto"},
        # a captured search replayed (a launch-bound serving loop)
        {"name": "graph-100k-fp32", "entry": "graph", "precision": "fp32", "docs": 100_003, "queries": 16,
         "law": "plain", "k": 100, "kernel": "auto"},
        # queries in host memory, one synchronous call (scripts, evaluation)
        {"name": "host-200k-bf16", "entry": "host", "precision": "bf16", "docs": 200_000, "queries": 4, "law": "plain",
         "k": 1000, "kernel": "auto"},
        # one step of a serving loop: a reserved batch refilled with mixed-length queries and mixed k, then searched
        {"name": "step-300k-u8", "entry": "update", "precision": "u8", "docs": 299_999, "queries": 64, "law": "tailed",
         "k": 0, "kernel": "auto"},
        # the request loop itself: a burst of requests submitted and waited for
        {"name": "server-300k-u8", "entry": "server", "precision": "u8", "docs": 300_000, "queries": 128,
         "law": "tailed", "k": 100, "kernel": "auto"},
        # one query against a large collection, deep results for a re-ranker
        {"name": "single-4m-fp32", "entry": "search", "precision": "fp32", "docs": 4_000_000, "queries": 1,
         "law": "plain", "k": 1000, "kernel": "auto"},
        # keyword-like queries of one to four terms, many with fewer matches than k
        {"name": "short-262k-fp32", "entry": "search", "precision": "fp32", "docs": 262_147, "queries": 48,
         "law": "short", "k": 1000, "kernel": "auto"},
        # offline batches: 500 queries, top-1000
        {"name": "batch-1m-fp32", "entry": "search", "precision": "fp32", "docs": 1_000_000, "queries": 500,
         "law": "plain", "k": 1000, "kernel": "auto"},
        {"name": "batch-500k-bf16", "entry": "search", "precision": "bf16", "docs": 500_000, "queries": 500,
         "law": "plain", "k": 1000, "kernel": "auto"},
        # the per-query kernel chosen by the caller, on a collection well past the caches
        {"name": "perquery-2m-fp32", "entry": "search", "precision": "fp32", "docs": 2_000_000, "queries": 100,
         "law": "plain", "k": 1000, "kernel": "tiled"},
        # a large uneven batch (query lengths long-tailed, k of 10, 100 and 1000 mixed)
        {"name": "uneven-250k-u8", "entry": "search", "precision": "u8", "docs": 250_000, "queries": 4096,
         "law": "tailed", "k": 0, "kernel": "auto"},
    ]


def draw(rng):
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    docs = spread(5_000, 4_000_000)
    entry = rng.choice(["search", "search", "search", "update", "host", "graph", "noalloc", "server"])
    queries = spread(1, 500)
    if entry in ("update", "graph", "host", "server"):
        queries = spread(1, 128)
    queries = min(queries, 500_000_000 // docs)
    return {"entry": entry, "precision": rng.choice(["fp32", "bf16", "u8"]), "docs": docs, "queries": queries,
            "law": rng.choice(["plain", "plain", "tailed", "short"]),
            "k": rng.choice([10, 100, 1000, rng.randint(1, 2000)] if entry == "server" else
                            [0, 10, 100, 1000, rng.randint(1, 4096)]),
            "kernel": rng.choice(["auto", "auto", "tiled", "shared"])}


# ------------------------------------------------------------------ inputs --


@functools.lru_cache(maxsize=None)
def _zipf():
    p = np.arange(1, VOCAB + 1, dtype=np.float64) ** -1.1
    return p / p.sum()


@functools.lru_cache(maxsize=None)
def _draw_table():
    """Mean distinct terms of a row for a Poisson number of draws with replacement, over a grid of that mean."""
    lam = np.exp(np.linspace(math.log(0.5), math.log(4000.0), 200))
    p = _zipf()
    return lam, np.array([-np.expm1(-x * p).sum() for x in lam])


def _draws_for(distinct):
    lam, mean = _draw_table()
    return np.interp(distinct, mean, lam)


def _rows(n, draws, gen, perm, cdf, most):
    """CSR rows of distinct terms (ascending), weights of the same law. draws: mean draws per row (number or tensor)."""
    dev = torch.device("cuda")
    ptr, terms = [torch.zeros(1, dtype=torch.int64, device=dev)], []
    step, at = 131072, 0
    for a in range(0, n, step):
        b = min(n, a + step)
        lam = draws[a:b] if torch.is_tensor(draws) else torch.full((b - a,), float(draws), device=dev, dtype=torch.float32)
        cnt = torch.poisson(lam.float(), generator=gen).long().clamp_(min=1)
        row = torch.repeat_interleave(torch.arange(b - a, device=dev), cnt)
        u = torch.rand(row.numel(), generator=gen, device=dev, dtype=torch.float64)
        t = perm[torch.searchsorted(cdf, u).clamp_(max=VOCAB - 1)]
        key = torch.unique_consecutive(torch.sort(row * VOCAB + t)[0])
        row, t = key // VOCAB, key % VOCAB
        n_row = torch.bincount(row, minlength=b - a)
        start = torch.cumsum(n_row, 0) - n_row
        keep = torch.arange(key.numel(), device=dev) - start[row] < most
        terms.append(t[keep].int())
        ptr.append(torch.cumsum(n_row.clamp(max=most), 0) + at)
        at = int(ptr[-1][-1])
    ptr, terms = torch.cat(ptr), torch.cat(terms)
    z = torch.randn(terms.numel(), generator=gen, device=dev)
    w = torch.log1p(torch.exp(0.8 * z)).clamp_(max=3.0)
    return ptr, terms, w


def _inputs(case, seed):
    """(document rows, query rows, k per query) on the GPU."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(1_000_003 * seed + 17)
    perm = torch.randperm(VOCAB, generator=gen, device=dev)
    cdf = torch.cumsum(torch.as_tensor(_zipf(), device=dev), 0)
    docs = _rows(case["docs"], _draws_for(DOC_TERMS), gen, perm, cdf, VOCAB)
    n = case["queries"]
    if case["law"] == "tailed":
        z = torch.randn(n, generator=gen, device=dev, dtype=torch.float64).cpu().numpy()
        want = np.clip(25.0 * np.exp(0.8 * z), 5, 220)
    elif case["law"] == "short":
        want = 1.0 + torch.randint(0, 4, (n,), generator=gen, device=dev).cpu().numpy()
        # keywords are not the commonest words: flatter term frequencies
        cdf = torch.cumsum(torch.as_tensor(_short_law(), device=dev), 0)
    else:
        want = np.full(n, 30.0)
    lam = want if case["law"] == "short" else _draws_for(want)
    queries = _rows(n, torch.as_tensor(lam, device=dev), gen, perm, cdf, MAX_QUERY_TERMS)
    if case["k"]:
        k = np.full(n, case["k"], dtype=np.int32)
    else:
        pick = torch.randint(0, 3, (n,), generator=gen, device=dev).cpu().numpy()
        k = np.array([10, 100, 1000], dtype=np.int32)[pick]
        k[0] = 1000
    return docs, queries, k


@functools.lru_cache(maxsize=None)
def _short_law():
    p = _zipf() ** 0.6
    return p / p.sum()


def _host(rows):
    ptr, terms, w = rows
    return types.SimpleNamespace(row_ptr=ptr.cpu().numpy(), terms=terms.cpu().numpy(), weights=w.cpu().numpy(),
                                 vocab=VOCAB)


# -------------------------------------------------------------------- runs --


def prepare(case, seed):
    import paper_2606_26441_amd as gs

    docs, queries, k = _inputs(case, seed)
    s = types.SimpleNamespace(entry=case["entry"], queries=_host(queries), k=k, n=case["queries"])
    s.index = gs.Index.from_rows(_host(docs), case["precision"])
    s.opts = gs.make_opts(kernel=case["kernel"])
    k_max = int(k.max())
    if s.entry == "server":
        s.server = gs.Server(s.index, max_batch=64, n_slots=4, k_max=k_max, opts=s.opts)
        s.parts = [(s.queries.terms[a:b], s.queries.weights[a:b])
                   for a, b in zip(s.queries.row_ptr[:-1], s.queries.row_ptr[1:])]
        return s
    if s.entry == "update":
        s.batch = gs.Batch.reserve(s.index, s.n, s.n * gs.GS_MAX_QUERY_NNZ, k_max)
    elif s.entry != "host":
        s.batch = s.index.batch(s.queries, k)
    if s.entry != "noalloc":
        s.workspace = s.index.workspace(s.n, s.opts)
    if s.entry != "host":
        s.out = (torch.empty((s.n, k_max), dtype=torch.int32, device="cuda"),
                 torch.empty((s.n, k_max), dtype=gs.SCORE_DTYPES[s.index.precision], device="cuda"))
    if s.entry == "graph":
        s.graph = gs.Graph(s.index, s.batch, s.workspace, s.out[0], s.out[1], s.opts)
    return s


def run(s):
    if s.entry == "search":
        ids, scores = s.index.search(s.batch, s.workspace, s.opts, out=s.out)
    elif s.entry == "update":
        s.batch.update(s.queries, s.k)
        ids, scores = s.index.search(s.batch, s.workspace, s.opts, out=s.out)
    elif s.entry == "host":
        ids, scores = s.index.search_host(s.queries, s.k, workspace=s.workspace, opts=s.opts)
    elif s.entry == "graph":
        s.graph.launch()
        ids, scores = s.out
    elif s.entry == "noalloc":
        ids, scores = s.index.search_noalloc(s.batch, s.out, s.opts)
    else:
        k = int(s.k[0])
        tickets = [s.server.submit(t, w, k) for t, w in s.parts]
        got = [s.server.wait(t, k) for t in tickets]
        ids, scores = np.stack([g[0] for g in got]), np.stack([g[1] for g in got])
    return {"ids": ids, "scores": scores}


def work(case):
    """Postings of the batch's terms read once (the weight and a byte for the gap to the next document), the queries
    read and the results written; one multiply-add per (query, posting of its terms)."""
    p = _zipf()
    n, b = case["docs"], case["queries"]
    in_doc = -np.expm1(-_draws_for(DOC_TERMS) * p)
    if case["law"] == "short":
        terms = 2.5
        in_query = -np.expm1(-terms * _short_law())
    else:
        terms = 30.0 if case["law"] == "plain" else 25.0 * math.exp(0.32)
        in_query = -np.expm1(-_draws_for(terms) * p)
    in_batch = -np.expm1(b * np.log1p(-np.minimum(in_query, 1 - 1e-12)))
    weight = {"fp32": 4, "bf16": 2, "u8": 1}[case["precision"]]
    score = {"fp32": 4, "bf16": 8, "u8": 4}[case["precision"]]
    k = min(case["k"] or 370, n)
    return {"bytes": n * float((in_doc * in_batch).sum()) * (1 + weight) + b * (8 * terms + (4 + score) * k),
            "flops": 2.0 * b * n * float((in_doc * in_query).sum())}


# ------------------------------------------------------------------- exact --


def exact(case, seed):
    """Scores of the k best documents per query in float64 (u8: integer impacts); ids have no such value."""
    (ptr, terms, w), (qptr, qterms, qw), k = _inputs(case, seed)
    dev, n = terms.device, case["docs"]
    impacts = case["precision"] == "u8"

    def value(x):
        x = x.double()
        return torch.round(x * 85.0).clamp(0, 255) if impacts else x

    doc = torch.repeat_interleave(torch.arange(n, device=dev), ptr[1:] - ptr[:-1])
    order = torch.argsort(terms, stable=True)  # term-major
    doc, w = doc[order], value(w[order])
    at = torch.searchsorted(terms[order].contiguous(), torch.arange(VOCAB + 1, device=dev, dtype=terms.dtype)).tolist()
    qptr, qterms, qw = qptr.tolist(), qterms.tolist(), value(qw).tolist()
    k_max = int(k.max())
    scores = torch.zeros((case["queries"], k_max), dtype=torch.float64, device=dev)
    row = torch.zeros(n, dtype=torch.float64, device=dev)
    for q in range(case["queries"]):
        row.zero_()
        for t, x in zip(qterms[qptr[q]:qptr[q + 1]], qw[qptr[q]:qptr[q + 1]]):
            d = doc[at[t]:at[t + 1]]  # a document holds a term once
            row[d] += x * w[at[t]:at[t + 1]]
        kq = min(int(k[q]), n)
        scores[q, :kq] = torch.topk(row, kq)[0]
    return {"ids": None, "scores": scores.long() if impacts else scores}
