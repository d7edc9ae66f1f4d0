"""Searches captured by their caller (torch.cuda.graph) and replayed after refills of the batch.

The launches are captured while the batch holds ordinary queries and replayed after updates
with wide-range ones (scores many orders of magnitude below the query's largest product),
which need the fp64 pass. Every replay follows unrelated eager work and a synchronisation,
and is checked against the oracle.
"""
import numpy as np
import pytest

from helpers import csr
from parity_rules import check_batch

pytestmark = pytest.mark.gpu

A, B, C = 0, 1, 2


def _gs():
    import torch
    assert torch.cuda.is_available(), "GPU test run without a GPU"
    import paper_2606_26441_amd as gs
    return gs, torch


def _docs(n):
    rng = np.random.default_rng(n)
    rows = []
    for d in range(n):
        r = []
        if d % 200 == 0:
            r.append((A, float(rng.uniform(0.5, 3.0))))
        if d % 8 == 3:
            r.append((B, float(1e-5 * rng.uniform(0.5, 2.0))))
        if d % 13 == 5:
            r.append((C, float(1e-9 * rng.uniform(0.5, 2.0))))
        for t in rng.choice(np.arange(3, 12), size=int(rng.integers(0, 4)), replace=False):
            r.append((int(t), float(rng.uniform(0.2, 3.0))))
        rows.append(sorted(r))
    return csr(rows, 12)


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("n_docs", [20_000, 50_000])
@pytest.mark.parametrize("noalloc", [False, True])
def test_replays_after_a_refill_with_wide_range_queries(precision, n_docs, noalloc):
    gs, torch = _gs()
    docs = _docs(n_docs)
    ordinary = csr([[(3, 1.0), (5, 2.0)], [(4, 0.5)], [(7, 1.5), (8, 1.0), (9, 0.25)]], 12)
    # k above the documents of A: the k-th score is among the tiny ones
    wide = csr([[(A, 3.0), (B, 1e-5), (C, 1e-9)], [(4, 0.5)], [(A, 2.5), (C, 1e-9)]], 12)
    k = 1000
    idx = gs.Index.from_rows(docs, precision)
    batch = gs.Batch.reserve(idx, 3, max(ordinary.nnz, wide.nnz), k)
    ws = idx.workspace(3)
    ids = torch.empty((3, k), dtype=torch.int32, device="cuda")
    sc = torch.empty((3, k), dtype=gs.SCORE_DTYPES[idx.precision], device="cuda")

    def search():
        if noalloc:
            idx.search_noalloc(batch, (ids, sc))
        else:
            idx.search(batch, ws, out=(ids, sc))

    batch.update(ordinary, k)
    search()  # one-time set-up outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        search()
    scratch = torch.randn(256, 256, device="cuda")
    for rep, (name, qs) in enumerate([("wide", wide), ("ordinary", ordinary), ("wide", wide), ("wide", wide)]):
        scratch = scratch @ scratch.T / 256.0  # unrelated eager work between replays
        torch.cuda.synchronize()
        batch.update(qs, k)
        ids.fill_(-7)
        sc.zero_()
        graph.replay()
        torch.cuda.synchronize()
        check_batch(precision, docs, qs, ids.cpu().numpy(), sc.cpu().numpy(), k, what="replay %d (%s)" % (rep, name))
        d = batch.diagnostics()
        if name == "wide":
            assert d[0, 4] == 2 and d[2, 4] == 2, "replay %d: no fp64 pass" % rep
    del graph
    batch.close()
    idx.close()
