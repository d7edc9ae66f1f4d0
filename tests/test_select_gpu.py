"""Selection kernels at the sizes where their paths change, against the oracle.

Collections around the candidate buffer (32,768 documents: up to it the score row itself
is the candidate set), k from 1 to the largest, queries that fewer than k documents match
(the answer then holds zero-score documents in id order), rows where every document ties,
bands of the bf16 form past what its ranking kernel holds in LDS, and batches with enough
queries for fused candidate filtering.
"""
import numpy as np
import pytest

from helpers import csr, dyadic, random_rows
from parity_rules import check_batch

pytestmark = pytest.mark.gpu


def _gs():
    import torch
    assert torch.cuda.is_available(), "GPU test run without a GPU"
    import paper_2606_26441_amd as gs
    return gs, torch


def _docs(n, seed, ties):
    rng = np.random.default_rng(seed)
    one = (lambda r, m: np.ones(m)) if ties else dyadic
    base = random_rows(rng, 2048, 80, 0, 5, weight_fn=one)
    pick = rng.integers(0, 2048, n)
    return base.subset(pick)


def _queries(n, seed, ties):
    # every third query has one term; term 79 is the rarest kind here (a few documents in a thousand)
    rng = np.random.default_rng(seed)
    one = (lambda r, m: np.ones(m)) if ties else dyadic
    rows = [random_rows(rng, 1, 80, 1, 1 if q % 3 == 0 else 6, weight_fn=one) for q in range(n)]
    return csr([list(zip(r.terms.tolist(), r.weights.tolist())) for r in rows], 80)


@pytest.mark.parametrize("precision", ["fp32", "u8", "bf16"])
@pytest.mark.parametrize("n_docs", [1, 63, 32_767, 32_768, 32_769, 140_001])
@pytest.mark.parametrize("n_queries,k", [(1, 1), (5, 1000), (33, 4096)])
@pytest.mark.parametrize("ties", [False, True])
def test_selection_edges(precision, n_docs, n_queries, k, ties):
    gs, torch = _gs()
    docs, qs = _docs(n_docs, 7 + n_docs, ties), _queries(n_queries, 11 + n_queries, ties)
    idx = gs.Index.from_rows(docs, precision)
    ks = np.where(np.arange(n_queries) % 4 == 3, np.minimum(k, 10), k).astype(np.int32)
    b = idx.batch(qs, ks, k_max=k)
    ids, sc = idx.search(b, idx.workspace(n_queries))
    torch.cuda.synchronize()
    ids, sc, over = ids.cpu().numpy(), sc.cpu().numpy(), b.diagnostics()[:, 3] != 0
    # massive ties may put more documents than its buffer holds into the bf16 band: flagged, not wrong
    assert not over.any() or (precision == "bf16" and ties and n_docs > 32_768)
    keep = np.flatnonzero(~over)
    check_batch(precision, docs, qs.subset(keep), ids[keep], sc[keep], ks[keep],
                what="%s N=%d nq=%d k=%d" % (precision, n_docs, n_queries, k))


@pytest.mark.parametrize("precision", ["fp32", "u8", "bf16"])
@pytest.mark.parametrize("n_queries", [2, 40])
def test_fewer_matches_than_k(precision, n_queries):
    # one term per query, held by 0, 1, 700 or 40,000 documents (the last past the appended
    # candidates' cap): the rest of the answer is the lowest ids without it
    gs, torch = _gs()
    n = 150_000
    rows = [[] for _ in range(n)]
    rng = np.random.default_rng(5)
    for t, m in ((0, 0), (1, 1), (2, 700), (3, 40_000)):
        for d in rng.choice(n, size=m, replace=False):
            rows[int(d)].append((t, float(rng.integers(1, 49)) / 16.0))
    docs = csr(rows, 5)
    qs = csr([[((q % 4 + 2) % 4, 1.5)] for q in range(n_queries)], 5)
    idx = gs.Index.from_rows(docs, precision)
    b = idx.batch(qs, 1000)
    ids, sc = idx.search(b, idx.workspace(n_queries))
    torch.cuda.synchronize()
    check_batch(precision, docs, qs, ids.cpu().numpy(), sc.cpu().numpy(), 1000, what="few matches " + precision)
