"""k-th scores far below the largest possible one, against the oracle.

One heavy term, held by fewer than k documents, and light terms held by many: the k-th score
is about a thousandth to a ten-thousandth of the largest possible, and more documents than
the candidate buffer holds (32,768) have a positive score. A few documents hold the terms with
tiny weights, so that every query has a wide-range limit, below its k-th score.
"""
import numpy as np
import pytest

from helpers import csr
from parity_rules import check_batch
from workload import SparseRows

pytestmark = pytest.mark.gpu

N, TERMS = 270_000, 11


def _gs():
    import torch
    assert torch.cuda.is_available(), "GPU test run without a GPU"
    import paper_2606_26441_amd as gs
    return gs, torch


@pytest.fixture(scope="module")
def docs():
    rng = np.random.default_rng(4)
    doc, term, w = [rng.choice(N, 500, replace=False)], [np.zeros(500, int)], [np.full(500, 3.0)]
    for t in range(1, TERMS):
        d = np.flatnonzero(rng.random(N) < (0.30 if t < 6 else 0.1))
        x = 0.1 + 0.4 * rng.random(len(d))
        x[:5] = 1e-7
        doc.append(d)
        term.append(np.full(len(d), t))
        w.append(x)
    doc, term, w = np.concatenate(doc), np.concatenate(term), np.concatenate(w)
    order = np.lexsort((term, doc))
    rp = np.zeros(N + 1, np.int64)
    np.cumsum(np.bincount(doc, minlength=N), out=rp[1:])
    return SparseRows(rp, term[order].astype(np.int32), w[order].astype(np.float32), TERMS)


def _queries(n, light):
    rng = np.random.default_rng(n)
    return csr([[(0, 3.0)] + [(t, float(light * (1.0 + rng.random()))) for t in range(1, TERMS) if rng.random() < 0.8]
                for _ in range(n)], TERMS)


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("kernel", ["tiled", "group", "atomic"])
@pytest.mark.parametrize("n_queries,light", [(3, 3e-3), (40, 3e-3), (40, 1e-3)])
def test_low_scores_need_no_fp64_pass(docs, precision, kernel, n_queries, light):
    gs, torch = _gs()
    qs = _queries(n_queries, light)
    idx = gs.Index.from_rows(docs, precision, keep_doc_ids=kernel == "atomic")
    b = idx.batch(qs, 1000)
    ids, sc = idx.search(b, idx.workspace(qs.n_rows), gs.make_opts(kernel))
    torch.cuda.synchronize()
    d = b.diagnostics()
    check_batch(precision, docs, qs, ids.cpu().numpy(), sc.cpu().numpy(), 1000, what="%s %s" % (precision, kernel))
    assert np.all(d[:, 4] != 2), "%d queries were summed in fp64 without need" % np.sum(d[:, 4] == 2)
    b.close()
    idx.close()
