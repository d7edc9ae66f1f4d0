"""Terms summed from rows, against the oracle.

A term held by at least a quarter of the documents has a row with its weight for every
document, which the doc-tiled kernel sums in registers; the other terms' postings are
scatter-added. Collections sit around the row threshold (N / 4 documents), the grain
(8,192) and the doc tiles, and queries hold only row terms, only posting terms, more row
terms than a wavefront has lanes, and zero weights.
"""
import numpy as np
import pytest

from helpers import csr, dyadic
from parity_rules import check_batch

pytestmark = pytest.mark.gpu

VOCAB = 300
COMMON = 100  # terms 0 .. 99 are held by at least a quarter of the documents, the others by fewer


def _gs():
    import torch
    assert torch.cuda.is_available(), "GPU test run without a GPU"
    import paper_2606_26441_amd as gs
    return gs, torch


def _docs(n):
    rng = np.random.default_rng(n)
    held = []
    for t in range(VOCAB):
        if t == 0:
            d = np.arange(n)                                       # every document
        elif t == 1:
            d = np.arange((n + 3) // 4)                            # exactly at the threshold
        elif t < COMMON:
            d = rng.choice(n, size=min(n, max((n + 3) // 4, n * (26 + t % 40) // 100)), replace=False)
        elif t == COMMON:
            d = np.arange(max((n + 3) // 4 - 1, 0))                # one short of it
        else:
            d = rng.choice(n, size=n * (t % 20) // 100, replace=False)
        held.append(np.sort(d))
    doc = np.concatenate(held)
    term = np.repeat(np.arange(VOCAB, dtype=np.int32), [len(d) for d in held])
    order = np.lexsort((term, doc))
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(doc, minlength=n), out=rp[1:])
    from workload import SparseRows
    return SparseRows(rp, term[order], dyadic(rng, len(order)).astype(np.float32), VOCAB)


def _queries():
    rng = np.random.default_rng(3)
    rows = [
        [(t, 0.5 + t / 64.0) for t in range(COMMON)],                   # 100 rows: more than 64
        [(t, 1.0) for t in range(200)],                                 # rows and postings past 64 terms
        [(t, 1.25) for t in range(COMMON, 180)],                        # postings only
        [(0, 2.0)], [(1, 2.0)], [(COMMON, 2.0)],                        # the threshold, either side
        [(0, 0.0), (2, 0.0), (150, 0.0)],                               # nothing weighs
        [(3, 0.0), (4, 1.0), (120, 0.0), (121, 1.0)],
        [],
    ]
    while len(rows) < 36:
        t = sorted(rng.choice(VOCAB, size=int(rng.integers(1, 40)), replace=False).tolist())
        rows.append([(int(x), float(rng.integers(1, 49)) / 16.0) for x in t])
    return csr(rows, VOCAB)


@pytest.mark.parametrize("precision", ["fp32", "u8", "bf16"])
@pytest.mark.parametrize("n_docs", [1, 5, 8_191, 8_193, 16_385, 41_000])
@pytest.mark.parametrize("tile_docs", [0, 8192, 16384, 32768])
def test_rows_and_postings(precision, n_docs, tile_docs):
    gs, torch = _gs()
    if precision == "fp32" and tile_docs == 32768:
        pytest.skip("no such tile for fp32")
    docs, qs = _docs(n_docs), _queries()
    idx = gs.Index.from_rows(docs, precision)
    for chunk in (64, 256, 512, 1024):
        opts = gs.make_opts("tiled", tile_docs=tile_docs, chunk=chunk)
        b = idx.batch(qs, 50, k_max=50)
        ids, sc = idx.search(b, idx.workspace(qs.n_rows, opts), opts)
        torch.cuda.synchronize()
        check_batch(precision, docs, qs, ids.cpu().numpy(), sc.cpu().numpy(), 50,
                    what="%s N=%d tile=%d chunk=%d" % (precision, n_docs, tile_docs, chunk))
        b.close()
    idx.close()


@pytest.mark.parametrize("precision", ["fp32", "u8", "bf16"])
def test_rows_match_the_group_kernel(precision):
    # the group kernel reads postings alone: the sums must agree bit for bit, by query tiles too
    gs, torch = _gs()
    docs, qs = _docs(150_001), _queries()
    idx = gs.Index.from_rows(docs, precision)
    got = []
    for kernel, tile in (("group", 0), ("tiled", 0), ("shared", 0), ("tiled", 7)):
        opts = gs.make_opts(kernel, query_tile=tile)
        b = idx.batch(qs, 300)
        ids, sc = idx.search(b, idx.workspace(qs.n_rows, opts), opts)
        torch.cuda.synchronize()
        got.append((ids.cpu().numpy(), sc.cpu().numpy()))
        b.close()
    for ids, sc in got[1:]:
        assert np.array_equal(ids, got[0][0]) and np.array_equal(sc, got[0][1])
    idx.close()


@pytest.mark.parametrize("precision", ["u8", "bf16"])
@pytest.mark.parametrize("n_docs,query_tile", [(114_688, 0), (114_689, 0), (114_689, 31), (114_689, 32)])
def test_tile_left_to_the_library(precision, n_docs, query_tile):
    # 36 queries x 7 tiles of 16,384 documents: 252 items; with 8 tiles 288, 248 and 256 (below 256
    # items the library halves the tile). Either tile gives the same ids and scores.
    gs, torch = _gs()
    docs, qs = _docs(n_docs), _queries()
    idx = gs.Index.from_rows(docs, precision)
    got = []
    for tile_docs in (0, 8192, 16384):
        opts = gs.make_opts("tiled", tile_docs=tile_docs, query_tile=query_tile)
        b = idx.batch(qs, 100)
        ids, sc = idx.search(b, idx.workspace(qs.n_rows, opts), opts)
        torch.cuda.synchronize()
        got.append((ids.cpu().numpy(), sc.cpu().numpy()))
        b.close()
    for ids, sc in got[1:]:
        assert np.array_equal(ids, got[0][0]) and np.array_equal(sc, got[0][1])
    idx.close()


@pytest.mark.parametrize("precision", ["fp32", "u8", "bf16"])
def test_rows_of_a_tiny_collection_stay_small(precision):
    # 3 documents of 3,000 terms each, none shared: a row of whole grains for each term would take
    # 74 to 295 MB
    gs, torch = _gs()
    rng = np.random.default_rng(5)
    vocab = 9_000
    rows = [[(t, float(rng.integers(1, 49)) / 16.0) for t in range(d, vocab, 3)] for d in range(3)]
    docs = csr(rows, vocab)
    qs = csr([[(t, 1.0) for t in range(0, vocab, 40)], [(vocab - 1, 2.0)], [(0, 1.0), (8_500, 1.0)]], vocab)
    idx = gs.Index.from_rows(docs, precision)
    assert idx.info().device_bytes < (64 << 20) + 16 * idx.info().padded_nnz
    b = idx.batch(qs, 3)
    ids, sc = idx.search(b, idx.workspace(qs.n_rows))
    torch.cuda.synchronize()
    check_batch(precision, docs, qs, ids.cpu().numpy(), sc.cpu().numpy(), 3, what="3 documents " + precision)
    b.close()
    idx.close()
