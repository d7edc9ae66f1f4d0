"""Forward rows with 2-byte and 4-byte term ids, against the oracle.

Up to 65,536 terms the forward rows keep 2-byte ids, above that 4-byte ones. bf16 scores are
summed again from these rows in fp64; the document-parallel kernel reads them for every score
(its table holds at most 40,960 terms).
"""
import numpy as np
import pytest

from helpers import csr, dyadic
from parity_rules import check_batch

pytestmark = pytest.mark.gpu


def _gs():
    import torch
    assert torch.cuda.is_available(), "GPU test run without a GPU"
    import paper_2606_26441_amd as gs
    return gs, torch


def _rows(rng, n, vocab, most):
    """Rows with terms around 65,535 and at both ends of the vocabulary, and empty ones."""
    edge = np.unique([t for t in (0, 1, 32767, 32768, 65534, 65535, 65536, vocab - 1) if t < vocab])
    out = []
    for i in range(n):
        if i % 17 == 3:
            out.append([])
            continue
        t = np.union1d(rng.choice(vocab, size=int(rng.integers(1, most)), replace=False),
                       rng.choice(edge, size=int(rng.integers(1, edge.size + 1)), replace=False))
        out.append(list(zip(t.tolist(), dyadic(rng, t.size).tolist())))
    return csr(out, vocab)


@pytest.mark.parametrize("precision,kernel,vocab", [
    ("bf16", "tiled", 40_960), ("bf16", "tiled", 65_536), ("bf16", "tiled", 65_537), ("bf16", "tiled", 131_073),
    ("bf16", "docpar", 40_960), ("fp32", "docpar", 40_960), ("u8", "docpar", 40_960)])
def test_term_id_widths(precision, kernel, vocab):
    gs, torch = _gs()
    rng = np.random.default_rng(vocab)
    docs, qs = _rows(rng, 3_000, vocab, 300), _rows(rng, 40, vocab, 200)
    idx = gs.Index.from_rows(docs, precision, keep_forward=True)
    opts = gs.make_opts(kernel)
    b = idx.batch(qs, 100)
    ids, sc = idx.search(b, idx.workspace(qs.n_rows, opts), opts)
    torch.cuda.synchronize()
    check_batch(precision, docs, qs, ids.cpu().numpy(), sc.cpu().numpy(), 100,
                what="%s %s vocabulary %d" % (precision, kernel, vocab))
    b.close()
    idx.close()
