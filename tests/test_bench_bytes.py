"""The bytes that bench.py counts for terms with rows (CPU only)."""
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402
from workload import SparseRows  # noqa: E402


@pytest.mark.parametrize("wbytes", [1, 2, 4])
def test_layout_bytes_with_rows(wbytes):
    # terms: a row at exactly a quarter of the documents, one short of it, empty, every document with a
    # row, every document without one (an index that had no room for it)
    n = 400
    df = np.array([100, 99, 0, 400, 400], np.int64)
    row = np.array([1, 0, 0, 1, 0], np.uint8)
    q = SparseRows(np.array([0, 5, 6], np.int64), np.array([0, 1, 2, 3, 4, 3], np.int32), np.ones(6, np.float32), 5)
    idb = bench.row_id_bytes(df, n, wbytes, row)
    p_q, score, _ = bench.algorithmic_bytes(df, q, n, wbytes, idb, written_docs=0)
    assert list(p_q) == [999, 400]
    assert score == 3 * n * wbytes + (99 + 400) * (2 + wbytes)  # three row reads, two lists, no rows of scores
