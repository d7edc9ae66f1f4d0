"""Synchronous searches from host memory: the batches an index keeps for them.

Calls of different sizes, k and options one after another and from several threads and
streams at once must each give what a prepared batch gives, also after a call that was
refused, and past the sizes that are kept or uploaded in one launch.
"""
import threading

import numpy as np
import pytest

import workload

pytestmark = pytest.mark.gpu


def _gs():
    import torch
    assert torch.cuda.is_available(), "GPU test run without a GPU"
    import paper_2606_26441_amd as gs
    return gs, torch


@pytest.fixture(scope="module")
def docs():
    return workload.collection(40_000, seed=91)


def _prepared(gs, torch, idx, qs, k, k_max):
    b = idx.batch(qs, k, k_max)
    ids, sc = idx.search(b, idx.workspace(max(qs.n_rows, 1)))
    torch.cuda.synchronize()
    b.close()
    return ids.cpu().numpy(), sc.cpu().numpy()


@pytest.mark.parametrize("precision", ["fp32", "u8", "bf16"])
def test_calls_of_many_sizes(docs, precision):
    gs, torch = _gs()
    idx = gs.Index.from_rows(docs, precision)
    for n, k in ((1, 10), (40, 100), (3, 1000), (1, 10), (700, 5), (6000, 7), (2, 4096), (40, 100)):
        qs = workload.queries_lognormal(n, seed=100 + n)
        want = _prepared(gs, torch, idx, qs, k, k)
        got = idx.search_host(qs, k)
        assert np.array_equal(got[0].cpu().numpy(), want[0]) and np.array_equal(got[1].cpu().numpy(), want[1]), (n, k)
        bad = workload.SparseRows(qs.row_ptr, np.full_like(qs.terms, -1), qs.weights, qs.vocab)
        with pytest.raises(gs.GsError) as e:
            idx.search_host(bad, k)
        assert e.value.code == gs.GS_EINVAL
    idx.close()


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_calls_from_threads_and_streams(docs, precision):
    gs, torch = _gs()
    idx = gs.Index.from_rows(docs, precision)
    jobs = [(n, k, workload.queries_poisson(n, seed=200 + n)) for n, k in ((1, 50), (4, 10), (9, 300), (33, 100), (64, 20), (2, 700))]
    want = [_prepared(gs, torch, idx, qs, k, k) for n, k, qs in jobs]
    errors = []

    def work(i):
        try:
            torch.cuda.set_device(0)
            stream = torch.cuda.Stream()
            n, k, qs = jobs[i]
            with torch.cuda.stream(stream):
                for _ in range(15):
                    ids, sc = idx.search_host(qs, k, stream=stream)
                    assert np.array_equal(ids.cpu().numpy(), want[i][0]) and np.array_equal(sc.cpu().numpy(), want[i][1])
        except Exception as e:  # reported below
            errors.append((i, repr(e)))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    idx.close()
