"""Insertion of large batches through bins of rows: from 2^21 half-edges on, half-edges of a batch that is on the device as a
whole are put together by bins of rows before they are counted and written.  The same batch sent in chunks
(dynlp_options.ingest_chunk_edges) takes an atomic per half-edge instead; appended entries are sorted either way, so that graph
and labels agree bit for bit."""
import numpy as np
import pytest

import paper_2604_06596_amd as P
from test_gpu_allocator import TorchAllocator

pytestmark = pytest.mark.gpu


def _edges(rng, m, lo, hi, n, hub=None):
    """m edges from [lo, hi) to anywhere below n, weights of few values (equal entries of a row too); `hub`: every 300th ends there."""
    u = rng.integers(lo, hi, m).astype(np.int32)
    v = rng.integers(0, n, m).astype(np.int32)
    if hub is not None:
        v[::300] = hub
    v = np.where(u == v, (v + 1) % n, v).astype(np.int32)
    return u, v, rng.integers(1, 9, m).astype(np.float32) / np.float32(8)


def _batches(n, extra, m, seed):
    """Two batches: all of the graph, then new vertices whose edges meet rows that have entries (and slack) already."""
    rng = np.random.default_rng(seed)
    first = _edges(rng, m, 0, n, n, hub=n // 2)
    second = _edges(rng, max(m // 2, (1 << 20) + 5), n if extra else 0, n + extra, n + extra)
    sv = np.arange(0, n, 97, dtype=np.int32)
    return first, second, sv, (sv % 2).astype(np.int32)


def _run(n, extra, first, second, sv, sc, rounds, delete=(), bad=None, **options):
    none = np.zeros(0, np.int32)
    with P.DynLP(0, np.zeros(1, np.int64), none, np.zeros(0, np.float32), 2, none, none, binary_scalar=True, **options) as d:
        d.set_params(1e-6, rounds)
        st = [d.apply_batch(n, *first, sv, sc)[0]]
        if bad is not None:
            worse = tuple(x.copy() for x in second)
            worse[1][bad] = n + extra
            with pytest.raises(P.DynLPError) as ei:
                d.apply_batch(extra, *worse, none, none)
            assert str(bad) in ei.value.message
        st.append(d.apply_update(np.asarray(delete, np.int32), extra, *second, none, none)[0])
        soft, hard = d.get_labels()
        return st, soft, hard, d.export_graph()


# rows: fewer than a bin holds (one bin of many slices), a ragged last bin, a last bin of one row, more bins (of 2^12 rows)
@pytest.mark.parametrize("n,extra", [(1500, 0), (300_001, 700), ((1 << 20) + 1, 2048), (2_200_000, 100_003)])
def test_bins_and_atomics_give_the_same_graph_and_labels(n, extra):
    m = (1 << 20) + 4099
    parts = _batches(n, extra, m, 7 + n)
    a = _run(n, extra, *parts, 3, ingest_chunk_edges=1 << 28)
    b = _run(n, extra, *parts, 3, ingest_chunk_edges=(1 << 20) + 1)
    assert a[0] == b[0]
    for x, y in zip((a[1], a[2], *a[3]), (b[1], b[2], *b[3])):
        assert np.array_equal(x, y)


def test_a_refused_batch_leaves_no_count_behind():
    n, extra, m = 300_001, 700, (1 << 20) + 4099
    parts = _batches(n, extra, m, 3)
    a = _run(n, extra, *parts, 2, bad=m // 2 - 5, ingest_chunk_edges=1 << 28)
    b = _run(n, extra, *parts, 2, ingest_chunk_edges=(1 << 20) + 1)
    for x, y in zip((a[1], a[2], *a[3]), (b[1], b[2], *b[3])):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("without", ["bins", "bins when the pool grows"])
def test_without_memory_for_the_bins_the_insertion_takes_atomics(without):
    n, extra, m = 300_001, 700, (1 << 20) + 4099
    parts = _batches(n, extra, m, 11)
    used = np.concatenate([parts[1][0], parts[1][1]])
    gone = np.setdiff1d(np.arange(n // 2 - 3000, n // 2 + 3000, dtype=np.int32), used)  # (no new edge may end at a deleted vertex)
    assert gone.size > 0
    runs = []
    for limited in (False, True):
        al = TorchAllocator()
        if limited and without == "bins":
            al.refuse = lambda nbytes: nbytes == 2 * m * 2 or nbytes == 2 * parts[1][0].shape[0] * 2
        elif limited:  # no pool beside the bins' arrays: three of the sizes that only they have
            al.refuse = lambda nbytes: nbytes > 16 * m and any(t.numel() == 4 * m for t in al.live.values())
        runs.append(_run(n, extra, *parts, 2, delete=gone, allocator=al, ingest_chunk_edges=1 << 28) + (al.refused, ))
        assert not al.live
    a, b = runs
    assert a[4] == 0 and b[4] > 0
    for x, y in zip((a[1], a[2], *a[3]), (b[1], b[2], *b[3])):
        assert np.array_equal(x, y)
