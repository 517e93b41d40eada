"""Batches of up to 2,048 half-edges and 128 deleted vertices go through Step 1 in launches of one workgroup.  The same batch takes the
ordinary launches where its deleted vertices are listed often enough (a vertex listed twice is deleted once) or, without any, where
its edges are sent in chunks.  Appended entries are sorted either way, so that graph and labels agree bit for bit."""
import numpy as np
import pytest
import torch

import paper_2604_06596_amd as P

pytestmark = pytest.mark.gpu

N, C = 3000, 5


def _base(seed):
    rng = np.random.default_rng(seed)
    m = 4 * N
    u = rng.integers(0, N, m).astype(np.int32)
    v = rng.integers(0, N, m).astype(np.int32)
    u[:400] = 17  # a row longer than 128 entries
    keep = u != v
    u, v = u[keep], v[keep]
    return u, v, rng.random(u.shape[0], dtype=np.float32) + np.float32(0.1)


def _batch(rng, m, nd, k, s):
    """Edges from new vertices (any vertex without them), some of them parallel and to a hub; deleted vertices are not used again."""
    gone = rng.permutation(np.arange(20, N, dtype=np.int32))[:nd]
    if nd > 1:
        gone[0] = 17
    old = np.setdiff1d(np.arange(N, dtype=np.int32), gone)
    u = rng.integers(N, N + k, m).astype(np.int32) if k else rng.choice(old[old >= 10], m).astype(np.int32)
    v = rng.choice(old, m).astype(np.int32)
    v[: m // 3] = old[3]
    v = np.where(u == v, old[4], v).astype(np.int32)
    w = rng.integers(1, 9, m).astype(np.float32) / np.float32(8)
    sv = np.union1d(u, v)
    sv = rng.permutation(sv[sv >= 100])[:s].astype(np.int32)
    return gone, u, v, w, sv, (sv % C).astype(np.int32)


def _run(device, ordinary, batches, k, reserve, bad=None):
    u, v, w = _base(1)
    labelled = np.arange(0, 10, dtype=np.int32)
    order = np.argsort(np.concatenate([u, v]), kind="stable")
    rp = np.concatenate([[0], np.cumsum(np.bincount(np.concatenate([u, v]), minlength=N))]).astype(np.int64)
    arrays = [rp, np.concatenate([v, u])[order], np.concatenate([w, w])[order]]

    def arg(x):
        return torch.as_tensor(x).cuda() if device else x

    with P.DynLP(N, *map(arg, arrays), C, arg(labelled), arg(labelled % C), device_ptrs=device, slack_factor=1.0,
                 ingest_chunk_edges=1 if ordinary else 1 << 20, **({"reserve_edges": 20000} if reserve else {})) as d:
        d.set_params(1e-6, 4)
        out = []
        for i, (gone, eu, ev, ew, sv, sc) in enumerate(batches):
            if ordinary and gone.size:
                gone = np.resize(gone, 129 + gone.size)
            a = [arg(x) for x in (eu, ev, ew, sv, sc)]
            if bad is not None and i == 0:
                which, value = bad
                wrong = [x.clone() if device else x.copy() for x in a]
                wrong[which][-1] = value
                with pytest.raises(P.DynLPError):
                    d.apply_update(arg(gone), k, *wrong)
            st, s = d.apply_update(arg(gone), k if i == 0 else 0, *a)
            out.append((st, s.frontier_initial, s.rows_updated, s.rows_relocated))
        soft, hard = d.get_labels()
        graph = d.export_graph()

        def host(x):
            return x.cpu().numpy() if torch.is_tensor(x) else x

        return out, [host(x) for x in (soft, hard, *graph)]


# half-edges: one edge, around a workgroup's threads, at the limit and beyond it; deleted rows: around the 64 that are taken at a time
# (without deleted vertices only a host batch can be sent in chunks)
_CASES = [(2, 0, 0, 0), (2, 1, 1, 1), (511, 63, 7, 40), (513, 64, 0, 40), (1023, 65, 900, 300), (1024, 127, 3, 0), (1024, 128, 1000, 1000),
          (1025, 128, 100, 5), (900, 0, 30, 20), (0, 5, 4, 0)]


@pytest.mark.parametrize("m,nd,k,s,device", [(*x, device) for x in _CASES for device in (False, True) if x[1] or not device])
def test_shared_and_ordinary_launches_give_the_same_graph_and_labels(m, nd, k, s, device):
    rng = np.random.default_rng(m + nd)
    batches = [_batch(rng, m, nd, k, s), _batch(rng, m, nd, 0, 0)]
    # without room in the pool both batches are planned before the pool is large enough for them
    a = _run(device, False, batches, k, reserve=True)
    for other in (_run(device, True, batches, k, reserve=True), _run(device, False, batches, k, reserve=False)):
        assert a[0] == other[0]
        for x, y in zip(a[1], other[1]):
            assert np.array_equal(x, y)


# (position of the argument, its last value): an end out of range, a weight, a seed's vertex, its class
@pytest.mark.parametrize("bad", [(1, N + 50), (2, -1.0), (3, -4), (4, C)])
def test_a_refused_batch_changes_nothing(bad):
    rng = np.random.default_rng(5)
    batches = [_batch(rng, 600, 70, 20, 30)]
    a = _run(True, False, batches, 20, reserve=True)
    b = _run(True, False, batches, 20, reserve=True, bad=bad)
    assert a[0] == b[0]
    for x, y in zip(a[1], b[1]):
        assert np.array_equal(x, y)
