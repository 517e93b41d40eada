"""GPU tests of a batch whose steps are queued without waiting for its checks or for the plan of its relocations: a pool that
turns out too small (the steps that insert run again after it has grown, the deletions do not), an argument that turns out
invalid on the device (nothing has changed, deletions included), and rows of more than 1,024 entries, which whole workgroups
handle, on either side of that length."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import reference as R
import paper_2604_06596_amd as P
from test_gpu_deletions import _check_graph, _make

pytestmark = pytest.mark.gpu

TOL = 1e-6


def _graph(p):
    return R.Graph(p.n, p.row_ptr, p.col, p.w, p.C, p.seed_vertex, p.seed_class)


@pytest.mark.parametrize("dead", [0, 40])
@pytest.mark.parametrize("rounds", [1, 3])
def test_a_pool_that_is_too_small_for_the_plan(dead, rounds):
    """slack 1.01 and batches of as many edges as the graph holds: every batch moves nearly every row."""
    rng = np.random.default_rng(3)
    p = W.small_random(3000, 5, 40.0, 150, 901)
    g = _graph(p)
    with _make(p, slack_factor=1.01) as d:
        assert d.static_solve(TOL, 20000)[0] == 0
        cap = d.storage_info()[1]
        for t in range(rounds):
            gone = rng.choice(p.n, dead, replace=False).astype(np.int32)
            m = 90000 * (t + 1)
            eu, ev = rng.integers(0, p.n + 10, m).astype(np.int32), rng.integers(0, p.n + 10, m).astype(np.int32)
            keep = (eu != ev) & (eu < g.n + 10) & (ev < g.n + 10)
            eu, ev = eu[keep], ev[keep]
            ew = rng.uniform(0.1, 1, eu.size).astype(np.float32)
            sv = np.array([g.n + 3], np.int32)
            st, s = d.apply_update(gone, 10, eu, ev, ew, sv, np.array([4], np.int32))
            assert st == 0 and s.rows_relocated > 0
            g.delete(gone)
            g.insert(10, eu, ev, ew, sv, np.array([4], np.int32))
            _check_graph(d, g, ordered=False)
        assert d.storage_info()[1] > cap, "the case is meant to outgrow the pool"
        soft, _ = d.get_labels()
        assert soft[sv[0], 4] == 1.0 and np.max(np.abs(soft.sum(1) - 1)) < 2e-5


@pytest.mark.parametrize("wrong", ["edge", "weight", "seed", "deleted", "conflict"])
def test_an_invalid_argument_found_on_the_device_changes_nothing(wrong):
    """Arrays on the GPU are only checked there, after the deletions have been queued."""
    p = W.small_random(2000, 3, 8.0, 100, 902)
    cu = lambda a, t: torch.as_tensor(np.asarray(a, t), device="cuda")
    arrays = dict(row_ptr=cu(p.row_ptr, np.int64), col=cu(p.col, np.int32), w=cu(p.w, np.float32),
                  sv=cu(p.seed_vertex, np.int32), sc=cu(p.seed_class, np.int32))
    free = np.setdiff1d(np.arange(p.n), p.seed_vertex)
    dead, seeds = list(free[:20]), [int(free[30]), int(free[31])]
    classes, eu, ev, ew = [0, 1], list(free[40:60]), list(free[60:80]), [0.5] * 20
    good = (list(dead), list(eu), list(ev), list(ew), list(seeds), list(classes))
    if wrong == "edge":
        eu[7] = p.n
    elif wrong == "weight":
        ew[3] = -1.0
    elif wrong == "seed":
        seeds[1] = -5
    elif wrong == "deleted":
        dead[19] = p.n
    else:
        seeds[1] = seeds[0]
    pack = lambda q: (cu(q[0], np.int32), 0, cu(q[1], np.int32), cu(q[2], np.int32), cu(q[3], np.float32), cu(q[4], np.int32), cu(q[5], np.int32))
    with P.DynLP(p.n, arrays["row_ptr"], arrays["col"], arrays["w"], 3, arrays["sv"], arrays["sc"], device_ptrs=True) as d:
        assert d.static_solve(TOL, 20000)[0] == 0
        before = [x.cpu().numpy() for x in d.export_graph()] + [x.cpu().numpy() for x in d.get_labels()]
        with pytest.raises(P.DynLPError) as ei:
            d.apply_update(*pack((dead, eu, ev, ew, seeds, classes)))
        assert ei.value.status == -1
        after = [x.cpu().numpy() for x in d.export_graph()] + [x.cpu().numpy() for x in d.get_labels()]
        for x, y in zip(before, after):
            assert np.array_equal(x, y)
        assert d.num_vertices == p.n
        st, s = d.apply_update(*pack(good))  # the context is as good as before, no mark or count is left behind
        assert st == 0 and s.frontier_initial > 0
        g = _graph(p)
        g.delete(np.array(good[0]))
        g.insert(0, np.array(good[1]), np.array(good[2]), np.array(good[3], np.float32), np.array(good[4]), np.array(good[5]))
        rp, col, w, deg, sc = (x.cpu().numpy() for x in d.export_graph())
        orp, ocol, _ = g.csr()
        assert rp.tolist() == orp.tolist() and sc.tolist() == g.seed_class.tolist()
        assert all(sorted(col[rp[u]:rp[u + 1]]) == sorted(ocol[orp[u]:orp[u + 1]]) for u in range(p.n))


@pytest.mark.parametrize("hub", [127, 128, 129, 1023, 1024, 1025, 2049, 9000])
def test_rows_about_the_lengths_that_change_hands(hub):
    """A row of `hub` entries loses some to deleted neighbours, receives some, and is deleted itself."""
    rng = np.random.default_rng(hub)
    n = 10000
    eu = np.concatenate([np.zeros(hub, np.int64), rng.integers(1, n, 4 * n)])
    ev = np.concatenate([1 + np.arange(hub), rng.integers(1, n, 4 * n)])
    keep = eu != ev
    rp, col, w = W.edges_to_csr(n, eu[keep], ev[keep], rng.uniform(0.1, 1, int(keep.sum())).astype(np.float32))
    assert rp[1] - rp[0] == hub
    sv = rng.permutation(np.arange(1, n))[:300].astype(np.int32)
    sc = rng.integers(0, 3, 300).astype(np.int32)
    g = R.Graph(n, rp, col, w, 3, sv, sc)
    with P.DynLP(n, rp, col, w, 3, sv, sc) as d:
        assert d.static_solve(TOL, 20000)[0] == 0
        gone = np.unique(np.concatenate([[1, hub], 1 + rng.choice(hub, hub // 3, replace=False)])).astype(np.int32)
        assert d.apply_update(gone)[0] == 0
        g.delete(gone)
        _check_graph(d, g)  # the order of the entries that stay is kept
        add = rng.choice(np.setdiff1d(np.arange(1, n), gone), 200, replace=False).astype(np.int32)
        for part in (add[:5], add[5:]):  # a few entries, and more than a group sorts
            assert d.apply_batch(0, np.zeros(part.size, np.int32), part, np.full(part.size, 0.25, np.float32))[0] == 0
            g.insert(0, np.zeros(part.size, np.int64), part, np.full(part.size, 0.25, np.float32), [], [])
            _check_graph(d, g, ordered=False)
        assert d.apply_update(np.array([0, 0], np.int32))[0] == 0
        g.delete(np.array([0]))
        _check_graph(d, g, ordered=False)


@pytest.mark.parametrize("n,per_row,hub", [(140001, 2, 63), (140001, 2, 64), (140001, 2, 65), (140001, 1, 129), (140001, 6, 3000), (9001, 2, 65)])
def test_rows_of_a_batch_that_touches_many(n, per_row, hub):
    """Where a batch touches many rows they are listed by a pass over the vertices, and from 131,072 rows on segments are
    sorted with 8 lanes: up to 64 entries per row, more are sorted by a workgroup.  Entries in order of id and weight, and
    degrees summed in the order of a fresh context, bit for bit."""
    rng = np.random.default_rng(hub)
    m = per_row * n // 2
    eu = np.concatenate([rng.integers(0, n, m), np.full(hub, 7)]).astype(np.int32)
    ev = np.concatenate([rng.integers(0, n, m), 8 + np.arange(hub)]).astype(np.int32)
    keep = (eu != ev) & ((eu != 7) & (ev != 7) | (np.arange(eu.size) >= m))
    eu, ev = eu[keep], ev[keep]
    ew = rng.uniform(0.1, 1, eu.size).astype(np.float32)
    base = np.arange(n - 1)
    rp0, col0, w0 = W.edges_to_csr(n, base[base % 3 == 0], base[base % 3 == 0] + 1, np.full(int(np.sum(base % 3 == 0)), 0.5, np.float32))
    sv, sc = np.arange(5, dtype=np.int32), np.array([0, 1, 0, 1, 0], np.int32)
    with P.DynLP(n, rp0, col0, w0, 2, sv, sc, slack_factor=1.01) as d:
        d.set_params(1e-3, 1)
        assert d.apply_batch(0, eu, ev, ew)[0] in (0, 1)
        rp, col, w, deg, _ = d.export_graph()
    src, dst = np.concatenate([eu, ev]), np.concatenate([ev, eu])
    ww = np.concatenate([ew, ew])
    order = np.lexsort((ww.view(np.uint32), dst, src))
    counts = np.bincount(src, minlength=n)
    old = np.diff(rp0)
    assert np.array_equal(np.diff(rp), old + counts)
    start = np.concatenate([[0], np.cumsum(counts)])[:-1]
    at = np.repeat(rp[:-1] + old - start, counts) + np.arange(src.size)  # where the appended entries belong
    assert np.array_equal(col[at], dst[order]) and np.array_equal(w[at], ww[order])
    with P.DynLP(n, rp, col, w, 2, sv, sc) as fresh:
        deg2 = fresh.export_graph()[3]
    assert np.array_equal(deg, deg2)


def test_edges_for_a_context_without_vertices_are_refused():
    """No vertex can be touched, so no launch may take its size from their number; the context is as good as before."""
    cu = lambda a, t: torch.as_tensor(np.asarray(a, t), device="cuda")
    none = (cu([], np.int32), cu([], np.int32))
    edge = (cu([0], np.int32), cu([1], np.int32), cu([0.5], np.float32))
    with P.DynLP(0, cu([0], np.int64), cu([0], np.int32), cu([1], np.float32), 2, *none, device_ptrs=True) as d:
        for seeds in ((None, None), (cu([0], np.int32), cu([1], np.int32))):
            with pytest.raises(P.DynLPError) as ei:
                d.apply_batch(0, *edge, *seeds)
            assert ei.value.status == -1 and d.num_vertices == 0 and d.num_entries == 0
        st, _ = d.apply_batch(2, *edge, cu([0], np.int32), cu([1], np.int32))
        assert st == 0
        assert d.get_labels()[1].cpu().tolist() == [1, 1]


@pytest.mark.parametrize("kinds,message", [
    (("deleted", "edge", "seed"), "deleted vertex out of range (item 3)"), (("edge", "seed"), "self loop (item 5)"),
    (("weight", "seed"), "weight must be finite and > 0 (item 11)"), (("seed",), "seed class out of range (seed 2)")])
def test_which_of_several_invalid_arguments_is_reported(kinds, message):
    """Found in one launch by whichever thread comes first; reported is, as when each kind had a launch of its own, a deleted
    vertex before an edge before a seed, and of one kind the first in the list."""
    p = W.small_random(2000, 3, 8.0, 100, 903)
    cu = lambda a, t: torch.as_tensor(np.asarray(a, t), device="cuda")
    m = 40000
    dead, sv, sc = np.arange(1000), np.arange(3000) % 2000, np.zeros(3000, np.int64)
    eu, ev, ew = np.arange(m) % 1000, 1000 + np.arange(m) % 1000, np.full(m, 0.5)
    if "deleted" in kinds:
        dead[3:] = -1
    if "edge" in kinds:
        ev[5:] = eu[5:]
        ev[6:] = 2000
    if "weight" in kinds:
        ew[11:] = np.nan
    sc[2:] = 3
    with P.DynLP(p.n, cu(p.row_ptr, np.int64), cu(p.col, np.int32), cu(p.w, np.float32), 3, cu([], np.int32), cu([], np.int32),
                 device_ptrs=True) as d:
        for _ in range(5):
            with pytest.raises(P.DynLPError) as ei:
                d.apply_update(cu(dead, np.int32), 0, cu(eu, np.int32), cu(ev, np.int32), cu(ew, np.float32), cu(sv, np.int32), cu(sc, np.int32))
            assert ei.value.status == -1 and ei.value.message == message


@pytest.mark.parametrize("slack", [1.01, 3.0])
def test_rows_that_receive_more_than_eight_lanes_hold(slack):
    """A batch that touches more than 131,072 rows, 1,500 of which (runs of neighbours, so that many meet in one workgroup) receive 60
    to 140 entries and a few of those already hold 1,100: sorted by 8 lanes, by 16 and by workgroups, each row alike."""
    rng = np.random.default_rng(4)
    n, far = 150000, 3000
    heavy = np.arange(500, 2000)
    count = rng.integers(60, 141, heavy.size)
    hub = heavy[::50]
    b0 = np.concatenate([np.repeat(hub, 1100), np.arange(n - 1)[::3]])
    b1 = np.concatenate([far + (np.arange(1100 * hub.size) * 7) % (n - far), np.arange(n - 1)[::3] + 1])
    rp0, col0, w0 = W.edges_to_csr(n, b0, b1, rng.uniform(0.1, 1, b0.size).astype(np.float32))
    light = rng.integers(far, n, (2, 140000))
    eu = np.concatenate([np.repeat(heavy, count), light[0]])
    ev = np.concatenate([rng.integers(far, n, int(count.sum())), np.where(light[0] == light[1], far + (light[1] + 1 - far) % (n - far), light[1])])
    order = rng.permutation(eu.size)
    eu, ev = eu[order].astype(np.int32), ev[order].astype(np.int32)
    ew = rng.uniform(0.1, 1, eu.size).astype(np.float32)
    sv, sc = np.arange(5, dtype=np.int32), np.array([0, 1, 0, 1, 0], np.int32)
    with P.DynLP(n, rp0, col0, w0, 2, sv, sc, slack_factor=slack) as d:
        d.set_params(1e-3, 1)
        assert d.apply_batch(0, eu, ev, ew)[0] in (0, 1)
        rp, col, w, deg, _ = d.export_graph()
    src, dst, ww = np.concatenate([eu, ev]), np.concatenate([ev, eu]), np.concatenate([ew, ew])
    order = np.lexsort((ww.view(np.uint32), dst, src))
    counts, old = np.bincount(src, minlength=n), np.diff(rp0)
    assert 2 * eu.size < 8 * n and np.count_nonzero(counts) > 131072, "the case is meant to be sorted with 8 lanes"
    assert np.array_equal(np.diff(rp), old + counts)
    start = np.concatenate([[0], np.cumsum(counts)])[:-1]
    at = np.repeat(rp[:-1] + old - start, counts) + np.arange(src.size)
    assert np.array_equal(col[at], dst[order]) and np.array_equal(w[at], ww[order])
    before = np.repeat(rp[:-1] - rp0[:-1], old) + np.arange(col0.size)
    assert np.array_equal(col[before], col0) and np.array_equal(w[before], w0)
    with P.DynLP(n, rp, col, w, 2, sv, sc) as fresh:
        assert np.array_equal(deg, fresh.export_graph()[3])
