"""GPU parity of the packed rounds (label rows of graphs of 32,768 updatable vertices or more: entries ordered by
neighbour id, sums of a part's rows in LDS): sweeps of the static solve and the rounds of a batch against the oracle,
for every way a label row is read (1 to 16 lanes, odd column counts, the scalar layout), odd sizes and hub rows.

Tolerances: one round rounds w / d to float32 and the sum of d terms to about 0.41 * sqrt(d) units of 2^-31, less than the
1e-6 that a float32 round is allowed; the bars of the ordinary rounds (test_gpu_parity) apply.
"""
import numpy as np
import pytest

import workloads as W
from oracle import native as ON
from oracle import reference as R
import paper_2604_06596_amd as P

pytestmark = pytest.mark.gpu

TOL = 1e-6
ROUNDS_ATOL = 5e-6


def _problem(kind, n, C, deg, seed):
    if kind == "hub":
        return W.chung_lu(n, C, deg, 2.1, 1200, 0.8, 0.03, seed)
    return W.sbm(n, C, deg, 8.0, 0.03, seed)


def _batch(kind, p, k, deg):
    return W.chung_lu_vertex_batch(p, k, 0.02) if kind == "hub" else W.sbm_vertex_batch(p, k, deg, 0.02)


def _make(p, **kw):
    return P.DynLP(p.n, p.row_ptr, p.col, p.w, p.C, p.seed_vertex, p.seed_class, **kw)


def _is_packed(r):
    return r.group_lanes == 0


@pytest.mark.parametrize("kind,n,C,deg,scalar", [
    ("sbm", 36001, 2, 12, True), ("sbm", 36001, 2, 12, False), ("sbm", 35213, 3, 12, False), ("sbm", 36000, 5, 12, False),
    ("sbm", 34817, 10, 20, False), ("sbm", 36007, 12, 20, False), ("sbm", 36007, 16, 20, False), ("sbm", 36000, 17, 20, False),
    ("sbm", 36000, 24, 20, False), ("sbm", 36000, 29, 20, False), ("sbm", 35000, 33, 20, False), ("sbm", 35000, 50, 24, False),
    ("sbm", 34999, 64, 24, False), ("hub", 40000, 20, 30, False)])
def test_packed_rounds_match_the_oracle(kind, n, C, deg, scalar):
    p, p0 = _problem(kind, n, C, deg, 31 + C), _problem(kind, n, C, deg, 31 + C)
    b = _batch(kind, p, 2500, deg)
    g = R.Graph(p0.n, p0.row_ptr, p0.col, p0.w, C, p0.seed_vertex, p0.seed_class)
    rp, col, w = g.csr()
    F = R.initial_labels(g.seed_class, C)
    for _ in range(20):
        F, _ = ON.itlp_sweep(rp, col, w, F, g.seed_class)
    runs = []
    for _ in range(2):
        with _make(p0, binary_scalar=scalar) as d:
            st, s = d.static_solve(1e-9, 20)
            assert st == 1 and s.iterations == 20
            assert [_is_packed(r) for r in d.round_log_full()] == [False] * 8 + [True] * 12
            cold, _ = d.get_labels()
            d.static_solve(TOL, 20000)
            soft0, _ = d.get_labels()
            d.set_params(TOL, 14)
            st, s = d.apply_batch(b.num_new_vertices, b.eu, b.ev, b.ew, b.seed_vertex, b.seed_class)
            soft, hard = d.get_labels()
            log = d.round_log_full()
            sizes, deltas = d.round_log()
        runs.append((cold, soft0, soft))
    assert np.max(np.abs(cold - F)) <= ROUNDS_ATOL
    assert any(_is_packed(r) and r.staged == 2 for r in log), "the case is meant to reach packed rounds"
    n_old = g.n
    g.insert(b.num_new_vertices, b.eu, b.ev, b.ew, b.seed_vertex, b.seed_class)
    rp, col, w = g.csr()
    A0 = ON.affected_set(rp, col, g.seed_class, n_old, b.eu, b.ev, b.seed_vertex)
    F = np.concatenate([soft0.astype(np.float64), np.full((b.num_new_vertices, C), 1.0 / C)])
    F[b.seed_vertex] = np.eye(C)[b.seed_class]
    o2 = ON.step3_propagate(rp, col, w, F, g.seed_class, A0, TOL, 14)
    print(kind, C, "packed rounds", sum(map(_is_packed, log)), "sizes", sizes.tolist(), "oracle", o2["frontier_sizes"].tolist())
    assert s.iterations == o2["rounds"]
    # a row that moves by almost exactly the threshold may fall on either side of it: float32 against float64
    assert np.all(np.abs(sizes - o2["frontier_sizes"]) <= 2e-3 * np.maximum(o2["frontier_sizes"], 1000))
    np.testing.assert_allclose(deltas, o2["max_changes"], atol=1e-6)
    assert np.max(np.abs(soft - o2["F"])) <= ROUNDS_ATOL
    assert soft.min() >= 0 and np.max(np.abs(soft.sum(1) - 1)) < 1e-5
    for x, y in zip(*runs):
        assert np.array_equal(x, y), "the order of the LDS atomics must not show"


def test_a_part_with_most_of_the_entries_keeps_the_ordinary_rounds():
    """A hub that holds many times a part's share of the entries: the round must not wait for one workgroup."""
    rng = np.random.default_rng(5)
    n = 40000
    eu = np.concatenate([np.arange(n - 1), np.zeros(30000, dtype=np.int64), rng.integers(0, n, 4 * n)])
    ev = np.concatenate([np.arange(1, n), rng.permutation(np.arange(2, n))[:30000], rng.integers(0, n, 4 * n)])
    keep = eu != ev
    rp, col, w = W.edges_to_csr(n, eu[keep], ev[keep], rng.uniform(0.1, 1, int(keep.sum())).astype(np.float32))
    sv = rng.permutation(np.arange(1, n))[:800].astype(np.int32)
    sc = rng.integers(0, 5, 800).astype(np.int32)
    with P.DynLP(n, rp, col, w, 5, sv, sc) as d:
        d.static_solve(1e-9, 14)
        assert not any(_is_packed(r) for r in d.round_log_full())
        soft, _ = d.get_labels()
    seed_class = np.full(n, -1, dtype=np.int32)
    seed_class[sv] = sc
    F = R.initial_labels(seed_class, 5)
    for _ in range(14):
        F, _ = ON.itlp_sweep(rp, col, w.astype(np.float64), F, seed_class)
    assert np.max(np.abs(soft - F)) <= ROUNDS_ATOL


@pytest.mark.parametrize("C,scalar,tol", [(10, False, 1e-4), (2, True, 1e-4), (3, False, 2e-5)])
def test_loose_thresholds_keep_the_sums_of_the_row_update(C, scalar, tol):
    """Where the last bits of a row show in the result, a synchronous run is the same whether or not packed rounds are
    possible (a fixed number of lanes per row excludes them)."""
    p0 = _problem("sbm", 36001, C, 20, 131 + C)
    runs = []
    for kw in ({}, dict(group_lanes=16)):
        p = _problem("sbm", 36001, C, 20, 131 + C)
        b = _batch("sbm", p, 2500, 20)
        with _make(p0, binary_scalar=scalar, **kw) as d:
            d.static_solve(tol, 20000)
            out = [d.get_labels()]
            assert not any(_is_packed(r) for r in d.round_log_full()) and len(d.round_log_full()) > 8
            d.apply_batch(b.num_new_vertices, b.eu, b.ev, b.ew, b.seed_vertex, b.seed_class)
            out.append(d.get_labels())
            assert not any(_is_packed(r) for r in d.round_log_full())
        runs.append(out)
    for x, y in zip(*runs):
        assert np.array_equal(x[0], y[0]) and np.array_equal(x[1], y[1])


@pytest.mark.parametrize("hub,C", [(8000, 20), (8000, 3), (8000, 64), (9000, 20)])
def test_hub_rows_whose_neighbours_are_alike(hub, C):
    """A hub of equal weights whose neighbours are nearly alike: rounding every term to the nearest unit would be off the
    same way in all of them (8,000 terms: up to 2e-6).  Rows too long for the unit stay unpacked.
    One sweep against the float64 sweep of the labels before.  Bar: four standard deviations of 0.41 * sqrt(d) units, and
    w / d (degree, quotient) and the stored value rounded to float32, 2^-24 of the value each."""
    rng = np.random.default_rng(7)
    n = 36000
    m = 65 * n
    eu = np.concatenate([np.zeros(hub, dtype=np.int64), rng.integers(1, n, m)])
    ev = np.concatenate([rng.permutation(np.arange(2, n))[:hub], rng.integers(1, n, m)])
    key = np.unique(np.minimum(eu, ev)[eu != ev] * n + np.maximum(eu, ev)[eu != ev])
    rp, col, w = W.edges_to_csr(n, key // n, key % n, np.full(key.size, 0.7, dtype=np.float32))
    assert rp[1] - rp[0] == hub
    sv = np.array([1], dtype=np.int32)  # one labelled vertex: the rows stay close to 1 / C
    seed_class = np.full(n, -1, dtype=np.int32)
    seed_class[sv] = 0

    def sweeps(k):
        with P.DynLP(n, rp, col, w, C, sv, np.zeros(1, dtype=np.int32)) as d:
            d.static_solve(1e-12, k)
            assert [_is_packed(r) for r in d.round_log_full()] == [hub <= 8192 and t >= 8 for t in range(k)]
            return d.get_labels()[0].astype(np.float64)

    before, worst, worst_sum = sweeps(9), 0.0, 0.0
    for k in range(10, 14):
        after = sweeps(k)
        F, _ = ON.itlp_sweep(rp, col, w.astype(np.float64), before, seed_class)
        worst = max(worst, float(np.max(np.abs(after - F)[0])))
        worst_sum = max(worst_sum, abs(float(after[0].sum() - F[0].sum())))
        before = after
    dither, value = 4 * 0.41 * np.sqrt(hub) * 2.0 ** -31, 3 * 2.0 ** -24
    print(hub, C, "hub's row: error", worst, "bar", dither + value * F[0].max(), "sum", worst_sum, "bar", C * dither + value)
    if hub <= 8192:
        assert worst <= dither + value * F[0].max() and worst_sum <= C * dither + value


def test_rows_that_take_several_generations_of_parts():
    """64 columns: the sums of 155,648 rows fit the chip at a time, a graph of 158,001 takes two workgroups per CU one
    after the other.  Sweeps and the rounds of a batch against the oracle."""
    C, n = 64, 158001
    p, p0 = (W.sbm(n, C, 34, 8.0, 0.03, 95) for _ in range(2))
    b = W.sbm_vertex_batch(p, 1500, 34, 0.02)
    g = R.Graph(p0.n, p0.row_ptr, p0.col, p0.w, C, p0.seed_vertex, p0.seed_class)
    rp, col, w = g.csr()
    F = R.initial_labels(g.seed_class, C)
    for _ in range(12):
        F, _ = ON.itlp_sweep(rp, col, w, F, g.seed_class)
    with _make(p0) as d:
        d.static_solve(1e-9, 12)
        assert [_is_packed(r) for r in d.round_log_full()] == [False] * 8 + [True] * 4
        cold, _ = d.get_labels()
        d.set_params(TOL, 10)
        d.apply_batch(b.num_new_vertices, b.eu, b.ev, b.ew, b.seed_vertex, b.seed_class)
        assert any(_is_packed(r) for r in d.round_log_full())
        soft, _ = d.get_labels()
        sizes, _ = d.round_log()
    assert np.max(np.abs(cold - F)) <= ROUNDS_ATOL
    g.insert(b.num_new_vertices, b.eu, b.ev, b.ew, b.seed_vertex, b.seed_class)
    rp, col, w = g.csr()
    A0 = ON.affected_set(rp, col, g.seed_class, n, b.eu, b.ev, b.seed_vertex)
    F = np.concatenate([cold.astype(np.float64), np.full((b.num_new_vertices, C), 1.0 / C)])
    F[b.seed_vertex] = np.eye(C)[b.seed_class]
    o2 = ON.step3_propagate(rp, col, w, F, g.seed_class, A0, TOL, 10)
    assert np.all(np.abs(sizes - o2["frontier_sizes"]) <= 2e-3 * np.maximum(o2["frontier_sizes"], 1000))
    assert np.max(np.abs(soft - o2["F"])) <= ROUNDS_ATOL


@pytest.mark.parametrize("kind,C,scalar", [("random", 2, True), ("random", 2, False), ("sbm", 10, False)])
def test_packed_stretches_begin_while_nearly_all_rows_move(kind, C, scalar):
    """Rows that did not move themselves look their neighbours up in a packed round: a V_aff of nearly all rows of which
    fewer and fewer move is left to the ordinary rounds."""
    def make():
        return W.small_random(60000, 2, 6.0, 3000, 57) if kind == "random" else W.sbm(60000, C, 16.0, 8.0, 0.05, 58)

    late = 0
    for tol in (1e-6, 3e-6, 1e-5):
        p, p0 = make(), make()
        b = W.small_random_batch(p, 100, 6, 5) if kind == "random" else W.sbm_vertex_batch(p, 100, 16, 0.02)
        with _make(p0, binary_scalar=scalar) as d:
            d.static_solve(1e-6, 20000)
            d.set_params(tol, 20000)
            assert d.apply_batch(b.num_new_vertices, b.eu, b.ev, b.ew, b.seed_vertex, b.seed_class)[0] == 0
            log = d.round_log_full()
        rows = max(r.rows_short + r.rows_long for r in log)
        for t, r in enumerate(log):
            start = t - t % 8
            if _is_packed(r) and not _is_packed(log[t - 1]):
                assert start > 0 and log[start - 1].rows_moved >= 0.969 * rows, (tol, t)
            if t == start and t > 0 and r.rows_short + r.rows_long > 0.6 * rows and log[t - 1].rows_moved < 0.9 * rows:
                late += 1
        print(kind, C, scalar, tol, "rounds", len(log), "packed", sum(map(_is_packed, log)))
    print(kind, C, scalar, "chains with a large V_aff of which few rows move:", late)
    assert late > 0 or kind == "sbm", "the case is meant to have chains that are left to ordinary rounds"


@pytest.mark.parametrize("C,heavy,extra,isolated", [(20, 3000, 60, 9001), (29, 2000, 60, 0), (3, 500, 20, 20000), (64, 37, 60, 1)])
def test_parts_of_unequal_numbers_of_rows(C, heavy, extra, isolated):
    """Parts are cut by their entries: the first `heavy` vertices have several times the mean (few rows per part), the last `isolated` none (many rows per part; with 64 columns as many as fit, so that
    the cut is by rows).  Sweeps and the rounds of a batch against the oracle."""
    rng = np.random.default_rng(17)
    n = 36000 + isolated
    m = 8 * 36000
    eu = np.concatenate([rng.integers(0, 36000, m), rng.integers(0, heavy, extra * heavy)])
    ev = rng.integers(0, 36000, eu.size)
    keep = eu != ev
    rp, col, w = W.edges_to_csr(n, eu[keep], ev[keep], rng.uniform(0.1, 1, int(keep.sum())).astype(np.float32))
    sv = rng.permutation(36000)[:900].astype(np.int32)
    sc = rng.integers(0, C, 900).astype(np.int32)
    g = R.Graph(n, rp, col, w, C, sv, sc)
    F = R.initial_labels(g.seed_class, C)
    for _ in range(13):
        F, _ = ON.itlp_sweep(rp, col, w.astype(np.float64), F, g.seed_class)
    with P.DynLP(n, rp, col, w, C, sv, sc) as d:
        d.static_solve(1e-9, 13)
        assert [_is_packed(r) for r in d.round_log_full()] == [False] * 8 + [True] * 5
        assert np.max(np.abs(d.get_labels()[0] - F)) <= ROUNDS_ATOL
        log = d.round_log_full()
        assert len({(r.rows_short + r.rows_long, r.entries_short + r.entries_long) for r in log}) == 1
        d.set_update_mode(P.UPDATE_IN_PLACE)
        assert d.static_solve(TOL, 20000)[0] == 0
        soft = d.get_labels()[0]
    mean, _ = ON.itlp_sweep(rp, col, w.astype(np.float64), soft.astype(np.float64), g.seed_class)
    assert np.max(np.abs(mean - soft)) <= 2 * TOL


@pytest.mark.parametrize("live", [112000, 106000, 99000])
def test_parts_of_so_many_rows_that_their_entries_pass_through_smaller_tiles(live):
    """Heavy rows fill 255 parts, the vertices without edges the last: tiles of 8,192, 4,096 and 2,048 entries."""
    import scipy.sparse as sp
    import torch

    g = torch.Generator(device="cuda")
    g.manual_seed(live)
    n, m = 131072, live * 150
    u = torch.randint(live, (m,), device="cuda", generator=g)
    v = torch.randint(live, (m,), device="cuda", generator=g)
    v = torch.where(u == v, (v + 1) % live, v)
    w = 0.1 + 0.9 * torch.rand(m, device="cuda", generator=g)
    src, order = torch.sort(torch.cat([u, v]), stable=True)
    rp = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), torch.bincount(src, minlength=n).cumsum(0)])
    col, ww = torch.cat([v, u])[order].int(), torch.cat([w, w])[order]
    sv = torch.arange(1000, device="cuda", dtype=torch.int32)
    with P.DynLP(n, rp, col, ww, 2, sv, sv % 2, device_ptrs=True, binary_scalar=True) as d:
        d.static_solve(1e-9, 11)
        assert [_is_packed(r) for r in d.round_log_full()] == [False] * 8 + [True] * 3
        soft = d.get_labels()[0].cpu().numpy()
    A = sp.csr_matrix((ww.double().cpu().numpy(), col.cpu().numpy(), rp.cpu().numpy()), shape=(n, n))
    deg = np.asarray(A.sum(1)).ravel()
    f = np.full(n, 0.5)
    f[:1000] = np.arange(1000) % 2
    for _ in range(11):
        f[1000:live] = (A @ f)[1000:live] / deg[1000:live]
    assert np.max(np.abs(soft[:, 1] - f)) <= ROUNDS_ATOL
