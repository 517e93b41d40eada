"""GPU parity of the rounds over a small V_aff that run many per launch on one workgroup (k_tail_rounds): same V_aff every
round, same labels as the oracle's Step 3 and as the ordinary launches (a fixed number of lanes per row keeps those), in
batches whose V_aff stays small, outgrows the launch and comes back, or is cut by the round cap inside a launch.  The
round log says which rounds shared a launch (launch_rounds).
"""
import numpy as np
import pytest

import workloads as W
from oracle import native as ON
from oracle import reference as R
import paper_2604_06596_amd as P

pytestmark = pytest.mark.gpu

ROUNDS_ATOL = 5e-6  # as for the first rounds of a batch in test_gpu_parity


def _run(p, b, tol, cap, mode, **kw):
    with P.DynLP(p.n, p.row_ptr, p.col, p.w, p.C, p.seed_vertex, p.seed_class, **kw) as d:
        d.static_solve(1e-7, 20000)
        start, _ = d.get_labels()
        d.set_update_mode(mode)
        d.set_params(tol, cap)
        st, s = d.apply_batch(b.num_new_vertices, b.eu, b.ev, b.ew, b.seed_vertex, b.seed_class)
        soft, hard = d.get_labels()
        sizes, deltas = d.round_log()
        log = d.round_log_full()
        st2, s2 = d.apply_batch(0, None, None, None)  # no mark may be left behind
        assert cap < 20000 or (st2 == 0 and s2.iterations == 0)
    assert len(log) == s.iterations
    return start, st, s, soft, hard, sizes, deltas, log


# deg: frontier rows of about that many entries, far from 8, where narrow rows change between 4 and 16 lanes
@pytest.mark.parametrize("kind,C,scalar,deg,lanes", [
    ("random", 1, False, 16, 16), ("random", 2, True, 16, 16), ("random", 2, True, 3, 4), ("random", 2, False, 3, 4),
    ("random", 3, False, 3, 4), ("random", 3, False, 16, 16), ("random", 7, False, 5, 16), ("random", 16, False, 5, 16),
    ("hub", 20, False, 10, 16), ("hub", 50, False, 10, 16), ("hub", 64, False, 10, 16)])
@pytest.mark.parametrize("tol,cap", [(1e-3, 20000), (1e-4, 20000), (1e-4, 3), (1e-4, 7)])
def test_small_rounds_match_the_oracle_and_the_ordinary_launches(kind, C, scalar, deg, lanes, tol, cap):
    def make():
        return W.chung_lu(4000, C, 10.0, 2.1, 600, 0.8, 0.05, 55) if kind == "hub" else W.small_random(3001, C, float(deg), 200, 55 + C)

    p, p0 = make(), make()
    b = W.chung_lu_vertex_batch(p, 2, 0.0) if kind == "hub" else W.small_random_batch(p, 1, deg, 0, num_extra_edges=3, num_revealed=1)
    start, st, s, soft, hard, sizes, deltas, log = _run(p0, b, tol, cap, P.UPDATE_SYNCHRONOUS, binary_scalar=scalar)
    _, st1, s1, soft1, hard1, sizes1, _, log1 = _run(p0, b, tol, cap, P.UPDATE_SYNCHRONOUS, binary_scalar=scalar, group_lanes=lanes)
    shared = np.array([r.launch_rounds for r in log])
    print(kind, C, tol, cap, "rounds that shared launches", shared.astype(int).tolist())
    # a first V_aff that may bring its neighbours runs in a shared launch if those fit it
    rows = 1024 if C <= 2 else 512 if C <= 16 else 256
    mean = (p0.row_ptr[-1] + 2 * len(b.eu)) / (p0.n + b.num_new_vertices)
    assert (shared[0] > 0) == (sizes[0] * mean <= rows)
    if cap == 3 and lanes == 4:
        assert shared.tolist() == [3, 3, 3], "the cap is meant to fall inside a launch"
    assert not any(r.launch_rounds for r in log1)
    assert (st, s.iterations, s.rows_updated, s.edges_traversed) == (st1, s1.iterations, s1.rows_updated, s1.edges_traversed)
    assert sizes.tolist() == sizes1.tolist() and np.array_equal(soft, soft1)
    g = R.Graph(p0.n, p0.row_ptr, p0.col, p0.w, C, p0.seed_vertex, p0.seed_class)
    n_old = g.n
    g.insert(b.num_new_vertices, b.eu, b.ev, b.ew, b.seed_vertex, b.seed_class)
    rp, col, w = g.csr()
    A0 = ON.affected_set(rp, col, g.seed_class, n_old, b.eu, b.ev, b.seed_vertex)
    F = np.concatenate([start.astype(np.float64), np.full((b.num_new_vertices, C), 1.0 / C)])
    if len(b.seed_vertex):
        F[b.seed_vertex] = np.eye(C)[b.seed_class]
    if cap < 20000:
        # (the end of a run is left to the comparison above: a row that moves by the threshold to within float32 rounding
        # stays in V_aff on one side only, against the float64 oracle, and the runs part there)
        o2 = ON.step3_propagate(rp, col, w, F, g.seed_class, A0, tol, cap)
        osz = o2["frontier_sizes"][:o2["rounds"]]
        assert s.iterations == o2["rounds"] and (s.iterations == cap or C == 1)
        # (the same row-at-the-threshold effect within the first rounds: such a row and the neighbours it brings)
        assert np.all(np.abs(sizes.astype(np.int64) - osz.astype(np.int64)) <= 10 + osz // 500)
        np.testing.assert_allclose(deltas, o2["max_changes"][:o2["rounds"]], atol=1e-6)
        # (a row that stays out of V_aff keeps a value within tol of its new one)
        assert np.max(np.abs(soft - o2["F"])) <= (ROUNDS_ATOL if sizes.tolist() == osz.tolist() else ROUNDS_ATOL + 2 * tol)
    else:
        # rows updated in place take another path to labels that stopped under the same rule
        _, st2, s2, soft2, _, sizes2, _, log2 = _run(p0, b, tol, cap, P.UPDATE_IN_PLACE, binary_scalar=scalar)
        assert (log2[0].launch_rounds > 0) == (shared[0] > 0)
        assert st2 == 0 and sizes2[0] == sizes[0] and np.max(np.abs(soft2 - soft)) <= 100 * tol


@pytest.mark.parametrize("C,scalar", [(2, True), (2, False), (3, False), (10, False)])
def test_lanes_per_row_change_where_a_chain_of_rounds_begins(C, scalar):
    """Rounds that share a launch sum their rows as ordinary rounds would: the lanes per row are chosen from the mean row
    length of the round before, every 8 rounds (narrow rows: 4 lanes below a mean length of 8, else 16)."""
    changes = 0
    for deg, tol in [(deg, tol) for deg in (4.0, 4.5, 5.0, 5.5, 6.0) for tol in (1e-4, 1e-6)]:
        p, p0 = W.small_random(3001, C, deg, 200, 155 + C), W.small_random(3001, C, deg, 200, 155 + C)
        b = W.small_random_batch(p, 1, 3, 0)
        with P.DynLP(p0.n, p0.row_ptr, p0.col, p0.w, C, p0.seed_vertex, p0.seed_class, binary_scalar=scalar) as d:
            d.static_solve(1e-7, 20000)
            d.set_params(tol, 20000)
            assert d.apply_batch(b.num_new_vertices, b.eu, b.ev, b.ew)[0] == 0
            mean = d.num_entries / d.num_vertices
            log = d.round_log_full()
        for t, r in enumerate(log):
            if t % 8 == 0:
                want = 4 if C <= 4 and mean < 8 else 16
                changes += t > 0 and want != log[t - 1].group_lanes
            assert r.group_lanes == want, (deg, tol, t, len(log), mean)
            mean = (r.entries_short + r.entries_long) / (r.rows_short + r.rows_long)
    print(C, scalar, "changes of the lanes per row", changes)
    assert changes > 0 or C > 4, "the case is meant to change the lanes per row"


@pytest.mark.parametrize("C", [5, 20])
def test_averaged_rows_begin_where_ordinary_launches_begin_them(C):
    """Two new vertices tied to each other by weight 1 and to two seeds by weight 0.001: rounds that repeat themselves
    exactly.  The rows are averaged from the same round on as with ordinary launches."""
    p = W.small_random(400, C, 6.0, 40, 4242)
    a = int(p.seed_vertex[np.flatnonzero(p.seed_class == 0)[0]])
    b = int(p.seed_vertex[np.flatnonzero(p.seed_class == 1)[0]])
    u, v = p.n, p.n + 1
    runs = []
    for lanes in (0, 16):
        with P.DynLP(p.n, p.row_ptr, p.col, p.w, C, p.seed_vertex, p.seed_class, group_lanes=lanes) as d:
            d.static_solve(1e-6, 20000)
            d.set_params(1e-6, 20000)
            st, s = d.apply_batch(2, np.array([u, u, v], np.int32), np.array([v, a, b], np.int32),
                                  np.array([1.0, 0.001, 0.001], np.float32))
            assert st == 0
            runs.append(d.get_labels() + d.round_log() + (s.iterations,))
    (soft, hard, sizes, deltas, rounds), (soft1, hard1, sizes1, deltas1, rounds1) = runs
    print(C, "rounds", rounds, rounds1)
    assert rounds == rounds1 and sizes.tolist() == sizes1.tolist() and np.array_equal(deltas, deltas1)
    assert np.array_equal(soft, soft1) and np.array_equal(hard, hard1)


@pytest.mark.parametrize("C", [2, 20, 50])
def test_long_rows_leaving_and_coming_back(C):
    """V_aff with rows of more than 128 entries, and one that outgrows the launch and comes back."""
    p0 = W.chung_lu(4000, C, 10.0, 2.1, 600, 0.8, 0.05, 55)
    hubs = np.argsort(-np.diff(p0.row_ptr), kind="stable")
    is_seed = np.zeros(p0.n, dtype=bool)
    is_seed[p0.seed_vertex] = True
    hub = int(next(h for h in hubs if not is_seed[h] and p0.row_ptr[h + 1] - p0.row_ptr[h] <= 500))
    assert p0.row_ptr[hub + 1] - p0.row_ptr[hub] > 128
    seen = dict(long=False, back=False)
    for tol in (3e-3, 1e-3, 3e-4, 1e-4):
        for w in (0.01, 0.1, 1.0):
            for cap in (20000, 3, 11):
                runs = []
                for lanes in (0, 16):
                    with P.DynLP(p0.n, p0.row_ptr, p0.col, p0.w, C, p0.seed_vertex, p0.seed_class, group_lanes=lanes) as d:
                        d.static_solve(1e-7, 20000)
                        d.set_params(tol, cap)
                        d.apply_batch(1, np.array([p0.n], np.int32), np.array([hub], np.int32), np.array([w], np.float32),
                                      np.array([p0.n], np.int32), np.array([C - 1], np.int32))
                        runs.append((d.get_labels()[0], d.round_log()[0], d.round_log_full()))
                assert np.array_equal(runs[0][0], runs[1][0]) or C <= 4  # narrow rows may take 4 lanes in the first run
                assert runs[0][1].tolist() == runs[1][1].tolist() or C <= 4
                log = runs[0][2]
                shared = [r.launch_rounds > 0 for r in log]
                seen["long"] |= any(r.rows_long > 0 and q for r, q in zip(log, shared))
                first_out = shared.index(False) if False in shared else len(log)
                seen["back"] |= any(shared[:first_out]) and any(shared[first_out:])
    print(C, seen)
    assert all(seen.values())


@pytest.mark.parametrize("C,limit", [(2, 8192), (10, 3072), (50, 1536)])
def test_a_few_hubs_are_not_left_to_one_workgroup(C, limit):
    """A small V_aff of hubs holds far more entries than its number of rows says: such a round does not share a launch."""
    p0 = W.chung_lu(20000, C, 30.0, 2.1, 6000, 0.8, 0.02, 56)
    is_seed = np.zeros(p0.n, dtype=bool)
    is_seed[p0.seed_vertex] = True
    lens = np.diff(p0.row_ptr)
    hubs = [int(h) for h in np.argsort(-lens, kind="stable") if not is_seed[h]][:8]
    assert lens[hubs].sum() > limit
    runs = []
    for lanes in (0, 16):
        with P.DynLP(p0.n, p0.row_ptr, p0.col, p0.w, C, p0.seed_vertex, p0.seed_class, group_lanes=lanes) as d:
            d.static_solve(1e-7, 20000)
            for tol in (1e-1, 1e-3, 1e-4):
                new = d.num_vertices
                d.set_params(tol, 20000)
                d.apply_batch(1, np.full(8, new, np.int32), np.array(hubs, np.int32), np.full(8, 0.05, np.float32),
                              np.array([new], np.int32), np.array([0], np.int32))
                log = d.round_log_full()
                assert all(r.entries_short + r.entries_long <= limit for r in log if r.launch_rounds > 0)
                assert log[0].entries_long > limit
            runs.append((d.get_labels()[0], d.round_log()[0]))
    if C > 4:
        assert np.array_equal(runs[0][0], runs[1][0]) and runs[0][1].tolist() == runs[1][1].tolist()
