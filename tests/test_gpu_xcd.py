"""Rounds of small graphs that share launches on the CUs of one XCD (k_xcd_rounds): the same V_aff, moves and labels, bit for
bit, as ordinary launches (a fixed number of lanes per row keeps those), over the edges of what the kernel cuts the graph into:
words of 32 rows, one word or many per workgroup, rows of 1 to 128 entries (longer ones end it), one to sixteen columns, 240
rounds to a launch.  With kernel timing on, all rounds of a launch have the same time.
"""
import threading
import time

import numpy as np
import pytest

import workloads as W
import paper_2604_06596_amd as P

pytestmark = pytest.mark.gpu


def _shared(log):
    """Rounds whose time is that of the round before: they shared its launch."""
    t = np.array([r.ms_update for r in log])
    return int(np.count_nonzero(t[1:] == t[:-1])) if len(t) > 1 else 0


def _run(make, lanes, tol, cap, mode, scalar=False, want_lanes=0):
    p, batches = make()
    out, shared, rounds, used = [], 0, 0, set()
    with P.DynLP(p.n, p.row_ptr, p.col, p.w, p.C, p.seed_vertex, p.seed_class, group_lanes=lanes, time_kernels=True,
                 binary_scalar=scalar) as d:
        d.set_update_mode(mode)
        st, s = d.static_solve(tol, cap)
        out.append((st, s.iterations, s.edges_traversed) + tuple(d.get_labels()) + tuple(d.round_log()))
        d.set_params(tol, cap)
        for b in batches:
            st, s = d.apply_batch(b.num_new_vertices, b.eu, b.ev, b.ew, b.seed_vertex, b.seed_class)
            out.append((st, s.iterations, s.rows_updated, s.edges_traversed, s.frontier_initial, s.frontier_peak) +
                       tuple(d.get_labels()) + tuple(d.round_log()))
            log = d.round_log_full()
            shared, rounds, used = shared + _shared(log), rounds + len(log), used | {int(r.group_lanes) for r in log}
    if lanes == 0 and want_lanes:
        assert used == {want_lanes}, "the case is meant to keep its lanes per row"
    return out, shared, rounds


def _random(n, C, deg):
    def make():
        p = W.small_random(n, C, deg, max(2, n // 50), 31 * n + C)
        q = W.small_random(n, C, deg, max(2, n // 50), 31 * n + C)
        return q, [W.small_random_batch(p, max(1, n // 40), max(1, int(deg)), 1, num_extra_edges=4, num_revealed=1),
                   W.small_random_batch(p, 1, 2, 0, num_extra_edges=1)]
    return make


def _star(n, C, length):
    """A vertex of `length` entries among short rows, and a batch that touches it."""
    def make():
        p, q = (W.small_random(n, C, 12.0, 40, 77 + length) for _ in range(2))
        u = int(np.setdiff1d(np.arange(n), p.seed_vertex)[0])
        near = p.col[p.row_ptr[u]:p.row_ptr[u + 1]]
        others = np.setdiff1d(np.arange(n), np.append(near, u))[:length - len(near)].astype(np.int32)
        none = np.zeros(0, np.int32)
        first = W.Batch(0, np.full(len(others), u, np.int32), others, np.linspace(0.1, 1.0, len(others)).astype(np.float32), none, none)
        return p, [first, W.small_random_batch(q, 2, 3, 0)]
    return make


# (n, C, mean degree, one float per vertex): lanes per row are 4 below a mean of 8 entries and up to four columns, else 16
@pytest.mark.parametrize("n,C,deg,scalar,lanes", [
    (5, 2, 2, True, 4), (31, 3, 3, False, 4), (33, 2, 3, False, 4), (64, 1, 12, False, 16), (65, 4, 12, False, 16),
    (2047, 2, 12, True, 16), (2048, 5, 6, False, 16), (2049, 16, 6, False, 16), (2049, 3, 3, False, 4), (6001, 2, 3, True, 4),
    (9001, 4, 12, False, 16), (9001, 9, 12, False, 16), (9001, 2, 12, False, 16), (22000, 8, 9, False, 16), (31500, 2, 3, True, 4)])
@pytest.mark.parametrize("tol,cap", [(1e-4, 20000), (1e-6, 300), (1e-6, 13)])
def test_the_same_rounds_as_ordinary_launches(n, C, deg, scalar, lanes, tol, cap):
    one, shared, rounds = _run(_random(n, C, float(deg)), 0, tol, cap, P.UPDATE_SYNCHRONOUS, scalar, lanes)
    own, shared0, _ = _run(_random(n, C, float(deg)), lanes, tol, cap, P.UPDATE_SYNCHRONOUS, scalar)
    print(n, C, deg, "rounds", rounds, "that shared launches", shared, shared0)
    assert rounds < 20 or 2 * shared > rounds, "the case is meant to share launches"
    assert shared0 < shared or rounds < 20
    for a, b in zip(one, own):
        for x, y in zip(a, b):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("length,shares", [(112, True), (127, True), (128, True), (129, False), (300, False)])
@pytest.mark.parametrize("C", [1, 3, 6, 12])
def test_rows_of_up_to_128_entries(length, shares, C):
    one, shared, rounds = _run(_star(1500, C, length), 0, 1e-5, 20000, P.UPDATE_SYNCHRONOUS)
    own, _, _ = _run(_star(1500, C, length), 16, 1e-5, 20000, P.UPDATE_SYNCHRONOUS)
    assert not shares or shared > rounds // 2 or rounds < 20
    for a, b in zip(one, own):
        for x, y in zip(a, b):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("n,C,scalar", [(40, 2, False), (3001, 2, True), (12000, 12, False)])
def test_rows_updated_in_place_end_under_the_same_rule(n, C, scalar):
    """In place the path differs; where it ends is within the threshold times the steps of a walk to a labelled vertex."""
    one, shared, _ = _run(_random(n, C, 9.0), 0, 1e-6, 20000, P.UPDATE_IN_PLACE, scalar)
    own, _, _ = _run(_random(n, C, 9.0), 16, 1e-6, 20000, P.UPDATE_SYNCHRONOUS, scalar)
    assert shared > 0
    for i, (a, b) in enumerate(zip(one, own)):
        k = 3 if i == 0 else 6  # the soft labels in the tuple
        assert a[0] == b[0] == 0 and np.max(np.abs(a[k] - b[k])) <= 400 * 1e-6


def test_two_contexts_take_turns_and_launches_are_told_apart():
    """Each context numbers its launches; what one leaves behind is not taken for the other's, on whichever XCD they run."""
    make = _random(2500, 4, 9.0)
    want, _, _ = _run(make, 16, 1e-5, 20000, P.UPDATE_SYNCHRONOUS)
    runs = []
    ctx = []
    for _ in range(2):
        p, batches = make()
        ctx.append((P.DynLP(p.n, p.row_ptr, p.col, p.w, p.C, p.seed_vertex, p.seed_class), batches))
    for d, _ in ctx:
        d.static_solve(1e-5, 20000)
        d.set_params(1e-5, 20000)
    for i in range(2):
        for d, batches in ctx:
            b = batches[i]
            d.apply_batch(b.num_new_vertices, b.eu, b.ev, b.ew, b.seed_vertex, b.seed_class)
            runs.append(d.get_labels()[0])
            assert np.array_equal(runs[-1], want[1 + i][6])
    for d, _ in ctx:
        d.__exit__(None, None, None)


def _solve_and_batches(make, lanes, tol, cap, mode, before=None, **options):
    """Static solve and batches; before[i] is called with the context ahead of step i.  Results, and the round logs."""
    p, batches = make()
    out, logs = [], []
    with P.DynLP(p.n, p.row_ptr, p.col, p.w, p.C, p.seed_vertex, p.seed_class, group_lanes=lanes, time_kernels=True,
                 **options) as d:
        d.set_update_mode(mode)
        for i, b in enumerate([None, *batches]):
            if before and i in before:
                before[i](d)
            if b is None:
                st, s = d.static_solve(tol, cap)
                d.set_params(tol, cap)
            else:
                st, s = d.apply_batch(b.num_new_vertices, b.eu, b.ev, b.ew, b.seed_vertex, b.seed_class)
            out.append((st, s.iterations, s.rows_updated, s.edges_traversed, s.frontier_initial, s.frontier_peak) +
                       tuple(d.get_labels()) + tuple(d.round_log()))
            logs.append(d.round_log_full())
    return out, logs


def _most_share(log):
    """(Two launches of their own may take the same time too, and the last rounds of a batch share those of one workgroup.)"""
    print("rounds", len(log), "that shared launches", _shared(log))
    return 2 * _shared(log) > len(log)


def _same(a, b):
    for x, y in zip(a, b):
        for u, v in zip(x, y):
            assert np.array_equal(u, v)


def test_a_launch_that_is_refused_before_it_takes_place_leaves_no_gap_in_the_numbers():
    """The sign-in list of a launch is cleared by the launch before it: after a refusal the next one finds it open all the same."""
    make = _random(2500, 4, 9.0)
    want, _ = _solve_and_batches(make, 16, 1e-6, 20000, P.UPDATE_SYNCHRONOUS)
    got, logs = _solve_and_batches(make, 0, 1e-6, 20000, P.UPDATE_SYNCHRONOUS,
                                   {1: lambda d: d.set_shared_rounds(-1), 2: lambda d: d.set_shared_rounds(0)})
    _same(got, want)
    assert [_most_share(log) for log in logs] == [True, False, True]


def _longest_launch(log):
    """Rounds in a row with the same time: those of one launch (of two, where both took the same)."""
    best = run = 1
    for a, b in zip(log, log[1:]):
        run = run + 1 if a.ms_update == b.ms_update else 1
        best = max(best, run)
    return best


def _crowded(n, C, hubs):
    """`hubs` vertices of some 100 entries come first, the others have a few: the first workgroup's entries outgrow its LDS though the
    graph as a whole is small enough for rounds on one XCD."""
    def make():
        rng = np.random.default_rng(n + C)
        a = rng.integers(0, hubs, 44 * hubs)
        b = (a + 1 + rng.integers(0, hubs - 1, 44 * hubs)) % hubs
        u = np.concatenate([a, np.arange(n - 1)])
        v = np.concatenate([b, np.arange(1, n)])
        w = (rng.integers(1, 17, len(u)) / 16).astype(np.float32)
        order = np.argsort(np.concatenate([u, v]), kind="stable")
        row_ptr = np.concatenate([[0], np.cumsum(np.bincount(np.concatenate([u, v]), minlength=n))]).astype(np.int64)
        assert np.diff(row_ptr).max() <= 128
        seeds = np.arange(0, n, 11).astype(np.int32)
        p = W.Problem(n, C, row_ptr, np.concatenate([v, u])[order].astype(np.int32), np.concatenate([w, w])[order], seeds,
                      (seeds % C).astype(np.int32), np.zeros(n, np.int32))
        none = np.zeros(0, np.int32)
        x = rng.integers(hubs, n - 1, 300).astype(np.int32)
        return p, [W.Batch(0, x[:150], x[150:][::-1] + (x[:150] == x[150:][::-1]), np.full(150, 0.5, np.float32), none, none)]
    return make


@pytest.mark.parametrize("C", [2, 3, 12])
@pytest.mark.parametrize("mode", [P.UPDATE_SYNCHRONOUS, P.UPDATE_IN_PLACE])
def test_a_graph_that_one_workgroup_has_no_room_for(C, mode):
    make = _crowded(20000, C, 600)
    want, logs0 = _solve_and_batches(make, 0, 1e-6, 20000, mode, {0: lambda d: d.set_shared_rounds(-1)})
    got, logs = _solve_and_batches(make, 0, 1e-6, 20000, mode)
    print([(len(a), _shared(a), len(b), _shared(b)) for a, b in zip(logs, logs0)])
    assert all(_shared(a) <= _shared(b) + len(a) // 4 for a, b in zip(logs, logs0)), "the kernel is meant to refuse"
    assert any(len(a) >= 40 for a in logs)
    if mode == P.UPDATE_SYNCHRONOUS:
        _same(got, want)
    for a, b in zip(got, want):
        k = 3 if len(a) < 8 else 6
        assert a[0] == b[0] == 0 and np.max(np.abs(a[k] - b[k])) <= 400 * 1e-6


# (24,000 entries: 70 KB for three workgroups, too much for one)
@pytest.mark.parametrize("workgroups,from_launch,shared", [(3, 0, 240), (31, 0, 240), (1, 0, 0), (1, 1, 240), (-1, 1, 240), (2, 1, 240)])
@pytest.mark.parametrize("C,deg", [(4, 9.0), (2, 9.5), (9, 9.0)])
def test_fewer_workgroups_than_wanted_and_launches_refused_amid_a_call(workgroups, from_launch, shared, C, deg):
    """From launch `from_launch` of each call on: where the entries do not fit, the call goes on with ordinary rounds from the lists,
    the counters and the label buffers that the launches before have left."""
    make = _random(2600, C, deg)
    want, _ = _solve_and_batches(make, 16, 1e-6, 20000, P.UPDATE_SYNCHRONOUS)
    few = lambda d: d.set_shared_rounds(workgroups, from_launch)
    got, logs = _solve_and_batches(make, 0, 1e-6, 20000, P.UPDATE_SYNCHRONOUS, {0: few, 1: few, 2: few})
    print([(len(log), _longest_launch(log)) for log in logs])
    for log in logs[:2]:
        assert len(log) > 240 + 64 and (_longest_launch(log) >= 240) == (shared == 240)
        if from_launch == 1 and workgroups != 2:
            assert _longest_launch(log[240:]) < 64
    _same(got, want)


def test_launches_are_numbered_anew_after_the_last_number():
    make = _random(2600, 4, 9.0)
    want, _ = _solve_and_batches(make, 16, 1e-6, 20000, P.UPDATE_SYNCHRONOUS)
    for last in ((1 << 24) - 1, (1 << 24) - 2, (1 << 24) - 3, 254, 255):
        number = lambda d: d.set_shared_rounds(last_launch=last)
        got, logs = _solve_and_batches(make, 0, 1e-6, 20000, P.UPDATE_SYNCHRONOUS, {0: number, 1: number})
        assert all(_longest_launch(log) >= 240 for log in logs[:2])
        _same(got, want)


def test_calls_of_several_contexts_at_the_same_time():
    """While other calls are at work a launch has fewer rounds than alone.  Wherever it ends, rounds and labels are those of a call on
    its own."""
    import torch

    cases = [(_random(2500, 4, 9.0), 1e-6), (_random(9001, 2, 12.0), 1e-6), (_random(20011, 3, 8.0), 1e-4), (_random(6001, 2, 3.0), 1e-6)]
    want = [_solve_and_batches(make, 0, tol, 20000, P.UPDATE_SYNCHRONOUS)[0] for make, tol in cases]
    wrong = []

    def work(k):
        stream = torch.cuda.Stream()
        for i in range(6):
            j = (k + i * (k + 1)) % len(cases)
            got = _solve_and_batches(cases[j][0], 0, cases[j][1], 20000, P.UPDATE_SYNCHRONOUS, stream=stream.cuda_stream)[0]
            for a, b in zip(got, want[j]):
                if not all(np.array_equal(x, y) for x, y in zip(a, b)):
                    wrong.append((k, i, j, [q for q, (x, y) in enumerate(zip(a, b)) if not np.array_equal(x, y)]))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


def test_a_call_does_not_keep_its_xcd_for_long_while_others_are_at_work():
    """Every launch of another context has workgroups for that XCD, which wait for the launch that holds it."""
    import torch

    make = _random(2500, 4, 9.0)
    time.sleep(0.3)  # (for a tenth of a second after calls have met, more of them are expected)
    _, alone = _solve_and_batches(make, 0, 1e-6, 20000, P.UPDATE_SYNCHRONOUS)
    assert _longest_launch(alone[0]) > 150
    enough, at_work = threading.Event(), threading.Event()

    def work():
        stream = torch.cuda.Stream()
        p, _ = _random(3001, 2, 6.0)()
        with P.DynLP(p.n, p.row_ptr, p.col, p.w, p.C, p.seed_vertex, p.seed_class, stream=stream.cuda_stream) as d:
            while not enough.is_set():
                d.static_solve(1e-5, 20000)
                at_work.set()

    other = threading.Thread(target=work)
    other.start()
    try:
        assert at_work.wait(60)
        stream = torch.cuda.Stream()
        logs = [_solve_and_batches(make, 0, 1e-6, 20000, P.UPDATE_SYNCHRONOUS, stream=stream.cuda_stream)[1] for _ in range(4)][-1]
    finally:
        enough.set()
        other.join()
    print("rounds of the longest launch", _longest_launch(alone[0]), [_longest_launch(log) for log in logs])
    assert _longest_launch(logs[0]) <= 48
