"""GPU tests of the conjugate rounds of the in-place mode: every kernel that forms their product (packed, row by row, binned)
at the column counts where its layout changes, hub rows among them, against the exact labels; where there is no memory for
their arrays, and where the round cap leaves them too little room, the relaxed rounds run as before; iterations that the round
cap cuts or that make no progress, on 2D grids, where they are slow."""
import functools

import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W
from oracle import reference as R
import certify as Cf
import paper_2604_06596_amd as P
from test_gpu_allocator import TorchAllocator
from test_gpu_relaxed import TOL, _check, _make, _problem

pytestmark = pytest.mark.gpu


def _graph(p):
    return R.Graph(p.n, p.row_ptr, p.col, p.w, p.C, p.seed_vertex, p.seed_class)


@pytest.mark.parametrize("kind,C,kw", [
    ("sbm", 1, {}), ("sbm", 2, {}), ("sbm", 4, {}), ("hub", 5, {}), ("sbm", 8, {}), ("sbm", 9, {}), ("sbm", 16, {}), ("hub", 17, {}),
    ("sbm", 25, {}), ("hub", 32, {}), ("sbm", 33, {}), ("sbm", 41, {}), ("sbm", 53, {}), ("sbm", 64, {}),
    ("hub", 1, dict(group_lanes=4)), ("hub", 2, dict(group_lanes=8)), ("sbm", 7, dict(group_lanes=64)),
    ("hub", 31, dict(group_lanes=8)), ("hub", 64, dict(group_lanes=16)),
    ("hub", 2, dict(binary_scalar=True, group_lanes=16)), ("hub", 2, dict(binary_scalar=True)),
    ("hub", 2, dict(binary_scalar=True, binned_rounds=8)), ("sbm", 2, dict(binary_scalar=True, binned_rounds=15))])
def test_every_product_kernel_reaches_the_exact_labels(kind, C, kw):
    p = _problem(kind, C)
    with _make(p, **kw) as d:
        st, s = d.static_solve(TOL, 20000)
        assert st == 0 and s.final_max_delta <= TOL
        log = d.round_log_full()
        assert s.iterations == len(log) and s.edges_traversed == sum(r.entries_short + r.entries_long for r in log)
        soft, hard = d.get_labels()
        cap = s.iterations
        d.static_solve(TOL, 20000)  # labels that are there already
    _check(soft, hard, _graph(p), Cf.stop_rule_residual(TOL), f"{kind} {C} {kw}")
    # relaxed rounds need 50 and more on these graphs
    print(kind, C, kw, "rounds", cap)
    assert cap < 45


def test_without_memory_for_their_arrays_the_relaxed_rounds_run():
    p = _problem("sbm", 10)
    a = TorchAllocator()
    with _make(p, allocator=a) as d:
        rows = d.num_vertices + max(1024, p.n // 8)
        a.refuse = lambda nbytes: nbytes == rows * 16 * 4
        st, s = d.static_solve(TOL, 20000)
        assert st == 0 and a.refused > 0
        soft, hard = d.get_labels()
        a.refuse = lambda nbytes: False
        st, s2 = d.static_solve(TOL, 20000)
        assert st == 0
    assert not a.live
    _check(soft, hard, _graph(p), Cf.stop_rule_residual(TOL), "no memory")
    print("rounds", s.iterations)
    assert s.iterations > 40


@pytest.mark.parametrize("cap", [63, 64, 65])
def test_round_caps_on_either_side_of_the_smallest_budget(cap):
    p = _problem("sbm", 6)
    with _make(p) as d:
        st, s = d.static_solve(TOL, cap)
        assert s.iterations <= cap and (st == 0) == (s.converged == 1)
        soft, hard = d.get_labels()
        if st == 0:
            _check(soft, hard, _graph(p), Cf.stop_rule_residual(TOL), f"cap {cap}")
        assert st == 0 or cap < 64
        assert soft.min() >= 0 and soft.max() <= 1 and np.max(np.abs(soft.sum(1) - 1)) < 2e-5


def test_scarce_labels_settle():
    """One vertex in 2,000 labelled: a small smallest eigenvalue, where relaxation takes hundreds of rounds."""
    p = W.sbm(40000, 4, 12.0, 6.0, 0.0005, 5)
    with _make(p) as d:
        st, s = d.static_solve(TOL, 20000)
        assert st == 0
        soft, hard = d.get_labels()
    print("rounds", s.iterations)
    _check(soft, hard, _graph(p), Cf.stop_rule_residual(TOL), "scarce labels")


@pytest.mark.parametrize("kind,C,kw,power", [
    ("sbm", 10, {}, 122), ("sbm", 10, {}, -70), ("sbm", 3, {}, -119), ("sbm", 7, dict(group_lanes=16), 122), ("hub", 5, {}, -95),
    ("hub", 20, dict(group_lanes=8), -110), ("sbm", 2, dict(binary_scalar=True, binned_rounds=8), 122),
    ("sbm", 2, dict(binary_scalar=True, binned_rounds=8), -119), ("hub", 2, dict(binary_scalar=True), -100)])
def test_the_scale_of_the_weights_does_not_matter(kind, C, kw, power):
    """All weights times 2^power, with degrees that stay normal float32 numbers: every quotient is the same, so the labels are
    and so is the number of rounds (but for the order in which the sums of an iteration are added)."""
    p = _problem(kind, C)
    g = _graph(p)
    rounds = []
    for scale in (1.0, 2.0 ** power):
        w = p.w * np.float32(scale)
        assert np.all(np.isfinite(w)) and w.min() >= np.finfo(np.float32).tiny
        with P.DynLP(p.n, p.row_ptr, p.col, w, C, p.seed_vertex, p.seed_class, **kw) as d:
            d.set_update_mode(P.UPDATE_IN_PLACE)
            st, s = d.static_solve(TOL, 20000)
            assert st == 0
            rounds.append(s.iterations)
            soft, hard = d.get_labels()
        _check(soft, hard, g, Cf.stop_rule_residual(TOL), f"{kind} {C} {kw} {scale}")
    print(kind, C, kw, power, "rounds", rounds)
    assert rounds[1] < 45


def test_a_part_with_light_weights_settles_too():
    """Two graphs without an edge between them, the weights of one 2^-60 of the other's: what the light one adds to the sums of an
    iteration is beneath their last bit."""
    p = _problem("sbm", 6)
    n, e = p.n, len(p.col)
    w = np.concatenate([p.w, p.w * np.float32(2.0 ** -60)])
    rp = np.concatenate([p.row_ptr, p.row_ptr[1:] + e])
    col = np.concatenate([p.col, p.col + n]).astype(np.int32)
    sv, sc = np.concatenate([p.seed_vertex, p.seed_vertex + n]).astype(np.int32), np.concatenate([p.seed_class, p.seed_class])
    with P.DynLP(2 * n, rp, col, w, 6, sv, sc) as d:
        d.set_update_mode(P.UPDATE_IN_PLACE)
        st, s = d.static_solve(TOL, 20000)
        assert st == 0
        soft, hard = d.get_labels()
    print("rounds", s.iterations)
    for half in (slice(0, n), slice(n, 2 * n)):
        _check(soft[half], hard[half], _graph(p), Cf.stop_rule_residual(TOL), "light and heavy")


def test_degrees_beyond_float32_leave_numbers():
    """Every weight is finite, the sums of most rows are not: no result is promised, but the iteration ends, and with labels."""
    p = _problem("sbm", 4)
    with P.DynLP(p.n, p.row_ptr, p.col, p.w * np.float32(2.0 ** 126), 4, p.seed_vertex, p.seed_class) as d:
        d.set_update_mode(P.UPDATE_IN_PLACE)
        assert d.static_solve(TOL, 300)[0] in (0, 1)
        soft, _ = d.get_labels()
    assert np.all(np.isfinite(soft)) and soft.min() >= 0 and soft.max() <= 1
    assert np.array_equal(soft[p.seed_vertex].argmax(1), p.seed_class) and np.all(soft[p.seed_vertex].max(1) == 1)


@pytest.mark.parametrize("C,kw,how", [(10, {}, (2, True)), (7, dict(group_lanes=16), (2, False)),
                                      (2, dict(binary_scalar=True, binned_rounds=8), (3, False))])
def test_the_round_log_tells_iterations_from_rounds(C, kw, how):
    """An ordinary round, the iterations, an ordinary round: only those in between are marked as iterations; the last one's
    residual is beneath the threshold by the recurrence, and by the round that follows within what float32 labels allow."""
    p = _problem("sbm", C)
    with _make(p, time_kernels=True, **kw) as d:
        st, s = d.static_solve(TOL, 20000)
        assert st == 0
        log = d.round_log_full()
    marked = [r.launch_rounds < 0 for r in log]
    last = max(i for i, m in enumerate(marked) if m)
    assert marked == [False] + [True] * last + [False] * (len(log) - 1 - last)
    assert all((r.staged, r.group_lanes == 0) == how for r in log[:last + 2])
    assert all(r.ms_update > 0 for r in log)
    assert len({(r.rows_short, r.rows_long, r.entries_short, r.entries_long) for r in log[:last + 1]}) == 1
    assert log[last].max_delta <= 0.5 * TOL < log[last - 1].max_delta and log[last].rows_moved == 0
    # the labels differ from what the iteration holds in 64 bits by a rounding per iteration, and a mean by its own
    assert log[last + 1].max_delta <= 0.5 * TOL + (len(log) + 2) * 2.0 ** -24
    assert sum(r.ms_update for r in log) <= s.ms_update_kernel * (1 + 1e-5)  # (which has the launches that found the end reached)


SIDE, GRID_CLASSES = 200, 3


@functools.lru_cache(maxsize=None)
def _grid(labelled):
    """A weighted 2D grid of 200 x 200 vertices, `labelled` of them labelled: CSR, labels, degrees."""
    rng = np.random.default_rng(labelled)
    i = np.arange(SIDE * SIDE).reshape(SIDE, SIDE)
    eu, ev = np.concatenate([i[:, :-1].ravel(), i[:-1].ravel()]), np.concatenate([i[:, 1:].ravel(), i[1:].ravel()])
    rp, col, w = W.edges_to_csr(i.size, eu, ev, rng.uniform(0.1, 1, eu.size).astype(np.float32))
    sv = rng.permutation(i.size)[:labelled].astype(np.int32)
    sc = (np.arange(labelled) % GRID_CLASSES).astype(np.int32)
    return rp, col, w, sv, sc


@functools.lru_cache(maxsize=None)
def _iterates(labelled, C, most):
    """{rounds: labels} of a call cut after so many rounds, up to `most`, and the fixed point: the definition in 64 bits.  An ordinary round
    gives the first residual, conjugate iterations, rows made distributions, an ordinary round."""
    rp, col, w, sv, sc = _grid(labelled)
    n = len(rp) - 1
    A = sp.csr_matrix((w.astype(np.float64), col, rp), shape=(n, n))
    deg = np.asarray(A.sum(1)).ravel()
    P = (sp.diags(1.0 / deg) @ A).tocsr()
    free = np.ones((n, 1), bool)
    free[sv] = False
    x = np.full((n, C), 1.0 / C)
    x[sv] = 0.0
    x[sv, sc % C] = 1.0
    d = np.where(free, deg[:, None], 0.0)
    z = np.where(free, P @ x, x) - x
    p, zz, out = z.copy(), float((d * z * z).sum()), {}
    for rounds in range(3, 5000):
        v = np.where(free, p - P @ p, 0.0)
        alpha = zz / float((d * p * v).sum())
        x = x + alpha * p
        z = z - alpha * v
        new = float((d * z * z).sum())
        p, zz = z + new / zz * p, new
        if rounds <= most:
            y = np.clip(x, 0.0, 1.0)
            y = np.where(free, y / y.sum(1, keepdims=True), y)
            out[rounds] = np.where(free, P @ y, y)
        if np.abs(z).max() < 1e-13:
            break
    return out, x


def _solve_grid(labelled, C, cap, **kw):
    rp, col, w, sv, sc = _grid(labelled)
    with P.DynLP(len(rp) - 1, rp, col, w, C, sv, sc % C, **kw) as d:
        d.set_update_mode(P.UPDATE_IN_PLACE)
        st, s = d.static_solve(TOL, cap)
        log = d.round_log_full()
        assert s.iterations == len(log) and s.edges_traversed == sum(r.entries_short + r.entries_long for r in log)
        soft, hard = d.get_labels()
    assert soft.min() >= 0 and soft.max() <= 1 and np.max(np.abs(soft.sum(1) - 1)) < 2e-5
    assert np.array_equal(hard[sv], sc % C)
    return st, s, log, soft


@pytest.mark.parametrize("C,kw", [(3, {}), (3, dict(group_lanes=16)), (2, dict(binary_scalar=True, binned_rounds=8))])
@pytest.mark.parametrize("labelled", [400, 40])
def test_a_round_cap_amid_the_iteration(labelled, C, kw):
    """Caps next to each other end where a step still owes its share to the labels and where it does not.  The labels are those of as many
    iterations in 64 bits: a model of them in float32 is 2e-6 away, the kernels up to 1.1e-5, a step more or less 3e-3 and more.  As
    a whole they are nearer to the fixed point than the relaxed rounds of a smaller cap leave them."""
    iterates, exact = _iterates(labelled, C, 67)
    far = lambda f: float(np.linalg.norm(f - exact) / np.linalg.norm(exact))
    st, s, log, soft = _solve_grid(labelled, C, 63, **kw)
    assert st == 1 and s.iterations == 63 and not any(r.launch_rounds < 0 for r in log)
    relaxed = far(soft)
    for cap in (64, 65, 66, 67):
        st, s, log, soft = _solve_grid(labelled, C, cap, **kw)
        assert st == 1 and s.converged == 0 and s.iterations == cap
        assert [r.launch_rounds < 0 for r in log] == [False] + [True] * (cap - 2) + [False]
        off, step = np.max(np.abs(soft - iterates[cap])), np.max(np.abs(iterates[cap] - iterates[cap - 1]))
        print(labelled, C, kw, cap, f"off {off:.1e}, a step {step:.1e}, from the fixed point {far(soft):.1e}, relaxed {relaxed:.1e}")
        assert off < 5e-5 < 0.05 * step
        assert far(soft) < relaxed


def test_iterations_without_progress_give_way_to_relaxed_rounds():
    """Four labelled vertices: the largest residual stays where it is for more than 96 iterations while the labels are on
    their way; relaxed rounds go on from there, to the round cap."""
    _, exact = _iterates(4, 3, 3)
    far = lambda f: float(np.linalg.norm(f - exact) / np.linalg.norm(exact))
    off = {cap: far(_solve_grid(4, 3, cap)[3]) for cap in (63, 200)}
    st, s, log, soft = _solve_grid(4, 3, 900)
    marked = [r.launch_rounds < 0 for r in log]
    k = sum(marked)
    print("iterations", k, "of", s.iterations, "distances", off, far(soft))
    assert st == 1 and s.iterations == 900 and 96 < k < 800
    assert marked == [False] + [True] * k + [False] * (len(log) - k - 1)
    assert far(soft) < off[200] < off[63]


@pytest.mark.parametrize("mode", [P.UPDATE_SYNCHRONOUS, P.UPDATE_IN_PLACE])
def test_every_sweep_of_a_static_solve_is_timed(mode):
    """The events of the last sweeps are read after the stream is done, not when their counters have arrived."""
    p = _problem("sbm", 4)
    for _ in range(20):
        with P.DynLP(p.n, p.row_ptr, p.col, p.w, p.C, p.seed_vertex, p.seed_class, time_kernels=True) as d:
            d.set_update_mode(mode)
            _, s = d.static_solve(TOL, 200)
            log = d.round_log_full()
        assert len(log) == s.iterations and all(r.ms_update > 0 for r in log)
        assert s.ms_update_kernel >= sum(r.ms_update for r in log) * (1 - 1e-5)


def test_their_arrays_are_given_back():
    """After four calls in a row that cannot use them, not before, and by compact_storage; the next call that wants them gets
    them again."""
    p = _problem("sbm", 10)
    a = TorchAllocator()
    with _make(p, allocator=a) as d:
        size = (d.num_vertices + max(1024, p.n // 8)) * 16 * 4
        held = lambda: sum(t.numel() == size for t in a.live.values())
        plain = held()
        first = d.static_solve(TOL, 20000)[1].iterations
        assert held() == plain + 2
        rule_out = [lambda: d.set_update_mode(P.UPDATE_SYNCHRONOUS), lambda: d.set_params(1e-4, 20000), lambda: d.set_params(TOL, 40)]
        for change in rule_out:
            d.set_update_mode(P.UPDATE_IN_PLACE)
            assert d.static_solve(TOL, 20000)[1].iterations <= first and held() == plain + 2
            change()
            for call in range(1, 5):
                assert held() == plain + 2
                d.apply_batch(0, np.array([call], np.int32), np.array([call + 100], np.int32), np.array([1e-3], np.float32))
                if call == 2:  # one call in between that can use them
                    d.set_update_mode(P.UPDATE_IN_PLACE)
                    d.static_solve(TOL, 20000)
                    change()
            for call in range(2):
                assert held() == plain + 2
                d.apply_batch(0, np.array([call + 9], np.int32), np.array([call + 900], np.int32), np.array([1e-3], np.float32))
            assert held() == plain
        d.set_update_mode(P.UPDATE_IN_PLACE)
        assert d.static_solve(TOL, 20000)[0] == 0 and held() == plain + 2
        d.compact_storage()
        assert held() == plain
        assert d.static_solve(TOL, 20000)[0] == 0
        soft, _ = d.get_labels()
    assert not a.live and np.max(np.abs(soft.sum(1) - 1)) < 2e-5
