"""The first list of a batch: every updatable vertex, and of these the flagged ones, found 64 vertices a step and 4, 8, 16 or 64
steps a wave (by the number of vertices).  Sizes at the ends of waves and workgroups, and at the sizes where the steps change."""
import numpy as np
import pytest

import paper_2604_06596_amd as P

pytestmark = pytest.mark.gpu

K = 1 << 10


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 257, 1023, 1024, 1025, 4097, 512 * K - 1, 512 * K, 512 * K + 1, 2048 * K - 1,
                               2048 * K + 3, 16384 * K - 1, 16384 * K + 65])
def test_the_first_list_holds_every_updatable_end_of_a_new_edge(n):
    rng = np.random.default_rng(n)
    none = np.zeros(0, np.int32)
    m = min(4 * n, 20000)
    u = rng.integers(0, n, m).astype(np.int32)
    v = rng.integers(0, n, m).astype(np.int32)
    if n > 1:  # the last vertices have edges too, one of them many (a long row)
        u[-1], v[-1] = n - 1, 0
        u[: min(m, 300)] = n - 1 - (n > 100)
    u, v = u[u != v], v[u != v]
    labelled = np.unique(rng.integers(0, n, max(1, n // 5))).astype(np.int32)
    ends = np.setdiff1d(np.union1d(u, v), labelled)
    with P.DynLP(0, np.zeros(1, np.int64), none, np.zeros(0, np.float32), 2, none, none, binary_scalar=True) as d:
        d.set_params(1e-4, 1)
        _, s = d.apply_batch(n, u, v, np.ones(u.shape[0], np.float32), labelled, labelled % 2)
        assert s.frontier_initial == ends.shape[0]
        log = d.round_log_full()
        if ends.size:  # the first round takes every listed row once
            assert log[0].rows_short + log[0].rows_long == ends.shape[0]
        # one more edge between two unlabelled vertices: only its ends are listed, whatever the list held before
        if ends.size > 1:
            a, b = ends[[0]], ends[[-1]]
            _, s = d.apply_batch(0, a, b, np.ones(1, np.float32), none, none)
            assert s.frontier_initial == 2
