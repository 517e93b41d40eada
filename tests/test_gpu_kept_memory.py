"""Device memory of destroyed contexts waits for the next context of the process: several threads and streams at once get the
results of one, a context like the last takes no new memory, and what waits goes back when the program or an allocation asks for it.
(Which block, how many and for how long: test_kept_memory.py.)"""
import threading

import numpy as np
import pytest

import workloads as W
import paper_2604_06596_amd as P
from test_gpu_allocator import TorchAllocator

pytestmark = pytest.mark.gpu


def _problem(n, C):
    p, q = (W.small_random(n, C, 8.0, n // 20, 600 + C) for _ in range(2))
    return p, W.small_random_batch(q, n // 10, 7, 3, num_extra_edges=20)


def _pass(p, b, stream=None, **options):
    with P.DynLP(p.n, p.row_ptr, p.col, p.w, p.C, p.seed_vertex, p.seed_class, stream=stream, **options) as d:
        d.static_solve(1e-6, 20000)
        d.apply_batch(b.num_new_vertices, b.eu, b.ev, b.ew, b.seed_vertex, b.seed_class)
        return d.get_labels()


def test_threads_and_streams_share_it():
    import torch

    cases = [_problem(n, C) for n, C in ((3000, 4), (40000, 3), (9000, 12), (40000, 2))]
    want = [_pass(p, b) for p, b in cases]
    wrong = []

    def work(k):
        stream = torch.cuda.Stream()
        for i in range(8):
            p, b = cases[(k + i) % len(cases)]
            got = _pass(p, b, stream.cuda_stream)
            if not all(np.array_equal(x, y) for x, y in zip(got, want[(k + i) % len(cases)])):
                wrong.append((k, i))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


def test_it_is_used_again_and_given_back():
    import torch

    p, b = _problem(200000, 10)
    _pass(p, b)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    for _ in range(4):
        _pass(p, b)
    torch.cuda.synchronize()
    after = torch.cuda.mem_get_info()[0]
    assert before - after <= 32 << 20, "a context like the last takes no new memory"
    assert P.release_kept_memory() > 32 << 20 and P.release_kept_memory() == 0
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] - after > 32 << 20


def test_what_a_living_context_gives_back_is_the_device_s_again():
    """The old pool of a compaction or of a batch that outgrows it does not wait for another context."""
    import torch

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    p = W.small_random(20000, 4, 8.0, 500, 81)
    P.release_kept_memory()
    with P.DynLP(p.n, p.row_ptr, p.col, p.w, p.C, p.seed_vertex, p.seed_class, reserve_edges=40_000_000) as d:
        reserved = free()
        d.compact_storage()
        assert free() - reserved > 500 << 20  # (16 bytes to a reserved edge)
        before = free()
        rng = np.random.default_rng(5)
        none = np.zeros(0, np.int32)
        pools = []
        for m in (300_000, 600_000, 900_000, 1_000_000):
            u = rng.integers(0, p.n, m).astype(np.int32)
            v = ((u + 1 + rng.integers(0, p.n - 1, m)) % p.n).astype(np.int32)
            d.set_params(1e-2, 1)
            d.apply_batch(0, u, v, np.ones(m, np.float32), none, none)
            pools.append(8 * d.storage_info()[1])
        # the pool, the batch's arrays (12 bytes to an edge, 12 for its half-edges' ranks), some more for short rows
        assert before - free() < pools[-1] + (64 << 20), (before - free(), pools)
    assert P.release_kept_memory() > 0


def test_an_allocator_that_has_no_memory_is_asked_again_after_kept_memory_went_back():
    """What destroyed contexts left waiting stands on the same device as the allocator of the next one."""
    import torch

    p, b = _problem(200000, 10)
    want = _pass(p, b)
    torch.cuda.synchronize()
    held = torch.cuda.mem_get_info()[0]
    a = TorchAllocator()
    a.refuse = lambda nbytes: a.refused == 0 and a.calls > 5
    got = _pass(p, b, allocator=a)
    torch.cuda.synchronize()
    assert a.refused == 1 and not a.live
    assert all(np.array_equal(x, y) for x, y in zip(got, want))
    torch.cuda.empty_cache()
    assert torch.cuda.mem_get_info()[0] - held > 32 << 20
