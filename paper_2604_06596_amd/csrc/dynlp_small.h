// Step 1 of small batches: several steps of a batch in one launch.
//
// A batch of a few items goes through some fifteen launches whose work is a trip or two to memory each: what it waits for is the
// launches (4 to 6 us each, whatever they do).  One workgroup goes from one of these steps to the next over a barrier.  Two
// launches therefore stand for nine and a copy:
//
//   k_small_check    the batch from pinned memory, counters cleared, checks, marks, deleted rows
//   k_small_insert   half-edges counted and listed, places planned, rows relocated, half-edges written
//
// Rows that lose entries, sorting and long rows keep their launches: they take a chain of trips to memory per row, and a workgroup
// has room for 64 rows at a time.  So does the first list: with it and the seeds as a third launch of one workgroup 3,001 vertices
// took 14 us instead of 8 and two launches, 20,000 vertices 40 instead of 9.  The steps are those of the ordinary kernels
// (dynlp_kernels.h), so that graph and labels are the same bits.  What is small: see small_batch in dynlp.hip.
// Measured (whole calls, before / after, with the counters sent by k_compact_start): one item into 3,001 vertices 182 / 164 us, 37
// into 20,011 285 / 274, 100 into 2,000 1,195 / 1,180.
#pragma once

#include "dynlp_kernels.h"

namespace dynlp {

constexpr int kSmallThreads = 1024;
constexpr int kSmallItems = 2;                                    // half-edges per thread
constexpr int64_t kSmallHalfEdges = kSmallThreads * kSmallItems;  // of a batch
constexpr int kSmallClear = 16;                                   // workgroups of k_small_check that clear the rounds' counters

struct SmallBatch {
    const uint4* from;  // the batch in pinned memory, `pieces` of 16 bytes, and where it goes (0: it is on the device)
    uint4* to;
    unsigned int pieces;
    uint4* ring;  // the rounds' counters, ring_pieces of 16 bytes; bc lies behind them
    unsigned int ring_pieces;
    unsigned long long pool_tail;
    int64_t nd, m, s, k, n0, n1;
    const int32_t *del, *eu, *ev, *sv, *sc;
    const float* ew;
    int C, Cs, coff, CP;
    float slack;
    BatchCtr* bc;
    RowMeta* meta;
    Edge* pool;
    unsigned long long pool_cap;
    int32_t *seed_class, *add_cnt, *touched, *dropping, *rank;  // rank: of 2m half-edges, or NULL
    int64_t* reloc_off;
    uint8_t* flag;
    float *deg, *F;
};

// Workgroups from 1 on clear the rounds' counters, which nothing else here looks at.
__global__ void __launch_bounds__(kSmallThreads) k_small_check(SmallBatch b) {
    const unsigned int tid = threadIdx.x;
    if (blockIdx.x > 0) {
        for (unsigned int i = (blockIdx.x - 1) * kSmallThreads + tid; i < b.ring_pieces; i += (gridDim.x - 1) * kSmallThreads)
            b.ring[i] = make_uint4(0u, 0u, 0u, 0u);
        return;
    }
    for (unsigned int i = tid; i < b.pieces; i += kSmallThreads) b.to[i] = b.from[i];
    batch_begin(tid, kSmallThreads, reinterpret_cast<unsigned int*>(b.bc), kBatchClear, b.bc, b.pool_tail);
    __syncthreads();
    for (int64_t i = tid; i < b.nd + b.m + b.s; i += kSmallThreads)
        validate_batch_item(i, b.nd, b.del, b.m, b.eu, b.ev, b.ew, b.s, b.sv, b.sc, b.n1, b.n0, b.C, b.seed_class, b.add_cnt, b.bc);
    __syncthreads();
    for (int64_t i = tid; i < b.nd + b.s + b.k; i += kSmallThreads)
        batch_prepare_item(i, b.bc, b.nd, b.del, b.s, b.sv, b.n1, b.add_cnt, b.n0, b.k, b.meta, b.deg, b.seed_class);
    if (b.nd == 0) return;
    __syncthreads();
    if (b.bc->err) return;
    for (unsigned int block = 0; (int64_t)block * (kSmallThreads / 16) < b.nd; ++block)
        delete_rows<kSmallThreads>(block, b.nd, b.del, b.C, b.Cs, b.CP, b.meta, b.pool, b.seed_class, b.flag, b.add_cnt, b.dropping, b.deg,
                                   b.F, b.bc);
}

// (Half-edges with an end out of range are not counted; after a failed check nothing else happens here.)
__global__ void __launch_bounds__(kSmallThreads) k_small_insert(SmallBatch b) {
    const unsigned int tid = threadIdx.x;
    const BatchGate gate{b.bc, b.pool_cap};
    for (int64_t i = tid; i < b.nd; i += kSmallThreads)
        if (b.bc->err == 0) b.seed_class[b.del[i]] = -1;
    if (b.m > 0) {
        count_halfedges<kSmallThreads, kSmallItems>(0, b.m, b.n1, b.eu, b.ev, b.add_cnt, b.touched, b.bc, b.rank,
                                                    b.rank ? b.rank + b.m : nullptr);
        __syncthreads();
        plan_reserve<kSmallThreads, 1>(b.touched, b.meta, b.add_cnt, b.slack, b.reloc_off, b.bc);
        __syncthreads();
    }
    for (int64_t i = tid; i < b.k * b.CP; i += kSmallThreads) init_label(i, b.n0, b.n1, b.C, b.Cs, b.coff, b.CP, b.seed_class, b.F);
    if (b.m == 0 || gate.closed()) return;
    relocate_rows<kSmallThreads>(b.touched, b.meta, b.add_cnt, b.slack, b.reloc_off, b.pool, gate);
    __syncthreads();
    for (int64_t i = tid; i < 2 * b.m; i += kSmallThreads) write_halfedge(i, b.m, b.eu, b.ev, b.ew, b.meta, b.pool, b.rank);
}

}  // namespace dynlp
