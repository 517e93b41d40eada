// HIP kernels of the DynLP hot path for gfx950 (wave64, no MFMA: the path is a sparse gather).
#pragma once

#include "dynlp_device.h"

namespace dynlp {

// =================================================================================================
// Slack-CSR construction (mutable CSR with per-row slack)
// =================================================================================================
__host__ __device__ inline int32_t row_capacity(int64_t len, float slack) {
    int64_t a = (int64_t)((double)len * (double)slack + 0.999999);
    int64_t b = len + 4;
    int64_t c = a > b ? a : b;
    c = (c + (kRowAlign - 1)) / kRowAlign * kRowAlign;
    return (int32_t)c;
}

// row_ptr must start at 0, never decrease and end at nnz.
__global__ void __launch_bounds__(kBlock) k_validate_row_ptr(int64_t n, const int64_t* __restrict__ row_ptr,
                                                            int64_t nnz, BatchCtr* bc) {
    const int64_t u = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (u >= n) return;
    const int64_t a = row_ptr[u], b = row_ptr[u + 1];
    if ((u == 0 && a != 0) || a > b || b > nnz || a < 0 || (b - a) > 0x7fffffff - 64) report_error(bc, kErrRowPtr, u);
}

// len, cap of every row and the per-block sums of the capacities.
__global__ void __launch_bounds__(kBlock) k_row_caps(int64_t n, const int64_t* __restrict__ row_ptr, float slack,
                                                    RowMeta* __restrict__ meta, int64_t* __restrict__ block_sums) {
    __shared__ int64_t sm[kBlock / kWave + 1];
    const int64_t u = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    int64_t cap = 0;
    if (u < n) {
        const int64_t len = row_ptr[u + 1] - row_ptr[u];
        cap = row_capacity(len, slack);
        meta[u].len = (int32_t)len;
        meta[u].cap = (int32_t)cap;
    }
    int64_t total;
    block_exclusive_scan<int64_t>(cap, sm, &total);
    if (threadIdx.x == 0) block_sums[blockIdx.x] = total;
}

// Exclusive scan of nb values in place by one workgroup; *grand_total receives the sum.
__global__ void __launch_bounds__(kBlock) k_scan_block_sums(int64_t nb, int64_t* __restrict__ sums,
                                                           unsigned long long* grand_total) {
    __shared__ int64_t sm[kBlock / kWave + 1];
    const int64_t per = (nb + kBlock - 1) / kBlock;
    const int64_t lo = (int64_t)threadIdx.x * per;
    const int64_t hi = lo + per < nb ? lo + per : nb;
    int64_t local = 0;
    for (int64_t i = lo; i < hi; ++i) local += sums[i];
    int64_t total;
    int64_t run = block_exclusive_scan<int64_t>(local, sm, &total);
    for (int64_t i = lo; i < hi; ++i) {
        const int64_t t = sums[i];
        sums[i] = run;
        run += t;
    }
    if (threadIdx.x == 0 && grand_total) *grand_total = (unsigned long long)total;
}

__global__ void __launch_bounds__(kBlock) k_row_offsets(int64_t n, RowMeta* __restrict__ meta,
                                                       const int64_t* __restrict__ block_offsets) {
    __shared__ int64_t sm[kBlock / kWave + 1];
    const int64_t u = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t cap = u < n ? meta[u].cap : 0;
    int64_t total;
    const int64_t ex = block_exclusive_scan<int64_t>(cap, sm, &total);
    if (u < n) meta[u].off = block_offsets[blockIdx.x] + ex;
}

// One thread per CSR entry: find its row, check it, store it in the pool.
__global__ void __launch_bounds__(kBlock) k_scatter_entries(int64_t nnz, int64_t n, const int64_t* __restrict__ row_ptr,
                                                           const int32_t* __restrict__ col,
                                                           const float* __restrict__ w,
                                                           const RowMeta* __restrict__ meta, Edge* __restrict__ pool,
                                                           BatchCtr* bc) {
    const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (j >= nnz) return;
    int64_t lo = 0, hi = n;  // largest u with row_ptr[u] <= j
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (row_ptr[mid] <= j) lo = mid; else hi = mid;
    }
    const int64_t u = lo;
    const int32_t c = col[j];
    const float ww = w[j];
    if (c < 0 || c >= n) { report_error(bc, kErrColRange, j); return; }
    if (c == u) { report_error(bc, kErrSelfLoop, j); return; }
    if (!(ww > 0.f) || !isfinite(ww)) { report_error(bc, kErrWeight, j); return; }
    Edge e;
    e.col = c;
    e.w = ww;
    pool[meta[u].off + (j - row_ptr[u])] = e;
}

// Degree d(u) = sum of the row's weights, in stored order (deterministic for a given order).
__global__ void __launch_bounds__(kBlock) k_row_degree(int64_t n, const RowMeta* __restrict__ meta,
                                                      const Edge* __restrict__ pool, float* __restrict__ deg) {
    constexpr int G = 16;
    const int64_t u = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / G;
    const int gl = threadIdx.x % G;
    if (u >= n) return;
    const RowMeta m = meta[u];
    float s = 0.f;
    for (int j = gl; j < m.len; j += G) s += pool[m.off + j].w;
#pragma unroll
    for (int d = G / 2; d > 0; d >>= 1) s += __shfl_xor(s, d, G);
    if (gl == 0) deg[u] = s;
}

// =================================================================================================
// Labels: initialisation, seed clamping, argmax, packing
// =================================================================================================
// Rows [u0, u1): seed rows one-hot, others uniform 1/C, padding columns 0.
// Stored column c holds class c + coff: coff = 0 and Cs = C normally; the binary scalar layout
// (C = 2) stores only class 1 (Cs = 1, coff = 1), class 0 being 1 - F_u.
__device__ inline void init_label(int64_t i, int64_t u0, int64_t u1, int C, int Cs, int coff, int CP,
                                  const int32_t* __restrict__ seed_class, float* __restrict__ F) {
    const int64_t u = u0 + i / CP;
    const int c = (int)(i % CP);
    if (u >= u1) return;
    const int sc = seed_class[u];
    float v = 0.f;
    if (c < Cs) v = sc < 0 ? 1.0f / (float)C : (c + coff == sc ? 1.0f : 0.0f);
    F[u * CP + c] = v;
}

__global__ void __launch_bounds__(kBlock) k_init_labels(int64_t u0, int64_t u1, int C, int Cs, int coff, int CP,
                                                       const int32_t* __restrict__ seed_class,
                                                       float* __restrict__ F) {
    init_label((int64_t)blockIdx.x * kBlock + threadIdx.x, u0, u1, C, Cs, coff, CP, seed_class, F);
}

__global__ void __launch_bounds__(kBlock) k_fill_i32(int64_t u0, int64_t u1, int32_t* __restrict__ a, int32_t v) {
    const int64_t i = u0 + (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < u1) a[i] = v;
}

// Seed i: range checks, clash with an existing label, two classes for one vertex in this list.
// tmp is an all-zero int32 scratch (n_total entries) that k_clear_seed_tmp or k_batch_prepare restores afterwards.
__device__ inline void validate_seed(int64_t i, int64_t n_total, int64_t n_existing, int C, const int32_t* __restrict__ sv,
                                     const int32_t* __restrict__ sc, const int32_t* __restrict__ seed_class,
                                     int32_t* __restrict__ tmp, BatchCtr* bc) {
    const int32_t v = sv[i], c = sc[i];
    if (v < 0 || v >= n_total) { report_error(bc, kErrSeedVertex, i); return; }
    if (c < 0 || c >= C) { report_error(bc, kErrSeedClass, i); return; }
    if (v < n_existing && seed_class[v] >= 0 && seed_class[v] != c) { report_error(bc, kErrRelabel, i); return; }
    const int32_t old = atomicCAS(&tmp[v], 0, c + 1);
    if (old != 0 && old != c + 1) report_error(bc, kErrSeedConflict, i);
}

__global__ void __launch_bounds__(kBlock) k_validate_seeds(int64_t s, int64_t n_total, int64_t n_existing, int C,
                                                          const int32_t* __restrict__ sv,
                                                          const int32_t* __restrict__ sc,
                                                          const int32_t* __restrict__ seed_class,
                                                          int32_t* __restrict__ tmp, BatchCtr* bc) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < s) validate_seed(i, n_total, n_existing, C, sv, sc, seed_class, tmp, bc);
}

__global__ void __launch_bounds__(kBlock) k_clear_seed_tmp(int64_t s, int64_t n_total, const int32_t* __restrict__ sv,
                                                          int32_t* __restrict__ tmp) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= s) return;
    const int32_t v = sv[i];
    if (v >= 0 && v < n_total) tmp[v] = 0;
}

__global__ void __launch_bounds__(kBlock) k_set_seed_class(int64_t s, const int32_t* __restrict__ sv,
                                                          const int32_t* __restrict__ sc,
                                                          int32_t* __restrict__ seed_class) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < s) seed_class[sv[i]] = sc[i];
}

// New seeds of a batch: clamp the row one-hot (the row is never updated again) and put the
// neighbours into V_aff.  16 lanes per seed.
__global__ void __launch_bounds__(kBlock) k_apply_seeds(int64_t s, const int32_t* __restrict__ sv,
                                                       const int32_t* __restrict__ sc, int Cs, int coff, int CP,
                                                       int32_t* __restrict__ seed_class, float* __restrict__ F,
                                                       const RowMeta* __restrict__ meta,
                                                       const Edge* __restrict__ pool, uint8_t* __restrict__ flag,
                                                       BatchGate gate) {
    constexpr int G = 16;
    if (gate.closed()) return;
    const int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / G;
    const int gl = threadIdx.x % G;
    if (i >= s) return;
    const int32_t v = sv[i], c = sc[i];
    if (gl == 0) seed_class[v] = c;
    for (int k = gl; k < CP; k += G) F[(int64_t)v * CP + k] = (k < Cs && k + coff == c) ? 1.0f : 0.0f;
    const RowMeta m = meta[v];
    for (int j = gl; j < m.len; j += G) flag[pool[m.off + j].col] = 1;
}

// Labels in the caller's format from one pass over the rows (either output may be NULL): soft without the padding columns, and
// hard[u] = argmax_c F[u][c], lowest index on ties.  A row of CP >= 4 floats is read by CP/4 adjacent lanes as one float4
// each (a coalesced 16*L-byte segment per row); the lanes' (value, index) pairs are merged with xor shuffles.  CP < 4 rows
// are read by one lane.  (1,000,000 rows of 10 columns: 25 + 13 us as two kernels.)  The soft rows leave through LDS as one run of
// words per workgroup: whole lines to memory (whole calls, us: 1,000,000 rows of 10 columns 39 -> 36, of 50 126 -> 113) and over
// the bus.
__global__ void __launch_bounds__(kBlock) k_labels(int64_t n, int C, int CP, const float* __restrict__ F,
                                                  float* __restrict__ soft, int32_t* __restrict__ hard) {
    const int L = CP >= 4 ? CP / 4 : 1;  // lanes per row: 1, 2, 4, 8 or 16
    const int64_t u = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / L;
    const int sub = threadIdx.x & (L - 1);
    const bool live = u < n;
    __shared__ float tile[4 * kBlock];  // the block's rows without padding: kBlock / L rows of C <= 4 * L columns
    const int R = kBlock / L;
    const int64_t u0 = (int64_t)blockIdx.x * R;
    float bv = -1.0f;  // label values are >= 0
    int best = 0;
    if (live) {
        const float* row = F + u * CP;
        float* const out = soft ? tile + (int)(u - u0) * C : nullptr;
        if (CP >= 4) {
            const float4 q = *reinterpret_cast<const float4*>(row + 4 * sub);
            const float v[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int c = 4 * sub + k;
                if (c >= C) continue;
                if (v[k] > bv) { bv = v[k]; best = c; }
                if (out) out[c] = v[k];
            }
        } else {
            bv = row[0];
            for (int c = 0; c < C; ++c) {
                const float x = row[c];
                if (x > bv) { bv = x; best = c; }
                if (out) out[c] = x;
            }
        }
    }
    if (soft) {
        __syncthreads();
        const int words = (int)(n - u0 < R ? n - u0 : R) * C;
        for (int i = threadIdx.x; i < words; i += kBlock) soft[u0 * C + i] = tile[i];
    }
    if (!hard) return;
    for (int d = L >> 1; d > 0; d >>= 1) {
        const float ov = __shfl_xor(bv, d);
        const int ob = __shfl_xor(best, d);
        if (ov > bv || (ov == bv && ob < best)) { bv = ov; best = ob; }
    }
    if (live && sub == 0) hard[u] = best;
}

// Binary scalar layout: hard label = the paper's 0.5 cut-off (class 1 iff F_u > 0.5, i.e. iff class 1
// beats class 0; a tie goes to class 0 like the argmax), soft row = (1 - F_u, F_u).
__global__ void __launch_bounds__(kBlock) k_scalar_labels(int64_t n, const float* __restrict__ F, float* __restrict__ soft,
                                                         int32_t* __restrict__ hard) {
    const int64_t u = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (u >= n) return;
    const float f = F[u];
    if (soft) {  // (two stores: the caller's array need not be aligned to 8 bytes)
        soft[2 * u] = 1.0f - f;
        soft[2 * u + 1] = f;
    }
    if (hard) hard[u] = f > 0.5f ? 1 : 0;
}

// =================================================================================================
// Edge insertion (Alg. 2 Step 1 for insertions) into the slack CSR
// =================================================================================================
__device__ inline void validate_edge(int64_t i, int64_t n_total, const int32_t* __restrict__ eu, const int32_t* __restrict__ ev,
                                     const float* __restrict__ ew, BatchCtr* bc, int64_t index_base) {
    const int32_t a = eu[i], b = ev[i];
    const float ww = ew[i];
    if (a < 0 || a >= n_total || b < 0 || b >= n_total) { report_error(bc, kErrEndpoint, index_base + i); return; }
    if (a == b) { report_error(bc, kErrSelfLoop, index_base + i); return; }
    if (!(ww > 0.f) || !isfinite(ww)) report_error(bc, kErrWeight, index_base + i);
}

// index_base: position of eu[0] in the caller's batch (the arrays may be one chunk of it), for the error report.
__global__ void __launch_bounds__(kBlock) k_validate_edges(int64_t m, int64_t n_total, const int32_t* __restrict__ eu,
                                                          const int32_t* __restrict__ ev,
                                                          const float* __restrict__ ew, BatchCtr* bc,
                                                          int64_t index_base = 0) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < m) validate_edge(i, n_total, eu, ev, ew, bc, index_base);
}

// ---- the steps of a batch that come before its edges are inserted -----------------------------------------------------
// All counters a batch uses: `words` 32-bit words from `zero` on are cleared, then the pool's tail is set.
__device__ inline void batch_begin(unsigned int first, unsigned int step, unsigned int* __restrict__ zero, unsigned int words, BatchCtr* bc,
                                   unsigned long long pool_tail) {
    for (unsigned int i = first; i < words; i += step) {
        const unsigned int* tail = reinterpret_cast<const unsigned int*>(&bc->pool_tail);
        zero[i] = zero + i == tail ? (unsigned int)pool_tail : zero + i == tail + 1 ? (unsigned int)(pool_tail >> 32) : 0u;
    }
    if (first == 0) bc->clock[0] = wall_clock64();
}

__global__ void __launch_bounds__(kBlock) k_batch_begin(unsigned int* __restrict__ zero, unsigned int words,
                                                       BatchCtr* bc, unsigned long long pool_tail) {
    batch_begin(blockIdx.x * kBlock + threadIdx.x, gridDim.x * kBlock, zero, words, bc, pool_tail);
}

// Every argument of a batch: nd deleted vertices, then m edges, then s seeds.
__device__ inline void validate_batch_item(int64_t i, int64_t nd, const int32_t* __restrict__ del, int64_t m,
                                           const int32_t* __restrict__ eu, const int32_t* __restrict__ ev, const float* __restrict__ ew,
                                           int64_t s, const int32_t* __restrict__ sv, const int32_t* __restrict__ sc, int64_t n_total,
                                           int64_t n_existing, int C, const int32_t* __restrict__ seed_class, int32_t* __restrict__ tmp,
                                           BatchCtr* bc) {
    if (i < nd) {
        if (del[i] < 0 || del[i] >= n_existing) report_error(bc, kErrDeleted, i);
        return;
    }
    i -= nd;
    if (i < m) {
        validate_edge(i, n_total, eu, ev, ew, bc, 0);
        return;
    }
    i -= m;
    if (i < s) validate_seed(i, n_total, n_existing, C, sv, sc, seed_class, tmp, bc);
}

__global__ void __launch_bounds__(kBlock) k_validate_batch(int64_t nd, const int32_t* __restrict__ del, int64_t m,
                                                          const int32_t* __restrict__ eu, const int32_t* __restrict__ ev,
                                                          const float* __restrict__ ew, int64_t s,
                                                          const int32_t* __restrict__ sv, const int32_t* __restrict__ sc,
                                                          int64_t n_total, int64_t n_existing, int C,
                                                          const int32_t* __restrict__ seed_class, int32_t* __restrict__ tmp,
                                                          BatchCtr* bc) {
    validate_batch_item((int64_t)blockIdx.x * kBlock + threadIdx.x, nd, del, m, eu, ev, ew, s, sv, sc, n_total, n_existing, C, seed_class,
                        tmp, bc);
}

constexpr int32_t kDeletedMark = -2;  // seed_class value of a vertex while its batch deletes it

// Deleted vertices marked (nd of them, if the checks have passed), the seeds' scratch cleared (s), empty rows for the new ids
// n0 .. n0 + k - 1 (they are nobody's until the batch is done).
__device__ inline void batch_prepare_item(int64_t i, const BatchCtr* bc, int64_t nd, const int32_t* __restrict__ del, int64_t s,
                                          const int32_t* __restrict__ sv, int64_t n_total, int32_t* __restrict__ tmp, int64_t n0, int64_t k,
                                          RowMeta* __restrict__ meta, float* __restrict__ deg, int32_t* __restrict__ seed_class) {
    if (i < nd) {
        if (bc->err == 0) seed_class[del[i]] = kDeletedMark;
        return;
    }
    i -= nd;
    if (i < s) {
        const int32_t v = sv[i];
        if (v >= 0 && v < n_total) tmp[v] = 0;
        return;
    }
    i -= s;
    if (i < k) {
        RowMeta m;
        m.off = 0;
        m.len = 0;
        m.cap = 0;
        meta[n0 + i] = m;
        deg[n0 + i] = 0.f;
        seed_class[n0 + i] = -1;
    }
}

__global__ void __launch_bounds__(kBlock) k_batch_prepare(const BatchCtr* bc, int64_t nd, const int32_t* __restrict__ del,
                                                         int64_t s, const int32_t* __restrict__ sv, int64_t n_total,
                                                         int32_t* __restrict__ tmp, int64_t n0, int64_t k,
                                                         RowMeta* __restrict__ meta, float* __restrict__ deg,
                                                         int32_t* __restrict__ seed_class) {
    batch_prepare_item((int64_t)blockIdx.x * kBlock + threadIdx.x, bc, nd, del, s, sv, n_total, tmp, n0, k, meta, deg, seed_class);
}

// Half-edge i < m has source eu[i]; half-edge m + i has source ev[i].  Count the entries each row
// will receive and list every row that receives any ("touched" rows).  Out-of-range sources are
// skipped (the validation kernel reports them).  A workgroup takes kAppendItems * kBlock half-edges
// and appends its first-touched rows with one counter atomic.
// rank_u / rank_v (both or neither): what the counting atomic returned for half-edge i / m + i, i.e. the
// half-edge's place among the entries this batch appends to its row; k_write_halfedges then needs no second atomic.
// touched NULL: only counted, the rows are listed afterwards (k_list_touched).
// One step of one workgroup: ITEMS * NT half-edges from `base` on.
template <int NT, int ITEMS>
__device__ inline void count_halfedges(int64_t base, int64_t m, int64_t n_total, const int32_t* __restrict__ eu,
                                       const int32_t* __restrict__ ev, int32_t* __restrict__ add_cnt, int32_t* __restrict__ touched,
                                       BatchCtr* bc, int32_t* __restrict__ rank_u, int32_t* __restrict__ rank_v) {
    __shared__ unsigned int smem[NT / kWave + 1];
    int32_t srcs[ITEMS];
    unsigned int firstmask = 0;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int64_t i = base + (int64_t)k * NT + threadIdx.x;
        int32_t src = -1;
        if (i < 2 * m) {
            src = i < m ? eu[i] : ev[i - m];
            if (src >= 0 && src < n_total) {
                const int32_t r = atomicAdd(&add_cnt[src], 1);
                if (r == 0 && touched) firstmask |= 1u << k;
                if (rank_u) (i < m ? rank_u[i] : rank_v[i - m]) = r;
            }
        }
        srcs[k] = src;
    }
    if (!touched) return;
    unsigned int slot = block_reserve<NT>(&bc->touched, (unsigned int)__popc(firstmask), smem);
#pragma unroll
    for (int k = 0; k < ITEMS; ++k)
        if ((firstmask >> k) & 1u) touched[slot++] = srcs[k];
}

// Workgroups from count_blocks on take the marks from the nd deleted vertices again (if the checks have passed).
__global__ void __launch_bounds__(kBlock) k_count_halfedges(int64_t m, int64_t n_total, const int32_t* __restrict__ eu,
                                                           const int32_t* __restrict__ ev,
                                                           int32_t* __restrict__ add_cnt,
                                                           int32_t* __restrict__ touched, BatchCtr* bc,
                                                           int32_t* __restrict__ rank_u, int32_t* __restrict__ rank_v,
                                                           unsigned int count_blocks, int64_t nd,
                                                           const int32_t* __restrict__ del, int32_t* __restrict__ seed_class) {
    if (blockIdx.x >= count_blocks) {
        const int64_t i = (int64_t)(blockIdx.x - count_blocks) * kBlock + threadIdx.x;
        if (i < nd && bc->err == 0) seed_class[del[i]] = -1;
        return;
    }
    count_halfedges<kBlock, kAppendItems>((int64_t)blockIdx.x * kBlock * kAppendItems, m, n_total, eu, ev, add_cnt, touched, bc, rank_u,
                                          rank_v);
}

// The rows that receive entries, in runs of ascending ids: rows that move to the pool's tail then lie there in the order of
// their vertices, and everything that goes through the list or through the rows finds neighbours next to each other (listed
// as they were touched first, 50M vertices and 250M half-edges lay in random order).  A workgroup lists 4,096 vertices.
__global__ void __launch_bounds__(kBlock) k_list_touched(int64_t n, const int32_t* __restrict__ add_cnt,
                                                        int32_t* __restrict__ touched, BatchCtr* bc) {
    __shared__ unsigned int smem[kBlock / kWave + 1];
    constexpr int PER = 16;
    const int64_t v0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * PER;
    unsigned int mask = 0;
    if (v0 + PER <= n) {
        int4 c[PER / 4];
#pragma unroll
        for (int q = 0; q < PER / 4; ++q) c[q] = reinterpret_cast<const int4*>(add_cnt + v0)[q];
#pragma unroll
        for (int q = 0; q < PER / 4; ++q)
            mask |= ((c[q].x ? 1u : 0u) | (c[q].y ? 2u : 0u) | (c[q].z ? 4u : 0u) | (c[q].w ? 8u : 0u)) << (4 * q);
    } else {
        for (int k = 0; k < PER && v0 + k < n; ++k)
            if (add_cnt[v0 + k]) mask |= 1u << k;
    }
    unsigned int slot = block_reserve(&bc->touched, (unsigned int)__popc(mask), smem);
    while (mask) {
        const int k = __ffs(mask) - 1;
        mask &= mask - 1;
        touched[slot++] = (int32_t)(v0 + k);
    }
}

// Rows whose slack cannot take the new entries get room at the pool tail (one tail atomic per workgroup: atomics
// on one address run at about 1e8 per second); reloc_off[t] is the new offset or -1.  Touches no row: bc->pool_tail
// afterwards tells the host how large the pool has to be before k_relocate may run.
template <int NT, int ITEMS>
__device__ inline void plan_reserve(const int32_t* __restrict__ touched, const RowMeta* __restrict__ meta,
                                    const int32_t* __restrict__ add_cnt, float slack, int64_t* __restrict__ reloc_off, BatchCtr* bc) {
    __shared__ unsigned long long smem[NT / kWave + 1];
    __shared__ unsigned long long sbase;
    if (bc->err) return;
    const unsigned int nt = bc->touched;
    // ITEMS rows per thread: with one, 195,000 workgroups queue for the tail when 50M rows are touched (4.6 ms, with 8 1.4);
    // with 8, a few hundred thousand rows keep too few lanes busy (400,000: 6 us with one, 14 with 8)
    for (unsigned int t0 = blockIdx.x * NT * ITEMS; t0 < nt; t0 += gridDim.x * NT * ITEMS) {  // uniform in the workgroup
        unsigned int caps[ITEMS];
        unsigned long long cap = 0;
        unsigned int moved = 0;
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const unsigned int t = t0 + threadIdx.x * ITEMS + k;
            caps[k] = 0;
            if (t < nt) {
                const int32_t u = touched[t];
                const RowMeta m = meta[u];
                const int64_t need = (int64_t)m.len + add_cnt[u];
                if (need > m.cap) caps[k] = (unsigned int)row_capacity(need, slack);
            }
            cap += caps[k];
            moved += caps[k] ? 1u : 0u;
        }
        unsigned long long total, rows;
        unsigned long long at = block_exclusive_scan<unsigned long long, NT>(cap, smem, &total);
        (void)block_exclusive_scan<unsigned long long, NT>(moved, smem, &rows);
        if (threadIdx.x == 0) {
            sbase = total ? atomicAdd(&bc->pool_tail, total) : 0ull;
            if (rows) atomicAdd(&bc->relocated, (unsigned int)rows);
        }
        __syncthreads();
        at += sbase;
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const unsigned int t = t0 + threadIdx.x * ITEMS + k;
            if (t < nt) reloc_off[t] = caps[k] ? (int64_t)at : -1;
            at += caps[k];
        }
        __syncthreads();
    }
}

template <int ITEMS>
__global__ void __launch_bounds__(kBlock) k_plan_reserve(const int32_t* __restrict__ touched,
                                                        const RowMeta* __restrict__ meta,
                                                        const int32_t* __restrict__ add_cnt, float slack,
                                                        int64_t* __restrict__ reloc_off, BatchCtr* bc) {
    plan_reserve<kBlock, ITEMS>(touched, meta, add_cnt, slack, reloc_off, bc);
}

// Give every relocated row its new place.  One lane per touched row; rows that already hold entries (few, but
// hubs among them) are copied by the whole wave, one row after the other.
template <int NT>
__device__ inline void relocate_rows(const int32_t* __restrict__ touched, RowMeta* __restrict__ meta, const int32_t* __restrict__ add_cnt,
                                     float slack, const int64_t* __restrict__ reloc_off, Edge* __restrict__ pool, const BatchGate& gate) {
    if (gate.closed()) return;
    const unsigned int nt = gate.bc->touched;
    const int lane = lane_id();
    for (unsigned int t0 = blockIdx.x * NT; t0 < nt; t0 += gridDim.x * NT) {
        const unsigned int t = t0 + threadIdx.x;
        const int64_t noff = t < nt ? reloc_off[t] : -1;
        int64_t ooff = 0;
        int len = 0;
        if (noff >= 0) {
            const int32_t u = touched[t];
            const RowMeta m = meta[u];
            ooff = m.off;
            len = m.len;
            RowMeta r;
            r.off = noff;
            r.len = m.len;
            r.cap = row_capacity((int64_t)m.len + add_cnt[u], slack);
            meta[u] = r;
        }
        unsigned long long todo = __ballot(len > 0);
        while (todo) {
            const int l = __ffsll((long long)todo) - 1;
            todo &= todo - 1;
            const int64_t from = __shfl(ooff, l), to = __shfl(noff, l);
            const int n = __shfl(len, l);
            for (int j = lane; j < n; j += kWave) pool[to + j] = pool[from + j];
        }
    }
}

__global__ void __launch_bounds__(kBlock) k_relocate(const int32_t* __restrict__ touched,
                                                    RowMeta* __restrict__ meta, const int32_t* __restrict__ add_cnt,
                                                    float slack, const int64_t* __restrict__ reloc_off,
                                                    Edge* __restrict__ pool, BatchGate gate) {
    relocate_rows<kBlock>(touched, meta, add_cnt, slack, reloc_off, pool, gate);
}

// Append both directions of every new edge.  With ranks (k_count_halfedges): the entry goes to position
// len + rank of its row and the row's length stays as it was (k_sort_finish adds the batch's count); without: the
// position comes from an atomic on the length.  Either way the order of one batch's entries inside a row is
// unspecified until they are sorted.
__device__ inline void write_halfedge(int64_t i, int64_t m, const int32_t* __restrict__ eu, const int32_t* __restrict__ ev,
                                      const float* __restrict__ ew, RowMeta* __restrict__ meta, Edge* __restrict__ pool,
                                      const int32_t* __restrict__ rank) {
    const int64_t k = i < m ? i : i - m;
    const int32_t src = i < m ? eu[k] : ev[k];
    const int32_t dst = i < m ? ev[k] : eu[k];
    Edge e;
    e.col = dst;
    e.w = ew[k];
    if (rank) {
        const RowMeta r = meta[src];
        pool[r.off + r.len + rank[i]] = e;
    } else {
        const int slot = atomicAdd(&meta[src].len, 1);
        pool[meta[src].off + slot] = e;
    }
}

__global__ void __launch_bounds__(kBlock) k_write_halfedges(int64_t m, const int32_t* __restrict__ eu,
                                                           const int32_t* __restrict__ ev,
                                                           const float* __restrict__ ew, RowMeta* __restrict__ meta,
                                                           Edge* __restrict__ pool, const int32_t* __restrict__ rank,
                                                           BatchGate gate) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= 2 * m || gate.closed()) return;
    write_halfedge(i, m, eu, ev, ew, meta, pool, rank);
}

// d(u) of a row by a whole workgroup, added in the order in which a 16-lane group adds it (lane j mod 16 takes entry j, then
// the lanes' sums by halves): the weights pass through LDS in tiles, so that the 16 chains of additions wait for nothing.  A
// hub of 50,000 entries: 390 dependent trips to memory of 16 lanes took 100 to 200 us.  Thread 0 has the sum.
constexpr int kHubRow = 1024;    // rows longer than this are handled by a workgroup in the passes of a batch
constexpr int kDegTile = 4096;   // weights per tile, a multiple of 16

template <int T>
__device__ inline float block_row_degree(const Edge* row, int len, float* tile) {
    constexpr int G = 16, UN = 8;
    float s = 0.f;
    for (int t0 = 0; t0 < len; t0 += kDegTile) {
        const int m = len - t0 < kDegTile ? len - t0 : kDegTile;
        for (int i = threadIdx.x; i < m; i += T) tile[i] = row[t0 + i].w;
        __syncthreads();
        if (threadIdx.x < G)
            for (int j0 = threadIdx.x; j0 < m; j0 += UN * G) {
                float wv[UN];
#pragma unroll
                for (int q = 0; q < UN; ++q) wv[q] = j0 + q * G < m ? tile[j0 + q * G] : 0.f;
#pragma unroll
                for (int q = 0; q < UN; ++q)
                    if (j0 + q * G < m) s += wv[q];
            }
        __syncthreads();
    }
    if (threadIdx.x < G) {
#pragma unroll
        for (int d = G / 2; d > 0; d >>= 1) s += __shfl_xor(s, d, G);
    }
    return s;
}

// The entries one batch appends to a row land in the order their atomics happened to take.  Sorting
// the appended segment by (neighbour id, weight bits) makes the stored row, and with it every sum
// over the row, a function of the batch alone.  G lanes per touched row (16; 8 where rows receive a few entries each, whose
// other lanes would have nothing to do: 50M rows of 5, 9.8 -> 5.5 ms; 330,000 of 1 to 20, 45 -> 30 us); segments of up to
// G * kSortRegs entries are rank-sorted in registers (every key is broadcast to the group once),
// longer ones than 16 lanes hold are queued for k_sort_long_segments.
__device__ inline unsigned long long edge_key(const Edge& e) {
    return ((unsigned long long)(unsigned int)e.col << 32) | (unsigned long long)__float_as_uint(e.w);
}

__device__ inline Edge key_edge(unsigned long long k) {
    Edge e;
    e.col = (int32_t)(unsigned int)(k >> 32);
    e.w = __uint_as_float((unsigned int)(k & 0xffffffffull));
    return e;
}

// ... and, for the same rows, what ends Step 1: d(u) recomputed from the stored row (entries added in position
// order, lane j mod 16 takes entry j), the counting scratch cleared, the row put into V_aff (both endpoints of every
// inserted edge are affected).  The sorted weights go through LDS so that the sum needs no second pass over the row.
// len_is_old: the rows' lengths do not yet include the appended entries (k_write_halfedges with ranks); the kernel
// then stores the new length.  Rows with long appended segments only get their length and are listed (long_list), hubs that
// received a few entries are sorted and listed for k_sort_long_segments (hub_list), which ends Step 1 for both.
struct SortFinish {
    RowMeta* meta;
    Edge* pool;
    int32_t* add_cnt;
    int len_is_old;
    int32_t *long_list, *hub_list;
    int64_t list_cap;  // entries of long_list: at least the rows that are touched
    BatchCtr* bc;
    float* deg;
    uint8_t* flag;
};

// One row per group of G lanes (own: the group has one, at *row), all threads of the workgroup take part.  sorted_w: a group's
// part stays with its wave.
template <int G>
__device__ inline void sort_finish_row(const SortFinish& f, bool own, const int32_t* __restrict__ row, float (*sorted_w)[G * kSortRegs]) {
    constexpr int L = 16, P = L / G;  // sums: entry j goes to sum j mod L, P sums per lane
    const int gl = threadIdx.x % G;
    const int grp = threadIdx.x / G;
    int32_t u = 0;
    int a = 0, len_old = 0;
    RowMeta m;
    m.off = 0;
    m.len = 0;
    m.cap = 0;
    bool is_long = false;
    if (own) {
        u = *row;
        a = f.add_cnt[u];
        m = f.meta[u];
        len_old = f.len_is_old ? m.len : m.len - a;
        is_long = a > G * kSortRegs;
    }
    Edge* seg = f.pool + m.off + len_old;
    if (own && !is_long) {
        const int slots = (a + G - 1) / G;  // uniform in the group
        unsigned long long key[kSortRegs];
#pragma unroll
        for (int r = 0; r < kSortRegs; ++r) {
            const int j = r * G + gl;
            key[r] = (r < slots && j < a) ? edge_key(seg[j]) : ~0ull;
        }
        int rank[kSortRegs];
#pragma unroll
        for (int r = 0; r < kSortRegs; ++r) rank[r] = r * G + gl;
        if (a > 1) {
#pragma unroll
            for (int r = 0; r < kSortRegs; ++r) rank[r] = 0;
#pragma unroll
            for (int r2 = 0; r2 < kSortRegs; ++r2) {
                if (r2 < slots) {
                    for (int l = 0; l < G; ++l) {
                        const unsigned int hi = __shfl((unsigned int)(key[r2] >> 32), l, G);
                        const unsigned int lo = __shfl((unsigned int)(key[r2] & 0xffffffffull), l, G);
                        const unsigned long long other = ((unsigned long long)hi << 32) | lo;
                        const int oj = r2 * G + l;
#pragma unroll
                        for (int r = 0; r < kSortRegs; ++r) {
                            const int j = r * G + gl;
                            rank[r] += (other < key[r] || (other == key[r] && oj < j)) ? 1 : 0;
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int r = 0; r < kSortRegs; ++r) {
            const int j = r * G + gl;
            if (r < slots && j < a) {
                const Edge e = key_edge(key[r]);
                if (a > 1) seg[rank[r]] = e;
                sorted_w[grp][rank[r]] = e.w;
            }
        }
    }
    __syncthreads();
    if (!own) return;
    const int len_new = len_old + a;
    if (is_long) {
        if (gl == 0) {
            if (G < 16 && a <= 16 * kSortRegs && len_new <= kHubRow) {
                f.long_list[f.list_cap - 1 - (int64_t)atomicAdd(&f.bc->sort_wide, 1u)] = u;
            } else {
                if (f.len_is_old) f.meta[u].len = len_new;
                f.long_list[atomicAdd(&f.bc->sort_long, 1u)] = u;
            }
        }
        return;
    }
    if (len_new > kHubRow) {
        if (gl == 0) {
            if (f.len_is_old) f.meta[u].len = len_new;
            f.hub_list[atomicAdd(&f.bc->finish_hubs, 1u)] = u;
        }
        return;
    }
    float sum[P];
#pragma unroll
    for (int p = 0; p < P; ++p) sum[p] = 0.f;
    constexpr int UN = 4;  // rounds of L entries whose loads are in flight, added in order
    for (int j0 = gl; j0 < len_new; j0 += UN * L) {
        float wv[UN][P];
#pragma unroll
        for (int q = 0; q < UN; ++q)
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const int j = j0 + q * L + p * G;
                wv[q][p] = j < len_old ? f.pool[m.off + j].w : (j < len_new ? sorted_w[grp][j - len_old] : 0.f);
            }
#pragma unroll
        for (int q = 0; q < UN; ++q)
#pragma unroll
            for (int p = 0; p < P; ++p)
                if (j0 + q * L + p * G < len_new) sum[p] += wv[q][p];
    }
    // the sums by halves: l and l + 8, l and l + 4, ...
    float s = sum[0];
    if constexpr (P == 2) s += sum[1];
#pragma unroll
    for (int d = G / 2; d > 0; d >>= 1) s += __shfl_xor(s, d, G);
    if (gl == 0) {
        if (f.len_is_old) f.meta[u].len = len_new;
        f.deg[u] = s;
        f.add_cnt[u] = 0;
        if (f.flag) f.flag[u] = 1;
    }
}

// With 8 lanes per row, rows of 65 to 128 appended entries are listed for 16 lanes of k_sort_long_segments (from the end of
// long_list), not for whole workgroups: a power law has many of them (1M vertices of mean degree 38, 10,000 / 50,000 / 100,000
// of them replaced; k_sort_finish + k_sort_long_segments, us: all with 16 lanes 84 + 369 / 211 + 664 / 316 + 960, 8 lanes and
// workgroups 69 + 402 / 147 + 777 / 209 + 1183, 8 and 16 lanes 66 + 372 / 146 + 697 / 197 + 1007; 200,000 of mean degree 30, 10,000
// replaced: 47 + 76, 37 + 97, 36 + 88).  16 lanes in a second pass of this kernel take its registers up (planted blocks, 100,000
// of 1M replaced, 116 -> 135).
template <int G>
__global__ void __launch_bounds__(kBlock) k_sort_finish(const int32_t* __restrict__ touched, SortFinish f, BatchGate gate) {
    __shared__ float sorted_w[kBlock / G][G * kSortRegs];
    if (gate.closed()) return;
    const unsigned int nt = f.bc->touched;
    for (unsigned int t0 = blockIdx.x * (kBlock / G); t0 < nt; t0 += gridDim.x * (kBlock / G)) {  // uniform in the workgroup
        const unsigned int t = t0 + threadIdx.x / G;
        sort_finish_row<G>(f, t < nt, touched + t, sorted_w);
    }
}

// Long appended segments: one workgroup of kSortThreads per row sorts the segment with a bitonic network whose
// compare-exchanges all point the same way (the first step of every merge pairs i with its mirror image inside
// the block), so positions past the end act as +infinity.  The network runs on tiles of kSortTile keys in LDS:
// a segment of one tile (a power-law hub that receives a few thousand entries from one batch) never goes to memory
// in between; a longer one (a new hub vertex arriving with tens of thousands of entries) is first sorted tile by
// tile, and of every later merge only the steps whose partners lie in different tiles run in memory (6 of 136 steps
// for 50,000 entries), UN disjoint pairs in flight per lane.
constexpr int kSortThreads = 1024;
constexpr int kSortTile = 8192;

// steps j = j_first, j_first / 2, ..., 1 of the network on the first `len` positions (a power of two) of a tile held
// in LDS; mirror: the first of them pairs i with its mirror image inside blocks of 2 * j_first
__device__ inline void sort_tile_steps(unsigned long long* keys, unsigned int len, unsigned int j_first, bool mirror) {
    for (unsigned int j = j_first; j > 0; j >>= 1) {
        const unsigned int mask = (mirror && j == j_first) ? (2 * j_first - 1) : j;
        for (unsigned int i = threadIdx.x; i < len; i += kSortThreads) {
            const unsigned int l = i ^ mask;
            if (l > i) {
                const unsigned long long x = keys[i], y = keys[l];
                if (y < x) {
                    keys[i] = y;
                    keys[l] = x;
                }
            }
        }
        __syncthreads();
    }
}

__global__ void __launch_bounds__(kSortThreads) k_sort_long_segments(SortFinish f) {
    __shared__ unsigned long long keys[kSortTile];
    constexpr unsigned int T = kSortTile;
    const unsigned int count = f.bc->sort_long, hubs = f.bc->finish_hubs, wide = f.bc->sort_wide;
    Edge* const pool = f.pool;
    // ... and then, as k_sort_finish does for the others: d(u) from the stored row, the counting scratch cleared, the row
    // put into V_aff
    auto finish = [&](int32_t u, const RowMeta& m) {
        const float d = block_row_degree<kSortThreads>(pool + m.off, m.len, reinterpret_cast<float*>(keys));
        if (threadIdx.x == 0) {
            f.deg[u] = d;
            f.add_cnt[u] = 0;
            if (f.flag) f.flag[u] = 1;
        }
    };
    for (unsigned int q = blockIdx.x; q < count + hubs; q += gridDim.x) {  // uniform per workgroup
        const int32_t u = q < count ? f.long_list[q] : f.hub_list[q - count];
        const RowMeta m = f.meta[u];
        if (q >= count) {
            finish(u, m);
            continue;
        }
        const unsigned int a = (unsigned int)f.add_cnt[u];
        Edge* seg = pool + m.off + (m.len - (int)a);
        unsigned int P = 2;
        while (P < a) P <<= 1;
        const unsigned int L = P < T ? P : T;  // positions of a tile the network works on (all of it from T keys on)
        const unsigned int tiles = (a + T - 1) / T;
        auto load_tile = [&](unsigned int t) {
            for (unsigned int i = threadIdx.x; i < L; i += kSortThreads)
                keys[i] = t * T + i < a ? edge_key(seg[t * T + i]) : ~0ull;
            __syncthreads();
        };
        auto store_tile = [&](unsigned int t) {
            for (unsigned int i = threadIdx.x; i < L; i += kSortThreads)
                if (t * T + i < a) seg[t * T + i] = key_edge(keys[i]);
            __syncthreads();
        };
        // every tile on its own: merges of blocks of 2, 4, ..., L keys
        for (unsigned int t = 0; t < tiles; ++t) {
            load_tile(t);
            for (unsigned int k = 2; k <= L; k <<= 1) sort_tile_steps(keys, L, k >> 1, true);
            store_tile(t);
        }
        // merges of blocks of 2T, 4T, ..., P keys: partners in different tiles meet in memory, the rest in LDS
        for (unsigned int k = 2 * T; k <= P; k <<= 1) {
            for (unsigned int j = k >> 1; j >= T; j >>= 1) {
                const unsigned int mask = (j == (k >> 1)) ? (k - 1) : j;
                constexpr int UN = 8;
                for (unsigned int i0 = threadIdx.x; i0 < a; i0 += UN * kSortThreads) {
                    Edge x[UN], y[UN];
                    bool pair[UN];
#pragma unroll
                    for (int r = 0; r < UN; ++r) {
                        const unsigned int i = i0 + r * kSortThreads, l = i ^ mask;
                        pair[r] = i < a && l > i && l < a;
                        if (pair[r]) {
                            x[r] = seg[i];
                            y[r] = seg[l];
                        }
                    }
#pragma unroll
                    for (int r = 0; r < UN; ++r) {
                        const unsigned int i = i0 + r * kSortThreads, l = i ^ mask;
                        if (pair[r] && edge_key(y[r]) < edge_key(x[r])) {
                            seg[i] = y[r];
                            seg[l] = x[r];
                        }
                    }
                }
                __syncthreads();
            }
            for (unsigned int t = 0; t < tiles; ++t) {
                load_tile(t);
                sort_tile_steps(keys, T, T >> 1, false);
                store_tile(t);
            }
        }
        finish(u, m);
    }
    __syncthreads();
    // rows for 16 lanes, from the workgroups that have no long row on
    constexpr unsigned int ROWS = kSortThreads / 16;
    static_assert(kSortThreads * kSortRegs * sizeof(float) <= sizeof keys, "the weights of the rows");
    for (unsigned int i0 = (gridDim.x - 1 - blockIdx.x) * ROWS; i0 < wide; i0 += gridDim.x * ROWS) {  // uniform in the workgroup
        const unsigned int i = i0 + threadIdx.x / 16;
        sort_finish_row<16>(f, i < wide, f.long_list + f.list_cap - 1 - (int64_t)i, reinterpret_cast<float(*)[16 * kSortRegs]>(keys));
    }
}

// Undo k_count_halfedges after a failed validation.
__global__ void __launch_bounds__(kBlock) k_clear_counts(unsigned int nt, const int32_t* __restrict__ touched,
                                                        int32_t* __restrict__ add_cnt) {
    const unsigned int t = blockIdx.x * kBlock + threadIdx.x;
    if (t < nt) add_cnt[touched[t]] = 0;
}

// =================================================================================================
// Vertex deletion (Alg. 2 Step 1 for Delta^Del): V_aff <- V_aff U N(u), then u and its edges go
// =================================================================================================
// One 16-lane group per listed vertex.  The group that swaps the row length to 0 owns the row (a
// vertex listed twice is handled once): every surviving neighbour v is put into V_aff (flag) and, on
// first touch, into the list of rows that must drop their entries towards deleted vertices.  The
// deleted row keeps its place and capacity in the pool (a later batch may give the id edges again);
// its label row becomes the neutral 1/C.
// Rows of up to kLongRow entries are held in registers, and a workgroup appends what its 16 rows touch first with one
// atomic (atomics on one address run at 1e8 per second; one per 64 entries: 30,000 vertices of degree 32 took 190 us);
// longer rows are left to the whole workgroup (a hub of 50,000 entries walked by 16 lanes took 1.2 ms).
constexpr int kDeleteRegs = 8;  // entries per lane: rows of up to 128

template <int NT>
__device__ inline void delete_rows(unsigned int block, int64_t nd, const int32_t* __restrict__ del, int C, int Cs, int CP, RowMeta* meta,
                                   const Edge* __restrict__ pool, const int32_t* __restrict__ seed_class, uint8_t* __restrict__ flag,
                                   int32_t* __restrict__ add_cnt, int32_t* __restrict__ dropping, float* __restrict__ deg,
                                   float* __restrict__ F, BatchCtr* bc) {
    constexpr int G = 16;
    __shared__ unsigned int smem[NT / kWave + 1];
    __shared__ int64_t long_off[NT / G];
    __shared__ int long_len[NT / G];
    __shared__ unsigned int nlong;
    if (threadIdx.x == 0) nlong = 0u;
    __syncthreads();
    const int64_t i = ((int64_t)block * NT + threadIdx.x) / G;
    const int gl = threadIdx.x % G;
    int len = 0;
    int64_t off = 0;
    if (i < nd) {
        const int32_t u = del[i];
        if (gl == 0) len = atomicExch(&meta[u].len, 0);
        len = __shfl(len, 0, G);
        off = meta[u].off;
        // also for a vertex that had no edges, or is listed twice: the same values again
        if (gl == 0) deg[u] = 0.f;
        for (int c = gl; c < CP; c += G) F[(size_t)u * CP + c] = c < Cs ? 1.0f / (float)C : 0.f;
        if (len > G * kDeleteRegs) {
            if (gl == 0) {
                const unsigned int k = atomicAdd(&nlong, 1u);
                long_off[k] = off;
                long_len[k] = len;
            }
            len = 0;
        }
    }
    unsigned long long removed = 0;
    int32_t v[kDeleteRegs];
    // the entries of one step: item q of this thread is entry at + q * stride (below end)
    auto take = [&](int64_t row, int at, int stride, int end) {
        unsigned int first = 0;
#pragma unroll
        for (int q = 0; q < kDeleteRegs; ++q) v[q] = at + q * stride < end ? pool[row + at + q * stride].col : -1;
#pragma unroll
        for (int q = 0; q < kDeleteRegs; ++q) {
            if (v[q] < 0) continue;
            removed += 1;
            if (seed_class[v[q]] == kDeletedMark) continue;
            flag[v[q]] = 1;
            removed += 1;  // the entry v -> u goes as well
            if (atomicAdd(&add_cnt[v[q]], 1) == 0) first |= 1u << q;
        }
        unsigned int slot = block_reserve<NT>(&bc->dropping, (unsigned int)__popc(first), smem);
#pragma unroll
        for (int q = 0; q < kDeleteRegs; ++q)
            if ((first >> q) & 1u) dropping[slot++] = v[q];
    };
    take(off, gl, G, len);
    for (unsigned int k = 0; k < nlong; ++k)  // uniform in the workgroup (block_reserve has barriers)
        for (int base = 0; base < long_len[k]; base += kDeleteRegs * NT) take(long_off[k], base + (int)threadIdx.x, NT, long_len[k]);
    removed = wave_sum(removed);
    __shared__ unsigned long long block_removed;
    if (threadIdx.x == 0) block_removed = 0ull;
    __syncthreads();
    if (lane_id() == 0) atomicAdd(&block_removed, removed);
    __syncthreads();
    if (threadIdx.x == 0 && block_removed) atomicAdd(&bc->removed, block_removed);
}

__global__ void __launch_bounds__(kBlock) k_delete_rows(int64_t nd, const int32_t* __restrict__ del, int C, int Cs, int CP,
                                                       RowMeta* meta, const Edge* __restrict__ pool,
                                                       const int32_t* __restrict__ seed_class,
                                                       uint8_t* __restrict__ flag, int32_t* __restrict__ add_cnt,
                                                       int32_t* __restrict__ dropping, float* __restrict__ deg,
                                                       float* __restrict__ F, BatchCtr* bc) {
    if (bc->err) return;
    delete_rows<kBlock>(blockIdx.x, nd, del, C, Cs, CP, meta, pool, seed_class, flag, add_cnt, dropping, deg, F, bc);
}

// Rows that lose entries (listed by k_delete_rows): drop the entries that point at deleted vertices, keeping the order of the others,
// then recompute d(v) from the stored row (same summation order as k_sort_finish) and clear the
// counting scratch.  16 lanes per row; a chunk is loaded completely before any of it is written
// back, and the write position never passes the read position.  Hubs are left to the whole workgroup.
__global__ void __launch_bounds__(kBlock) k_drop_deleted_entries(const BatchCtr* bc, const int32_t* __restrict__ dropping,
                                                                RowMeta* __restrict__ meta, Edge* __restrict__ pool,
                                                                const int32_t* __restrict__ seed_class,
                                                                int32_t* __restrict__ add_cnt,
                                                                float* __restrict__ deg) {
    constexpr int G = 16;
    __shared__ float tile[kDegTile];
    __shared__ unsigned int smem[kBlock / kWave + 1];
    __shared__ int32_t hub[kBlock / G];
    __shared__ unsigned int nhubs;
    const unsigned int nt = bc->dropping;
    const int gl = threadIdx.x % G;
    const int gshift = (lane_id() / G) * G;
    for (unsigned int t0 = blockIdx.x * (kBlock / G); t0 < nt; t0 += gridDim.x * (kBlock / G)) {  // uniform in the workgroup
        if (threadIdx.x == 0) nhubs = 0u;
        __syncthreads();
        const unsigned int t = t0 + threadIdx.x / G;
        int32_t v = 0;
        RowMeta m;
        m.off = 0;
        m.len = 0;
        m.cap = 0;
        bool own = t < nt;
        if (own) {
            v = dropping[t];
            m = meta[v];
            if (m.len > kHubRow) {
                if (gl == 0) hub[atomicAdd(&nhubs, 1u)] = v;
                own = false;
            }
        }
        if (own) {
            int out = 0;
            // UN chunks of G entries per step: their loads and the lookups of their neighbours are in flight together; the
            // kept ones are written in order, always to positions that lie before everything the step has read
            constexpr int UN = 4;
            for (int base = 0; base < m.len; base += UN * G) {
                Edge e[UN];
                bool keep[UN];
#pragma unroll
                for (int q = 0; q < UN; ++q) {
                    const int j = base + q * G + gl;
                    e[q].col = 0;
                    e[q].w = 0.f;
                    if (j < m.len) e[q] = pool[m.off + j];
                }
#pragma unroll
                for (int q = 0; q < UN; ++q) keep[q] = base + q * G + gl < m.len && seed_class[e[q].col] != kDeletedMark;
#pragma unroll
                for (int q = 0; q < UN; ++q) {
                    const unsigned int mask = (unsigned int)((__ballot(keep[q]) >> gshift) & 0xffffull);
                    if (keep[q]) pool[m.off + out + __popc(mask & ((1u << gl) - 1u))] = e[q];
                    out += __popc(mask);
                }
            }
            float s = 0.f;
            for (int j0 = gl; j0 < out; j0 += 8 * G) {  // the same order of additions as k_sort_finish
                float wv[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) wv[q] = j0 + q * G < out ? pool[m.off + j0 + q * G].w : 0.f;
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (j0 + q * G < out) s += wv[q];
            }
#pragma unroll
            for (int d = G / 2; d > 0; d >>= 1) s += __shfl_xor(s, d, G);
            if (gl == 0) {
                meta[v].len = out;
                deg[v] = s;
                add_cnt[v] = 0;
            }
        }
        __syncthreads();
        for (unsigned int k = 0; k < nhubs; ++k) {  // uniform in the workgroup
            const int32_t h = hub[k];
            const RowMeta r = meta[h];
            constexpr int UN = 8;  // neighbouring entries per thread
            unsigned int out = 0;
            for (int base = 0; base < r.len; base += UN * kBlock) {
                const int j0 = base + (int)threadIdx.x * UN;
                Edge e[UN];
                unsigned int keep = 0;
#pragma unroll
                for (int q = 0; q < UN; ++q) {
                    e[q].col = -1;
                    e[q].w = 0.f;
                    if (j0 + q < r.len) e[q] = pool[r.off + j0 + q];
                }
#pragma unroll
                for (int q = 0; q < UN; ++q)
                    if (e[q].col >= 0 && seed_class[e[q].col] != kDeletedMark) keep |= 1u << q;
                // (the barriers of the scan: the whole step has been read before any of it is written)
                unsigned int total;
                unsigned int at = out + block_exclusive_scan<unsigned int>((unsigned int)__popc(keep), smem, &total);
#pragma unroll
                for (int q = 0; q < UN; ++q)
                    if ((keep >> q) & 1u) pool[r.off + at++] = e[q];
                out += total;
            }
            __syncthreads();
            const float s = block_row_degree<kBlock>(pool + r.off, (int)out, tile);
            if (threadIdx.x == 0) {
                meta[h].len = (int)out;
                deg[h] = s;
                add_cnt[h] = 0;
            }
        }
        __syncthreads();  // hub, nhubs
    }
}

// =================================================================================================
// Storage compaction: rows laid out again in id order with fresh slack (reclaims what relocations
// and deletions left behind)
// =================================================================================================
__global__ void __launch_bounds__(kBlock) k_recap_rows(int64_t n, const RowMeta* __restrict__ meta_old, float slack,
                                                      RowMeta* __restrict__ meta_new,
                                                      int64_t* __restrict__ block_sums) {
    __shared__ int64_t sm[kBlock / kWave + 1];
    const int64_t u = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    int64_t cap = 0;
    if (u < n) {
        const int32_t len = meta_old[u].len;
        cap = row_capacity(len, slack);
        meta_new[u].len = len;
        meta_new[u].cap = (int32_t)cap;
    }
    int64_t total;
    block_exclusive_scan<int64_t>(cap, sm, &total);
    if (threadIdx.x == 0) block_sums[blockIdx.x] = total;
}

__global__ void __launch_bounds__(kBlock) k_copy_rows(int64_t n, const RowMeta* __restrict__ meta_old,
                                                     const RowMeta* __restrict__ meta_new,
                                                     const Edge* __restrict__ pool_old, Edge* __restrict__ pool_new) {
    constexpr int G = 16;
    const int64_t u = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / G;
    const int gl = threadIdx.x % G;
    if (u >= n) return;
    const RowMeta a = meta_old[u], b = meta_new[u];
    for (int j = gl; j < a.len; j += G) pool_new[b.off + j] = pool_old[a.off + j];
}

// =================================================================================================
// Counters to the host
// =================================================================================================
// Copies up to two runs of 16-byte pieces to pinned host memory and then sets *flag there.  The host waits by reading the flag:
// a copy by the runtime and a wait for the stream take 25 to 40 us of idle GPU after every chain of rounds, this 10.
__global__ void __launch_bounds__(kBlock) k_to_host(const uint4* __restrict__ a, unsigned int na, const uint4* __restrict__ b,
                                                   unsigned int nb, uint4* __restrict__ to, unsigned int* flag, unsigned int value) {
    for (unsigned int i = threadIdx.x; i < na + nb; i += kBlock) to[i] = i < na ? a[i] : b[i - na];
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(flag, value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// =================================================================================================
// Yardstick: a plain streaming copy (what this chip sustains when every byte is used once)
// =================================================================================================
__global__ void __launch_bounds__(kBlock) k_stream_copy(int64_t n16, const float4* __restrict__ src,
                                                       float4* __restrict__ dst) {
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
}

// Read-only counterpart (the row update reads about 40 times what it writes): every thread sums what
// it reads and stores one float, so that the loads cannot be dropped.
__global__ void __launch_bounds__(kBlock) k_stream_read(int64_t n16, const float4* __restrict__ src,
                                                       float* __restrict__ sink) {
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    float acc = 0.f;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n16; i += stride) {
        const float4 v = src[i];
        acc += (v.x + v.y) + (v.z + v.w);
    }
    sink[(int64_t)blockIdx.x * kBlock + threadIdx.x] = acc;
}

// Yardstick for the gathers of the row update: every group of LPN adjacent lanes reads whole rows of 16 * LPN
// bytes at pseudo-random places of a table (the row number is a multiplicative hash of a running index, so the
// kernel reads no index array: its only memory traffic is the gathers), eight independent rows in flight per
// group, the values summed so that the loads cannot be dropped.  What it sustains is the ceiling of "one
// neighbour row per CSR entry" for rows of that size in a table of that footprint.
template <int LPN>
__global__ void __launch_bounds__(kBlock) k_gather_probe(const float4* __restrict__ table, unsigned int rows,
                                                        unsigned long long gathers, float* __restrict__ sink) {
    constexpr int UN = 8;
    const unsigned long long groups = (unsigned long long)gridDim.x * (kBlock / LPN);
    const unsigned long long g = (unsigned long long)blockIdx.x * (kBlock / LPN) + threadIdx.x / LPN;
    const unsigned int part = threadIdx.x % LPN;
    float acc = 0.f;
    for (unsigned long long i = g; i < gathers; i += groups * UN) {
        float4 v[UN];
#pragma unroll
        for (int t = 0; t < UN; ++t) {
            const unsigned long long idx = i + (unsigned long long)t * groups;
            const unsigned int h = (unsigned int)((idx * 0x9E3779B97F4A7C15ull) >> 32);
            const unsigned int r = (unsigned int)(((unsigned long long)h * rows) >> 32);
            v[t] = idx < gathers ? table[(unsigned long long)r * LPN + part] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int t = 0; t < UN; ++t) acc += (v[t].x + v[t].y) + (v[t].z + v[t].w);
    }
    sink[(unsigned long long)blockIdx.x * kBlock + threadIdx.x] = acc;
}

// =================================================================================================
// Export (inspection / tests)
// =================================================================================================
__global__ void __launch_bounds__(kBlock) k_row_lens(int64_t n, const RowMeta* __restrict__ meta,
                                                    int64_t* __restrict__ lens, int64_t* __restrict__ block_sums) {
    __shared__ int64_t sm[kBlock / kWave + 1];
    const int64_t u = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t len = u < n ? meta[u].len : 0;
    if (u < n) lens[u] = len;
    int64_t total;
    block_exclusive_scan<int64_t>(len, sm, &total);
    if (threadIdx.x == 0) block_sums[blockIdx.x] = total;
}

// lens[] (in) becomes the exclusive prefix (out); row_ptr[n] is written by the host.
__global__ void __launch_bounds__(kBlock) k_lens_to_row_ptr(int64_t n, int64_t* __restrict__ lens,
                                                           const int64_t* __restrict__ block_offsets) {
    __shared__ int64_t sm[kBlock / kWave + 1];
    const int64_t u = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t len = u < n ? lens[u] : 0;
    int64_t total;
    const int64_t ex = block_exclusive_scan<int64_t>(len, sm, &total);
    if (u < n) lens[u] = block_offsets[blockIdx.x] + ex;
}

__global__ void __launch_bounds__(kBlock) k_export_rows(int64_t n, const RowMeta* __restrict__ meta,
                                                       const Edge* __restrict__ pool,
                                                       const int64_t* __restrict__ row_ptr, int32_t* __restrict__ col,
                                                       float* __restrict__ w) {
    constexpr int G = 16;
    const int64_t u = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / G;
    const int gl = threadIdx.x % G;
    if (u >= n) return;
    const RowMeta m = meta[u];
    const int64_t o = row_ptr[u];
    for (int j = gl; j < m.len; j += G) {
        const Edge e = pool[m.off + j];
        col[o + j] = e.col;
        w[o + j] = e.w;
    }
}

// Every step-th updatable row (list: short rows from the front, long rows from the back): out[0] += weight of its edges to
// labelled vertices, out[1] += weight of all its edges (the first 128 of a longer row's).  16 lanes per row.
__global__ void __launch_bounds__(kBlock) k_labelled_share(unsigned int ns, unsigned int nl, unsigned int step,
                                                          const int32_t* __restrict__ front, const int32_t* __restrict__ back,
                                                          const RowMeta* __restrict__ meta, const Edge* __restrict__ pool,
                                                          const int32_t* __restrict__ seed_class, float* __restrict__ out) {
    __shared__ float sm[2][kBlock / kWave];
    const unsigned long long pos = (unsigned long long)((blockIdx.x * kBlock + threadIdx.x) / 16u) * step;
    float labelled = 0.f, all = 0.f;
    if (pos < (unsigned long long)ns + nl) {
        const int32_t u = pos < ns ? front[pos] : back[-(long long)(pos - ns)];
        const RowMeta m = meta[u];
        for (int j = (int)(threadIdx.x & 15u); j < (m.len < 128 ? m.len : 128); j += 16) {
            const Edge e = pool[m.off + j];
            all += e.w;
            if (seed_class[e.col] >= 0) labelled += e.w;
        }
    }
    labelled = wave_sum(labelled);
    all = wave_sum(all);
    if (lane_id() == 0) {
        sm[0][threadIdx.x / kWave] = labelled;
        sm[1][threadIdx.x / kWave] = all;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kBlock / kWave; ++i) {
            labelled += sm[0][i];
            all += sm[1][i];
        }
        if (all > 0.f) {
            atomicAdd(&out[0], labelled);
            atomicAdd(&out[1], all);
        }
    }
}

}  // namespace dynlp
