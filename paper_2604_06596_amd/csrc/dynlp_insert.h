// Insertion of large batches through bins of rows.
//
// A half-edge counted and written on its own costs an atomic on its row's counter and, later, the row's record and a store, each
// on a line of its own somewhere in memory: 125M edges into 50M rows took 9.5 ms to count and 17.8 to write.  Here the half-edges
// are first put together by bins of 2^bin_bits rows, whose counters and places fit the LDS of a CU; both passes then stream, and
// only the stores into the rows of one bin are spread (over a megabyte).
//
//   k_hb_count   half-edges per (chunk of kHbChunk, bin)
//   (k_pb_seg_sums ... k_pb_offsets: where the runs of every chunk begin)
//   k_hb_place   a chunk's half-edges sorted by bin in LDS, and out as one run per bin: row in its bin, neighbour, weight
//   k_hb_rows    a workgroup per bin (and kHbSlice of its half-edges): half-edges per row, counted in LDS
//   k_hb_write   likewise: every half-edge to the next place of its row, the places in LDS
//
// Between the last two the plan of the rows that have to move, as for any batch.  The order of a row's new entries is that of the
// atomics; k_sort_finish makes it a function of the batch.  Half-edges whose row is out of range are left out (the checks report
// them and the batch ends there).
// Measured (us, 125M edges into 50M rows / 7.5M into 3M): count 9,550 / 598 -> k_hb_count 410 / 17, k_hb_place 2,230 / 86, k_hb_rows
// 160 / 16; write 17,770 / 592 -> 5,450 / 307 (the stores into rows are transactions of 8 bytes: 46 G/s of the 55 G/s that this
// card's fabric takes; bins whose rows stay in L2 while they fill would need 2^11 rows and a second pass to sort so finely).
#pragma once

#include "dynlp_binned.h"

namespace dynlp {

constexpr int kHbChunk = 8192;      // half-edges sorted at a time
constexpr int kHbThreads = 1024;
constexpr int kHbMaxBits = 14;      // 128 KB of places
constexpr unsigned int kHbSlice = 1u << 17;  // half-edges of one workgroup: a bin of hubs or of a batch's own vertices has many

__device__ inline int32_t half_edge_row(int64_t i, int64_t m, const int32_t* __restrict__ eu, const int32_t* __restrict__ ev) {
    return i < m ? eu[i] : ev[i - m];
}

__global__ void __launch_bounds__(kHbThreads) k_hb_count(int64_t m, int64_t n, int bin_bits, int nbins, const int32_t* __restrict__ eu,
                                                        const int32_t* __restrict__ ev, unsigned int* __restrict__ table) {
    __shared__ unsigned int hist[kPbMaxBins];
    for (int b = threadIdx.x; b < nbins; b += kHbThreads) hist[b] = 0u;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kHbChunk;
#pragma unroll
    for (int k = 0; k < kHbChunk; k += kHbThreads) {
        const int64_t i = base + k + threadIdx.x;
        const int32_t u = i < 2 * m ? half_edge_row(i, m, eu, ev) : -1;
        if (u >= 0 && u < n) atomicAdd(&hist[u >> bin_bits], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < nbins; b += kHbThreads) table[(size_t)blockIdx.x * nbins + b] = hist[b];
}

__global__ void __launch_bounds__(kHbThreads) k_hb_place(int64_t m, int64_t n, int bin_bits, int nbins, int lg_group,
                                                        const int32_t* __restrict__ eu, const int32_t* __restrict__ ev,
                                                        const float* __restrict__ ew, const unsigned int* __restrict__ table,
                                                        const unsigned int* __restrict__ bin_off, unsigned short* __restrict__ row,
                                                        int32_t* __restrict__ col, float* __restrict__ w) {
    constexpr int T = kHbThreads;
    __shared__ int32_t st_c[kHbChunk];
    __shared__ float st_w[kHbChunk];
    __shared__ unsigned short st_r[kHbChunk];
    __shared__ unsigned int cur[kPbMaxBins];
    __shared__ unsigned int first_slot[kPbMaxBins];
    __shared__ unsigned short loff[kPbMaxBins + 2];
    __shared__ unsigned int wave_tot[T / kWave + 1];
    // (chunks of one eighth of the batch on one XCD: what consecutive chunks write into a bin lies side by side)
    const unsigned int chunks = (unsigned int)((2 * m + kHbChunk - 1) / kHbChunk), per_xcd = (chunks + 7u) / 8u;
    const unsigned int chunk = (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    if ((blockIdx.x >> 3) >= per_xcd || chunk >= chunks) return;
    pb_chunk_runs<T>(nbins, table + (size_t)chunk * nbins, bin_off, loff, first_slot, wave_tot);
    for (int b = threadIdx.x; b < nbins; b += T) cur[b] = loff[b];
    __syncthreads();
    const int64_t base = (int64_t)chunk * kHbChunk;
    constexpr int UN = 4;
    for (int k0 = 0; k0 < kHbChunk; k0 += UN * T) {
        int32_t u[UN], v[UN];
        float x[UN];
#pragma unroll
        for (int q = 0; q < UN; ++q) {
            const int64_t i = base + k0 + q * T + threadIdx.x;
            const bool ok = i < 2 * m;
            u[q] = ok ? half_edge_row(i, m, eu, ev) : -1;
            v[q] = ok ? half_edge_row(i, m, ev, eu) : 0;
            x[q] = ok ? ew[i < m ? i : i - m] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < UN; ++q) {
            if (u[q] < 0 || u[q] >= n) continue;
            const unsigned int pos = atomicAdd(&cur[u[q] >> bin_bits], 1u);
            st_c[pos] = v[q];
            st_w[pos] = x[q];
            st_r[pos] = (unsigned short)(u[q] & ((1 << bin_bits) - 1));
        }
    }
    __syncthreads();
    const int gl = (int)threadIdx.x & ((1 << lg_group) - 1);
    const int G = 1 << lg_group;
    for (int b = (int)threadIdx.x >> lg_group; b < nbins; b += T >> lg_group) {
        const unsigned int lo = loff[b], hi = loff[b + 1], s0 = first_slot[b];
        for (unsigned int p = lo + gl; p < hi; p += G) {
            row[s0 + (p - lo)] = st_r[p];
            col[s0 + (p - lo)] = st_c[p];
            w[s0 + (p - lo)] = st_w[p];
        }
    }
}

// Where the slices of every bin begin, kHbSlice half-edges to a slice (nbins + 1 values).  One workgroup.
__global__ void __launch_bounds__(kBlock) k_hb_slices(int nbins, const unsigned int* __restrict__ bin_count,
                                                     unsigned int* __restrict__ slice_off) {
    __shared__ unsigned int smem[kBlock / kWave + 1];
    unsigned int carry = 0;
    for (int base = 0; base < nbins; base += kBlock) {
        const int i = base + (int)threadIdx.x;
        const unsigned int v = i < nbins ? (bin_count[i] + (kHbSlice - 1)) / kHbSlice : 0u;
        unsigned int total;
        const unsigned int ex = block_exclusive_scan(v, smem, &total);
        if (i < nbins) slice_off[i] = carry + ex;
        carry += total;
    }
    if (threadIdx.x == 0) slice_off[nbins] = carry;
}

// The slice of a workgroup: its bin, its half-edges, and whether the bin has others.
struct HbSlice {
    int bin;
    unsigned int lo, hi;
    bool shared;
    __device__ inline bool find(int nbins, const unsigned int* __restrict__ bin_off, const unsigned int* __restrict__ slice_off) {
        const unsigned int x = blockIdx.x;
        if (x >= slice_off[nbins]) return false;
        int a = 0, b = nbins;  // slice_off[a] <= x < slice_off[b]
        while (b - a > 1) {
            const int mid = (a + b) >> 1;
            if (slice_off[mid] <= x) a = mid;
            else b = mid;
        }
        bin = a;
        lo = bin_off[a] + (x - slice_off[a]) * kHbSlice;
        hi = min(bin_off[a + 1], lo + kHbSlice);
        shared = slice_off[a + 1] - slice_off[a] > 1;
        return true;
    }
};

// add_cnt[u] = half-edges of row u, for every row of the bin (it is all zero between batches).
__global__ void __launch_bounds__(kHbThreads) k_hb_rows(int64_t n, int bin_bits, int nbins, const unsigned int* __restrict__ bin_off,
                                                       const unsigned int* __restrict__ slice_off,
                                                       const unsigned short* __restrict__ row, int32_t* __restrict__ add_cnt) {
    __shared__ int32_t cnt[1 << kHbMaxBits];
    HbSlice sl;
    if (!sl.find(nbins, bin_off, slice_off)) return;
    const int size = 1 << bin_bits;
    const int64_t first = (int64_t)sl.bin << bin_bits;
    for (int d = threadIdx.x; d < size; d += kHbThreads) cnt[d] = 0;
    __syncthreads();
    constexpr unsigned int UN = 8;
    for (unsigned int i0 = sl.lo; i0 < sl.hi; i0 += UN * kHbThreads) {
        int r[UN];
#pragma unroll
        for (unsigned int q = 0; q < UN; ++q) {
            const unsigned int i = i0 + q * kHbThreads + threadIdx.x;
            r[q] = i < sl.hi ? (int)row[i] : -1;
        }
#pragma unroll
        for (unsigned int q = 0; q < UN; ++q)
            if (r[q] >= 0) atomicAdd(&cnt[r[q]], 1);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < size; d += kHbThreads) {
        if (first + d >= n || !cnt[d]) continue;
        if (sl.shared) atomicAdd(&add_cnt[first + d], cnt[d]);
        else add_cnt[first + d] = cnt[d];
    }
}

// As k_write_halfedges without ranks: the entries go behind the row's old ones and its length grows, by one atomic per row and
// slice where the bin has several slices (which counts first).
__global__ void __launch_bounds__(kHbThreads) k_hb_write(int64_t n, int bin_bits, int nbins, const unsigned int* __restrict__ bin_off,
                                                        const unsigned int* __restrict__ slice_off,
                                                        const unsigned short* __restrict__ row, const int32_t* __restrict__ col,
                                                        const float* __restrict__ w, RowMeta* __restrict__ meta,
                                                        Edge* __restrict__ pool, BatchGate gate) {
    extern __shared__ __align__(16) unsigned long long hb_place[];  // 1 << bin_bits
    HbSlice sl;
    if (gate.closed() || !sl.find(nbins, bin_off, slice_off)) return;
    const int size = 1 << bin_bits;
    const int64_t first = (int64_t)sl.bin << bin_bits;
    const int rows = n - first < size ? (int)(n - first) : size;
    if (sl.shared) {
        for (int d = threadIdx.x; d < rows; d += kHbThreads) hb_place[d] = 0ull;
        __syncthreads();
        constexpr unsigned int UN = 8;
        for (unsigned int i0 = sl.lo; i0 < sl.hi; i0 += UN * kHbThreads) {
            int r[UN];
#pragma unroll
            for (unsigned int q = 0; q < UN; ++q) {
                const unsigned int i = i0 + q * kHbThreads + threadIdx.x;
                r[q] = i < sl.hi ? (int)row[i] : -1;
            }
#pragma unroll
            for (unsigned int q = 0; q < UN; ++q)
                if (r[q] >= 0) atomicAdd(&hb_place[r[q]], 1ull);
        }
        __syncthreads();
        for (int d = threadIdx.x; d < rows; d += kHbThreads) {
            const int mine = (int)hb_place[d];
            if (mine) hb_place[d] = (unsigned long long)(meta[first + d].off + atomicAdd(&meta[first + d].len, mine));
        }
    } else {
        for (int d = threadIdx.x; d < rows; d += kHbThreads) {
            const RowMeta m = meta[first + d];
            hb_place[d] = (unsigned long long)(m.off + m.len);
        }
    }
    __syncthreads();
    constexpr unsigned int UN = 4;
    for (unsigned int i0 = sl.lo; i0 < sl.hi; i0 += UN * kHbThreads) {
        int r[UN];
        Edge e[UN];
#pragma unroll
        for (unsigned int q = 0; q < UN; ++q) {
            const unsigned int i = i0 + q * kHbThreads + threadIdx.x;
            const bool ok = i < sl.hi;
            r[q] = ok ? (int)row[i] : -1;
            e[q].col = ok ? col[i] : 0;
            e[q].w = ok ? w[i] : 0.f;
        }
#pragma unroll
        for (unsigned int q = 0; q < UN; ++q)
            if (r[q] >= 0) pool[atomicAdd(&hb_place[r[q]], 1ull)] = e[q];
    }
    if (sl.shared) return;
    __syncthreads();
    for (int d = threadIdx.x; d < rows; d += kHbThreads) {
        const RowMeta m = meta[first + d];
        const int len = (int)((int64_t)hb_place[d] - m.off);
        if (len != m.len) meta[first + d].len = len;
    }
}

}  // namespace dynlp
