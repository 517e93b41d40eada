// Packed rounds for label rows: Alg. 2 Step 3 / Eq. (1) over nearly all vertices with the sums of all rows on the chip
// and the gathers served by the L2s.
//
// A gather of a random neighbour's row costs one 128-byte line whatever the kernel around it: about 250 G rows/s when
// the lines are in the L2s and 55 G rows/s when they come over the fabric (random whole-row reads of 64 bytes, nothing
// else, tables of 0.25 ... 4 MB against 64 MB; 8 / 16 / 32 MB: 203 / 104 / 68 G).  The ordinary row update walks a row
// at a time, so its gathers go all over the label matrix, and a row's chain of dependent reads (list, record, entries,
// neighbours, next entries, old row) keeps it below even that rate on graphs whose labels do fit the caches.
//
// While the graph does not change (all rounds of a batch, all sweeps of a static solve) the entries are laid out once
// for the order the chip wants to read them in:
//   parts    ranges of consecutive vertices with about the same number of entries, one workgroup each; the sums of all its rows stay in the workgroup's LDS
//            from the first entry to the last (256 CUs x 160 KB hold 1,000,000 rows of 10 columns);
//   buckets  a part's entries are in ascending order of neighbour id (512 ranges of ids).  Every workgroup goes through
//            the ids in the same order, and since all parts hold about the same number of entries per range, the
//            workgroups of an XCD read the same few hundred KB of label rows at about the same time: a line comes over
//            the fabric once per XCD and round instead of once per entry.  Nothing keeps the workgroups together
//            (those that lag find their lines in the L2 and catch up); drifting apart costs misses, never correctness.
// Entries are handled one by one, whatever row they belong to (no lanes idle at the ends of rows, a hub row costs what
// its entries cost): a wave reads 64 entries with one load, hands them round with shuffles, LANES lanes read one
// neighbour row, multiply it by w / deg and add it to the row's sums in LDS.
//
// The sums are 32-bit fixed-point numbers (unit 2^-31; the terms w / deg * F of a row add up to at most 1): integer
// additions commute, so a round is bit-reproducible although the order of the LDS atomics is not.
// Rounding a term to the nearest unit is off by up to 2^-32, and where a hub's neighbours are alike by the same amount in
// every term.  A fraction of a unit that depends on the neighbour's id is therefore added before rounding (pk_dither): the
// error of d terms is then about 0.41 * sqrt(d) units, 2e-9 for 100 entries and 1.7e-8 for the longest row that is packed
// (kPackedMaxRow in dynlp.hip).  Weights are divided by a degree summed in float32 over 16 lanes (rows of up to kLongRow
// entries) or in 64 bits (longer ones, k_pk_long_degrees).  Largest error of one sweep against 64 bits, a hub of 8,000
// equal weights with 20 nearly equal columns: 8.9e-7 with nearest units and float32 degrees, 3.7e-8 now; the row update
// (a hub of 9,000) 1.3e-7.  The additions cost nothing that can be measured.
//
// Bound: the vector memory path of the CUs (a line of 128 bytes per gather through the L1; leaving out the LDS atomics
// changes nothing, leaving out the gathers takes away half).  One round over all rows, row update -> packed round, us:
//   1,000,000 vertices, degree 20, 10 columns (64 MB of label rows)   400 -> 178   (lines read from memory 21.6M -> 6.3M)
//     400,000 vertices, degree 20, 10 columns                         147 ->  77
//     150,000 vertices, power law, degree 30, 20 columns              90 ->  62
//     300,000 vertices, degree 16, 29 columns                        109 ->  71
//     100,000 vertices, kNN, mean degree 18, 10 columns               38 ->  27
// What it took: without the barriers in the loop the oldest waves of a CU run ahead and the L2s hit 20% instead of 72%
// (1,000,000 vertices: 320 us); with every lane group loading its own entries the loads of entries cost as much as the
// gathers (195 us).
#pragma once

#include "dynlp_device.h"
#include "dynlp_conjugate.h"

namespace dynlp {

constexpr int kPkThreads = 1024;
constexpr int kPkLds = 160 * 1024;     // LDS of one workgroup, everything included: one workgroup per CU
constexpr int kPkFixedLds = 1024;      // of it: reductions at the end of the kernel (static arrays)
constexpr unsigned int kPkWindow = 2688;  // entries between barriers (see k_pk_round)
constexpr int kPkBuckets = 512;        // ranges of neighbour ids a part's entries are ordered by
constexpr float kPkUnit = 2147483648.0f;  // 2^31: a row of ones sums to 2^31 and a few units, far from 2^32
constexpr unsigned int kPkGolden = 3204163u;  // 0.382 * 2^23 (odd): multiples of it are spread evenly modulo 2^23

// One entry of the packed stream: receiving row (offset in its part) << col_bits | neighbour, and
// w / deg(row) * 2^31.
struct __attribute__((aligned(8))) PkEntry {
    unsigned int at;
    float wn;
};

// Reads through a buffer descriptor: addresses are 32-bit offsets, reads past the end return 0.
__device__ inline __amdgpu_buffer_rsrc_t pk_buffer(const void* p, unsigned int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

// Between -0.5 and 0.5, evenly spread over the neighbours of a row; `lane` tells the pieces of a row apart.
__device__ inline float pk_dither(unsigned int at, unsigned int lane) {
    return __uint_as_float(((__umul24(at, kPkGolden) + lane) & 0x7fffffu) | 0x3f800000u) - 1.5f;
}

// The entry stream is read once per round and should not push label rows out of the L2: non-temporal.
__device__ inline PkEntry pk_load_entry(__amdgpu_buffer_rsrc_t b, unsigned int at) {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(b, (int)at, 0, 2);
    return PkEntry{v.x, __uint_as_float(v.y)};
}

template <int V>
__device__ inline Vec<V> pk_load_piece(__amdgpu_buffer_rsrc_t b, unsigned int at) {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    Vec<V> r;
    if constexpr (V == 1) {
        r.v[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(b, (int)at, 0, 0));
    } else if constexpr (V == 2) {
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(b, (int)at, 0, 0);
        r.v[0] = __uint_as_float(v.x);
        r.v[1] = __uint_as_float(v.y);
    } else {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(b, (int)at, 0, 0);
        r.v[0] = __uint_as_float(v.x);
        r.v[1] = __uint_as_float(v.y);
        r.v[2] = __uint_as_float(v.z);
        r.v[3] = __uint_as_float(v.w);
    }
    return r;
}

__device__ inline void clear_round_slot(RoundCtr* slot) {  // called by one workgroup
    if (threadIdx.x == 0) {
        slot->next_count = 0;
        slot->next_long = 0;
        slot->executed = 0;
        slot->rows_short = 0;
        slot->rows_long = 0;
        slot->any_moved = 0;
    }
    if (threadIdx.x < kCtrLanes) {
        RoundPart* p = &slot->part[threadIdx.x];
        p->resid_bits = 0;
        p->changed = 0;
        p->edges = 0;
        p->edges_long = 0;
        p->rows_short = 0;
        p->rows_long = 0;
    }
}

// len[v] = row length of an updatable vertex (unlabelled, at least one entry), else 0; pk_deg[v] = its degree;
// gran[g] = the entries of such rows among 32 g .. 32 g + 31; *longest = the longest of all (0 at launch).
__global__ void __launch_bounds__(kBlock) k_pk_receivers(int64_t n, const RowMeta* __restrict__ meta,
                                                        const int32_t* __restrict__ seed_class,
                                                        const float* __restrict__ deg, int32_t* __restrict__ len,
                                                        float* __restrict__ pk_deg, unsigned int* __restrict__ gran,
                                                        unsigned int* longest) {
    __shared__ unsigned int sm[kBlock / kWave];
    const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    unsigned int l = 0;
    if (v < n) {
        l = seed_class[v] < 0 ? (unsigned int)meta[v].len : 0u;
        len[v] = (int32_t)l;
        pk_deg[v] = deg[v];
    }
    unsigned int sum = l, most = l;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        if (d < 32) sum += __shfl_xor(sum, d);
        const unsigned int o = __shfl_xor(most, d);
        most = most > o ? most : o;
    }
    if ((threadIdx.x & 31) == 0 && v < n) gran[v >> 5] = sum;
    if (lane_id() == 0) sm[threadIdx.x / kWave] = most;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / kWave; ++w) most = most > sm[w] ? most : sm[w];
        // (atomics on one address run at 1e8 per second: most workgroups find a longer row listed already)
        if (most > __atomic_load_n(longest, __ATOMIC_RELAXED)) atomicMax(longest, most);
    }
}

// Degrees of the long rows (listed backwards from `back`), summed in 64 bits; one workgroup per row.
__global__ void __launch_bounds__(kBlock) k_pk_long_degrees(unsigned int nl, const int32_t* __restrict__ back,
                                                           const RowMeta* __restrict__ meta, const Edge* __restrict__ pool,
                                                           float* __restrict__ pk_deg) {
    __shared__ double sm[kBlock / kWave];
    for (unsigned int i = blockIdx.x; i < nl; i += gridDim.x) {
        const int32_t u = back[-(long long)i];
        const RowMeta m = meta[u];
        double s = 0.0;
        for (int j = threadIdx.x; j < m.len; j += kBlock) s += (double)pool[m.off + j].w;
#pragma unroll
        for (int d = kWave / 2; d > 0; d >>= 1) s += __shfl_xor(s, d);
        if (lane_id() == 0) sm[threadIdx.x / kWave] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < kBlock / kWave; ++w) s += sm[w];
            pk_deg[u] = (float)s;
        }
        __syncthreads();
    }
}

// Cuts the granules into `parts` runs of about the same cost, row_cost entries per row and one per entry (a workgroup sums
// its entries, then finishes its rows): part p is granules bound[p] .. bound[p + 1] - 1 (maybe none) and the entries
// start[p] .. start[p + 1] - 1 of the stream.  Where that gives a part more than max_rows rows, cut by rows alone.
// largest[0], largest[1]: the most entries and rows of a part.
// With as many rows in every part a power law's hubs fall where they fall, and a round waits for the part that has most
// entries: 150,000 vertices, power law of mean degree 30, 20 columns: 1.46 times the mean and 60.6 us per round, cut by cost
// 1.11 times and 52.2 us; planted blocks 1.02 times either way.  One workgroup.
__global__ void __launch_bounds__(kPkThreads) k_pk_bounds(int64_t n, int granules, int parts, unsigned int row_cost,
                                                         unsigned int max_rows, const unsigned int* __restrict__ gran,
                                                         unsigned int* bound, unsigned int* start, unsigned int* __restrict__ largest) {
    constexpr int NW = kPkThreads / kWave;
    __shared__ unsigned long long sm_cost[NW];
    __shared__ unsigned int sm_ent[NW];
    __shared__ unsigned int most[2];
    const int per = (granules + kPkThreads - 1) / kPkThreads;
    const int g0 = (int)threadIdx.x * per < granules ? (int)threadIdx.x * per : granules;
    const int g1 = g0 + per < granules ? g0 + per : granules;
    for (unsigned int entry_cost = 1u;; entry_cost = 0u) {  // uniform in the workgroup
        auto cost_of = [&](int g, unsigned int ent) {
            const int64_t rows = n - (int64_t)g * 32 < 32 ? n - (int64_t)g * 32 : 32;
            return (unsigned long long)ent * entry_cost + (unsigned long long)rows * row_cost;
        };
        unsigned long long cost = 0;
        unsigned int ent = 0;
        for (int g = g0; g < g1; ++g) {
            const unsigned int e = gran[g];
            ent += e;
            cost += cost_of(g, e);
        }
        const unsigned long long cost_in = wave_inclusive_scan(cost);
        const unsigned int ent_in = wave_inclusive_scan(ent);
        if (lane_id() == kWave - 1) {
            sm_cost[threadIdx.x / kWave] = cost_in;
            sm_ent[threadIdx.x / kWave] = ent_in;
        }
        if (threadIdx.x < 2) most[threadIdx.x] = 0u;
        __syncthreads();
        unsigned long long c = cost_in - cost, total = 0;
        unsigned int e0 = ent_in - ent;
        for (int w = 0; w < NW; ++w) {
            if (w < (int)threadIdx.x / kWave) {
                c += sm_cost[w];
                e0 += sm_ent[w];
            }
            total += sm_cost[w];
        }
        auto part_of = [&](unsigned long long middle) {
            const unsigned long long p = middle * (unsigned long long)parts / total;
            return (int)(p < (unsigned long long)parts ? p : (unsigned long long)(parts - 1));
        };
        if (g0 < g1) {
            int before = g0 > 0 ? part_of(c - (cost_of(g0 - 1, gran[g0 - 1]) + 1) / 2) : -1;
            for (int g = g0; g < g1; ++g) {
                const unsigned int e = gran[g];
                const unsigned long long w = cost_of(g, e);
                const int p = part_of(c + w - (w + 1) / 2);
                for (int q = before + 1; q <= p; ++q) {
                    bound[q] = (unsigned int)g;
                    start[q] = e0;
                }
                before = p;
                c += w;
                e0 += e;
            }
            if (g1 == granules)
                for (int q = before + 1; q <= parts; ++q) {
                    bound[q] = (unsigned int)granules;
                    start[q] = e0;
                }
        }
        __syncthreads();
        for (int p = threadIdx.x; p < parts; p += kPkThreads) {
            atomicMax(&most[0], start[p + 1] - start[p]);
            atomicMax(&most[1], (bound[p + 1] - bound[p]) * 32u);
        }
        __syncthreads();
        if (most[1] <= max_rows || entry_cost == 0u) break;
        __syncthreads();
    }
    if (threadIdx.x < 2) largest[threadIdx.x] = most[threadIdx.x];
}

// Place of the i-th entry of a bucket of L: entries of one row arrive one after the other and would meet at the row's
// sums in LDS; steps of about 0.618 L (coprime to L) spread them over the bucket.
__device__ inline unsigned int pk_spread(unsigned int L) {
    for (unsigned int s = (unsigned int)(0.618 * (double)L) | 1u;; s += 2u) {
        unsigned int x = L, y = s;
        while (y) {
            const unsigned int t = x % y;
            x = y;
            y = t;
        }
        if (x == 1u) return s;
    }
}

// The entries of part p to its stretch of the stream, start[p] .. start[p + 1] - 1, in
// ascending order of neighbour >> bucket_bits.  Which of a bucket's places an entry gets depends on timing and has no
// influence on results.  One workgroup per part, one lane per entry (running row lengths in LDS tell its row): the reads
// of eight entries per lane are in flight together and a hub row is as quick as any other (1,000,000 vertices of degree
// 20, 16 lanes per row: 667 us).
// The entries go through LDS in tiles, where they are ordered by bucket, and leave as one run of neighbouring places per tile
// and bucket (us, placed one by one, 8 bytes each at 512 places at a time, and now: 1,000,000 vertices of degree 20 588, 282;
// 400,000 177, 100; 300,000 of degree 16 136, 77).  Tile t of T takes every T-th group of 16 entries, in steps of 0.618 of the
// tile's groups, so that entries of one row that fall into one bucket do not come one after the other.
// A part of more than 20,991 rows leaves room for a smaller tile; its threads then read no more entries than it holds (30M
// entries among 100,000 vertices beside 31,072 without edges, tiles of 2,048: 691 us reading MOST per thread, 472 now; placed one by
// one 828).
// spread: a row holds so much of a part that several of its entries are added at once wherever they lie; they then go to the
// places that pk_spread gives, each on its own (150,000 vertices, a power law whose longest row is a sixth of a part: rounds
// of 52.0 us, 52.8 to 54.2 with runs).
constexpr int kPkMaxRows = 32768;  // their running lengths fit the LDS beside a tile of 1,024 entries
constexpr unsigned int kPkTile = 8192;
constexpr int kPkPlaceLds = 146 * 1024;  // dynamic LDS of k_pk_place
static_assert((kPkMaxRows + 1) * 4 + 1024 * sizeof(PkEntry) <= kPkPlaceLds, "the smallest tile");

// Rows of the workgroup's part (0: an empty part).
__device__ inline int pk_part_rows(int64_t n, const unsigned int* __restrict__ bound) {
    const int64_t base = (int64_t)bound[blockIdx.x] * 32, end = (int64_t)bound[blockIdx.x + 1] * 32;
    return (int)((end < n ? end : n) - (base < n ? base : n));
}

__global__ void __launch_bounds__(kPkThreads) k_pk_place(int64_t n, const unsigned int* __restrict__ bound, int col_bits, int bucket_bits,
                                                        unsigned int tile, int spread, const RowMeta* __restrict__ meta,
                                                        const Edge* __restrict__ pool, const int32_t* __restrict__ len,
                                                        const float* __restrict__ deg, const unsigned int* __restrict__ start,
                                                        PkEntry* __restrict__ ent) {
    constexpr int T = kPkThreads;
    constexpr int NW = T / kWave;
    constexpr int UN = 4;
    extern __shared__ __align__(16) unsigned int pk_lds[];  // a tile of entries; rows + 1 words: entries in the part's rows before
    __shared__ unsigned int next[kPkBuckets];               // entries per bucket, then the next place of the bucket
    __shared__ unsigned int cnt[kPkBuckets], off[kPkBuckets];  // of the tile: entries per bucket, their first place in the tile
    __shared__ unsigned int seg0[kPkBuckets], seg_len[kPkBuckets], step[kPkBuckets];  // spread: of the bucket
    __shared__ unsigned int wave_tot[NW];
    static_assert(kPkBuckets <= T && kPkBuckets % kWave == 0, "one thread per bucket");
    PkEntry* const sorted = reinterpret_cast<PkEntry*>(pk_lds);
    unsigned int* const pre = pk_lds + 2 * tile;
    const int64_t base = (int64_t)bound[blockIdx.x] * 32;
    const int nr = pk_part_rows(n, bound);
    const unsigned int mask = (1u << col_bits) - 1u;
    if (threadIdx.x < kPkBuckets) next[threadIdx.x] = 0u;
    // running row lengths: every thread sums a run of rows, the runs are scanned
    const int per = (nr + T - 1) / T;
    const int r0 = (int)threadIdx.x * per < nr ? (int)threadIdx.x * per : nr;
    const int r1 = r0 + per < nr ? r0 + per : nr;
    unsigned int sum = 0;
    for (int r = r0; r < r1; ++r) sum += (unsigned int)len[base + r];
    const unsigned int scan = wave_inclusive_scan(sum);
    if (lane_id() == kWave - 1) wave_tot[threadIdx.x / kWave] = scan;
    __syncthreads();
    unsigned int before = scan - sum;
    for (unsigned int w = 0; w < threadIdx.x / kWave; ++w) before += wave_tot[w];
    for (int r = r0; r < r1; ++r) {
        pre[r] = before;
        before += (unsigned int)len[base + r];
    }
    const unsigned int count = start[blockIdx.x + 1] - start[blockIdx.x];
    if (threadIdx.x == 0) pre[nr] = count;
    __syncthreads();
    if (count == 0) return;
    auto row_of = [&](unsigned int i) {  // the last row r with pre[r] <= i (rows without entries share their start with the next)
        int lo = 0, hi = nr;             // pre[lo] <= i < pre[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (pre[mid] <= i) lo = mid;
            else hi = mid;
        }
        return lo;
    };
    for (unsigned int i0 = threadIdx.x; i0 < count; i0 += UN * T) {
        unsigned int b[UN];
#pragma unroll
        for (int t = 0; t < UN; ++t) {
            const unsigned int i = i0 + t * T < count ? i0 + t * T : count - 1;
            const int r = row_of(i);
            b[t] = (unsigned int)pool[meta[base + r].off + (i - pre[r])].col >> bucket_bits;
        }
#pragma unroll
        for (int t = 0; t < UN; ++t)
            if (i0 + t * T < count) atomicAdd(&next[b[t]], 1u);
    }
    __syncthreads();
    // exclusive scan over the buckets: every thread of the first kPkBuckets gives its value and takes its prefix
    auto scan_buckets = [&](unsigned int v) {
        unsigned int inc = 0;
        if (threadIdx.x < kPkBuckets) {
            inc = wave_inclusive_scan(v);
            if (lane_id() == kWave - 1) wave_tot[threadIdx.x / kWave] = inc;
        }
        __syncthreads();
        unsigned int at = inc - v;
        if (threadIdx.x < kPkBuckets)
            for (unsigned int w = 0; w < threadIdx.x / kWave; ++w) at += wave_tot[w];
        __syncthreads();
        return at;
    };
    {
        const unsigned int at = scan_buckets(threadIdx.x < kPkBuckets ? next[threadIdx.x] : 0u);
        if (threadIdx.x < kPkBuckets) {
            if (spread) {
                const unsigned int v = next[threadIdx.x];
                seg0[threadIdx.x] = start[blockIdx.x] + at;
                seg_len[threadIdx.x] = v;
                step[threadIdx.x] = v > 0u ? pk_spread(v) : 1u;
            }
            next[threadIdx.x] = start[blockIdx.x] + at;
        }
    }
    constexpr unsigned int GRP = 16;
    constexpr int MOST = 8;  // entries per thread and tile: a tile holds at most MOST * T
    const unsigned int groups = (count + GRP - 1) / GRP, tiles = (groups + tile / GRP - 1) / (tile / GRP);
    for (unsigned int q = 0; q < tiles; ++q) {
        if (threadIdx.x < kPkBuckets) cnt[threadIdx.x] = 0u;
        __syncthreads();
        PkEntry x[MOST];
        unsigned int place[MOST];  // bucket << 16 | rank; ~0: none
#pragma unroll
        for (int k0 = 0; k0 < MOST; k0 += UN) {
            int r[UN];
            Edge e[UN];
            float d[UN];
            bool ok[UN];
#pragma unroll
            for (int t = 0; t < UN; ++t) {
                ok[t] = false;
                if ((unsigned int)(k0 + t) * T >= tile) continue;  // (a small tile: nothing for any thread)
                const unsigned int j = (unsigned int)(k0 + t) * T + threadIdx.x;
                const unsigned int g = (j / GRP) * 317u % (tile / GRP);
                const unsigned int i = GRP * (q + tiles * g) + j % GRP;
                ok[t] = j < tile && i < count;
                const unsigned int from = ok[t] ? i : count - 1;
                r[t] = row_of(from);
                e[t] = pool[meta[base + r[t]].off + (from - pre[r[t]])];
                d[t] = deg[base + r[t]];
            }
#pragma unroll
            for (int t = 0; t < UN; ++t) {
                place[k0 + t] = ~0u;
                if (!ok[t]) continue;
                x[k0 + t].at = ((unsigned int)r[t] << col_bits) | (unsigned int)e[t].col;
                x[k0 + t].wn = e[t].w / d[t] * kPkUnit;
                const unsigned int b = (unsigned int)e[t].col >> bucket_bits;
                place[k0 + t] = (b << 16) | atomicAdd(&cnt[b], 1u);
            }
        }
        __syncthreads();
        const unsigned int at = scan_buckets(threadIdx.x < kPkBuckets ? cnt[threadIdx.x] : 0u);
        if (threadIdx.x < kPkBuckets) off[threadIdx.x] = at;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < MOST; ++k)
            if (place[k] != ~0u) sorted[off[place[k] >> 16] + (place[k] & 0xffffu)] = x[k];
        __syncthreads();
        const unsigned int held = off[kPkBuckets - 1] + cnt[kPkBuckets - 1];
        for (unsigned int p = threadIdx.x; p < held; p += T) {
            const PkEntry e = sorted[p];
            const unsigned int b = (e.at & mask) >> bucket_bits;
            unsigned int to = next[b] + (p - off[b]);
            if (spread) {
                const unsigned int k = to - seg0[b], L = seg_len[b];
                to = seg0[b] + (L < 65536u ? k * step[b] % L : (unsigned int)((unsigned long long)k * step[b] % L));
            }
            ent[to] = e;
        }
        __syncthreads();
        if (threadIdx.x < kPkBuckets) next[threadIdx.x] += cnt[threadIdx.x];
    }
}

struct PkRound {
    const RoundCtr* prev;
    RoundCtr* ctr;
    RoundCtr* ctr_zero;
    int64_t n;
    int rows;  // of the largest part, a multiple of 32
    const unsigned int* bound;  // per part: its first row / 32
    int C;     // stored columns that are in use
    int stride;  // sums per row in LDS: C, rounded up to even where a row has several columns
    int col_bits;
    const PkEntry* ent;
    const unsigned int* start;  // per part: its first entry; the last word: the number of entries
    const int32_t* len;
    const RowMeta* meta;
    const Edge* pool;
    const float* F_in;
    float* F_out;
    const unsigned int* moved_prev;  // bitmap of the rows that moved in the previous round
    unsigned int* moved_cur;         // ... in this round (every word of a part is written by its workgroup)
    unsigned int* moved_clear;
    unsigned int words;
    float tol;
    int flags;    // kRoundAll, kRoundForce
    float omega;  // relaxation; 1: none, else F_out holds the rows of the round before the last
};

// The entries of one part on their way through a workgroup of kPkThreads: SLOTS neighbour rows per gather, LANES lanes each.
// SIGNED: the table holds numbers of either sign of at most 1 / (2 * scale) (k_pk_product); else labels, scale = 1.
template <int CP, int LANES, bool SIGNED>
struct PkStream {
    static constexpr int NW = kPkThreads / kWave;
    static constexpr int VEC = CP >= 4 ? 4 : CP;
    static constexpr int SLOTS = kWave / LANES;  // neighbour rows per gather
    static constexpr int GATHERS = kWave / SLOTS;
    static constexpr int TILE = SLOTS * GATHERS;  // entries a wave reads at once, one per lane
    static constexpr int TILES = GATHERS >= 3 ? 1 : 4 / GATHERS;
    static constexpr unsigned int kStep = NW * TILES * TILE;  // entries the workgroup takes at a time
    int mslot, mchunk, C, col_bits;
    unsigned int lane_part, mask, stride, piece, count, own;
    __amdgpu_buffer_rsrc_t ent, rows;
    PkEntry e[TILES];

    // asks for the first entries
    __device__ inline PkStream(int wave, int64_t n, int columns, int lds_stride, int bits, const PkEntry* entries,
                               const unsigned int* start, const float* table) {
        mslot = lane_id() / LANES;
        mchunk = lane_id() % LANES;
        C = columns;
        col_bits = bits;
        lane_part = (unsigned int)mchunk * 2779933u;
        mask = (1u << col_bits) - 1u;
        stride = (unsigned int)lds_stride * 4u;  // bytes of a row's sums
        piece = (unsigned int)mchunk * VEC * 4u;
        const unsigned int first = __builtin_amdgcn_readfirstlane(start[blockIdx.x]);
        count = __builtin_amdgcn_readfirstlane(start[blockIdx.x + 1]) - first;
        // buffer reads: one address register, and reads past the part's last entry return an entry of weight 0
        ent = pk_buffer(entries + first, count * (unsigned int)sizeof(PkEntry));
        rows = pk_buffer(table, (unsigned int)n * (unsigned int)(CP * 4));
        own = (unsigned int)(wave * TILES * TILE + (lane_id() < TILE ? lane_id() : TILE - 1)) * (unsigned int)sizeof(PkEntry);
#pragma unroll
        for (int q = 0; q < TILES; ++q) e[q] = pk_load_entry(ent, own + q * TILE * (unsigned int)sizeof(PkEntry));
    }

    // adds all entries to the sums in LDS
    __device__ inline void add(unsigned int* lds, float scale) {
        char* const sums = reinterpret_cast<char*>(lds) + piece;
        const bool second = mchunk * VEC + 2 < C;  // the upper two columns of a piece of four are in use
        unsigned int since = 0;
#pragma unroll 1
        for (unsigned int i0 = 0; i0 < count; i0 += kStep) {  // uniform in the workgroup
            since += kStep;
            if (since > kPkWindow) {  // keeps the waves of the workgroup within kPkWindow entries of each other
                __syncthreads();
                since = kStep;
            }
            PkEntry cur[TILES];
#pragma unroll
            for (int q = 0; q < TILES; ++q) {
                cur[q] = e[q];
                if constexpr (SIGNED) cur[q].wn *= scale;
                e[q] = pk_load_entry(ent, own + (i0 + kStep + q * TILE) * (unsigned int)sizeof(PkEntry));
            }
            constexpr int ALL = TILES * GATHERS;
            constexpr int UN = ALL <= 8 ? ALL : ALL % 8 == 0 ? 8 : ALL % 6 == 0 ? 6 : ALL % 5 == 0 ? 5 : ALL;
            static_assert(ALL % UN == 0, "whole groups of gathers");
#pragma unroll
            for (int g0 = 0; g0 < ALL; g0 += UN) {
                Vec<VEC> f[UN];
                unsigned int to[UN];
                float wn[UN], dither[UN];
#pragma unroll
                for (int t = 0; t < UN; ++t) {
                    const int q = (g0 + t) / GATHERS, src = (g0 + t) % GATHERS * SLOTS + mslot;
                    unsigned int at = cur[q].at;
                    wn[t] = cur[q].wn;
                    if constexpr (LANES > 1) {
                        at = __shfl(at, src);
                        wn[t] = __shfl(wn[t], src);
                    }
                    f[t] = pk_load_piece<VEC>(rows, (at & mask) * (unsigned int)(CP * 4) + piece);
                    to[t] = at >> col_bits;
                    dither[t] = pk_dither(at, lane_part);
                }
                if (mslot >= SLOTS) continue;  // the lanes left over
#pragma unroll
                for (int t = 0; t < UN; ++t) {
                    unsigned int byte = __umul24(to[t], stride);
                    asm("" : "+v"(byte));  // computed once, outside the masked half below
                    char* const dst = sums + byte;
                    unsigned int x[VEC];
#pragma unroll
                    for (int k = 0; k < VEC; ++k) {
                        const float r = __builtin_rintf(__builtin_fmaf(wn[t], f[t].v[k], dither[t]));
                        x[k] = SIGNED ? (unsigned int)(int)r : (unsigned int)r;
                    }
                    if constexpr (VEC == 1) {
                        atomicAdd(reinterpret_cast<unsigned int*>(dst), x[0]);
                    } else {
                        // two columns per atomic.  Labels: sums stay below 2^32, nothing carries over.  Signed: the sum of
                        // the two as one 64-bit number (pk_signed_sum takes it apart)
                        auto pair = [](unsigned int lo, unsigned int hi) {
                            if constexpr (SIGNED) hi += (unsigned int)((int)lo >> 31);
                            return lo | ((unsigned long long)hi << 32);
                        };
                        atomicAdd(reinterpret_cast<unsigned long long*>(dst), pair(x[0], x[1]));
                        if constexpr (VEC == 4)
                            if (second) atomicAdd(reinterpret_cast<unsigned long long*>(dst) + 1, pair(x[2], x[3]));
                    }
                }
            }
        }
        __syncthreads();
    }
};

// One round.  V_aff is decided per row as in k_row_update_pull: u is in it iff u or a neighbour moved in the previous
// round; rows outside it are copied to F_out.  Does nothing if the previous round did not run or moved no row.
// LANES: lanes that read one neighbour row (those of its CP columns that are in use).
template <int CP, int LANES>
__global__ void __launch_bounds__(kPkThreads, 4) k_pk_round(PkRound a) {
    constexpr int T = kPkThreads;
    constexpr int NW = T / kWave;
    constexpr int VEC = CP >= 4 ? 4 : CP;
    constexpr int LPN = CP / VEC;
    extern __shared__ __align__(16) unsigned int pk_lds[];
    __shared__ float sm_r[NW];
    __shared__ unsigned long long sm_e[NW], sm_c[NW];
    if (a.ctr_zero && blockIdx.x == 0) clear_round_slot(a.ctr_zero);
    // a static sweep finds the size of its row list in its predecessor's slot: hand it on (0 in batch rounds)
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.ctr->next_count = a.prev->next_count;
        a.ctr->next_long = a.prev->next_long;
    }
    // the first entries are asked for before anything that has to be waited for
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    PkStream<CP, LANES, false> stream(wave, a.n, a.C, a.stride, a.col_bits, a.ent, a.start, a.F_in);
    if (!(a.flags & kRoundForce) && (!a.prev->executed || a.prev->any_moved == 0u)) return;
#pragma unroll 1
    for (unsigned int w = blockIdx.x * T + threadIdx.x; w < a.words; w += gridDim.x * T) a.moved_clear[w] = 0u;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ctr->executed = 1;

    const int chunk = threadIdx.x % LPN;
    const int64_t base = (int64_t)a.bound[blockIdx.x] * 32;
    const int nr = pk_part_rows(a.n, a.bound);
    const int nwords = (nr + 31) / 32;
    unsigned int* const acc = pk_lds;
    unsigned int* const in = pk_lds + a.rows * a.stride;  // rows in V_aff
    unsigned int* const mv = in + a.rows / 32;            // rows that move in this round
#pragma unroll 1
    for (int i = threadIdx.x; i < a.rows * a.stride; i += T) acc[i] = 0u;
#pragma unroll 1
    for (int w = threadIdx.x; w < nwords; w += T) {
        in[w] = a.flags & kRoundAll ? ~0u : a.moved_prev[(base >> 5) + w];
        mv[w] = 0u;
    }
    __syncthreads();
    // rows that did not move themselves: 16 lanes look their neighbours up until one that moved is found
    if (!(a.flags & kRoundAll)) {
        const int gl = threadIdx.x & 15;
#pragma unroll 1
        for (int r = threadIdx.x >> 4; r < nr; r += T / 16) {
            if ((in[r >> 5] >> (r & 31)) & 1u) continue;
            const int l = a.len[base + r];
            if (l == 0) continue;
            const Edge* __restrict__ row = a.pool + a.meta[base + r].off;
            bool hit = false;
#pragma unroll 1
            for (int j0 = 0; j0 < l && !hit; j0 += 16) {  // uniform in the group of 16 lanes
                const int j = j0 + gl;
                const int32_t v = row[j < l ? j : l - 1].col;
                const unsigned long long b = __ballot((a.moved_prev[(unsigned int)v >> 5] >> ((unsigned int)v & 31u)) & 1u);
                hit = ((b >> (lane_id() & 48)) & 0xffffull) != 0ull;
            }
            if (hit && gl == 0) atomicOr(&in[r >> 5], 1u << (r & 31));
        }
    }
    stream.add(pk_lds, 1.f);
    const int cols = a.C - chunk * VEC;  // columns of this lane's piece of a row that are in use (may be <= 0)
    float rmax = 0.f;
    unsigned int edges = 0, edges_long = 0;
    unsigned int nchanged = 0, nrows = 0, nrows_long = 0;
    constexpr int RPP = T / LPN;  // rows per pass
    constexpr int UF = 4;         // passes whose reads are in flight together
#pragma unroll 1
    for (int r0 = 0; r0 < nr; r0 += UF * RPP) {
        int l[UF];
        Vec<VEC> old[UF];
#pragma unroll
        for (int q = 0; q < UF; ++q) {
            const int r = r0 + q * RPP + (int)threadIdx.x / LPN;
            l[q] = r < nr ? a.len[base + r] : 0;
            if (l[q] > 0) old[q] = load_vec<VEC>(a.F_in + (size_t)(base + r) * CP + chunk * VEC);
        }
#pragma unroll
        for (int q = 0; q < UF; ++q) {
            const int r = r0 + q * RPP + (int)threadIdx.x / LPN;
            if (l[q] == 0) continue;  // the same for the lanes of a row
            float* const out = a.F_out + (size_t)(base + r) * CP + chunk * VEC;
            if (!((in[r >> 5] >> (r & 31)) & 1u)) {
                if (a.F_out != a.F_in) store_vec<VEC>(out, old[q]);
                continue;
            }
            Vec<VEC> fn, before = old[q];
            float d = 0.f;
            if (a.omega != 1.f) before = load_vec<VEC>(out);
#pragma unroll
            for (int k = 0; k < VEC; ++k)
                fn.v[k] = k < cols ? fminf((float)acc[r * a.stride + chunk * VEC + k] * (1.0f / kPkUnit), 1.0f) : 0.f;
            if (a.omega != 1.f) relax_row<VEC, LPN>(fn, before, a.omega);
#pragma unroll
            for (int k = 0; k < VEC; ++k) d = fmaxf(d, fabsf(fn.v[k] - old[q].v[k]));
#pragma unroll
            for (int s = 1; s < LPN; s <<= 1) d = fmaxf(d, __shfl_xor(d, s, LPN));
            store_vec<VEC>(out, fn);
            if (chunk == 0) {
                rmax = fmaxf(rmax, d);
                if (d > a.tol) {
                    atomicOr(&mv[r >> 5], 1u << (r & 31));
                    nchanged += 1u;
                }
                if (l[q] > 128) {
                    edges_long += (unsigned int)l[q];
                    nrows_long += 1u;
                } else {
                    edges += (unsigned int)l[q];
                    nrows += 1u;
                }
            }
        }
    }
    // per workgroup: at most 2^31 entries and 2^16 rows
    unsigned long long both_edges = edges | ((unsigned long long)edges_long << 32);
    unsigned long long counts = nchanged | ((unsigned long long)nrows << 20) | ((unsigned long long)nrows_long << 40);
    rmax = wave_max(rmax);
    both_edges = wave_sum(both_edges);
    counts = wave_sum(counts);
    if (lane_id() == 0) {
        sm_r[wave] = rmax;
        sm_e[wave] = both_edges;
        sm_c[wave] = counts;
    }
    __syncthreads();
    for (int w = threadIdx.x; w < nwords; w += T) a.moved_cur[(base >> 5) + w] = mv[w];
    if (threadIdx.x >= NW) return;
    rmax = sm_r[threadIdx.x];
    both_edges = sm_e[threadIdx.x];
    counts = sm_c[threadIdx.x];
#pragma unroll
    for (int d = NW / 2; d > 0; d >>= 1) {
        rmax = fmaxf(rmax, __shfl_xor(rmax, d, NW));
        both_edges += __shfl_xor(both_edges, d, NW);
        counts += __shfl_xor(counts, d, NW);
    }
    if (threadIdx.x == 0) {
        edges = (unsigned int)both_edges;
        edges_long = (unsigned int)(both_edges >> 32);
        nchanged = (unsigned int)(counts & 0xfffffu);
        nrows = (unsigned int)((counts >> 20) & 0xfffffu);
        nrows_long = (unsigned int)(counts >> 40);
        RoundPart* p = &a.ctr->part[blockIdx.x & (kCtrLanes - 1)];
        if (rmax > 0.f) atomicMax(&p->resid_bits, __float_as_uint(rmax));
        if (edges) atomicAdd(&p->edges, (unsigned long long)edges);
        if (edges_long) atomicAdd(&p->edges_long, (unsigned long long)edges_long);
        if (nchanged) {
            atomicAdd(&p->changed, nchanged);
            a.ctr->any_moved = 1u;
        }
        if (nrows) atomicAdd(&p->rows_short, nrows);
        if (nrows_long) atomicAdd(&p->rows_long, nrows_long);
    }
}

// ---- one product of the conjugate rounds (dynlp_conjugate.h): v = p - (weighted mean of the neighbours' p) -------------
// The rows of p are numbers of either sign; they are scaled so that the largest in the whole table takes half of a sum's
// range.  Sums of one row: at most 2^30 units and half a unit per entry, either sign.
__device__ inline Vec<2> pk_signed_sum(unsigned long long s, float unit) {
    const int lo = (int)(unsigned int)s;
    const int hi = (int)(unsigned int)(s >> 32) - (lo >> 31);
    Vec<2> r;
    r.v[0] = (float)lo * unit;
    r.v[1] = (float)hi * unit;
    return r;
}

struct PkProduct {
    CgRun run;
    int64_t n;
    int rows;
    const unsigned int* bound;
    int C, stride, col_bits;
    const PkEntry* ent;
    const unsigned int* start;
    const int32_t* len;
    const float* deg;
    const float* p;
    float* v;  // 0 in rows that are not updated
};

template <int CP, int LANES>
__global__ void __launch_bounds__(kPkThreads, 4) k_pk_product(PkProduct a) {
    constexpr int T = kPkThreads;
    constexpr int VEC = CP >= 4 ? 4 : CP;
    constexpr int LPN = CP / VEC;
    extern __shared__ __align__(16) unsigned int pk_lds[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    PkStream<CP, LANES, true> stream(wave, a.n, a.C, a.stride, a.col_bits, a.ent, a.start, a.p);
    if (cg_done(a.run)) return;
    const float scale = cg_scale(a.run);
    const int chunk = threadIdx.x % LPN;
    const int64_t base = (int64_t)a.bound[blockIdx.x] * 32;
    const int nr = pk_part_rows(a.n, a.bound);
#pragma unroll 1
    for (int i = threadIdx.x; i < a.rows * a.stride; i += T) pk_lds[i] = 0u;
    __syncthreads();
    stream.add(pk_lds, scale);
    const int cols = a.C - chunk * VEC;
    const float unit = 1.0f / (scale * kPkUnit);
    double pv = 0.0, vv = 0.0;
    constexpr int RPP = T / LPN;
    constexpr int UF = 4;
#pragma unroll 1
    for (int r0 = 0; r0 < nr; r0 += UF * RPP) {
        int l[UF];
        float d[UF];
        Vec<VEC> own[UF];
#pragma unroll
        for (int q = 0; q < UF; ++q) {
            const int r = r0 + q * RPP + (int)threadIdx.x / LPN;
            l[q] = r < nr ? a.len[base + r] : 0;
            d[q] = 0.f;
            if (l[q] > 0) {
                own[q] = load_vec<VEC>(a.p + (size_t)(base + r) * CP + chunk * VEC);
                d[q] = a.deg[base + r];
            }
        }
#pragma unroll
        for (int q = 0; q < UF; ++q) {
            const int r = r0 + q * RPP + (int)threadIdx.x / LPN;
            if (l[q] == 0) continue;
            Vec<VEC> v;
            const unsigned int* const sum = pk_lds + r * a.stride + chunk * VEC;
#pragma unroll
            for (int k = 0; k < VEC; ++k) v.v[k] = 0.f;
            if constexpr (VEC == 1) {
                v.v[0] = own[q].v[0] - (float)(int)sum[0] * unit;
            } else {
#pragma unroll
                for (int k = 0; k < VEC; k += 2) {
                    if (k >= cols) continue;
                    const Vec<2> m = pk_signed_sum(*reinterpret_cast<const unsigned long long*>(sum + k), unit);
                    v.v[k] = own[q].v[k] - m.v[0];
                    v.v[k + 1] = k + 1 < cols ? own[q].v[k + 1] - m.v[1] : 0.f;
                }
            }
            float a1 = 0.f, a2 = 0.f;
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                a1 += own[q].v[k] * v.v[k];
                a2 += v.v[k] * v.v[k];
            }
            pv += (double)d[q] * (double)a1;
            vv += (double)d[q] * (double)a2;
            store_vec<VEC>(a.v + (size_t)(base + r) * CP + chunk * VEC, v);
        }
    }
    cg_add_product<T>(a.run, pv, vv);
}

}  // namespace dynlp
