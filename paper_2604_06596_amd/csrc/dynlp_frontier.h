// Frontier kernels of DynLP for gfx950: compaction of V_aff into queues, the frontier row update
// (the hot kernel), the Jacobi commit of staged rows and the expansion of V_aff (Alg. 2 Step 3).
#pragma once

#include "dynlp_device.h"
#include "dynlp_conjugate.h"

#include <type_traits>

namespace dynlp {

constexpr int kFlagsPerThread = 16;
constexpr int kFlagsPerBlock = kBlock * kFlagsPerThread;  // 4096
constexpr int kLongRow = 128;  // rows longer than this get a whole workgroup

#ifndef DYNLP_UN_CAP
#define DYNLP_UN_CAP 8
#endif

// A frontier is stored in one int32 array of n_cap entries: "short" rows (len <= kLongRow) from
// the front, position i at front[i]; "long" rows from the back, position j at back[-j] with
// back = front + n_cap - 1.  The two never meet because a frontier has at most n entries.
// Row i of the frontier (short rows first, then long rows) has *position* i; staged label rows
// are indexed by position.
__device__ inline int32_t frontier_vertex(const int32_t* front, const int32_t* back, unsigned int ns,
                                          unsigned int pos) {
    return pos < ns ? front[pos] : back[-(long long)(pos - ns)];
}

// =================================================================================================
// Compaction: flag bytes -> next frontier
// =================================================================================================
// Each workgroup scans SEG * kFlagsPerBlock flag bytes (SEG runs of kFlagsPerBlock, 16 consecutive bytes per
// thread and run), keeps the vertices that may be updated (unlabelled, at least one edge), reserves ranges of
// the short and the long queue with one atomic each, writes the ids inside its ranges, and clears the flags it
// read.  The order of a frontier list has no influence on results.  SEG: atomics on one address run at about 1e8
// per second, so the 12,000 workgroups of a 50M-vertex graph at SEG = 1 spend 0.12 ms queueing for the counter;
// the host picks SEG = 4 from 16M vertices on and SEG = 1 (more workgroups) below.
// all_rows != 0 ignores the flags and lists every updatable vertex (static solve, and the count of
// updatable vertices).  bid: number of the workgroup among those that compact.
template <int SEG>
__device__ inline void compact_flags(unsigned int bid, unsigned int n, uint8_t* __restrict__ flag,
                                     const int32_t* __restrict__ seed_class, const RowMeta* __restrict__ meta, int all_rows,
                                     int32_t* __restrict__ front, int32_t* __restrict__ back,
                                     unsigned int* __restrict__ count_short, unsigned int* __restrict__ count_long) {
    __shared__ unsigned long long sm[kBlock / kWave + 1];
    __shared__ unsigned int sbase[2];
    unsigned int keep[SEG], is_long[SEG];  // bit k: vertex v0+k enters the frontier / as a long row
    unsigned int n_short = 0, n_long = 0;
#pragma unroll
    for (int q = 0; q < SEG; ++q) {
        const unsigned int v0 = (bid * SEG + q) * kFlagsPerBlock + threadIdx.x * kFlagsPerThread;
        keep[q] = 0;
        is_long[q] = 0;
        if (v0 < n) {
            unsigned int cand = 0;
            if (all_rows) {
                cand = 0xffffu;
            } else {
                const uint4 f = *reinterpret_cast<const uint4*>(flag + v0);
                if ((f.x | f.y | f.z | f.w) != 0) {
                    const unsigned int wds[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
                    for (int k = 0; k < kFlagsPerThread; ++k)
                        if ((wds[k >> 2] >> ((k & 3) * 8)) & 0xffu) cand |= 1u << k;
                    *reinterpret_cast<uint4*>(flag + v0) = make_uint4(0, 0, 0, 0);
                }
            }
            while (cand) {
                const int k = __ffs(cand) - 1;
                cand &= cand - 1;
                const unsigned int v = v0 + k;
                if (v < n && seed_class[v] < 0) {
                    const int len = meta[v].len;
                    if (len > 0) {
                        keep[q] |= 1u << k;
                        if (len > kLongRow) is_long[q] |= 1u << k;
                    }
                }
            }
        }
        n_short += (unsigned int)__popc(keep[q] & ~is_long[q]);
        n_long += (unsigned int)__popc(is_long[q]);
    }
    const unsigned long long cnt = (unsigned long long)n_short | ((unsigned long long)n_long << 32);
    unsigned long long total;
    const unsigned long long ex = block_exclusive_scan<unsigned long long>(cnt, sm, &total);
    if (threadIdx.x == 0) {
        const unsigned int ts = (unsigned int)total, tl = (unsigned int)(total >> 32);
        sbase[0] = ts ? atomicAdd(count_short, ts) : 0u;
        sbase[1] = tl ? atomicAdd(count_long, tl) : 0u;
    }
    __syncthreads();
    unsigned int ps = sbase[0] + (unsigned int)ex;
    unsigned int pl = sbase[1] + (unsigned int)(ex >> 32);
#pragma unroll
    for (int q = 0; q < SEG; ++q) {
        const unsigned int v0 = (bid * SEG + q) * kFlagsPerBlock + threadIdx.x * kFlagsPerThread;
        unsigned int kp = keep[q];
        while (kp) {
            const int k = __ffs(kp) - 1;
            kp &= kp - 1;
            if ((is_long[q] >> k) & 1u) back[-(long long)(pl++)] = (int32_t)(v0 + k);
            else front[ps++] = (int32_t)(v0 + k);
        }
    }
}

template <int SEG>
__global__ void __launch_bounds__(kBlock) k_compact(unsigned int n, uint8_t* __restrict__ flag,
                                                   const int32_t* __restrict__ seed_class,
                                                   const RowMeta* __restrict__ meta, int all_rows,
                                                   int32_t* __restrict__ front, int32_t* __restrict__ back,
                                                   unsigned int* __restrict__ count_short,
                                                   unsigned int* __restrict__ count_long) {
    compact_flags<SEG>(blockIdx.x, n, flag, seed_class, meta, all_rows, front, back, count_short, count_long);
}

// The first frontier of a batch from the flags (cleared) and the list of all updatable vertices, in one pass.  A wave takes
// STEPS * 64 consecutive vertices, a lane one of 64 neighbours per step, and lane s keeps what step s found; the loads of eight
// steps are in flight together.  Bound by the rows' records (16 bytes a vertex), for small graphs by one trip to memory and the
// four counters.  (With 16 neighbouring vertices per thread every load of a wave touched 64 lines; us, before / now: 3,001 vertices
// 8.9 / 5.3, 20,000 11.1 / 6.1, 100,000 12.1 / 6.9, 1M 19.8 / 15.8, 3M 78 / 30, 50M 1,885 / 329.)
constexpr int start_block_rows(int steps) { return steps * kBlock; }

// `words` words of 8 bytes from the start slot on for the host (pinned memory), then *flag = value; flag NULL: nothing.
struct StartToHost {
    unsigned long long* host;
    unsigned int words;
    unsigned int* flag;
    unsigned int value;
};

// The last workgroup of a launch to get here sends what k_to_host otherwise sends in a launch of its own.  (The others' counters
// have been added by then: each workgroup has waited for what its additions returned.  They are read at device scope.)
__device__ inline void send_start(RoundCtr* start, BatchCtr* bc, const StartToHost& to, unsigned long long began) {
    __shared__ bool last;
    if (threadIdx.x == 0) last = atomicAdd(&bc->lists_done, 1u) == gridDim.x - 1;
    __syncthreads();
    if (!last) return;
    unsigned long long* const from = reinterpret_cast<unsigned long long*>(start);
    for (unsigned int i = threadIdx.x; i < to.words; i += kBlock)
        to.host[i] = from + i == &bc->clock[1] ? began : __hip_atomic_load(from + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) {
        bc->lists_done = 0u;  // (the lists are made again where the pool was too small)
        __hip_atomic_store(to.flag, to.value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

template <int STEPS>
__device__ inline void compact_start(unsigned int n, uint8_t* __restrict__ flag, const int32_t* __restrict__ seed_class,
                                     const RowMeta* __restrict__ meta, int32_t* __restrict__ front, int32_t* __restrict__ back,
                                     RoundCtr* __restrict__ start, int32_t* __restrict__ ufront, int32_t* __restrict__ uback, BatchCtr* bc) {
    constexpr int UN = STEPS < 8 ? STEPS : 8;
    static_assert(STEPS <= kWave && STEPS % UN == 0, "a lane per step");
    static_assert(start_block_rows(STEPS) < 65536, "four counts in one 64-bit scan");
    __shared__ unsigned long long sm[kBlock / kWave + 1];
    __shared__ unsigned int sbase[4];
    const int lane = lane_id();
    const unsigned int w0 = (blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave) * (STEPS * kWave) + lane;
    unsigned long long listed = 0, keep = 0, is_long = 0;  // of step `lane`; bit l: lane l's vertex is updatable / flagged too / a long row
#pragma unroll 1
    for (int s0 = 0; s0 < STEPS; s0 += UN) {
        int32_t seed[UN];
        int len[UN];
        uint8_t f[UN];
#pragma unroll
        for (int q = 0; q < UN; ++q) {
            const unsigned int v = w0 + (unsigned int)(s0 + q) * kWave;
            seed[q] = v < n ? seed_class[v] : 0;
            len[q] = v < n ? meta[v].len : 0;
            f[q] = v < n ? flag[v] : (uint8_t)0;
        }
#pragma unroll
        for (int q = 0; q < UN; ++q) {
            const unsigned int v = w0 + (unsigned int)(s0 + q) * kWave;
            const bool upd = seed[q] < 0 && len[q] > 0;
            const unsigned long long bl = __ballot(upd), bk = __ballot(upd && f[q]), bg = __ballot(upd && len[q] > kLongRow);
            if (f[q]) flag[v] = 0;
            if (lane == s0 + q) {
                listed = bl;
                keep = bk;
                is_long = bg;
            }
        }
    }
    // frontier short, long, updatable short, long
    const unsigned long long cnt = (unsigned long long)__popcll(keep & ~is_long) | ((unsigned long long)__popcll(keep & is_long) << 16) |
                                   ((unsigned long long)__popcll(listed & ~is_long) << 32) |
                                   ((unsigned long long)__popcll(listed & is_long) << 48);
    unsigned long long total;
    const unsigned long long ex = block_exclusive_scan<unsigned long long>(cnt, sm, &total);
    if (threadIdx.x < 4) {
        const unsigned int t = (unsigned int)(total >> (16 * threadIdx.x)) & 0xffffu;
        unsigned int* const counter = threadIdx.x == 0   ? &start->next_count
                                      : threadIdx.x == 1 ? &start->next_long
                                      : threadIdx.x == 2 ? &bc->upd_short
                                                         : &bc->upd_long;
        sbase[threadIdx.x] = t ? atomicAdd(counter, t) : 0u;
    }
    __syncthreads();
    unsigned int at[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) at[k] = sbase[k] + ((unsigned int)(ex >> (16 * k)) & 0xffffu);
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll 1
    for (int s = 0; s < STEPS; ++s) {
        const unsigned long long bl = __shfl(listed, s), bk = __shfl(keep, s), bg = __shfl(is_long, s);
        if (!bl) continue;  // uniform in the wave
        const unsigned int a0 = __shfl(at[0], s), a1 = __shfl(at[1], s), a2 = __shfl(at[2], s), a3 = __shfl(at[3], s);
        const int32_t v = (int32_t)(w0 + (unsigned int)s * kWave);
        if (!((bl >> lane) & 1ull)) continue;
        const bool f = (bk >> lane) & 1ull;
        if ((bg >> lane) & 1ull) {
            uback[-(long long)(a3 + __popcll(bl & bg & below))] = v;
            if (f) back[-(long long)(a1 + __popcll(bk & bg & below))] = v;
        } else {
            ufront[a2 + __popcll(bl & ~bg & below)] = v;
            if (f) front[a0 + __popcll(bk & ~bg & below)] = v;
        }
    }
}

template <int STEPS>
__global__ void __launch_bounds__(kBlock) k_compact_start(unsigned int n, uint8_t* __restrict__ flag,
                                                         const int32_t* __restrict__ seed_class,
                                                         const RowMeta* __restrict__ meta, int32_t* __restrict__ front,
                                                         int32_t* __restrict__ back, RoundCtr* start, int32_t* __restrict__ ufront,
                                                         int32_t* __restrict__ uback, BatchCtr* bc, BatchGate gate, StartToHost to) {
    const unsigned long long began = wall_clock64();
    if (!gate.closed()) compact_start<STEPS>(n, flag, seed_class, meta, front, back, start, ufront, uback, bc);
    if (to.flag) send_start(start, bc, to, began);
    else if (blockIdx.x == 0 && threadIdx.x == 0) bc->clock[1] = began;
}

// =================================================================================================
// Commit of staged rows (staged rounds) and the next frontier after a round
// =================================================================================================
// F[vertex at position i] = Fq[i] for all positions: the Jacobi commit of a staged round, by nblocks workgroups.
__device__ inline void commit_rows(unsigned int bid, unsigned int nblocks, const RoundCtr* __restrict__ prev,
                                   const int32_t* __restrict__ front, const int32_t* __restrict__ back,
                                   const float* __restrict__ Fq, float* __restrict__ F, int CP) {
    const unsigned int ns = prev->next_count, nl = prev->next_long;
    const unsigned int nq = ns + nl;
    if (CP >= 4) {
        const unsigned int vpr = CP / 4;
        const unsigned long long total = (unsigned long long)nq * vpr;
        const float4* src = reinterpret_cast<const float4*>(Fq);
        float4* dst = reinterpret_cast<float4*>(F);
        for (unsigned long long i = (unsigned long long)bid * kBlock + threadIdx.x; i < total;
             i += (unsigned long long)nblocks * kBlock) {
            const unsigned int pos = (unsigned int)(i / vpr);
            const unsigned int ch = (unsigned int)(i % vpr);
            dst[(unsigned long long)frontier_vertex(front, back, ns, pos) * vpr + ch] = src[i];
        }
    } else {
        const unsigned long long total = (unsigned long long)nq * CP;
        for (unsigned long long i = (unsigned long long)bid * kBlock + threadIdx.x; i < total;
             i += (unsigned long long)nblocks * kBlock) {
            const unsigned int pos = (unsigned int)(i / CP);
            F[(unsigned long long)frontier_vertex(front, back, ns, pos) * CP + (i % CP)] = Fq[i];
        }
    }
}

// What follows a staged round, in one launch: its rows are committed (workgroups from compact_blocks on) and the next list of
// rows is made from the marks.  (Two launches: a round over a few thousand rows spent 2 us in the commit, 5 in the
// compaction and 3 between them.)
template <int SEG>
__global__ void __launch_bounds__(kBlock) k_commit_compact(unsigned int compact_blocks, unsigned int n,
                                                          uint8_t* __restrict__ flag, const int32_t* __restrict__ seed_class,
                                                          const RowMeta* __restrict__ meta, int32_t* __restrict__ next_front,
                                                          int32_t* __restrict__ next_back, unsigned int* __restrict__ count_short,
                                                          unsigned int* __restrict__ count_long, const RoundCtr* __restrict__ prev,
                                                          const int32_t* __restrict__ front, const int32_t* __restrict__ back,
                                                          const float* __restrict__ Fq, float* __restrict__ F, int CP) {
    if (blockIdx.x < compact_blocks)
        compact_flags<SEG>(blockIdx.x, n, flag, seed_class, meta, 0, next_front, next_back, count_short, count_long);
    else
        commit_rows(blockIdx.x - compact_blocks, gridDim.x - compact_blocks, prev, front, back, Fq, F, CP);
}

__device__ inline void mark(uint8_t* __restrict__ flag, int32_t v) {
    if (!flag[v]) flag[v] = 1;
}

// Next V_aff after a ping-pong round, computed by *pulling* instead of marking, and written straight
// into the next frontier (no flag bytes, no separate compaction).  The update kernels of a ping-pong
// round set one bit per row that moved by more than tol (moved[], 1 bit per vertex: 125 KB per million
// vertices, so the neighbour look-ups below stay in cache).  Alg. 2 Step 3 puts u into the next V_aff
// iff u moved or one of its neighbours moved; this kernel evaluates exactly that for every updatable
// vertex u (the universe list, short rows first, long rows from the back): one bit read, and only
// when u itself did not move a scan of N(u)'s bits that stops at the first hit.  A row that does not
// make it into the next V_aff gets its current value copied into F_old if the two buffers differ
// (it was updated in this round), so that they keep agreeing on every row outside V_aff (the
// invariant ping-pong rounds rely on).  The kernel also clears the bitmap of the next round.
// Workgroups [0, long_blocks): long rows, one wave per row, 64 neighbours per step.  The others:
// short rows, one lane per row.  A workgroup handles chunks of consecutive universe positions and
// reserves the output range of a whole chunk with ONE atomic (atomics on one address run at only
// ~10^8 per second device-wide, so they are kept to a few hundred per launch); kept ids are written
// in universe order inside the chunk's range.
__device__ inline bool moved_bit(const unsigned int* __restrict__ moved, int32_t v) {
    return (moved[(unsigned int)v >> 5] >> ((unsigned int)v & 31u)) & 1u;
}

// COH: read past the caches (the bitmap was written by other workgroups earlier in the same launch)
template <bool COH>
__device__ inline bool moved_bit_c(const unsigned int* moved, int32_t v) {
    if constexpr (!COH) return moved_bit(moved, v);
    else
        return (__hip_atomic_load(&moved[(unsigned int)v >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >>
                ((unsigned int)v & 31u)) & 1u;
}

// kPullSub = sub-steps per workgroup chunk (one queue atomic per chunk of kPullSub * kBlock positions).
// Small chunks mean more workgroups (the kernel is latency-bound on small and on low-degree graphs),
// large chunks mean fewer atomics on the one queue counter (which run at about 1e8 per second and show
// once every row also scans tens of neighbours): the host picks 4 or 16.
template <int kPullSub>
__global__ void __launch_bounds__(kBlock) k_pull_frontier(unsigned int ns, unsigned int nl, unsigned int long_blocks,
                                                         const int32_t* __restrict__ ufront,
                                                         const int32_t* __restrict__ uback,
                                                         const unsigned int* __restrict__ moved,
                                                         unsigned int* __restrict__ moved_next, unsigned int words,
                                                         const float* __restrict__ F_new, float* __restrict__ F_old,
                                                         int CP, const RowMeta* __restrict__ meta,
                                                         const Edge* __restrict__ pool,
                                                         int32_t* __restrict__ front, int32_t* __restrict__ back,
                                                         unsigned int* __restrict__ count_short,
                                                         unsigned int* __restrict__ count_long) {
    constexpr int NW = kBlock / kWave;
    __shared__ unsigned int cnt[kPullSub][NW];  // kept items per sub-step and wave, then their offsets
    __shared__ unsigned int sbase;
    const int wave = threadIdx.x / kWave;
    const int lane = lane_id();
    for (unsigned int w = blockIdx.x * kBlock + threadIdx.x; w < words; w += gridDim.x * kBlock) moved_next[w] = 0u;

    if (blockIdx.x < long_blocks) {
        // long rows: one wave per row, kPullSub rows per wave and chunk
        constexpr unsigned int CH = NW * kPullSub;
        for (unsigned int c0 = blockIdx.x * CH; c0 < nl; c0 += long_blocks * CH) {  // uniform per workgroup
            unsigned int keepmask = 0;
            for (int sub = 0; sub < kPullSub; ++sub) {
                const unsigned int j = c0 + sub * NW + wave;
                bool keep = false;
                if (j < nl) {
                    const int32_t u = uback[-(long long)j];
                    keep = moved_bit(moved, u);
                    if (!keep) {
                        const RowMeta m = meta[u];
                        const Edge* __restrict__ row = pool + m.off;
                        for (int base = 0; base < m.len; base += kWave) {  // uniform per wave
                            const int idx = base + lane;
                            const bool hit = idx < m.len && moved_bit(moved, row[idx].col);
                            if (__ballot(hit)) {
                                keep = true;
                                break;
                            }
                        }
                        if (!keep && F_old) {
                            for (int k = lane; k < CP; k += kWave) {
                                const float a = F_new[(size_t)u * CP + k];
                                if (a != F_old[(size_t)u * CP + k]) F_old[(size_t)u * CP + k] = a;
                            }
                        }
                    }
                }
                if (keep) keepmask |= 1u << sub;
                if (lane == 0) cnt[sub][wave] = keep ? 1u : 0u;
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                unsigned int run = 0;
                for (int sub = 0; sub < kPullSub; ++sub)
                    for (int q = 0; q < NW; ++q) {
                        const unsigned int t = cnt[sub][q];
                        cnt[sub][q] = run;
                        run += t;
                    }
                sbase = run ? atomicAdd(count_long, run) : 0u;
            }
            __syncthreads();
            if (lane == 0) {
                for (int sub = 0; sub < kPullSub; ++sub)
                    if ((keepmask >> sub) & 1u)
                        back[-(long long)(sbase + cnt[sub][wave])] = uback[-(long long)(c0 + sub * NW + wave)];
            }
            __syncthreads();
        }
        return;
    }
    // short rows: one lane per row, kPullSub * kBlock consecutive universe positions per chunk
    constexpr unsigned int CH = kBlock * kPullSub;
    const unsigned int nb = gridDim.x - long_blocks;
    const unsigned int bid = blockIdx.x - long_blocks;
    for (unsigned int c0 = bid * CH; c0 < ns; c0 += nb * CH) {  // uniform per workgroup
        // all ids of the chunk first, then all their bits: two memory round trips instead of 2 * kPullSub
        int32_t us[kPullSub];
#pragma unroll
        for (int sub = 0; sub < kPullSub; ++sub) {
            const unsigned int pos = c0 + sub * kBlock + threadIdx.x;
            us[sub] = pos < ns ? ufront[pos] : -1;
        }
        unsigned int keepmask = 0;
#pragma unroll
        for (int sub = 0; sub < kPullSub; ++sub)
            if (us[sub] >= 0 && moved_bit(moved, us[sub])) keepmask |= 1u << sub;
#pragma unroll
        for (int sub = 0; sub < kPullSub; ++sub) {
            const int32_t u = us[sub];
            bool keep = (keepmask >> sub) & 1u;
            if (u >= 0 && !keep) {
                const RowMeta m = meta[u];
                const Edge* __restrict__ row = pool + m.off;
                // eight independent look-ups per step (the lane waits once per step, not once per entry)
                for (int j = 0; j < m.len && !keep; j += 8) {
                    unsigned int hit = 0;
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        const int jj = j + q < m.len ? j + q : m.len - 1;
                        hit |= moved_bit(moved, row[jj].col) ? 1u : 0u;
                    }
                    keep = hit != 0;
                }
                if (keep) {
                    keepmask |= 1u << sub;
                } else if (F_old) {
                    for (int k = 0; k < CP; ++k) {
                        const float a = F_new[(size_t)u * CP + k];
                        if (a != F_old[(size_t)u * CP + k]) F_old[(size_t)u * CP + k] = a;
                    }
                }
            }
            const unsigned long long b = __ballot(keep);
            if (lane == 0) cnt[sub][wave] = (unsigned int)__popcll(b);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned int run = 0;
            for (int sub = 0; sub < kPullSub; ++sub)
                for (int q = 0; q < NW; ++q) {
                    const unsigned int t = cnt[sub][q];
                    cnt[sub][q] = run;
                    run += t;
                }
            sbase = run ? atomicAdd(count_short, run) : 0u;
        }
        __syncthreads();
#pragma unroll
        for (int sub = 0; sub < kPullSub; ++sub) {
            const bool keep = (keepmask >> sub) & 1u;
            const unsigned long long b = __ballot(keep);
            if (keep) {
                const unsigned int rank = (unsigned int)__popcll(b & ((1ull << lane) - 1ull));
                front[sbase + cnt[sub][wave] + rank] = us[sub];
            }
        }
        __syncthreads();
    }
}

// =================================================================================================
// Frontier row update: the hot kernels (Alg. 2 Step 3 inner loop / one ItLP sweep of Eq. (1))
// =================================================================================================
// G lanes cooperate on one frontier row u.  A neighbour row of CP floats is read by LPN = CP/VEC
// adjacent lanes (VEC = 4 floats = 16 bytes per lane), so the group gathers SLOTS = G/LPN neighbour
// rows at once, each as one contiguous CP*4-byte segment.  The row's (col, w) pairs are read G at
// a time with one coalesced 8-byte load per lane and handed round with lane shuffles; UN gathers
// are issued back to back before their values are used.  Every lane keeps the partial sums of its
// slot; a butterfly over the slot bits finishes acc = sum_j w_j F[col_j] and s = sum_j w_j.
template <int CP>
struct RowShape {
    static constexpr int VEC = CP >= 4 ? 4 : CP;
    static constexpr int LPN = CP / VEC;
};

// Accumulate the chunks first_chunk, first_chunk + chunk_step, ... (G entries each) of one row.
// Lanes past the end of the row carry a stand-in entry (own row, weight 0).  On return e holds the
// last chunk this group loaded (or the stand-in if it loaded none).
template <int CP, int G, bool COH = false>
__device__ inline void accumulate_row(const Edge* __restrict__ row, int len, int first_chunk, int chunk_step,
                                      int32_t u, const float* F_in, int gl,
                                      Vec<RowShape<CP>::VEC>& acc, float& s, Edge& e) {
    constexpr int VEC = RowShape<CP>::VEC;
    constexpr int LPN = RowShape<CP>::LPN;
    constexpr int SLOTS = G / LPN;
    constexpr int UN = LPN < DYNLP_UN_CAP ? LPN : DYNLP_UN_CAP;
    static_assert(G % LPN == 0 && SLOTS >= 1, "group must hold whole neighbour rows");
    static_assert(G % (SLOTS * UN) == 0, "a chunk of G entries is a whole number of gather blocks");
    const int slot = gl / LPN;
    const int chunk = gl % LPN;
    for (int base = first_chunk * G; base < len; base += chunk_step * G) {
        const int idx = base + gl;
        if (idx < len) {
            e = row[idx];
        } else {
            e.col = u;
            e.w = 0.f;
        }
        const int cnt = len - base;
#pragma unroll
        for (int j0 = 0; j0 < G; j0 += SLOTS * UN) {
            if (j0 < cnt) {  // uniform across the group
                int32_t c[UN];
                float w[UN];
                Vec<VEC> f[UN];
#pragma unroll
                for (int t = 0; t < UN; ++t) {
                    c[t] = __shfl(e.col, j0 + t * SLOTS + slot, G);
                    w[t] = __shfl(e.w, j0 + t * SLOTS + slot, G);
                }
#pragma unroll
                for (int t = 0; t < UN; ++t) f[t] = load_row<VEC, COH>(F_in + (size_t)c[t] * CP + chunk * VEC);
#pragma unroll
                for (int t = 0; t < UN; ++t) {
#pragma unroll
                    for (int k = 0; k < VEC; ++k) acc.v[k] = fmaf(w[t], f[t].v[k], acc.v[k]);
                    s += w[t];
                }
            }
        }
    }
#pragma unroll
    for (int d = LPN; d < G; d <<= 1) {
#pragma unroll
        for (int k = 0; k < VEC; ++k) acc.v[k] += __shfl_xor(acc.v[k], d, G);
        s += __shfl_xor(s, d, G);
    }
}

// Per-workgroup totals -> one set of atomics on one of the round's partial records.
// Returns (in thread 0) the number of rows the workgroup moved.
__device__ inline unsigned int flush_round_counters(float rmax, unsigned long long edges, unsigned int changed,
                                                    RoundCtr* __restrict__ ctr, bool long_rows, unsigned int rows = 0) {
    __shared__ float sm_r[kBlock / kWave];
    __shared__ unsigned long long sm_e[kBlock / kWave];
    __shared__ unsigned int sm_c[kBlock / kWave];
    __shared__ unsigned int sm_n[kBlock / kWave];
    rmax = wave_max(rmax);
    edges = wave_sum(edges);
    changed = wave_sum(changed);
    rows = wave_sum(rows);
    if (lane_id() == 0) {
        sm_r[threadIdx.x / kWave] = rmax;
        sm_e[threadIdx.x / kWave] = edges;
        sm_c[threadIdx.x / kWave] = changed;
        sm_n[threadIdx.x / kWave] = rows;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kBlock / kWave; ++i) {
            rmax = fmaxf(rmax, sm_r[i]);
            edges += sm_e[i];
            changed += sm_c[i];
            rows += sm_n[i];
        }
        RoundPart* p = &ctr->part[blockIdx.x & (kCtrLanes - 1)];
        if (rmax > 0.f) atomicMax(&p->resid_bits, __float_as_uint(rmax));
        if (edges) atomicAdd(long_rows ? &p->edges_long : &p->edges, edges);
        if (changed) {
            atomicAdd(&p->changed, changed);
            ctr->any_moved = 1u;
        }
        if (rows) atomicAdd(long_rows ? &p->rows_long : &p->rows_short, rows);
    }
    return changed;
}

// Short rows: G lanes per row, grid-strided (body; k_row_update dispatches to it).
//   STAGED = false (static sweep / ping-pong round): F'_u is written to row u of F_out, the
//            ping-pong partner of F_in; a row that moved by more than tol sets its bit in moved[]
//            (if not NULL; see k_pull_frontier).
//   STAGED = true (partial round): F'_u is staged at row pos of F_out so that every row of this
//            round reads the round-start F (Jacobi); a row that moved by > tol marks itself and
//            its neighbours in flag[] for the next round.  by_vertex is a set of flags.  kRowByVertex: the
//            row is written to row u of F_out instead (in-place rounds, F_out == F_in: nothing to commit).
//            kRowLazy: the new row is the mean of the old row and the weighted mean of the neighbours (same
//            fixed point; the host asks for it when rounds repeat themselves exactly, a period-2 cycle
//            that float32 rounding keeps alive in a nearly bipartite, weakly tied component).
// F_in and F_out may be the same array (in-place mode): a row then reads whatever its neighbours
// hold at that moment.  Reads and writes are whole 16-byte segments, columns are independent linear
// systems, and the update is a contraction per column, so mixed old/new reads only change the path
// to the fixed point, not the fixed point.
//   PULL (with STAGED = false): front lists every updatable vertex and the round itself decides which of them
//            are in V_aff: u is updated iff u or one of its neighbours moved by more than tol in the previous
//            round (bitmap moved_prev) - Alg. 2 Step 3's V_aff, evaluated where the row is read anyway.  A row
//            outside V_aff is copied to F_out when that is another buffer, so the two keep agreeing there.
//   RELAX (with PULL): every listed row is updated, and relaxed by omega (F_out then holds the rows of the round before).
constexpr int kRowByVertex = 1, kRowLazy = 2;

template <int CP, int G, bool STAGED, bool PULL = false, bool COH = false, bool RELAX = false>
__device__ inline unsigned int row_update_short(unsigned int bid, unsigned int nblocks, const int32_t* __restrict__ front,
                                        unsigned int ns, const RowMeta* __restrict__ meta,
                                        const Edge* __restrict__ pool, const float* F_in,
                                        float* F_out, int by_vertex, uint8_t* __restrict__ flag,
                                        unsigned int* __restrict__ moved, float tol,
                                        RoundCtr* __restrict__ ctr,
                                        const unsigned int* moved_prev = nullptr, float omega = 1.f) {
    constexpr int VEC = RowShape<CP>::VEC;
    constexpr int LPN = RowShape<CP>::LPN;
    constexpr int GPB = kBlock / G;
    const int gl = threadIdx.x % G;
    const int slot = gl / LPN;
    const int chunk = gl % LPN;
    float rmax = 0.f;
    unsigned long long edges = 0;
    unsigned int nchanged = 0;
    unsigned int nrows = 0;

    for (unsigned int g = bid * GPB + threadIdx.x / G; g < ns; g += nblocks * GPB) {
        const int32_t u = front[g];
        const RowMeta m = meta[u];
        const Edge* __restrict__ row = pool + m.off;
        if (PULL) {
            bool in_front = RELAX || moved_bit_c<COH>(moved_prev, u);
            for (int base = 0; base < m.len && !in_front; base += G) {  // uniform in the group
                const int idx = base + gl;
                const bool hit = idx < m.len && moved_bit_c<COH>(moved_prev, row[idx].col);
                const unsigned long long b = __ballot(hit);
                const unsigned long long mine = G == kWave ? b : (b >> ((lane_id() / G) * G)) & ((1ull << (G & 63)) - 1ull);
                in_front = mine != 0ull;
            }
            if (!in_front) {
                if (F_out != F_in && slot == 0)
                    store_row<VEC, COH>(F_out + (size_t)u * CP + chunk * VEC, load_row<VEC, COH>(F_in + (size_t)u * CP + chunk * VEC));
                continue;
            }
            if (gl == 0) nrows += 1;
        }
        Vec<VEC> acc;
#pragma unroll
        for (int k = 0; k < VEC; ++k) acc.v[k] = 0.f;
        float s = 0.f;
        Edge e;
        e.col = u;
        e.w = 0.f;
        accumulate_row<CP, G, COH>(row, m.len, 0, 1, u, F_in, gl, acc, s, e);
        const Vec<VEC> old = load_row<VEC, COH>(F_in + (size_t)u * CP + chunk * VEC);
        Vec<VEC> fn, before = old;
        float r = 0.f;
        if (RELAX && omega != 1.f) before = load_row<VEC, COH>(F_out + (size_t)u * CP + chunk * VEC);
#pragma unroll
        for (int k = 0; k < VEC; ++k) fn.v[k] = acc.v[k] / s;
        if (RELAX && omega != 1.f) relax_row<VEC, LPN>(fn, before, omega);
#pragma unroll
        for (int k = 0; k < VEC; ++k) {
            if (by_vertex & kRowLazy) fn.v[k] = 0.5f * (fn.v[k] + old.v[k]);
            r = fmaxf(r, fabsf(fn.v[k] - old.v[k]));
        }
#pragma unroll
        for (int d = 1; d < LPN; d <<= 1) r = fmaxf(r, __shfl_xor(r, d, G));
        if (slot == 0) store_row<VEC, COH>(F_out + (size_t)(STAGED && !(by_vertex & kRowByVertex) ? g : (unsigned int)u) * CP + chunk * VEC, fn);
        const bool big = r > tol;
        if (STAGED) {
            if (big) {  // V_aff <- V_aff U {u} U N(u); the last chunk of the row is still in registers
                if (gl == 0) flag[u] = 1;
                if (e.w != 0.f) mark(flag, e.col);
                const int last_base = ((m.len - 1) / G) * G;
                for (int idx = gl; idx < last_base; idx += G) mark(flag, row[idx].col);
            }
        } else if (moved) {
            // one atomic per distinct bitmap word among the rows of this wave (consecutive list positions are mostly
            // consecutive vertices: the wave's kWave / G rows usually share a word)
            const unsigned int word = (unsigned int)u >> 5;
            unsigned int bits = (big && gl == 0) ? 1u << ((unsigned int)u & 31u) : 0u;
            bool lowest = true;
#pragma unroll
            for (int k = 0; k < kWave / G; ++k) {
                const unsigned int ow = __shfl(word, k * G);
                const unsigned int ob = __shfl((big && gl == 0) ? 1u << ((unsigned int)u & 31u) : 0u, k * G);
                if (ow == word && k * G != (lane_id() / G) * G) {
                    bits |= ob;
                    if (k * G < (lane_id() / G) * G && ob) lowest = false;
                }
            }
            if (gl == 0 && big && lowest) atomicOr(&moved[word], bits);
        }
        if (gl == 0) {
            rmax = fmaxf(rmax, r);
            edges += (unsigned long long)m.len;
            nchanged += big ? 1u : 0u;
        }
    }
    return flush_round_counters(rmax, edges, nchanged, ctr, false, nrows);
}

// Long rows: one workgroup per row (body; k_row_update dispatches to it).  Its kBlock/G groups take the row's chunks round-robin; their
// partial sums meet in LDS and are added in group order (a fixed order: results do not depend on
// timing).  Position of long row j is pos_base + j.
template <int CP, bool STAGED, bool PULL = false, bool COH = false, bool RELAX = false>
__device__ inline unsigned int row_update_long(unsigned int bid, unsigned int nblocks, const int32_t* __restrict__ back,
                                       unsigned int nl, unsigned int pos_base, const RowMeta* __restrict__ meta,
                                       const Edge* __restrict__ pool, const float* F_in,
                                       float* F_out, int by_vertex, uint8_t* __restrict__ flag,
                                       unsigned int* __restrict__ moved, float tol,
                                       RoundCtr* __restrict__ ctr,
                                       const unsigned int* moved_prev = nullptr, float omega = 1.f) {
    constexpr int VEC = RowShape<CP>::VEC;
    constexpr int LPN = RowShape<CP>::LPN;
    constexpr int G = LPN > 16 ? LPN : 16;
    constexpr int NG = kBlock / G;
    __shared__ float part[NG][CP + 1];
    __shared__ float part_s[NG];
    __shared__ int sh_big;
    const int gi = threadIdx.x / G;
    const int gl = threadIdx.x % G;
    const int slot = gl / LPN;
    const int chunk = gl % LPN;
    float rmax = 0.f;
    unsigned long long edges = 0;
    unsigned int nchanged = 0;

    unsigned int nrows = 0;
    for (unsigned int j = bid; j < nl; j += nblocks) {
        const int32_t u = back[-(long long)j];
        const RowMeta m = meta[u];
        const Edge* __restrict__ row = pool + m.off;
        if (PULL) {  // every decision below is uniform across the workgroup
            bool in_front = RELAX || moved_bit_c<COH>(moved_prev, u);
            for (int base = 0; base < m.len && !in_front; base += kBlock) {
                const int idx = base + (int)threadIdx.x;
                in_front = __syncthreads_or(idx < m.len && moved_bit_c<COH>(moved_prev, row[idx].col)) != 0;
            }
            if (!in_front) {
                if (F_out != F_in && gi == 0 && slot == 0)
                    store_row<VEC, COH>(F_out + (size_t)u * CP + chunk * VEC, load_row<VEC, COH>(F_in + (size_t)u * CP + chunk * VEC));
                continue;
            }
            if (threadIdx.x == 0) nrows += 1;
        }
        Vec<VEC> acc;
#pragma unroll
        for (int k = 0; k < VEC; ++k) acc.v[k] = 0.f;
        float s = 0.f;
        Edge e;
        e.col = u;
        e.w = 0.f;
        accumulate_row<CP, G, COH>(row, m.len, gi, NG, u, F_in, gl, acc, s, e);
        if (slot == 0) {
#pragma unroll
            for (int k = 0; k < VEC; ++k) part[gi][chunk * VEC + k] = acc.v[k];
            if (gl == 0) part_s[gi] = s;
        }
        __syncthreads();
        if (gi == 0 && slot == 0) {
            Vec<VEC> tot;
#pragma unroll
            for (int k = 0; k < VEC; ++k) tot.v[k] = 0.f;
            float st = 0.f;
            constexpr int UQ = CP >= 32 ? 4 : NG;  // all partial sums of wide rows at once would cost half the waves
#pragma unroll UQ
            for (int q = 0; q < NG; ++q) {
#pragma unroll
                for (int k = 0; k < VEC; ++k) tot.v[k] += part[q][chunk * VEC + k];
                st += part_s[q];
            }
            const Vec<VEC> old = load_row<VEC, COH>(F_in + (size_t)u * CP + chunk * VEC);
            Vec<VEC> fn, before = old;
            float r = 0.f;
            if (RELAX && omega != 1.f) before = load_row<VEC, COH>(F_out + (size_t)u * CP + chunk * VEC);
#pragma unroll
            for (int k = 0; k < VEC; ++k) fn.v[k] = tot.v[k] / st;
            if (RELAX && omega != 1.f) relax_row<VEC, LPN>(fn, before, omega);
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                if (by_vertex & kRowLazy) fn.v[k] = 0.5f * (fn.v[k] + old.v[k]);
                r = fmaxf(r, fabsf(fn.v[k] - old.v[k]));
            }
#pragma unroll
            for (int d = 1; d < LPN; d <<= 1) r = fmaxf(r, __shfl_xor(r, d, G));
            store_row<VEC, COH>(F_out + (size_t)(STAGED && !(by_vertex & kRowByVertex) ? pos_base + j : (unsigned int)u) * CP + chunk * VEC, fn);
            if (gl == 0) {
                const bool big = r > tol;
                sh_big = big ? 1 : 0;
                if (!STAGED && moved && big) atomicOr(&moved[(unsigned int)u >> 5], 1u << ((unsigned int)u & 31u));
                rmax = fmaxf(rmax, r);
                edges += (unsigned long long)m.len;
                nchanged += big ? 1u : 0u;
            }
        }
        __syncthreads();
        if (STAGED && sh_big) {
            if (threadIdx.x == 0) flag[u] = 1;
            for (int idx = threadIdx.x; idx < m.len; idx += kBlock) mark(flag, row[idx].col);
        }
        __syncthreads();
    }
    return flush_round_counters(rmax, edges, nchanged, ctr, true, nrows);
}

// One launch per round.  The frontier's size comes from the previous round's counter slot (prev), so
// that rounds can be queued back to back without the host reading anything.  Workgroups
// [0, long_blocks) take the long rows (started first: they are the long poles; long_blocks =
// min(long rows, long_blocks_max)), the rest take the short rows.  Workgroup 0 clears the counter slot of the next round and records what this round
// worked on.  stop_bits: a static sweep does nothing if the previous sweep already met the stop rule
// (max change <= tol, as float bits) or did not run; frontier rounds pass 0xffffffff... never stop.
template <int CP, int G, bool STAGED>
__global__ void __launch_bounds__(kBlock) k_row_update(const RoundCtr* __restrict__ prev, int static_stop,
                                                      unsigned int stop_bits, unsigned int long_blocks_max,
                                                      const int32_t* __restrict__ front,
                                                      const int32_t* __restrict__ back,
                                                      const RowMeta* __restrict__ meta,
                                                      const Edge* __restrict__ pool,
                                                      const float* F_in, float* F_out, int by_vertex,
                                                      uint8_t* __restrict__ flag, unsigned int* __restrict__ moved,
                                                      float tol,
                                                      RoundCtr* __restrict__ ctr,
                                                      RoundCtr* __restrict__ ctr_zero) {
    if (ctr_zero && blockIdx.x == 0) {
        if (threadIdx.x == 0) {
            ctr_zero->next_count = 0;
            ctr_zero->next_long = 0;
            ctr_zero->executed = 0;
            ctr_zero->rows_short = 0;
            ctr_zero->rows_long = 0;
            ctr_zero->any_moved = 0;
        }
        if (threadIdx.x < kCtrLanes) {
            RoundPart* p = &ctr_zero->part[threadIdx.x];
            p->resid_bits = 0;
            p->changed = 0;
            p->edges = 0;
            p->edges_long = 0;
            p->rows_short = 0;
            p->rows_long = 0;
        }
    }
    const unsigned int ns = prev->next_count, nl = prev->next_long;
    if (ns + nl == 0) return;
    if (static_stop) {
        unsigned int prev_resid = 0xffffffffu;
        if (static_stop == 2) {  // max change of the previous sweep: maximum over its partial records
            const int lane = lane_id();
            prev_resid = lane < kCtrLanes ? prev->part[lane].resid_bits : 0u;
#pragma unroll
            for (int d = kWave / 2; d > 0; d >>= 1) {
                const unsigned int o = __shfl_xor(prev_resid, d, kWave);
                prev_resid = o > prev_resid ? o : prev_resid;
            }
        }
        if (static_stop == 2 && (!prev->executed || prev_resid <= stop_bits)) {
            // keep the frontier for whoever reads this slot next
            if (blockIdx.x == 0 && threadIdx.x == 0) {
                ctr->next_count = ns;
                ctr->next_long = nl;
            }
            return;
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) {  // a static sweep's frontier never changes
            ctr->next_count = ns;
            ctr->next_long = nl;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ctr->executed = 1;
        ctr->rows_short = ns;
        ctr->rows_long = nl;
    }
    const unsigned int long_blocks = nl < long_blocks_max ? nl : long_blocks_max;
    if (blockIdx.x < long_blocks)
        row_update_long<CP, STAGED>(blockIdx.x, long_blocks, back, nl, ns, meta, pool, F_in, F_out, by_vertex, flag, moved,
                                    tol, ctr);
    else
        row_update_short<CP, G, STAGED>(blockIdx.x - long_blocks, gridDim.x - long_blocks, front, ns, meta, pool, F_in,
                                        F_out, by_vertex, flag, moved, tol, ctr);
}

// A round over nearly all updatable vertices that finds its own V_aff (no frontier list, no separate pull):
// (front, back, ns, nl) is the list of all updatable vertices; moved_prev has the bits of the rows that moved
// in the previous round, moved_cur receives this round's, moved_clear (the bitmap of the round after) is
// zeroed.  The round does nothing if the previous one did not run or moved no row (V_aff is empty then).
// RELAX: a round over all rows with relaxation (flags: kRoundForce); an instance of its own, because the second row per
// lane doubles the registers of the plain one (60 -> 121 with 16 columns: half the waves).
template <int CP, int G, bool RELAX>
__global__ void __launch_bounds__(kBlock) k_row_update_pull(const RoundCtr* __restrict__ prev, unsigned int long_blocks_max,
                                                           const int32_t* __restrict__ front,
                                                           const int32_t* __restrict__ back, unsigned int ns,
                                                           unsigned int nl, const RowMeta* __restrict__ meta,
                                                           const Edge* __restrict__ pool, const float* F_in,
                                                           float* F_out, const unsigned int* __restrict__ moved_prev,
                                                           unsigned int* __restrict__ moved_cur,
                                                           unsigned int* __restrict__ moved_clear, unsigned int words,
                                                           float tol, int flags, float omega,
                                                           RoundCtr* __restrict__ ctr, RoundCtr* __restrict__ ctr_zero) {
    if (ctr_zero && blockIdx.x == 0) {
        if (threadIdx.x == 0) {
            ctr_zero->next_count = 0;
            ctr_zero->next_long = 0;
            ctr_zero->executed = 0;
            ctr_zero->rows_short = 0;
            ctr_zero->rows_long = 0;
            ctr_zero->any_moved = 0;
        }
        if (threadIdx.x < kCtrLanes) {
            RoundPart* p = &ctr_zero->part[threadIdx.x];
            p->resid_bits = 0;
            p->changed = 0;
            p->edges = 0;
            p->edges_long = 0;
            p->rows_short = 0;
            p->rows_long = 0;
        }
    }
    // did the previous round move a row?  (one word of its header instead of its 32 partial records: thousands of
    // short-lived workgroups each reading 32 lines was a fifth of the launch on a 100K-vertex graph)
    if (!(flags & kRoundForce) && (!prev->executed || prev->any_moved == 0u)) return;
    for (unsigned int w = blockIdx.x * kBlock + threadIdx.x; w < words; w += gridDim.x * kBlock) moved_clear[w] = 0u;
    if (blockIdx.x == 0 && threadIdx.x == 0) ctr->executed = 1;
    const unsigned int long_blocks = nl < long_blocks_max ? nl : long_blocks_max;
    if (blockIdx.x < long_blocks)
        row_update_long<CP, false, true, false, RELAX>(blockIdx.x, long_blocks, back, nl, ns, meta, pool, F_in, F_out, 1, nullptr,
                                         moved_cur, tol, ctr, moved_prev, omega);
    else
        row_update_short<CP, G, false, true, false, RELAX>(blockIdx.x - long_blocks, gridDim.x - long_blocks, front, ns, meta, pool,
                                             F_in, F_out, 1, nullptr, moved_cur, tol, ctr, moved_prev, omega);
}

// =================================================================================================
// One product of the conjugate rounds (dynlp_conjugate.h), row by row
// =================================================================================================
// v[u] = p[u] - (weighted mean of the neighbours' rows of p) for every updatable row, and the sums (p, v), (v, v).  Rows are
// walked as in k_row_update (workgroups [0, long_blocks) take the long ones).
template <int CP, int G>
__device__ inline void row_product_short(unsigned int bid, unsigned int nblocks, const int32_t* __restrict__ front,
                                         unsigned int ns, const RowMeta* __restrict__ meta, const Edge* __restrict__ pool,
                                         const float* __restrict__ p, float* __restrict__ v, double& pv, double& vv) {
    constexpr int VEC = RowShape<CP>::VEC;
    constexpr int LPN = RowShape<CP>::LPN;
    constexpr int GPB = kBlock / G;
    const int gl = threadIdx.x % G;
    for (unsigned int g = bid * GPB + threadIdx.x / G; g < ns; g += nblocks * GPB) {
        const int32_t u = front[g];
        const RowMeta m = meta[u];
        Vec<VEC> acc;
#pragma unroll
        for (int k = 0; k < VEC; ++k) acc.v[k] = 0.f;
        float s = 0.f;
        Edge e;
        e.col = u;
        e.w = 0.f;
        accumulate_row<CP, G>(pool + m.off, m.len, 0, 1, u, p, gl, acc, s, e);
        if (gl >= LPN) continue;
        const size_t at = (size_t)u * CP + gl * VEC;
        const Vec<VEC> own = load_vec<VEC>(p + at);
        Vec<VEC> r;
        float a1 = 0.f, a2 = 0.f;
#pragma unroll
        for (int k = 0; k < VEC; ++k) {
            r.v[k] = own.v[k] - acc.v[k] / s;
            a1 += own.v[k] * r.v[k];
            a2 += r.v[k] * r.v[k];
        }
        pv += (double)s * (double)a1;
        vv += (double)s * (double)a2;
        store_vec<VEC>(v + at, r);
    }
}

template <int CP>
__device__ inline void row_product_long(unsigned int bid, unsigned int nblocks, const int32_t* __restrict__ back,
                                        unsigned int nl, const RowMeta* __restrict__ meta, const Edge* __restrict__ pool,
                                        const float* __restrict__ p, float* __restrict__ v, double& pv, double& vv) {
    constexpr int VEC = RowShape<CP>::VEC;
    constexpr int LPN = RowShape<CP>::LPN;
    constexpr int G = LPN > 16 ? LPN : 16;
    constexpr int NG = kBlock / G;
    __shared__ float part[NG][CP + 1];
    __shared__ float part_s[NG];
    const int gi = threadIdx.x / G;
    const int gl = threadIdx.x % G;
    for (unsigned int j = bid; j < nl; j += nblocks) {
        const int32_t u = back[-(long long)j];
        const RowMeta m = meta[u];
        Vec<VEC> acc;
#pragma unroll
        for (int k = 0; k < VEC; ++k) acc.v[k] = 0.f;
        float s = 0.f;
        Edge e;
        e.col = u;
        e.w = 0.f;
        accumulate_row<CP, G>(pool + m.off, m.len, gi, NG, u, p, gl, acc, s, e);
        if (gl < LPN) {
#pragma unroll
            for (int k = 0; k < VEC; ++k) part[gi][gl * VEC + k] = acc.v[k];
            if (gl == 0) part_s[gi] = s;
        }
        __syncthreads();
        if (threadIdx.x < LPN) {
            Vec<VEC> tot;
#pragma unroll
            for (int k = 0; k < VEC; ++k) tot.v[k] = 0.f;
            float st = 0.f;
#pragma unroll 4
            for (int q = 0; q < NG; ++q) {
#pragma unroll
                for (int k = 0; k < VEC; ++k) tot.v[k] += part[q][gl * VEC + k];
                st += part_s[q];
            }
            const size_t at = (size_t)u * CP + gl * VEC;
            const Vec<VEC> own = load_vec<VEC>(p + at);
            Vec<VEC> r;
            float a1 = 0.f, a2 = 0.f;
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                r.v[k] = own.v[k] - tot.v[k] / st;
                a1 += own.v[k] * r.v[k];
                a2 += r.v[k] * r.v[k];
            }
            pv += (double)st * (double)a1;
            vv += (double)st * (double)a2;
            store_vec<VEC>(v + at, r);
        }
        __syncthreads();
    }
}

template <int CP, int G>
__global__ void __launch_bounds__(kBlock) k_row_product(CgRun run, unsigned int long_blocks, const int32_t* __restrict__ front,
                                                       const int32_t* __restrict__ back, unsigned int ns, unsigned int nl,
                                                       const RowMeta* __restrict__ meta, const Edge* __restrict__ pool,
                                                       const float* __restrict__ p, float* __restrict__ v) {
    if (cg_done(run)) return;
    double pv = 0.0, vv = 0.0;
    if (blockIdx.x < long_blocks) row_product_long<CP>(blockIdx.x, long_blocks, back, nl, meta, pool, p, v, pv, vv);
    else row_product_short<CP, G>(blockIdx.x - long_blocks, gridDim.x - long_blocks, front, ns, meta, pool, p, v, pv, vv);
    cg_add_product<kBlock>(run, pv, vv);
}

// =================================================================================================
// Rounds over a small V_aff: many per launch, on one workgroup
// =================================================================================================
// A round over a few hundred rows is three launches (update, commit, and a compaction that scans the marks of every
// vertex) for one or two microseconds of work: 13 us on 2,000 vertices, 14 to 20 us on 3,000,000, and the last rounds of
// a batch are all of that kind.  One workgroup runs up to `rounds` of them in one launch: it reads a list of rows,
// updates them exactly as a flag-marking round does (same sums in the same order, new rows staged by position and
// committed after a barrier, or written in place), and appends the vertices it marks for the first time straight to the next list, so that nothing
// scans the marks; those it has set it clears again.  All data between rounds stays with one CU: a workgroup's own
// stores are visible to it after a barrier.  Measured: see tail_rounds_pay in dynlp.hip.
// The launch ends when V_aff is empty, after `rounds` rounds, when V_aff or its entries outgrow one CU (also before its
// first round: the host knows how many rows there are, but not that a few of them are hubs), or where a chain of
// ordinary rounds would go on with another number of lanes per row or with averaged rows (both decided by the host); the
// list of the next round is then where an ordinary round expects it.
constexpr int kTailThreads = 1024;

// On a graph whose labels, row records and lists fit the LDS of the CU beside the rest, they are brought there at the start of
// the launch (RES): a round is a chain of a dozen dependent accesses, and all but the entries' then stay on the CU.  3,001
// vertices with one label column, rounds of up to 850 rows: 14 -> 8 us per round, whole call 322 -> 244 us.
//
// A row's entries, cut where they are beyond every limit: the sum over all rows a round may list fits 32 bits.
__device__ inline unsigned int tail_entries(int len) { return len < 65536 ? (unsigned int)len : 65536u; }

struct TailArgs {
    RoundCtr* ring;
    int t0, rounds;               // rounds t0 .. t0 + rounds - 1 at most; rounds < kRing - 1
    int32_t* front[2];            // list of round t0: front[0] / back[0]; the two arrays take turns
    int32_t* back[2];
    const RowMeta* meta;
    const Edge* pool;
    const int32_t* seed_class;
    float* F;
    float* staged;                // rows by position (synchronous mode)
    int by_vertex;                // kRowByVertex: in place; kRowLazy
    uint8_t* flag;
    float tol;
    unsigned int max_rows, max_entries;
    int chain, chain_off;         // decisions are taken every `chain` rounds; the first comes after chain - chain_off rounds
    unsigned int len_lo, len_hi;  // mean row lengths [len_lo, len_hi) keep the lanes per row of this launch
    int same_run, same_max;       // rounds that repeated themselves before this launch, and how many make the rows averaged
    unsigned int sig[3];          // rows, rows moved, max change of the round before
    unsigned int n;               // RES: vertices, below 65,536; the pool's entries are numbered with 32 bits
};

// LDS of a RES launch, in bytes: row records (offset; length, top bit: labelled), label rows, staged rows, marks, two lists.
// (Records and rows of n rounded up to a multiple of four vertices, so that everything is aligned.)
__host__ __device__ inline unsigned int tail_resident_bytes(unsigned int n, int CP, unsigned int max_rows) {
    const unsigned int n4 = (n + 3u) & ~3u;
    return n4 * 8u + n4 * (unsigned int)CP * 4u + max_rows * (unsigned int)CP * 4u + (n + 31u) / 32u * 4u + 2u * n4 * 2u;
}

template <int CP, int G, bool RES>
__global__ void __launch_bounds__(kTailThreads) k_tail_rounds(TailArgs a) {
    constexpr int VEC = RowShape<CP>::VEC;
    constexpr int LPN = RowShape<CP>::LPN;
    constexpr int GL = LPN > 16 ? LPN : 16, NG = kBlock / GL;  // long rows: as in row_update_long
    constexpr int TEAMS = kTailThreads / kBlock;
    extern __shared__ __align__(16) unsigned int tail_lds[];
    __shared__ float part[TEAMS][NG][CP + 1];
    __shared__ float part_s[TEAMS][NG];
    __shared__ unsigned int big[TEAMS];
    __shared__ unsigned int count[2];       // rows of the running round: short, long
    __shared__ unsigned int next[3];        // of the next one: short, long, their entries
    __shared__ unsigned int moved, resid;
    __shared__ unsigned int entries[2];     // of the running round: in short rows, in long rows
    __shared__ bool leave;                  // the host has something to decide
    int same_run = a.same_run;              // (thread 0)
    bool repeats = false;
    unsigned int sig[3] = {a.sig[0], a.sig[1], a.sig[2]};
    // RES: the graph's label rows etc. in LDS (see tail_resident_bytes)
    const unsigned int lstride = (a.n + 3u) & ~3u;
    uint2* const lrow = reinterpret_cast<uint2*>(tail_lds);
    float* const lF = reinterpret_cast<float*>(lrow + lstride);
    float* const lstaged = lF + lstride * CP;
    unsigned int* const lmark = reinterpret_cast<unsigned int*>(lstaged + a.max_rows * CP);
    unsigned short* const llist = reinterpret_cast<unsigned short*>(lmark + (a.n + 31u) / 32u);
    auto listed = [&](int parity, unsigned int ns, unsigned int pos) -> int32_t {
        if constexpr (RES) return (int32_t)llist[parity * lstride + (pos < ns ? pos : a.n - 1u - (pos - ns))];
        else return frontier_vertex(a.front[parity], a.back[parity], ns, pos);
    };
    auto record = [&](int32_t u, int64_t* off, int* len) {
        if constexpr (RES) {
            const uint2 q = lrow[u];
            *off = (int64_t)q.x;
            *len = (int)(q.y & 0x7fffffffu);
        } else {
            const RowMeta m = a.meta[u];
            *off = m.off;
            *len = m.len;
        }
    };
    {
        // the slots of all rounds this launch may run, and of the round after
        constexpr int kWords = sizeof(RoundCtr) / 4;
        for (int i = threadIdx.x; i < (a.rounds + 1) * kWords; i += kTailThreads)
            reinterpret_cast<unsigned int*>(a.ring + (a.t0 + i / kWords) % kRing)[i % kWords] = 0u;
        if (threadIdx.x == 0) {
            const RoundCtr* prev = a.ring + (a.t0 + kRing - 1) % kRing;
            count[0] = (a.t0 == 0 ? a.ring + kRing : prev)->next_count;
            count[1] = (a.t0 == 0 ? a.ring + kRing : prev)->next_long;
            next[2] = 0u;
            leave = false;
        }
        if constexpr (RES) {
            constexpr unsigned int UN = 4;  // loads in flight
            for (unsigned int i0 = threadIdx.x; i0 < a.n * CP / VEC; i0 += UN * kTailThreads) {
                Vec<VEC> x[UN];
#pragma unroll
                for (unsigned int q = 0; q < UN; ++q)
                    if (i0 + q * kTailThreads < a.n * CP / VEC) x[q] = load_vec<VEC>(a.F + (size_t)(i0 + q * kTailThreads) * VEC);
#pragma unroll
                for (unsigned int q = 0; q < UN; ++q)
                    if (i0 + q * kTailThreads < a.n * CP / VEC) store_vec<VEC>(lF + (i0 + q * kTailThreads) * VEC, x[q]);
            }
            for (unsigned int v0 = threadIdx.x; v0 < a.n; v0 += UN * kTailThreads) {
                RowMeta m[UN];
                int32_t sc[UN];
#pragma unroll
                for (unsigned int q = 0; q < UN; ++q) {
                    const unsigned int v = v0 + q * kTailThreads < a.n ? v0 + q * kTailThreads : a.n - 1u;
                    m[q] = a.meta[v];
                    sc[q] = a.seed_class[v];
                }
#pragma unroll
                for (unsigned int q = 0; q < UN; ++q)
                    if (v0 + q * kTailThreads < a.n)
                        lrow[v0 + q * kTailThreads] = make_uint2((unsigned int)m[q].off, (unsigned int)m[q].len | (sc[q] >= 0 ? 0x80000000u : 0u));
            }
            for (unsigned int w = threadIdx.x; w < (a.n + 31u) / 32u; w += kTailThreads) lmark[w] = 0u;
        }
    }
    __syncthreads();
    // (the host knows the number of rows of the first round, not that a few of them are hubs)
    const bool fits = count[0] + count[1] <= a.max_rows;
    if (fits) {
        unsigned int e = 0;
        for (unsigned int i = threadIdx.x; i < count[0] + count[1]; i += kTailThreads) {
            const int32_t u = frontier_vertex(a.front[0], a.back[0], count[0], i);
            if constexpr (RES) llist[i < count[0] ? i : a.n - 1u - (i - count[0])] = (unsigned short)u;
            int64_t off;
            int len;
            record(u, &off, &len);
            e += tail_entries(len);
        }
        e = wave_sum(e);
        if (lane_id() == 0) atomicAdd(&next[2], e);
    }
    __syncthreads();
    int r = 0;
    for (; r < a.rounds; ++r) {
        const unsigned int ns = count[0], nl = count[1];  // uniform from here on
        if (ns + nl == 0u || leave || ns + nl > a.max_rows || next[2] > a.max_entries) break;
        __syncthreads();
        if (threadIdx.x == 0) {
            next[0] = next[1] = next[2] = 0u;
            moved = resid = 0u;
            entries[0] = entries[1] = 0u;
        }
        __syncthreads();
        const int cur = r & 1, nxt = cur ^ 1;
        float rmax = 0.f;
        unsigned int nmoved = 0, nent[2] = {0u, 0u};
        auto mark = [&](int32_t v) {  // v joins the next V_aff, once
            int len;
            if constexpr (RES) {
                const unsigned int q = lrow[v].y;
                if (q >> 31) return;
                len = (int)q;
                const unsigned int bit = 1u << ((unsigned int)v & 31u);
                if (atomicOr(&lmark[(unsigned int)v >> 5], bit) & bit) return;
            } else {
                // (both reads on their way together)
                const int32_t sc = a.seed_class[v];
                len = a.meta[v].len;
                if (sc >= 0) return;
                const unsigned int bit = 1u << (((unsigned int)v & 3u) * 8u);
                if (atomicOr(reinterpret_cast<unsigned int*>(a.flag) + ((unsigned int)v >> 2), bit) & bit) return;
            }
            atomicAdd(&next[2], tail_entries(len));
            if (len > kLongRow) {
                const unsigned int at = atomicAdd(&next[1], 1u);
                if constexpr (RES) llist[nxt * lstride + a.n - 1u - at] = (unsigned short)v;
                else a.back[nxt][-(long long)at] = v;
            } else {
                const unsigned int at = atomicAdd(&next[0], 1u);
                if constexpr (RES) llist[nxt * lstride + at] = (unsigned short)v;
                else a.front[nxt][at] = v;
            }
        };
        auto old_row = [&](int32_t u, int chunk) {
            if constexpr (RES) return load_vec<VEC>(lF + (unsigned int)u * CP + chunk * VEC);
            else return load_vec<VEC>(a.F + (size_t)u * CP + chunk * VEC);
        };
        auto accumulate = [&](auto lanes, const Edge* row, int len, int first, int step, int32_t u, int gl, Vec<VEC>& acc, float& s, Edge& e) {
            if constexpr (RES) accumulate_row<CP, decltype(lanes)::value>(row, len, first, step, u, lF, gl, acc, s, e);
            else accumulate_row<CP, decltype(lanes)::value>(row, len, first, step, u, a.F, gl, acc, s, e);
        };
        // the new row from the sums of its entries (the lanes of slot 0 hold acc and s), by the LPN lanes of one slot
        auto finish = [&](unsigned int pos, int32_t u, int chunk, const Vec<VEC>& acc, float s, const Vec<VEC>& old) {
            Vec<VEC> fn;
            float d = 0.f;
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                fn.v[k] = acc.v[k] / s;
                if (a.by_vertex & kRowLazy) fn.v[k] = 0.5f * (fn.v[k] + old.v[k]);
                d = fmaxf(d, fabsf(fn.v[k] - old.v[k]));
            }
#pragma unroll
            for (int k = 1; k < LPN; k <<= 1) d = fmaxf(d, __shfl_xor(d, k, LPN));
            if constexpr (RES) {
                store_vec<VEC>((a.by_vertex & kRowByVertex ? lF + (unsigned int)u * CP : lstaged + pos * CP) + chunk * VEC, fn);
            } else {
                float* const out = a.by_vertex & kRowByVertex ? a.F + (size_t)u * CP : a.staged + (size_t)pos * CP;
                store_vec<VEC>(out + chunk * VEC, fn);
            }
            return d;
        };
        // long rows: four at a time, 256 threads each, summed in the order k_row_update sums them
        for (unsigned int j0 = 0; j0 < nl; j0 += TEAMS) {
            const int team = threadIdx.x / kBlock, tid = threadIdx.x % kBlock;
            const unsigned int j = j0 + team;
            const int gi = tid / GL, gl = tid % GL, slot = gl / LPN, chunk = gl % LPN;
            const int32_t u = j < nl ? listed(cur, ns, ns + j) : 0;
            int64_t off;
            int len;
            record(u, &off, &len);
            if (j >= nl) len = 0;
            const Edge* __restrict__ row = a.pool + off;
            Vec<VEC> acc;
#pragma unroll
            for (int k = 0; k < VEC; ++k) acc.v[k] = 0.f;
            float s = 0.f;
            Edge e;
            e.col = u;
            e.w = 0.f;
            accumulate(std::integral_constant<int, GL>{}, row, len, gi, NG, u, gl, acc, s, e);
            if (slot == 0) {
#pragma unroll
                for (int k = 0; k < VEC; ++k) part[team][gi][chunk * VEC + k] = acc.v[k];
                if (gl == 0) part_s[team][gi] = s;
            }
            __syncthreads();
            if (gi == 0 && slot == 0 && j < nl) {
                Vec<VEC> tot;
#pragma unroll
                for (int k = 0; k < VEC; ++k) tot.v[k] = 0.f;
                float st = 0.f;
#pragma unroll 4
                for (int q = 0; q < NG; ++q) {
#pragma unroll
                    for (int k = 0; k < VEC; ++k) tot.v[k] += part[team][q][chunk * VEC + k];
                    st += part_s[team][q];
                }
                const float d = finish(ns + j, u, chunk, tot, st, old_row(u, chunk));
                if (gl == 0) {
                    rmax = fmaxf(rmax, d);
                    nent[1] += (unsigned int)len;
                    nmoved += d > a.tol ? 1u : 0u;
                    big[team] = d > a.tol ? 1u : 0u;
                }
            }
            __syncthreads();
            if (j < nl && big[team]) {
                if (tid == 0) mark(u);
                for (int k = tid; k < len; k += kBlock) mark(row[k].col);
            }
            __syncthreads();
        }
        for (unsigned int i = threadIdx.x / G; i < ns; i += kTailThreads / G) {
            const int32_t u = listed(cur, ns, i);
            const int gl = threadIdx.x % G, slot = gl / LPN, chunk = gl % LPN;
            int64_t off;
            int len;
            record(u, &off, &len);
            const Edge* __restrict__ row = a.pool + off;
            Vec<VEC> acc;
#pragma unroll
            for (int k = 0; k < VEC; ++k) acc.v[k] = 0.f;
            float s = 0.f;
            Edge e;
            e.col = u;
            e.w = 0.f;
            const Vec<VEC> old = old_row(u, chunk);
            accumulate(std::integral_constant<int, G>{}, row, len, 0, 1, u, gl, acc, s, e);
            float d = 0.f;
            if (slot == 0) d = finish(i, u, chunk, acc, s, old);
            d = __shfl(d, 0, G);
            if (gl == 0) {
                rmax = fmaxf(rmax, d);
                nent[0] += (unsigned int)len;
                nmoved += d > a.tol ? 1u : 0u;
            }
            if (d > a.tol) {  // the last chunk of the row is still in registers
                if (gl == 0) mark(u);
                if (e.w != 0.f) mark(e.col);
                const int last = ((len - 1) / G) * G;
                for (int j = gl; j < last; j += G) mark(row[j].col);
            }
        }
        rmax = wave_max(rmax);
        nmoved = wave_sum(nmoved);
        nent[0] = wave_sum(nent[0]);
        nent[1] = wave_sum(nent[1]);
        if (lane_id() == 0) {
            atomicMax(&resid, __float_as_uint(rmax));
            if (nmoved) atomicAdd(&moved, nmoved);
            if (nent[0]) atomicAdd(&entries[0], nent[0]);
            if (nent[1]) atomicAdd(&entries[1], nent[1]);
        }
        __syncthreads();
        if (!(a.by_vertex & kRowByVertex)) {
            constexpr unsigned int PER = CP / VEC;
            for (unsigned int i = threadIdx.x; i < (ns + nl) * PER; i += kTailThreads) {
                const unsigned int pos = i / PER;
                const unsigned int to = (unsigned int)listed(cur, ns, pos) * CP + (i % PER) * VEC;
                if constexpr (RES) store_vec<VEC>(lF + to, load_vec<VEC>(lstaged + pos * CP + (i % PER) * VEC));
                else
                    store_vec<VEC>(a.F + (size_t)listed(cur, ns, pos) * CP + (i % PER) * VEC,
                                   load_vec<VEC>(a.staged + (size_t)pos * CP + (i % PER) * VEC));
            }
        }
        if constexpr (RES) {
            for (unsigned int w = threadIdx.x; w < (a.n + 31u) / 32u; w += kTailThreads) lmark[w] = 0u;
        } else {
            for (unsigned int i = threadIdx.x; i < next[0] + next[1]; i += kTailThreads) a.flag[listed(nxt, next[0], i)] = 0;
        }
        if (threadIdx.x == 0) {
            RoundCtr* slot = a.ring + (a.t0 + r) % kRing;
            slot->next_count = next[0];
            slot->next_long = next[1];
            slot->executed = 1u;
            slot->rows_short = ns;
            slot->rows_long = nl;
            slot->any_moved = moved ? 1u : 0u;
            RoundPart* p = &slot->part[0];
            p->resid_bits = resid;
            p->changed = moved;
            p->edges = entries[0];
            p->edges_long = entries[1];
            count[0] = next[0];
            count[1] = next[1];
            same_run = ns + nl == sig[0] && moved == sig[1] && resid == sig[2] ? same_run + 1 : 0;
            sig[0] = ns + nl;
            sig[1] = moved;
            sig[2] = resid;
            repeats = repeats || (same_run >= a.same_max && !(a.by_vertex & kRowLazy));
            const unsigned long long e = (unsigned long long)entries[0] + entries[1], n = ns + nl;
            leave = (a.chain_off + r + 1) % a.chain == 0 && (repeats || e < n * a.len_lo || e >= n * a.len_hi);
        }
        __syncthreads();
    }
    if constexpr (RES) {
        if (r == 0) return;  // nothing has run: list and labels are as they were
        for (unsigned int i = threadIdx.x; i < a.n * CP / VEC; i += kTailThreads)
            store_vec<VEC>(a.F + (size_t)i * VEC, load_vec<VEC>(lF + i * VEC));
        const unsigned int ns = count[0], nl = count[1];
        for (unsigned int i = threadIdx.x; i < ns + nl; i += kTailThreads) {
            const int32_t u = listed(r & 1, ns, i);
            if (i < ns) a.front[r & 1][i] = u;
            else a.back[r & 1][-(long long)(i - ns)] = u;
        }
    }
}

// =================================================================================================
// Several rounds in one launch, for graphs whose rounds are too short to be worth a launch each
// =================================================================================================
// On a graph of a few hundred thousand rows a round over all rows takes tens of microseconds, of which the
// work is a small part: the rest is the launch, the ramp-up of thousands of short-lived workgroups and the
// drain before the next launch may start.  k_rounds_persistent runs up to `rounds` consecutive rounds of the kind
// k_row_update_pull runs (every updatable vertex decides from the previous round's bitmap whether it is in V_aff)
// with a grid of workgroups that are all resident at once and a barrier across the grid between rounds.
//
// What crosses the barrier (label rows, bitmap words, counters) is read and written with device-scope accesses
// (load_row / store_row / moved_bit_c with COH): every XCD has an L2 of its own, and writing back and invalidating
// whole caches at every barrier costs ten times the round.
//
// The barrier is a two-level tree, so that no address is polled by more than kBarGroup workgroups (a word polled by
// a thousand workgroups answers so slowly that the barrier alone took 100 us): a workgroup arrives at its group's
// counter; the last arrival of a group arrives at the global counter; the last arrival there writes the release
// word of every group, and every workgroup waits for the release word of its group only.  The arrivals carry along
// whether the workgroup moved a row in the round, so that the release word also says whether any row moved at all:
// if none did, V_aff is empty and every workgroup leaves the kernel.
//
// The wait is bounded.  After spin_limit polls a workgroup tries to give the barrier up for the whole grid: a
// compare-and-swap sets the top bit of the global counter, and only succeeds while the last group has not arrived
// there; the last arrival, in turn, does not release when it finds that bit set.  So either every workgroup is
// released from barrier k or none is, and no round is ever run by a part of the grid.  Every workgroup completes the
// work of a round before it looks at the barrier; whenever the kernel ends - all rounds done, V_aff empty, or a
// barrier given up - the rounds whose counter slots say "executed" have been executed in full, and the host goes
// on from there with ordinary launches.
constexpr unsigned int kBarGroup = 32;              // workgroups per group
constexpr unsigned int kBarWordsPerLine = 16;       // every counter and release word has a 64-byte line of its own
constexpr unsigned int kBarMaxGroups = 128;
constexpr unsigned int kBarGivenUp = 0x80000000u;   // global counter: the barrier was given up
constexpr unsigned int kBarMovedUnit = 0x10000u;    // counters: arrivals in the low 16 bits, arrivals that moved rows above
constexpr unsigned int kRelStop = 0x40000000u;      // release word: no row moved in the round
constexpr unsigned int kRelFail = 0x80000000u;      // release word: the barrier was given up
// words: [0] global counter, [1] "a barrier was given up" for the host, then one line per group counter, then one
// line per release word
constexpr unsigned int kBarWords = kBarWordsPerLine * (1 + 2 * kBarMaxGroups);

struct PersistArgs {
    RoundCtr* ring;               // kRing slots
    int t0;                       // round number of the first round (>= 1)
    int rounds;
    unsigned int long_blocks_max;
    const int32_t* front;         // list of all updatable vertices: short rows from the front, long rows from the back
    const int32_t* back;
    unsigned int ns, nl;
    const RowMeta* meta;
    const Edge* pool;
    float* buf0;                  // round t0 + r reads buf[r & 1] and writes buf[(r + 1) & 1] (one array in place)
    float* buf1;
    unsigned int* moved0;         // the three bitmaps; the round with stretch index q reads (q - 1) % 3, sets q % 3
    unsigned int* moved1;         // and clears (q + 1) % 3
    unsigned int* moved2;
    int q0;                       // stretch index of the first round (>= 1)
    unsigned int words;
    float tol;
    unsigned int* barrier;        // kBarWords words, all zero at launch
    unsigned int ngroups;         // ceil(gridDim.x / kBarGroup) <= kBarMaxGroups
    unsigned int spin_limit;
};

__device__ inline unsigned int load_fresh(const unsigned int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline void store_through(unsigned int* p, unsigned int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Barrier number k (1, 2, ...) of the launch.  moved: this workgroup moved at least one row in the round (thread 0's
// value counts).  Returns 1: released, some row moved; 2: released, no row moved anywhere; 0: given up.
__device__ inline int grid_barrier(unsigned int* bar, unsigned int k, unsigned int ngroups, bool moved,
                                   unsigned int spin_limit) {
    __shared__ int sh_res;
    // every wave: its stores and atomics of this round (all of them device-scope, write-through accesses) have been
    // acknowledged before the workgroup reports its arrival
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned int g = blockIdx.x / kBarGroup;
        const unsigned int first = g * kBarGroup;
        const unsigned int gsize = gridDim.x - first < kBarGroup ? gridDim.x - first : kBarGroup;
        unsigned int* global = bar;
        unsigned int* gctr = bar + kBarWordsPerLine * (1 + g);
        unsigned int* rel = bar + kBarWordsPerLine * (1 + ngroups + g);
        auto release_all = [&](unsigned int word) {
            for (unsigned int i = 0; i < ngroups; ++i) store_through(bar + kBarWordsPerLine * (1 + ngroups + i), word);
        };
        const unsigned int add = 1u + (moved ? kBarMovedUnit : 0u);
        const unsigned int in_group = atomicAdd(gctr, add) + add;
        if ((in_group & 0xffffu) == gsize * k) {
            // last of the group: take the group's "moved" count out again and arrive at the global counter
            const unsigned int group_moved = in_group & 0xffff0000u;
            if (group_moved) atomicSub(gctr, group_moved);
            const unsigned int gadd = 1u + (group_moved ? kBarMovedUnit : 0u);
            const unsigned int old = atomicAdd(global, gadd);
            const unsigned int now = old + gadd;
            if (old & kBarGivenUp) {
                release_all(kRelFail | k);
            } else if ((now & 0xffffu) == ngroups * k) {
                // last of all: nobody else touches the global counter until the next round's arrivals
                const unsigned int any_moved = now & 0x7fff0000u;
                if (any_moved) atomicSub(global, any_moved);
                release_all(k | (any_moved ? 0u : kRelStop));
            }
        }
        int res = -1;
        unsigned int spins = 0;
        while (res < 0) {
            const unsigned int w = load_fresh(rel);
            if (w & kRelFail) {
                res = 0;
            } else if ((w & 0xffffu) == k) {
                res = (w & kRelStop) ? 2 : 1;
            } else if (++spins > spin_limit) {
                // give up for everybody, unless the last group has arrived by now (then the release is on its way)
                const unsigned int v = load_fresh(global);
                if (v & kBarGivenUp) {
                    res = 0;
                } else if ((v & 0xffffu) >= ngroups * k) {
                    spins = 0;
                } else if (atomicCAS(global, v, v | kBarGivenUp) == v) {
                    release_all(kRelFail | k);
                    res = 0;
                }
            } else {
                __builtin_amdgcn_s_sleep(16);
            }
        }
        if (res == 0) store_through(&bar[1], 1u);  // for the host
        sh_res = res;
    }
    __syncthreads();
    const int res = sh_res;
    __syncthreads();  // sh_res may be rewritten by the next barrier
    return res;
}

template <int CP, int G>
__global__ void __launch_bounds__(kBlock) k_rounds_persistent(PersistArgs a) {
    __shared__ unsigned int sh_go;
    unsigned int* const moved[3] = {a.moved0, a.moved1, a.moved2};
    float* const buf[2] = {a.buf0, a.buf1};
    const unsigned int long_blocks = a.nl < a.long_blocks_max ? a.nl : a.long_blocks_max;
    {
        // the round before the launch: did it run, and did it move a row?  (every later round learns this from the
        // barrier)
        const RoundCtr* prev = a.ring + ((a.t0 - 1) % kRing);
        if (threadIdx.x < kWave) {
            unsigned int prev_changed = lane_id() < kCtrLanes ? load_fresh(&prev->part[lane_id()].changed) : 0u;
            prev_changed = wave_sum(prev_changed);
            if (threadIdx.x == 0) sh_go = (load_fresh(&prev->executed) != 0u && prev_changed != 0u) ? 1u : 0u;
        }
        __syncthreads();
        if (sh_go == 0u) return;  // the same for every workgroup
    }
    for (int r = 0; r < a.rounds; ++r) {
        const int t = a.t0 + r;
        RoundCtr* ctr = a.ring + (t % kRing);
        RoundCtr* ctr_zero = a.ring + ((t + 1) % kRing);
        if (blockIdx.x == 0) {  // write-through stores: the slot's next user may sit on another XCD
            auto put64 = [](unsigned long long* p, unsigned long long v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
            if (threadIdx.x == 0) {
                store_through(&ctr_zero->next_count, 0u);
                store_through(&ctr_zero->next_long, 0u);
                store_through(&ctr_zero->executed, 0u);
                store_through(&ctr_zero->rows_short, 0u);
                store_through(&ctr_zero->rows_long, 0u);
                store_through(&ctr_zero->any_moved, 0u);
                store_through(&ctr->executed, 1u);
            }
            if (threadIdx.x < kCtrLanes) {
                RoundPart* p = &ctr_zero->part[threadIdx.x];
                store_through(&p->resid_bits, 0u);
                store_through(&p->changed, 0u);
                put64(&p->edges, 0ull);
                put64(&p->edges_long, 0ull);
                store_through(&p->rows_short, 0u);
                store_through(&p->rows_long, 0u);
            }
        }
        const int q = a.q0 + r;
        unsigned int* moved_clear = moved[(q + 1) % 3];
        for (unsigned int w = blockIdx.x * kBlock + threadIdx.x; w < a.words; w += gridDim.x * kBlock)
            store_through(&moved_clear[w], 0u);
        const float* F_in = buf[r & 1];
        float* F_out = buf[(r + 1) & 1];
        unsigned int block_moved;
        if (blockIdx.x < long_blocks)
            block_moved = row_update_long<CP, false, true, true>(blockIdx.x, long_blocks, a.back, a.nl, a.ns, a.meta, a.pool,
                                                                 F_in, F_out, 1, nullptr, moved[q % 3], a.tol, ctr,
                                                                 moved[(q + 2) % 3]);
        else
            block_moved = row_update_short<CP, G, false, true, true>(blockIdx.x - long_blocks, gridDim.x - long_blocks, a.front,
                                                                     a.ns, a.meta, a.pool, F_in, F_out, 1, nullptr,
                                                                     moved[q % 3], a.tol, ctr, moved[(q + 2) % 3]);
        if (r + 1 == a.rounds) return;
        if (grid_barrier(a.barrier, (unsigned int)(r + 1), a.ngroups, block_moved != 0u, a.spin_limit) != 1) return;
    }
}

}  // namespace dynlp
