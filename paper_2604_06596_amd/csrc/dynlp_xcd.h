// Rounds over a small graph: many per launch, on the CUs of one XCD.
//
// A round over a few thousand to a few ten thousand vertices is one or two launches of 5 to 10 us each, whatever they do, with
// gaps of about as much between those of a marking round (2,000 vertices of degree 16 with 4 columns: 9 us per fused round, 14
// per marking one; 20,000 of degree 8: 17).  A barrier across the whole chip costs as much as a launch, because the XCDs have
// an L2 each and what they exchange has to get past those.  The 32 CUs of one XCD share an L2: whatever one of their
// workgroups has stored, the others read from there, and they wait for each other in about a microsecond.  k_xcd_rounds
// therefore runs up to kXcdRounds rounds in one launch on the workgroups of one XCD; those that start on the others leave at
// once.
//
// Which XCD, and which of its workgroups: see dynlp_signin.h.  Those that take part are running and agree on who they are, so
// every wait for the others ends, whatever else the chip does meanwhile; rows are cut among as many as came.  Where the entries
// of a workgroup's rows do not fit its LDS, no round is run and the host goes on with ordinary ones.
//
// Each workgroup keeps the entries and records of its rows in LDS, and one bit per vertex of the graph, "moved in the previous
// round"; from that it lists its rows of V_aff (u moved or a neighbour did: Alg. 2 Step 3), gathers their neighbours' label
// rows from the L2 and writes the new rows back there.  Sums are formed in the order of accumulate_row, so that a round's
// result is that of an ordinary launch bit for bit.  Synchronous mode: rounds take turns between the two label buffers; a row
// that leaves V_aff is copied once.
//
// Between two rounds every workgroup publishes the moved bits of its rows and its counters as 64-bit words, half of which is
// the number of the launch and of the exchange, and polls those of all others until they carry that number too: barrier and
// exchange in one trip (a barrier counter and the bits after it took 2.2 us).  What the workgroup has stored before is in the
// L2 by then (xcd_drain).  What crosses workgroups is read at device scope, past the L1 of the CU.
//
// What bounds a round: latency, some four dependent trips to the L2; beyond some 100,000 entries the gathers.
// Measured (whole calls, before / after): see xcd_rounds_pay in dynlp.hip; next to other contexts: xcd_rounds_at_once.
#pragma once

#include "dynlp_frontier.h"
#include "dynlp_signin.h"

namespace dynlp {

constexpr int kXcdThreads = 1024;
constexpr int kXcdGroups = 32;          // workgroups at most: one per CU of an XCD
constexpr int kXcdRounds = 240;         // rounds per launch at most; exchanges are numbered with 8 bits
constexpr int kXcdChain = 8;            // rounds between two decisions at most
constexpr unsigned int kXcdMaxRows = 32768;   // a moved word per thread
constexpr unsigned int kXcdLds = 140u << 10;  // dynamic LDS of a workgroup
constexpr int kXcdLooks = 64;           // at the list before it is closed with fewer workgroups than wanted
constexpr unsigned int kXcdLaunches = (1u << 24) - 1u;  // numbers of launches; the host clears XcdCtl before it starts again

// Counters of a round: of one workgroup, or of all.
struct __attribute__((aligned(16))) XcdPart {
    unsigned int resid_bits, changed, entries, rows;
};

// What a launch tells the host, in pinned memory.
struct __attribute__((aligned(16))) XcdResult {
    unsigned int rounds;  // executed
    unsigned int next;    // |V_aff| of the round after
    unsigned int groups;  // workgroups that shared them
    unsigned int pad;
    XcdPart round[kXcdRounds];
};

constexpr int kXcdPartWords = 3;  // a workgroup's counters in the exchange: max change; rows moved << 16 | rows; entries

struct __attribute__((aligned(64))) XcdCtl {
    unsigned int turn;       // launch << 8 | XCD
    unsigned int pad0[31];
    unsigned int signed_in[2][32];  // [0]: by parity of the launch, workgroups that came, kListClosed; 0 when its launch begins
    unsigned int groups;            // launch << 8 | workgroups that share its rounds
    unsigned int pad1[31];
    unsigned long long part[2][kXcdPartWords][kXcdGroups];  // by parity of the exchange: launch << 8 | exchange, and 32 bits
    unsigned long long moved[2][kXcdMaxRows / 32];
};

struct XcdArgs {
    XcdCtl* ctl;
    XcdResult* result;            // pinned
    unsigned int* flag;           // pinned: set to `value` when the result is there
    unsigned int value;
    unsigned int launch;          // number of the launch, 1 .. kXcdLaunches
    unsigned int want;            // workgroups wanted
    unsigned int zero;            // 0, unknown to the compiler: reads by atomic addition stay what they are
    RoundCtr* ring;
    int t0, rounds;               // rounds t0 .. t0 + rounds - 1 at most; rounds <= kXcdRounds
    int32_t* front[2];            // the first round's list: front[0] (no long rows); the one after r rounds: front[r & 1]
    const RowMeta* meta;
    const Edge* pool;
    const int32_t* seed_class;
    float* F[2];                  // round t0 + r reads F[r & 1] and writes F[(r + 1) & 1] (the same array in place)
    unsigned int n;               // <= kXcdMaxRows
    int all_rows;                 // static sweeps: every updatable row in every round
    int lazy;                     // averaged rows
    float tol;
    int chain, chain_off;         // as in TailArgs; chain <= kXcdChain
    unsigned int len_lo, len_hi;
    int same_run, same_max;
    unsigned int sig[3];
};

__device__ inline unsigned int xcd_id() { return __builtin_amdgcn_s_getreg((3 << 11) | 20); }  // HW_REG_XCC_ID, 4 bits

// Everything this wave has stored is in the L2.
__device__ inline void xcd_drain() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
}

typedef unsigned int xcd_u4 __attribute__((ext_vector_type(4)));
typedef unsigned int xcd_u2 __attribute__((ext_vector_type(2)));

// Label rows: written through to the L2 as all stores are, read at device scope (sc1): past the L1 of the CU.  (At workgroup
// scope, sc0, a read may find what an earlier round left in the L1.)  `at` in bytes, below 2^31.
constexpr int kXcdScope = 16;
struct XcdArray {
    __amdgpu_buffer_rsrc_t r;
    __device__ inline XcdArray(const void* p, unsigned int bytes)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00027000)) {}
    template <int V>
    __device__ inline Vec<V> load(unsigned int at) const {
        Vec<V> x;
        if constexpr (V == 4) {
            const xcd_u4 q = __builtin_amdgcn_raw_buffer_load_b128(r, (int)at, 0, kXcdScope);
            x.v[0] = __uint_as_float(q.x);
            x.v[1] = __uint_as_float(q.y);
            x.v[2] = __uint_as_float(q.z);
            x.v[3] = __uint_as_float(q.w);
        } else if constexpr (V == 2) {
            const xcd_u2 q = __builtin_amdgcn_raw_buffer_load_b64(r, (int)at, 0, kXcdScope);
            x.v[0] = __uint_as_float(q.x);
            x.v[1] = __uint_as_float(q.y);
        } else {
            x.v[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)at, 0, kXcdScope));
        }
        return x;
    }
    template <int V>
    __device__ inline void store(unsigned int at, const Vec<V>& x) const {
        if constexpr (V == 4) {
            const xcd_u4 q = {__float_as_uint(x.v[0]), __float_as_uint(x.v[1]), __float_as_uint(x.v[2]), __float_as_uint(x.v[3])};
            __builtin_amdgcn_raw_buffer_store_b128(q, r, (int)at, 0, 0);
        } else if constexpr (V == 2) {
            const xcd_u2 q = {__float_as_uint(x.v[0]), __float_as_uint(x.v[1])};
            __builtin_amdgcn_raw_buffer_store_b64(q, r, (int)at, 0, 0);
        } else {
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x.v[0]), r, (int)at, 0, 0);
        }
    }
};

// x of the lane whose number differs in bit D, for D < 16: by DPP moves, without the LDS unit that shuffles go through (16 waves
// that reduce 5 values over 16 lanes keep it busy for longer than their gathers take).
template <int D>
__device__ inline unsigned int lane_xor(unsigned int x) {
    static_assert(D == 1 || D == 2 || D == 4 || D == 8, "within a row of 16 lanes");
    auto dpp = [](unsigned int v, auto ctrl) {
        return (unsigned int)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xf, 0xf, true);
    };
    if constexpr (D == 1) return dpp(x, std::integral_constant<int, 0xb1>{});                  // quad_perm 1 0 3 2
    if constexpr (D == 2) return dpp(x, std::integral_constant<int, 0x4e>{});                  // quad_perm 2 3 0 1
    if constexpr (D == 4)                                                                      // row_half_mirror, quad_perm 3 2 1 0
        return dpp(dpp(x, std::integral_constant<int, 0x141>{}), std::integral_constant<int, 0x1b>{});
    return dpp(x, std::integral_constant<int, 0x128>{});                                       // row_ror 8
}
template <int D>
__device__ inline float lane_xor(float x) {
    return __uint_as_float(lane_xor<D>(__float_as_uint(x)));
}

// x + x of the lanes that differ in bits FROM, 2 FROM, ... below G, as a butterfly of shuffles sums them.
template <int FROM, int G>
__device__ inline float lanes_sum(float x) {
    if constexpr (FROM < G) return lanes_sum<2 * FROM, G>(x + lane_xor<FROM>(x));
    else return x;
}
template <int FROM, int G>
__device__ inline float lanes_max(float x) {
    if constexpr (FROM < G) return lanes_max<2 * FROM, G>(fmaxf(x, lane_xor<FROM>(x)));
    else return x;
}

// Over the 64 lanes of a wave.
__device__ inline unsigned int wave_total(unsigned int x) {
    x += lane_xor<1>(x);
    x += lane_xor<2>(x);
    x += lane_xor<4>(x);
    x += lane_xor<8>(x);
    return (unsigned int)(__builtin_amdgcn_readlane((int)x, 0) + __builtin_amdgcn_readlane((int)x, 16) + __builtin_amdgcn_readlane((int)x, 32) +
                          __builtin_amdgcn_readlane((int)x, 48));
}
__device__ inline unsigned int wave_top(unsigned int x) {
    x = max(x, lane_xor<1>(x));
    x = max(x, lane_xor<2>(x));
    x = max(x, lane_xor<4>(x));
    x = max(x, lane_xor<8>(x));
    return max(max((unsigned int)__builtin_amdgcn_readlane((int)x, 0), (unsigned int)__builtin_amdgcn_readlane((int)x, 16)),
               max((unsigned int)__builtin_amdgcn_readlane((int)x, 32), (unsigned int)__builtin_amdgcn_readlane((int)x, 48)));
}

__device__ inline void xcd_put(unsigned long long* p, unsigned int tag, unsigned int x) {
    __hip_atomic_store(p, (unsigned long long)tag << 32 | x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The word's 32 bits once it carries the tag.  (Its writer runs, and writes it before it waits for anything itself.)
__device__ inline unsigned int xcd_get(unsigned long long* p, unsigned int tag) {
    unsigned long long x;
    do x = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    while ((unsigned int)(x >> 32) != tag);
    return (unsigned int)x;
}

// The words of dynlp_signin.h.  `turn` is reached from all XCDs, the others from one.
struct XcdSignIn {
    XcdCtl* ctl;
    unsigned int zero;  // 0, unknown to the compiler
    __device__ inline unsigned int read_turn() { return __hip_atomic_fetch_add(&ctl->turn, zero, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ inline bool set_turn(unsigned int* seen, unsigned int value) {
        return __hip_atomic_compare_exchange_strong(&ctl->turn, seen, value, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ inline unsigned int add(int p) { return __hip_atomic_fetch_add(ctl->signed_in[p], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ inline unsigned int look(int p) { return __hip_atomic_fetch_add(ctl->signed_in[p], zero, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ inline unsigned int close(int p) {
        return __hip_atomic_fetch_or(ctl->signed_in[p], kListClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ inline void clear(int p) { __hip_atomic_store(ctl->signed_in[p], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ inline void publish(unsigned int word) {
        (void)__hip_atomic_exchange(&ctl->groups, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ inline unsigned int published() {
        return __hip_atomic_fetch_add(&ctl->groups, zero, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};

template <int CP, int G>
__global__ void __launch_bounds__(kXcdThreads) k_xcd_rounds(XcdArgs a) {
    constexpr int VEC = RowShape<CP>::VEC;
    constexpr int LPN = RowShape<CP>::LPN;
    constexpr int SLOTS = G / LPN;
    constexpr int NW = kXcdThreads / kWave;
    extern __shared__ __align__(16) unsigned char xcd_lds[];
    __shared__ int sh_place;
    __shared__ unsigned int sh_groups;
    __shared__ bool sh_leave;
    __shared__ unsigned int na;                              // rows listed in act
    __shared__ unsigned int sh_resid, sh_moved, sh_entries;  // of the running round
    __shared__ unsigned int sh_wave[NW];
    __shared__ XcdPart parts[kXcdChain][kXcdGroups];         // of the last rounds
    __shared__ XcdPart sums[kXcdChain];
    const int tid = (int)threadIdx.x;

    if (tid == 0) {
        XcdSignIn words{a.ctl, a.zero};
        const SignedIn in = sign_in(words, a.launch, xcd_id(), a.want, kXcdLooks);
        sh_place = in.place;
        sh_groups = in.groups;
        na = 0u;
        sh_resid = sh_moved = sh_entries = 0u;
    }
    __syncthreads();
    const int place = sh_place;
    if (place < 0) return;
    const unsigned int P = sh_groups;
    XcdCtl* const ctl = a.ctl;

    // ---- the workgroup's rows ----
    const unsigned int words = (a.n + 31u) / 32u, wper = (words + P - 1u) / P, per = wper * 32u;  // rows per workgroup
    const unsigned int v0 = min((unsigned int)place * per, a.n), rows = min(a.n - v0, per);
    const unsigned int words4 = (words + 3u) & ~3u, wper4 = (wper + 3u) & ~3u;
    unsigned int* const bits = reinterpret_cast<unsigned int*>(xcd_lds);         // words4: moved in the previous round
    unsigned int* const mine = bits + words4;                                    // wper4: moved in this one, of the own rows
    unsigned int* const was = mine + wper4;                                      // wper4: own rows updated in the previous round
    unsigned int* const rec = was + wper4;                                       // per: first entry << 8 | entries (0: never updated)
    unsigned short* const act = reinterpret_cast<unsigned short*>(rec + per);    // per: this round's rows, from v0 on
    Edge* const ent = reinterpret_cast<Edge*>(act + per);
    const unsigned int head = 4u * (words4 + 2u * wper4) + 6u * per;
    const unsigned int cap = head < kXcdLds ? (kXcdLds - head) / (unsigned int)sizeof(Edge) : 0u;
    const unsigned int bytes = a.n * (unsigned int)CP * 4u;
    const XcdArray Fa(a.F[0], bytes), Fb(a.F[1], bytes);
    const bool two = a.F[0] != a.F[1];
    const RoundCtr* const prev = a.t0 == 0 ? a.ring + kRing : a.ring + (a.t0 + kRing - 1) % kRing;
    const unsigned int listed = prev->next_count;
    bool refused = head > kXcdLds || (!a.all_rows && prev->next_long != 0u);  // (uniform)
    // records: lengths of the updatable rows, and where their entries go
    unsigned int total = 0, updatable = 0;
    int too_long = 0;
    for (unsigned int b = 0; b < rows && !refused; b += kXcdThreads) {
        const unsigned int i = b + tid;
        unsigned int len = 0;
        if (i < rows && a.seed_class[v0 + i] < 0) len = (unsigned int)a.meta[v0 + i].len;
        too_long |= len > (unsigned int)kLongRow ? 1 : 0;  // (the host does not launch this where there are any)
        const unsigned int inc = wave_inclusive_scan(len);
        if (lane_id() == kWave - 1) sh_wave[tid / kWave] = inc;
        updatable += (unsigned int)__syncthreads_count(len > 0u);
        unsigned int before = total;
        for (int w = 0; w < NW; ++w) {
            if (w < tid / kWave) before += sh_wave[w];
            total += sh_wave[w];
        }
        if (i < rows) rec[i] = (before + inc - len) << 8 | (len & 255u);
        __syncthreads();
    }
    refused = __syncthreads_or(too_long) != 0 || refused || total > cap;
    if (!refused) {
        for (unsigned int i = tid; i < wper; i += kXcdThreads) mine[i] = was[i] = 0u;
        for (unsigned int i = tid / 16; i < rows; i += kXcdThreads / 16) {
            const unsigned int q = rec[i];
            if (q & 255u) {
                const Edge* __restrict__ row = a.pool + a.meta[v0 + i].off;
                for (unsigned int j = tid % 16; j < (q & 255u); j += 16) ent[(q >> 8) + j] = row[j];
            }
        }
        if (two)
            for (unsigned int i = tid; i < rows * (CP / VEC); i += kXcdThreads)
                Fb.template store<VEC>((v0 * CP + i * VEC) * 4u, Fa.template load<VEC>((v0 * CP + i * VEC) * 4u));
        if (a.all_rows) {
            for (unsigned int i = tid; i < rows; i += kXcdThreads)
                if (rec[i] & 255u) act[atomicAdd(&na, 1u)] = (unsigned short)i;
        } else {
            for (unsigned int i = tid; i < listed; i += kXcdThreads) {
                const unsigned int v = (unsigned int)a.front[0][i] - v0;
                if (v < rows) act[atomicAdd(&na, 1u)] = (unsigned short)v;
            }
        }
    }

    // Exchange k: this workgroup's counters, and with_bits: the moved bits of its rows; then everybody's, into parts[at] and
    // bits.  Whether any workgroup has changed != 0.  Call from all threads, after a barrier.
    // (A word is written again two exchanges later, when all have read it: their words of the exchange between say so.)
    auto exchange = [&](unsigned int k, const XcdPart& p, bool with_bits, int at) -> bool {
        const unsigned int tag = a.launch << 8 | k;
        unsigned long long* const out = &ctl->part[k & 1][0][0];
        if (tid < kXcdPartWords)
            xcd_put(out + tid * kXcdGroups + place, tag, tid == 0 ? p.resid_bits : tid == 1 ? p.changed << 16 | p.rows : p.entries);
        if (with_bits && (unsigned int)tid < wper) {
            if ((unsigned int)place * wper + tid < words) xcd_put(&ctl->moved[k & 1][place * wper + tid], tag, mine[tid]);
            mine[tid] = 0u;
        }
        unsigned int any = 0;
        if (with_bits && (unsigned int)tid < words) bits[tid] = xcd_get(&ctl->moved[k & 1][tid], tag);
        const int q = kXcdThreads - 1 - tid;  // (the last waves: the first ones have the bits of small graphs)
        if (q < kXcdPartWords * kXcdGroups && (unsigned int)(q % kXcdGroups) < P) {
            const unsigned int x = xcd_get(out + q, tag);
            XcdPart* const to = &parts[at][q % kXcdGroups];
            if (q < kXcdGroups) {
                to->resid_bits = x;
            } else if (q < 2 * kXcdGroups) {
                to->changed = x >> 16;
                to->rows = x & 0xffffu;
                any = x >> 16;
            } else {
                to->entries = x;
            }
        }
        return __syncthreads_or(any != 0u ? 1 : 0) != 0;
    };
    xcd_drain();
    __syncthreads();
    refused = exchange(0u, XcdPart{0u, refused ? 1u : 0u, 0u, 0u}, false, 0);

    // The rows of V_aff among this workgroup's, from the moved bits of round r - 1; the others are settled.  One, two or four
    // lanes per row, eight entries each at a time.
    auto has_moved = [&](unsigned int v) -> bool { return (bits[v >> 5] >> (v & 31u)) & 1u; };
    auto list_rows = [&](int r, bool last) {
        const int lg = rows <= kXcdThreads / 4 ? 2 : rows <= kXcdThreads / 2 ? 1 : 0;
        const int sub = tid & ((1 << lg) - 1);
        for (unsigned int b = 0; b < rows; b += kXcdThreads >> lg) {
            const unsigned int i = b + ((unsigned int)tid >> lg);
            const unsigned int q = i < rows ? rec[i] : 0u;
            const int len = (int)(q & 255u);
            const Edge* const row = ent + (q >> 8);
            bool in = len > 0 && has_moved(v0 + i);
            for (int base = sub; base - sub < len && !in; base += 8 << lg) {  // uniform in the row's lanes
                int col[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) col[j] = row[min(base + (j << lg), len - 1)].col;
#pragma unroll
                for (int j = 0; j < 8; ++j) in = has_moved((unsigned int)col[j]) || in;
                if (lg > 0) in = lane_xor<1>(in ? 1u : 0u) != 0u || in;
                if (lg > 1) in = lane_xor<2>(in ? 1u : 0u) != 0u || in;
            }
            const unsigned long long first = __ballot(in && sub == 0);
            unsigned int at = 0;
            if (lane_id() == 0 && first) at = atomicAdd(&na, (unsigned int)__popcll(first));
            at = (unsigned int)__builtin_amdgcn_readfirstlane((int)at);
            if (in && sub == 0) act[at + (unsigned int)__popcll(first & ((1ull << lane_id()) - 1ull))] = (unsigned short)i;
            if (!in && len > 0 && sub == 0 && two && !last && ((was[i >> 5] >> (i & 31u)) & 1u)) {
                atomicAnd(&was[i >> 5], ~(1u << (i & 31u)));
#pragma unroll
                for (int c = 0; c < LPN; ++c) {
                    const unsigned int p = ((v0 + i) * CP + c * VEC) * 4u;
                    (r & 1 ? Fa : Fb).template store<VEC>(p, (r & 1 ? Fb : Fa).template load<VEC>(p));
                }
            }
        }
    };

    int r = 0, done = 0, same_run = a.same_run;  // rounds run; of those, folded
    unsigned int sig[3] = {a.sig[0], a.sig[1], a.sig[2]};
    bool repeats = false, more = true, keep = a.all_rows != 0;  // keep: the rows of the next round are those of this one
    // Counters of rounds done .. r - 1 over all workgroups, for the decisions the host takes between two chains of launches
    // (the same in every workgroup) and, from the workgroup at place 0, for the host.
    auto fold = [&]() {
        for (int q = done + tid / kWave; q < r; q += NW) {
            XcdPart p{0u, 0u, 0u, 0u};
            if ((unsigned int)lane_id() < P) p = parts[q % kXcdChain][lane_id()];
            const XcdPart f{wave_top(p.resid_bits), wave_total(p.changed), wave_total(p.entries), wave_total(p.rows)};
            if (lane_id() == 0) {
                sums[q % kXcdChain] = f;
                if (place == 0) a.result->round[q] = f;
            }
        }
        __syncthreads();
        if (tid == 0) {
            unsigned int e = 0, nr = 0;
            for (int q = done; q < r; ++q) {
                const XcdPart f = sums[q % kXcdChain];
                const bool same = f.resid_bits == sig[2] && (a.all_rows || (f.rows == sig[0] && f.changed == sig[1]));
                same_run = same ? same_run + 1 : 0;
                sig[0] = f.rows;
                sig[1] = f.changed;
                sig[2] = f.resid_bits;
                repeats = repeats || (same_run >= a.same_max && !a.lazy);
                e = f.entries;
                nr = f.rows;
            }
            sh_leave = repeats || (!a.all_rows && (e < nr * a.len_lo || e >= nr * a.len_hi));
        }
        done = r;
        __syncthreads();
    };
    while (!refused && more && r < a.rounds) {
        if (r > 0 && !keep) {
            list_rows(r, false);
            __syncthreads();
        }
        const unsigned int count = na;
        const XcdArray Fi = r & 1 ? Fb : Fa, Fo = r & 1 ? Fa : Fb;
        float rmax = 0.f;
        unsigned int nmoved = 0, nent = 0;
        // A lane sums S of the SLOTS partial sums that the 16 (or 4) lanes of a row share in accumulate_row, in the same order, and
        // those of the row's lanes meet in the same tree: what a sum is does not depend on S.  H gathers of a lane are in flight
        // together.  (Few rows wait for the longest of them: a lane per slot.  Many take as long as their instructions: 64 rows of 8
        // entries with 4 columns are 16 x 150 of them with 16 lanes per row, 2 x 230 with two.)
        auto update = [&](auto slots, auto in_flight) {
            constexpr int S = decltype(slots)::value, R = SLOTS / S, LR = LPN * R;  // lanes per row
            constexpr int H = decltype(in_flight)::value;
            static_assert(H % S == 0, "whole steps of a lane's slots");
            const int sub = tid % LR, chunk = sub % LPN, part = sub / LPN;
            for (unsigned int i = (unsigned int)(tid / LR); i < count; i += kXcdThreads / LR) {
                const unsigned int li = act[i], x = rec[li];
                const int len = (int)(x & 255u);
                const Edge* const row = ent + (x >> 8) + part * S;
                const Vec<VEC> old = Fi.template load<VEC>(((v0 + li) * CP + chunk * VEC) * 4u);
                Vec<VEC> acc[S];
                float s[S];
#pragma unroll
                for (int j = 0; j < S; ++j) {
#pragma unroll
                    for (int k = 0; k < VEC; ++k) acc[j].v[k] = 0.f;
                    s[j] = 0.f;
                }
#pragma unroll 1
                for (int base = 0; base < len; base += H / S * SLOTS) {  // (steps of SLOTS entries, S of them this lane's)
                    Edge e[H];
                    Vec<VEC> f[H];
#pragma unroll
                    for (int h = 0; h < H; ++h) {
                        const int idx = base + h / S * SLOTS + h % S;
                        e[h].col = 0;
                        e[h].w = 0.f;
                        if (idx + part * S < len) e[h] = row[idx];
                    }
#pragma unroll
                    for (int h = 0; h < H; ++h) {
#pragma unroll
                        for (int k = 0; k < VEC; ++k) f[h].v[k] = 0.f;
                        if (base + h / S * SLOTS + h % S + part * S < len)
                            f[h] = Fi.template load<VEC>(((unsigned int)e[h].col * CP + chunk * VEC) * 4u);
                    }
#pragma unroll
                    for (int h = 0; h < H; ++h) {
#pragma unroll
                        for (int k = 0; k < VEC; ++k) acc[h % S].v[k] = fmaf(e[h].w, f[h].v[k], acc[h % S].v[k]);
                        s[h % S] += e[h].w;
                    }
                }
#pragma unroll
                for (int d = 1; d < S; d <<= 1)
#pragma unroll
                    for (int j = 0; j < S; j += 2 * d) {
#pragma unroll
                        for (int k = 0; k < VEC; ++k) acc[j].v[k] += acc[j + d].v[k];
                        s[j] += s[j + d];
                    }
                const float sum = lanes_sum<LPN, LR>(s[0]);
                Vec<VEC> fn;
                float d = 0.f;
#pragma unroll
                for (int k = 0; k < VEC; ++k) {
                    fn.v[k] = lanes_sum<LPN, LR>(acc[0].v[k]) / sum;
                    if (a.lazy) fn.v[k] = 0.5f * (fn.v[k] + old.v[k]);
                    d = fmaxf(d, fabsf(fn.v[k] - old.v[k]));
                }
                d = lanes_max<1, LPN>(d);
                if (part == 0) Fo.template store<VEC>(((v0 + li) * CP + chunk * VEC) * 4u, fn);
                if (sub == 0) {
                    const bool big = d > a.tol;
                    const unsigned int word = li >> 5, bit = 1u << (li & 31u);
                    rmax = fmaxf(rmax, d);
                    nent += (unsigned int)len;
                    nmoved += big ? 1u : 0u;
                    if (big) atomicOr(&mine[word], bit);
                    if (two) atomicOr(&was[word], bit);
                }
            }
        };
        using std::integral_constant;
        if constexpr (G == 4) {
            if (count <= kXcdThreads / 4) update(integral_constant<int, 1>{}, integral_constant<int, 4>{});
            else update(integral_constant<int, 4>{}, integral_constant<int, 8>{});
        } else {
            constexpr int MANY = CP == 1 ? 16 : CP <= 4 ? 8 : 4;
            if (count <= 2 * kXcdThreads / 16) update(integral_constant<int, 1>{}, integral_constant<int, CP <= 8 ? 4 : 8>{});
            else if (MANY == 4 || count <= 2 * kXcdThreads / 4) update(integral_constant<int, 4>{}, integral_constant<int, 8>{});
            else update(integral_constant<int, MANY>{}, integral_constant<int, MANY>{});
        }
        const unsigned int top = wave_top(__float_as_uint(rmax));  // (non-negative floats order as integers)
        nmoved = wave_total(nmoved);
        nent = wave_total(nent);
        if (lane_id() == 0) {
            if (top) atomicMax(&sh_resid, top);
            if (nmoved) atomicAdd(&sh_moved, nmoved);
            if (nent) atomicAdd(&sh_entries, nent);
        }
        xcd_drain();
        __syncthreads();
        const XcdPart own{sh_resid, sh_moved, sh_entries, count};
        more = exchange((unsigned int)r + 1u, own, !a.all_rows, r % kXcdChain);
        // (all the workgroup's updatable rows have moved: they are in V_aff again)
        keep = a.all_rows != 0 || (own.changed == count && count == updatable);
        if (tid == 0) {
            sh_resid = sh_moved = sh_entries = 0u;
            if (!keep) na = 0u;
        }
        ++r;
        if ((a.chain_off + r) % a.chain == 0) {
            fold();
            if (sh_leave) break;
        } else {
            __syncthreads();
        }
    }
    fold();

    // ---- the list of the next round, and what the host and ordinary rounds look for ----
    const bool list = r > 0 && more && !a.all_rows;
    if (list && !keep) {
        list_rows(r, true);
        __syncthreads();
    }
    (void)exchange((unsigned int)r + 1u, XcdPart{0u, 0u, na, 0u}, false, 0);
    unsigned int before = 0, next = 0;
    for (unsigned int q = 0; q < P; ++q) {
        const unsigned int x = parts[0][q].entries;
        if (q < (unsigned int)place) before += x;
        next += x;
    }
    if (list)
        for (unsigned int i = tid; i < na; i += kXcdThreads) a.front[r & 1][before + i] = (int32_t)(v0 + act[i]);
    if (place != 0) return;
    if (r > 0) {
        RoundCtr* const end = a.ring + (a.t0 + r + kRing - 1) % kRing;
        constexpr int kWords = sizeof(RoundCtr) / 4;
        for (int i = tid; i < 2 * kWords; i += kXcdThreads)
            reinterpret_cast<unsigned int*>(i < kWords ? end : a.ring + (a.t0 + r) % kRing)[i % kWords] = 0u;
        xcd_drain();
        __syncthreads();
        if (tid == 0) {
            const XcdPart f = sums[(r - 1) % kXcdChain];
            end->next_count = next;
            end->executed = 1u;
            end->rows_short = f.rows;
            end->any_moved = f.changed ? 1u : 0u;
            end->part[0].resid_bits = f.resid_bits;
            end->part[0].changed = f.changed;
            end->part[0].edges = f.entries;
        }
    }
    if (tid == 0) {
        a.result->rounds = (unsigned int)r;
        a.result->next = next;
        a.result->groups = P;
    }
    __threadfence_system();
    __syncthreads();
    if (tid == 0) __hip_atomic_store(a.flag, a.value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace dynlp
