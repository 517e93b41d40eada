// Conjugate rounds of the in-place mode: the fixed point of Eq. (1) over all updatable rows by the method of conjugate
// gradients (Hestenes and Stiefel 1952).
//
// With D the rows' degrees, W the weights between updatable rows and b what the labelled neighbours contribute, every
// column x of the label matrix solves (D - W) x = b, a symmetric positive definite system (semidefinite where a component
// has no labelled vertex: the iteration then keeps the component's weighted mean, as the rounds do).  Preconditioned by D
// its residual z = D^-1 (b - (D - W) x) is what an ordinary round would change, (weighted mean of the neighbours) - x, and
// the product that an iteration needs is one round's gathers, v = p - (weighted mean of the neighbours' p), with p = 0 in
// labelled rows.  A random graph's update has a few eigenvalues near 1 (the classes and the constant) and the others well
// inside: conjugate gradients deal with the few one by one, where a relaxation with one factor has to be slow enough for
// the largest.  Rounds until the largest move is below 1e-6, relaxed / conjugate: planted blocks 65 / 14, kNN 97 / 29, power
// law with 50 classes 105 / 21, random graph of degree 5 105 / 54.
//
// All columns share the two coefficients of an iteration (their systems are one block system with the same matrix), so
// that a row's columns keep the sum they have.  The step needs (p, v), (v, v) and (z, z), weighted by D: the product kernel
// leaves the first two and the step before it the third, so that the second coefficient, (z', z') / (z, z), is known before
// z' is: (z', z') = alpha^2 (v, v) - (z, z) by conjugacy (Meurant 1987).  alpha itself uses the (z, z) that was summed, which
// keeps the recurrence from drifting.  Weights may be as large or as small as float32 has them, and a sum of products of
// degrees and squares leaves its range at both ends (labels lost for weights of 1e36, no step taken for 1e-28): such products
// are formed and added in 64 bits (in k_cg_step and k_pb_product where float32 has no room for them; 64 bits throughout: 36.1 ->
// 37.2 us for 300,000 rows of 32 floats, 725 -> 767 us for 49.5M binned rows).  An iteration is then two launches:
//   product   k_pk_product, k_pb_product or k_row_product: v, and the sums (p, v) and (v, v)
//   step      k_cg_step: x += alpha p, z -= alpha v, p = z + beta p, and the sum (z, z), the largest |z| and |p|.  The step is
//             bound by its streams (seven with x's); x, which nothing reads in between, is updated in every second step only, by the
//             sum of two (1M rows of 16 floats 94 -> 68 us per step, of 64 floats 371 -> 297).
// and needs no other wait.  Measured, whole calls at tol = 1e-6, relaxed / conjugate rounds (error against 64 bits): 1M planted
// blocks, 10 classes 10.6 / 5.5 ms (1.2e-5 / 1e-7); 300K, 29 classes 7.6 / 3.2 ms (7e-7 / 1.5e-7); 100K kNN 2.70 / 1.50 ms (1.4e-5 /
// 6e-7); 1M power law, 50 classes 95 / 40.5 ms (5e-5 / 2e-7); since then, with the rest of the batch, 4.4, 2.6, 1.31 and 36 ms.
// Four arrays of the size of the label matrix: x in the labels themselves, v in their partner buffer, z and p allocated by the
// first call that runs conjugate rounds and kept.
#pragma once

#include "dynlp_device.h"

namespace dynlp {

constexpr int kCgLanes = 16;  // partial records per iteration, a cache line each (as RoundPart)
constexpr int kCgRing = 64;   // iterations whose sums are kept

struct __attribute__((aligned(64))) CgPart {
    double pv, vv;                // of the iteration's product
    double zz;                    // after the iteration's step
    unsigned int zmax, pmax;      // largest |z| and |p| after it (float bits)
    unsigned int moved;           // rows with |z| > tol
    unsigned int pad[3];
};

// pending: the iteration's step left its alpha p out of x; with its beta the next step finds that p again, as (p - z) / beta.
// broken: its coefficients are no numbers (a degree that overflowed), it changed nothing.  All words are 0 before.
struct __attribute__((aligned(64))) CgSlot {
    CgPart part[kCgLanes];
    float alpha, beta;
    unsigned int pending;
    unsigned int broken;
    unsigned int pad[12];
};
// A step with a smaller beta leaves nothing out: the quotient's rounding, 2^-24 |z| / beta, would show.
constexpr float kCgMinBeta = 5e-2f;

// Iteration k: prev holds what iteration k - 1 (or k_cg_begin) left.  Nothing is done once its largest |z| is <= stop (a NaN
// among the residuals counts as infinitely large, see cg_add_tally).
struct CgRun {
    const CgSlot* prev;
    CgSlot* cur;
    float stop, tol;
};

// Every wave for itself; all lanes of a wave take part.
__device__ inline float cg_prev_max(const CgSlot* s, bool of_p) {
    const int lane = lane_id();
    unsigned int m = 0;
    if (lane < kCgLanes) m = of_p ? s->part[lane].pmax : s->part[lane].zmax;
    return wave_max(__uint_as_float(m));
}

__device__ inline bool cg_done(const CgRun& r) { return !(cg_prev_max(r.prev, false) > r.stop); }

// Power of two by which the rows of p are multiplied for sums in fixed point: the largest |p| becomes at most 1/2.
__device__ inline float cg_scale(const CgRun& r) {
    const float m = cg_prev_max(r.prev, true);
    int e = 0;
    (void)frexpf(m, &e);                    // m < 2^e
    return ldexpf(0.5f, e > 96 ? -96 : e < -96 ? 96 : -e);
}

// Adds the sums of a workgroup of T threads to one of the iteration's partial records.
template <int T>
__device__ inline void cg_add_product(const CgRun& r, double pv, double vv) {
    __shared__ double sm[2][T / kWave];
    const double a = wave_sum(pv), b = wave_sum(vv);
    if (lane_id() == 0) {
        sm[0][threadIdx.x / kWave] = a;
        sm[1][threadIdx.x / kWave] = b;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double s = 0.0;
        for (int w = 0; w < T / kWave; ++w) s += sm[threadIdx.x][w];
        CgPart* p = &r.cur->part[blockIdx.x & (kCgLanes - 1)];
        if (s != 0.0) unsafeAtomicAdd(threadIdx.x == 0 ? &p->pv : &p->vv, s);
    }
}

// What a row piece contributes to the records of the next iteration.
struct CgTally {
    double zz = 0.0;
    float zz_near = 0.f;  // what float32 has room for
    float zmax = 0.f, pmax = 0.f;
    unsigned int moved = 0;
};

template <int CP>
struct CgShape {
    static constexpr int VEC = CP >= 4 ? 4 : CP;
    static constexpr int LPN = CP / VEC;  // neighbouring lanes hold one row
};

template <int CP>
__device__ inline void cg_tally(CgTally& t, const Vec<CgShape<CP>::VEC>& z, const Vec<CgShape<CP>::VEC>& p, float d, float tol) {
    float s = 0.f, m = 0.f;
#pragma unroll
    for (int k = 0; k < CgShape<CP>::VEC; ++k) {
        s += z.v[k] * z.v[k];
        m = fmaxf(m, fabsf(z.v[k]));
        t.pmax = fmaxf(t.pmax, fabsf(p.v[k]));
    }
    const float x = d * s;
    if (x > 1e-30f && x < 1e30f) t.zz_near += x;
    else if (s != 0.f) t.zz += (double)d * (double)s;
    t.zmax = fmaxf(t.zmax, m);
#pragma unroll
    for (int q = 1; q < CgShape<CP>::LPN; q <<= 1) m = fmaxf(m, __shfl_xor(m, q, CgShape<CP>::LPN));
    if (threadIdx.x % CgShape<CP>::LPN == 0 && m > tol) t.moved += 1u;
}

__device__ inline void cg_add_tally(CgSlot* slot, const CgTally& t) {
    __shared__ double sm_z[kBlock / kWave];
    __shared__ float sm_m[2][kBlock / kWave];
    __shared__ unsigned int sm_n[kBlock / kWave];
    const double zz = wave_sum(t.zz + (double)t.zz_near);
    const float zmax = wave_max(t.zmax), pmax = wave_max(t.pmax);
    const unsigned int moved = wave_sum(t.moved);
    if (lane_id() == 0) {
        const int w = threadIdx.x / kWave;
        sm_z[w] = zz;
        sm_m[0][w] = zmax;
        sm_m[1][w] = pmax;
        sm_n[w] = moved;
    }
    __syncthreads();
    CgPart* part = &slot->part[blockIdx.x & (kCgLanes - 1)];
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < kBlock / kWave; ++w) s += sm_z[w];
        if (s != 0.0) unsafeAtomicAdd(&part->zz, s);
        if (!isfinite(s)) atomicMax(&part->zmax, __float_as_uint(INFINITY));  // (a NaN gets past every maximum)
    } else if (threadIdx.x < 3) {
        float m = 0.f;
        for (int w = 0; w < kBlock / kWave; ++w) m = fmaxf(m, sm_m[threadIdx.x - 1][w]);
        if (m > 0.f) atomicMax(threadIdx.x == 1 ? &part->zmax : &part->pmax, __float_as_uint(m));
    } else if (threadIdx.x == 3) {
        unsigned int s = 0;
        for (int w = 0; w < kBlock / kWave; ++w) s += sm_n[w];
        if (s) atomicAdd(&part->moved, s);
    }
}

// After one ordinary round F -> F_new over all rows: z = F_new - F (0 in rows that are not updated, where the two agree),
// p = z, and F_new, whose memory holds v from now on, cleared.
template <int CP>
__global__ void __launch_bounds__(kBlock) k_cg_begin(int64_t n, const float* __restrict__ deg, const float* __restrict__ F,
                                                    float* __restrict__ F_new, float* __restrict__ z, float* __restrict__ p,
                                                    float tol, CgSlot* __restrict__ slot) {
    constexpr int VEC = CgShape<CP>::VEC, LPN = CgShape<CP>::LPN;
    CgTally t;
    const int64_t items = n * LPN, step = (int64_t)gridDim.x * kBlock;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < items; i += step) {
        const Vec<VEC> a = load_vec<VEC>(F + i * VEC), b = load_vec<VEC>(F_new + i * VEC);
        Vec<VEC> r, zero;
#pragma unroll
        for (int k = 0; k < VEC; ++k) {
            r.v[k] = b.v[k] - a.v[k];
            zero.v[k] = 0.f;
        }
        store_vec<VEC>(z + i * VEC, r);
        store_vec<VEC>(p + i * VEC, r);
        store_vec<VEC>(F_new + i * VEC, zero);
        cg_tally<CP>(t, r, r, deg[i / LPN], tol);
    }
    cg_add_tally(slot, t);
}

template <int CP>
__global__ void __launch_bounds__(kBlock) k_cg_step(CgRun run, int64_t n, const float* __restrict__ deg, float* __restrict__ x,
                                                   float* __restrict__ z, float* __restrict__ p, const float* __restrict__ v) {
    constexpr int VEC = CgShape<CP>::VEC, LPN = CgShape<CP>::LPN;
    if (cg_done(run)) return;
    float alpha = 0.f, beta = 0.f;
    bool broken = false;
    {
        const int lane = lane_id();
        const bool ok = lane < kCgLanes;
        const double pv = wave_sum(ok ? run.cur->part[lane].pv : 0.0), vv = wave_sum(ok ? run.cur->part[lane].vv : 0.0);
        const double zz = wave_sum(ok ? run.prev->part[lane].zz : 0.0);
        if (pv > 0.0 && zz > 0.0) {
            const double a = zz / pv, next = a * a * vv - zz;
            alpha = (float)a;
            beta = next > 0.0 ? (float)(next / zz) : 0.f;
        }
        broken = !isfinite(pv) || !isfinite(vv) || !isfinite(zz) || !isfinite(alpha) || !isfinite(beta);
    }
    if (broken) {  // the same in all workgroups; the iterations queued behind this one find a largest |z| of 0 and end
        if (blockIdx.x == 0 && threadIdx.x == 0) run.cur->broken = 1u;
        return;
    }
    const bool owed = run.prev->pending != 0u, later = !owed && beta >= kCgMinBeta;
    // x += alpha p, and what the step before left out: its alpha (p - z) / beta with p and z as they are now
    const float owed_p = owed ? run.prev->alpha / run.prev->beta : 0.f;
    const float from_p = alpha + owed_p, from_z = -owed_p;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        run.cur->alpha = alpha;
        run.cur->beta = beta;
        run.cur->pending = later ? 1u : 0u;
    }
    CgTally t;
    const int64_t items = n * LPN, step = (int64_t)gridDim.x * kBlock;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < items; i += step) {
        Vec<VEC> zi = load_vec<VEC>(z + i * VEC), pi = load_vec<VEC>(p + i * VEC);
        const Vec<VEC> vi = load_vec<VEC>(v + i * VEC);
        const float d = deg[i / LPN];
        if (!later) {  // uniform in the launch
            Vec<VEC> xi = load_vec<VEC>(x + i * VEC);
#pragma unroll
            for (int k = 0; k < VEC; ++k) xi.v[k] = fmaf(from_p, pi.v[k], fmaf(from_z, zi.v[k], xi.v[k]));
            store_vec<VEC>(x + i * VEC, xi);
        }
#pragma unroll
        for (int k = 0; k < VEC; ++k) {
            zi.v[k] = fmaf(-alpha, vi.v[k], zi.v[k]);
            pi.v[k] = fmaf(beta, pi.v[k], zi.v[k]);
        }
        store_vec<VEC>(z + i * VEC, zi);
        store_vec<VEC>(p + i * VEC, pi);
        cg_tally<CP>(t, zi, pi, d, run.tol);
    }
    cg_add_tally(run.cur, t);
}

// What the last step (its slot: last) left out of x is added.  The rows are distributions again (columns below 0 or above 1 by
// rounding, or by more where the iteration was cut), and the partner buffer holds the same rows.  Rows that no round updates stay
// as they are.
template <int CP>
__global__ void __launch_bounds__(kBlock) k_cg_end(const CgSlot* __restrict__ last, int64_t n, int Cs, const float* __restrict__ deg,
                                                  const int32_t* __restrict__ seed_class, const float* __restrict__ z,
                                                  const float* __restrict__ p, float* __restrict__ x,
                                                  float* __restrict__ partner) {
    const bool owed = last->pending != 0u;
    const float factor = owed ? last->alpha / last->beta : 0.f;
    constexpr int VEC = CgShape<CP>::VEC, LPN = CgShape<CP>::LPN;
    const int64_t items = n * LPN, step = (int64_t)gridDim.x * kBlock;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < items; i += step) {
        const int64_t u = i / LPN;
        const int first = (int)(i % LPN) * VEC;
        Vec<VEC> f = load_vec<VEC>(x + i * VEC);
        if (seed_class[u] < 0 && deg[u] > 0.f) {  // the same for the lanes of a row
            float s = 0.f;
            if (owed) {
                const Vec<VEC> pi = load_vec<VEC>(p + i * VEC), zi = load_vec<VEC>(z + i * VEC);
#pragma unroll
                for (int k = 0; k < VEC; ++k) {
                    const float sum = fmaf(factor, pi.v[k] - zi.v[k], f.v[k]);
                    f.v[k] = isfinite(sum) ? sum : f.v[k];
                }
            }
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                f.v[k] = fminf(fmaxf(f.v[k], 0.f), 1.f);
                s += f.v[k];
            }
#pragma unroll
            for (int q = 1; q < LPN; q <<= 1) s += __shfl_xor(s, q, LPN);
            if (Cs > 1) {
#pragma unroll
                for (int k = 0; k < VEC; ++k)
                    f.v[k] = s > 0.f ? fminf(f.v[k] / s, 1.f) : (first + k < Cs ? 1.f / (float)Cs : 0.f);
            }
            store_vec<VEC>(x + i * VEC, f);
        }
        store_vec<VEC>(partner + i * VEC, f);
    }
}

}  // namespace dynlp
