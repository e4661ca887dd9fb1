// Per-ray FP64 re-evaluation, shared by the re-check kernels of single maps
// (recheck.hip, farfield.hip) and of batches.
//
// exact_ray_*: the plain definition, operation for operation —
//   ray position (Section 3.1 regular grid, cell-centred, or the ray's random point):
//       x1 = sx0 + ((double)i + 0.5) * (sw / nx)   or   x1 = sx0 + U1 * sw
//   Section 2, Eq. (sigma): a1 = sum_k (m_k / r2) * d1 in lens order,
//       d1 = x1 - X_k, r2 = d1*d1 + d2*d2; a ray with r2 == 0 is singular;
//   y1 = ((1 - gamma) - sigma_c) * x1 - a1, u = (y1 - tx0) / (tw / npx);
//   pixel floor(u), floor(v) if 0 <= u < npx and 0 <= v < npy, else out.
// Every operation is one IEEE-754 binary64 operation (no contraction: the
// library is compiled with -ffp-contract=off), so the result is the
// definition's, bit for bit.
//
// fast_ray: FP64 with fused multiply-adds and a Newton-refined v_rcp_f64,
// plus S = sum (|d1|+|d2|) |m|/r2. Its deviation from the exact real value,
// and the definition's own, are each at most (N+10) 2^-53 S + 8 2^-53
// (|c1 x1| + |a1| + |tx0|) in source units; a ray farther than twice that
// from every pixel edge is decided identically to the definition.
#pragma once

#include "rs_internal.h"
#include "philox.h"

namespace rs {

constexpr uint32_t UNRESOLVED = 0x80000000u;  // queue mark: stage A could not place the ray
constexpr uint32_t RESOLVED = 0x40000000u;    // queue mark: the far-field stage placed the ray

// A copy of a wave-uniform struct whose every 32-bit word goes through
// readfirstlane, so the compiler keeps it in scalar registers.
template <class T>
__device__ __forceinline__ T make_uniform(const T &v) {
    static_assert(sizeof(T) % 4 == 0, "word-sized struct");
    T out;
    const int *src = reinterpret_cast<const int *>(&v);
    int *dst = reinterpret_cast<int *>(&out);
#pragma unroll
    for (int k = 0; k < (int)(sizeof(T) / 4); ++k) dst[k] = __builtin_amdgcn_readfirstlane(src[k]);
    return out;
}
constexpr int CODE_OUT = -1;
constexpr int CODE_SINGULAR = -2;

// Lens reads through a global-address-space pointer. A batch's descriptors hold
// plain (generic) pointers; read through those, the lens loop compiles to flat
// loads that wait on every memory counter each iteration.
typedef __attribute__((address_space(1))) const double global_double;
typedef __attribute__((address_space(1))) const int32_t global_i32;
// Data that no kernel in flight writes, read at wave-uniform addresses: scalar loads.
typedef __attribute__((address_space(4))) const double const_double;

// Relaxed device-scope atomic adds through global (not flat) addressing, so a
// later wait on LDS results does not also wait for these to complete.
__device__ __forceinline__ void global_add(uint32_t *p, uint32_t v) {
    __hip_atomic_fetch_add((__attribute__((address_space(1))) uint32_t *)p, v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void global_add(unsigned long long *p, unsigned long long v) {
    __hip_atomic_fetch_add((__attribute__((address_space(1))) unsigned long long *)p, v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double lens_x(const RecheckArgs &a, int64_t k) {
    return ((global_double *)a.lens_xy)[2 * k];
}
__device__ __forceinline__ double lens_y(const RecheckArgs &a, int64_t k) {
    return ((global_double *)a.lens_xy)[2 * k + 1];
}
__device__ __forceinline__ double lens_mass(const RecheckArgs &a, int64_t k) {
    return ((global_double *)a.lens_m)[k];
}

// Image-plane position of ray (i, j): the regular grid's cell centre, or the
// ray's Philox-random point of the shooting rectangle.
__device__ __forceinline__ void ray_xy(const RecheckArgs &a, int64_t i, int64_t j, double &x1, double &x2) {
    if (a.random) {
        random_ray_xy(a.sx0, a.sy0, a.sw, a.sh, a.nx, a.seed, i, j, x1, x2);
    } else {
        x1 = a.sx0 + ((double)i + 0.5) * (a.sw / (double)a.nx);
        x2 = a.sy0 + ((double)j + 0.5) * (a.sh / (double)a.ny);
    }
}

// The pixel of the ray at (x1, x2) deflected by the definition's sums (a1, a2), or CODE_OUT.
__device__ __forceinline__ int definition_pixel(const RecheckArgs &a, double x1, double x2, double a1, double a2) {
    const double y1 = ((1.0 - a.gamma) - a.sigma_c) * x1 - a1;
    const double y2 = ((1.0 + a.gamma) - a.sigma_c) * x2 - a2;
    const double u = (y1 - a.tx0) / (a.tw / (double)a.npx);
    const double v = (y2 - a.ty0) / (a.th / (double)a.npy);
    if (isfinite(u) && isfinite(v) && u >= 0.0 && u < (double)a.npx && v >= 0.0 && v < (double)a.npy)
        return (int)((int64_t)floor(v) * a.npx + (int64_t)floor(u));
    return CODE_OUT;
}

template <bool UNIT>
__device__ inline int exact_ray_thread(const RecheckArgs &a, int64_t i, int64_t j) {
    double x1, x2;
    ray_xy(a, i, j, x1, x2);
    double a1 = 0.0, a2 = 0.0;
    for (int64_t k = 0; k < a.n_lens; ++k) {
        const double d1 = x1 - lens_x(a, k);
        const double d2 = x2 - lens_y(a, k);
        const double r2 = d1 * d1 + d2 * d2;
        if (r2 == 0.0) return CODE_SINGULAR;
        const double m = UNIT ? 1.0 : lens_mass(a, k);
        const double f = m / r2;
        a1 += f * d1;
        a2 += f * d2;
    }
    return definition_pixel(a, x1, x2, a1, a2);
}

__device__ __forceinline__ void wave_lds_fence() {
    // LDS accesses of one wave complete in order; keep the compiler from moving them across.
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Inclusive sums over the wave's lanes, in lane order, by DPP (row_shr within rows of 16
// lanes, then the rows' last lanes broadcast to the rows after them).
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ double shift_dpp(double v) {   // (0 where there is no source lane)
    const uint64_t w = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)w, CTRL, ROWS, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(w >> 32), CTRL, ROWS, 0xf, false);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double add_dpp(double v) {
    return v + shift_dpp<CTRL, ROWS>(v);
}
__device__ __forceinline__ double wave_scan(double v) {
    v = add_dpp<0x111, 0xf>(v);   // row_shr:1, 2, 4, 8
    v = add_dpp<0x112, 0xf>(v);
    v = add_dpp<0x114, 0xf>(v);
    v = add_dpp<0x118, 0xf>(v);
    v = add_dpp<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    return add_dpp<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
}
__device__ __forceinline__ double read_lane(double v, int lane) {
    const uint64_t w = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)w, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(w >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// s <- fl(...fl(fl(s + t_0) + t_1)...) over the terms of the wave, lane l holding terms
// l J .. l J + J - 1 of the sequence: each addition's rounding exactly as one after the
// other, many at a time.
//
// While every partial sum stays strictly inside one binade (2^e < |s| < 2^(e+1), unit in
// the last place g = 2^(e-52)), s is a multiple of g and an addition gives s + r, r = t
// rounded to a multiple of g: the roundings do not depend on s, and the r add up without
// rounding, in any order. r = fl(t + C) - C with C = 1.5 2^e, which stays in the binade for
// |t| < 2^(e-1). Where that does not hold - a partial sum leaves the binade, a larger t, a
// tie (t halfway between two multiples of g, whose rounding depends on s) - the first
// lane concerned is found from the exact partial sums; the lanes before it are added at
// once, its J terms one by one, and the rest starts over from the new s (the second time
// after two lanes one by one, then after four, ...: such places lie close together).

// One round, over the lanes from `from` on: the partial sum before each lane (exact up to
// the first lane concerned), the sum of every lane's terms, and the lanes concerned.
struct OrderedRound {
    double before, total;
    uint64_t where;
};
template <int J>
__device__ __forceinline__ OrderedRound ordered_round(double s, const double (&t)[J], int from) {
    const uint64_t bits = (uint64_t)__double_as_longlong(s);
    const uint64_t ex = bits & 0x7ff0000000000000ull, sign = bits & 0x8000000000000000ull;
    // (g has to be a normal number, 2^(e+1) finite; zero and denormals are not)
    bool bad = ex < (60ull << 52) || ex >= (2040ull << 52);
    const double p = __longlong_as_double((long long)ex);   // 2^e
    const double half_g = __longlong_as_double((long long)(ex - (53ull << 52)));
    const double C = __longlong_as_double((long long)((uint64_t)__double_as_longlong(1.5 * p) | sign));
    const bool mine = __lane_id() >= from;
    double sum = 0.0, lo = 0.0, hi = 0.0;   // this lane's partial sums
#pragma unroll
    for (int u = 0; u < J; ++u) {
        const double r = (t[u] + C) - C;
        bad |= !(fabs(t[u]) < 0.5 * p) || fabs(t[u] - r) == half_g;   // (t - r is exact)
        sum += r;
        lo = fmin(lo, sum);
        hi = fmax(hi, sum);
    }
    const double upto = wave_scan(mine ? sum : 0.0);
    OrderedRound o;
    o.before = s + shift_dpp<0x138>(upto);   // wave_shr:1
    o.total = read_lane(upto, 63);
    const double a0 = o.before + lo, a1 = o.before + hi;
    const double least = sign ? -a1 : a0, most = sign ? -a0 : a1;   // of |partial sum|
    bad |= !(least > p && most < 2.0 * p);
    o.where = __ballot(bad && mine);
    return o;
}

// starts: counts the starts over.
template <int J>
__device__ __forceinline__ double add_in_order(double s, const double (&t)[J], OrderedRound o, int &starts) {
    for (int run = 1; o.where; run *= 2, ++starts) {   // (the same in every lane)
        int next = __builtin_ctzll(o.where);
        s = read_lane(o.before, next);   // (exact: every lane before it is good)
        const int end = next + run < 64 ? next + run : 64;
#pragma unroll 1
        for (; next < end; ++next) {   // every lane adds its own terms; lane next's sum counts
#pragma unroll
            for (int u = 0; u < J; ++u) s += t[u];
            s = read_lane(s, next);
        }
        if (next == 64) return s;
        o = ordered_round(s, t, next);
    }
    return s + o.total;
}

// Stage B: the same definition evaluated by a whole wave for one ray (i, j wave-uniform),
// in two forms; the caller picks the form by the map's lenses.
//
// The chain: lanes form the per-lens terms (m/r2)*d1, (m/r2)*d2 of 64 lenses at a time and
// stage them in LDS; every lane then adds them in lens order (the same sum in every lane, so
// no lane-to-scalar moves sit on the dependent chain). Callers are blocks of at most 256
// threads.
template <bool UNIT, int P = 4, int B = 8>
__device__ inline int exact_ray_chain(const RecheckArgs &a, int64_t i, int64_t j) {
    __shared__ double2 terms[4][2][64];   // [wave][buffer][lens of the chunk]: (m/r2 d1, m/r2 d2)
    const int lane = __lane_id();
    const int w = (threadIdx.x >> 6) & 3;
    double x1, x2;
    ray_xy(a, i, j, x1, x2);
    double a1 = 0.0, a2 = 0.0;
    bool zero = false;
    if (a.n_lens > 0) {
        // Loads and terms have no branches (indices past the last lens read the last
        // lens, and their terms are replaced by zero, which adds nothing: the running
        // sums start at +0 and never become -0), so the compiler can count the loads
        // in flight and wait for the oldest only.
        const int64_t last = a.n_lens - 1;
        auto load = [&](int64_t k, double &X, double &Y, double &M) {
            const int64_t kc = k < a.n_lens ? k : last;
            X = lens_x(a, kc);
            Y = lens_y(a, kc);
            M = UNIT ? 1.0 : lens_mass(a, kc);
        };
        auto term = [&](int64_t k, double X, double Y, double M) {
            const double d1 = x1 - X;
            const double d2 = x2 - Y;
            const double r2 = d1 * d1 + d2 * d2;
            const bool real = k < a.n_lens;
            zero |= real && (r2 == 0.0);
            const double m = UNIT ? 1.0 : M;
            const double f = m / r2;
            return make_double2(real ? f * d1 : 0.0, real ? f * d2 : 0.0);
        };
        const int64_t n_chunks = (a.n_lens + 63) / 64;
        {
            double X, Y, M;
            load(lane, X, Y, M);
            terms[w][0][lane] = term(lane, X, Y, M);
        }
        // Lens positions are loaded P chunks ahead of their terms (slot s of the ring
        // holds chunk c + 1 while chunk c is summed, c = s mod P), and a chunk's terms
        // are formed while the previous chunk is summed, so neither the memory latency
        // nor the division sits on the dependent chain of additions.
        double SX[P], SY[P], SM[P];
#pragma unroll
        for (int s = 0; s < P; ++s) load(64 * (s + 1) + lane, SX[s], SY[s], SM[s]);
        wave_lds_fence();
        // Whole rounds of P chunks: the chunks past the last one hold zero terms.
        for (int64_t c0 = 0; c0 < n_chunks; c0 += P) {
#pragma unroll
            for (int s = 0; s < P; ++s) {
                const int64_t c = c0 + s;
                const double2 tn = term(64 * (c + 1) + lane, SX[s], SY[s], SM[s]);
                load(64 * (c + 1 + P) + lane, SX[s], SY[s], SM[s]);
                const double2 *T = terms[w][c & 1];
                // in lens order, B terms read ahead of their additions (LDS latency
                // is several times one addition's)
                double2 cur[B];
#pragma unroll
                for (int l = 0; l < B; ++l) cur[l] = T[l];
#pragma unroll
                for (int g = 0; g < 64 / B; ++g) {
                    double2 nxt[B];
#pragma unroll
                    for (int l = 0; l < B; ++l) nxt[l] = T[(B * (g + 1) + l) & 63];
#pragma unroll
                    for (int l = 0; l < B; ++l) {
                        a1 += cur[l].x;
                        a2 += cur[l].y;
                    }
#pragma unroll
                    for (int l = 0; l < B; ++l) cur[l] = nxt[l];
                }
                terms[w][(c + 1) & 1][lane] = tn;
                wave_lds_fence();   // every lane has read chunk c, and chunk c + 1 is written
            }
        }
    }
    if (__ballot(zero)) return CODE_SINGULAR;
    return definition_pixel(a, x1, x2, a1, a2);
}

// The sums many terms at a time: lanes form the terms of J consecutive lenses each, and
// add_in_order adds a chunk of 64 J of them in lens order. Where a sum starts at zero, or stays
// small beside its terms (near the field's centre, on the lenses' mirror axis), it starts over
// again and again and takes up to twice the chain's time, so the first 4096 lenses, and after a
// chunk of more than six starts over the next chunks too (more of them each time it happens
// again), are added one by one, both sums at once (PAUSE; not in maps of 131072 lenses or more,
// where that saves nothing). One ray among n lenses, chain / this
// form / this form without that pause, at 0.05, 0.3 and 0.7 of the field's radius and on a mirror
// axis, in us: 8000 lenses 81 / 104, 93, 67, 99 / 135, 106, 62, 153; 16000 158 / 165, 172, 104, 189 /
// 184, 184, 106, 273; 64000 619 / 553, 589, 229, 699 / 590, 603, 220, 988; 10^6 9.68 ms / 5.45, 4.37,
// 2.71, 7.01 / 5.46, 4.37, 2.72, 6.65. The line between the forms lies where they come out even.
constexpr int64_t EXACT_CHAIN_LENSES = 8192;
constexpr int64_t EXACT_PAUSE_LENSES = 131072;
// In batches the chain alone up to this many lenses: both forms in the scan's kernel leave it no
// registers for more than the two waves per SIMD it has, and its rays are spread over many waves.
constexpr int64_t BATCH_CHAIN_LENSES = 32768;
template <bool UNIT, int J, bool PAUSE>
__device__ inline int exact_ray_parallel(const RecheckArgs &a, int64_t i, int64_t j) {
    const int lane = __lane_id();
    double x1, x2;
    ray_xy(a, i, j, x1, x2);
    double a1 = 0.0, a2 = 0.0;   // the same in every lane
    bool zero = false;
    // Loads have no branches (indices past the last lens read the last lens, and their
    // terms are replaced by zero, which adds nothing: the running sums start at +0 and
    // never become -0), and the next lenses are loaded while these are summed.
    const int64_t last = a.n_lens - 1;
    double X[J], Y[J], M[J];
    constexpr int FIRST = 64 / J, STARTS_MAX = 6, PAUSE_MIN = 1, PAUSE_MAX = 64;
    int one_by_one = FIRST, pause = PAUSE_MIN;   // chunks
    auto load = [&](int64_t k0) {
#pragma unroll
        for (int u = 0; u < J; ++u) {
            const int64_t k = k0 + u < a.n_lens ? k0 + u : last;
            X[u] = lens_x(a, k);
            Y[u] = lens_y(a, k);
            M[u] = UNIT ? 1.0 : lens_mass(a, k);
        }
    };
    if (a.n_lens > 0) load((int64_t)lane * J);
    for (int64_t k0 = 0; k0 < a.n_lens; k0 += 64 * J) {
        const int64_t mine = k0 + (int64_t)lane * J;
        double t1[J], t2[J];
#pragma unroll
        for (int u = 0; u < J; ++u) {
            const double d1 = x1 - X[u];
            const double d2 = x2 - Y[u];
            const double r2 = d1 * d1 + d2 * d2;
            const bool real = mine + u < a.n_lens;
            zero |= real && (r2 == 0.0);
            const double f = (UNIT ? 1.0 : M[u]) / r2;
            t1[u] = real ? f * d1 : 0.0;
            t2[u] = real ? f * d2 : 0.0;
        }
        load(mine + 64 * J);
        if (PAUSE && one_by_one > 0) {
            --one_by_one;
            const int64_t lanes = (a.n_lens - k0 + J - 1) / J;
#pragma unroll 1
            for (int l = 0; l < (lanes < 64 ? (int)lanes : 64); ++l) {   // every lane adds its own terms; lane l's sums count
#pragma unroll
                for (int u = 0; u < J; ++u) {
                    a1 += t1[u];
                    a2 += t2[u];
                }
                a1 = read_lane(a1, l);
                a2 = read_lane(a2, l);
            }
        } else {
            int starts = 0;
            const OrderedRound o1 = ordered_round(a1, t1, 0), o2 = ordered_round(a2, t2, 0);
            a1 = add_in_order(a1, t1, o1, starts);
            a2 = add_in_order(a2, t2, o2, starts);
            if (starts > STARTS_MAX) {
                one_by_one = pause;
                pause = pause < PAUSE_MAX ? 4 * pause : PAUSE_MAX;
            } else {
                pause = PAUSE_MIN;
            }
        }
    }
    if (__ballot(zero)) return CODE_SINGULAR;
    return definition_pixel(a, x1, x2, a1, a2);
}

enum ExactForm { EXACT_CHAIN, EXACT_PAUSE, EXACT_PARALLEL };
template <bool UNIT, ExactForm FORM>
__device__ __forceinline__ int exact_ray_wave(const RecheckArgs &a, int64_t i, int64_t j) {
    if constexpr (FORM == EXACT_CHAIN) return exact_ray_chain<UNIT>(a, i, j);
    else return exact_ray_parallel<UNIT, 8, FORM == EXACT_PAUSE>(a, i, j);
}

// Maps of at most this many lenses and of one launch run stage B in stage A's kernel.
constexpr int64_t EXACT_INLINE_LENSES = 2048;

// Stage A's pixel decision. (a1, a2) is this stage's FP64 sum, S = sum (|d1| + |d2|) |m| / r^2
// over every lens, and t1, t2 bound |definition's a_i - this a_i| (both roundings added); the
// ray is decided when its position is farther than that, plus both epilogues' rounding, from
// every pixel edge.
__device__ inline bool stage_a_decide(const RecheckArgs &a, double x1, double x2, double a1, double a2, double S,
                                      double t1, double t2, bool tiny, int &code) {
    const double U64 = 1.1102230246251565e-16;  // 2^-53
    const double c1 = (1.0 - a.gamma) - a.sigma_c;
    const double c2 = (1.0 + a.gamma) - a.sigma_c;
    const double inv_pixw = (double)a.npx / a.tw;
    const double inv_pixh = (double)a.npy / a.th;
    const double u = (c1 * x1 - a1 - a.tx0) * inv_pixw;
    const double v = (c2 * x2 - a2 - a.ty0) * inv_pixh;
    const double Mu = (t1 + 2.002 * 8.0 * U64 * (fabs(c1 * x1) + fabs(a1) + fabs(a.tx0))) * inv_pixw;
    const double Mv = (t2 + 2.002 * 8.0 * U64 * (fabs(c2 * x2) + fabs(a2) + fabs(a.ty0))) * inv_pixh;
    const double fu = floor(u), fv = floor(v);
    const bool ok_u = (fmin(u - fu, fu + 1.0 - u) > Mu) && (fu >= 0.0) && (fu < (double)a.npx);
    const bool ok_v = (fmin(v - fv, fv + 1.0 - v) > Mv) && (fv >= 0.0) && (fv < (double)a.npy);
    const bool out_u = (u < -Mu) || (u > (double)a.npx + Mu);
    const bool out_v = (v < -Mv) || (v > (double)a.npy + Mv);
    const bool sane = !tiny && isfinite(S) && isfinite(Mu) && isfinite(Mv);
    if (sane && ok_u && ok_v) {
        code = (int)((int64_t)fv * a.npx + (int64_t)fu);
        return true;
    }
    if (sane && (out_u || out_v)) {
        code = CODE_OUT;
        return true;
    }
    return false;
}

// The bound t of stage_a_decide. Any summation order of N terms stays within (N + 10) 2^-53 S
// of the exact sum, so 2 (N + 10) 2^-53 S covers both evaluations (any_order). Tighter, from the
// partial sums: the definition adds its terms in lens order and the k-th addition's rounding is
// at most 2^-53 |s_k| (s_k its partial sum), so its sum is within 2^-53 sum_k |s_k| of its own
// terms' exact sum, and that within 8 2^-53 S of the exact one (per-term rounding). This stage
// estimates sum_k |s_k|; the two functions below add its error and this stage's own. Constants
// are rounded up; N 2^-53 < 1e-3 for every map the library takes.
__device__ inline double any_order_bound(int64_t n_lens, double S) {
    const double U64 = 1.1102230246251565e-16;  // 2^-53
    return 2.002 * ((double)n_lens + 10.0) * U64 * 1.001 * S;
}

// This stage summing in lens order itself (one thread per ray): Q = sum_k |running sum after
// lens k|. Its own sum is within 8 2^-53 S + 2^-53 Q, its partial sums within that of the
// definition's terms' partial sums, so sum_k |s_k| <= Q (1 + N 2^-53) + 16 N 2^-53 S.
__device__ inline double sequential_bound(int64_t n_lens, double S, double Q) {
    const double U64 = 1.1102230246251565e-16;  // 2^-53
    const double N = (double)n_lens;
    const double partial = 1.001 * (16.0 * U64 * S + 2.2 * U64 * Q + 17.0 * N * U64 * U64 * S);
    return fmin(any_order_bound(n_lens, S), partial);
}

// This stage summing lenses in blocks of B in lens order (one wave per ray, the lanes' sums
// combined at every block's end): Q = sum over block starts of |partial sum|. For lens k of a
// block, |s_k| <= |s at the block's start| + the block's sum of |terms|, so sum_k |s_k| <=
// B Q + B S plus each block start's error (its sum depth e: e 2^-53 S, plus 21 2^-53 S for the
// two term evaluations); this stage's own sum is within (e + 13) 2^-53 S (a term: 4 roundings
// in r^2, 6 of the shared reciprocal, the mass, d).
__device__ inline double block_bound(int64_t n_lens, double S, double Q, double B, double e) {
    const double U64 = 1.1102230246251565e-16;  // 2^-53
    const double N = (double)n_lens;
    const double partial = 1.001 * ((e + 40.0 + 1.05 * B) * U64 * S + 1.05 * B * U64 * Q +
                                    1.05 * (N + B) * (e + 40.0) * U64 * U64 * S);
    return fmin(any_order_bound(n_lens, S), partial);
}

// Stage A. Returns true (and the definition's code) when the ray is decided.
template <bool UNIT>
__device__ inline bool fast_ray(const RecheckArgs &a, int64_t i, int64_t j, int &code) {
    double x1, x2;
    ray_xy(a, i, j, x1, x2);
    double a1 = 0.0, a2 = 0.0, S = 0.0, Q1 = 0.0, Q2 = 0.0;
    bool tiny = false;
#pragma unroll 4
    for (int64_t k = 0; k < a.n_lens; ++k) {
        const double d1 = x1 - lens_x(a, k);
        const double d2 = x2 - lens_y(a, k);
        const double r2 = __builtin_fma(d1, d1, d2 * d2);
        tiny |= !(r2 > 1e-200);
        double rc = __builtin_amdgcn_rcp(r2);
        double e = __builtin_fma(-r2, rc, 1.0);
        rc = __builtin_fma(rc, e, rc);
        e = __builtin_fma(-r2, rc, 1.0);
        rc = __builtin_fma(rc, e, rc);
        if (!UNIT) rc = rc * lens_mass(a, k);
        a1 = __builtin_fma(d1, rc, a1);
        a2 = __builtin_fma(d2, rc, a2);
        S = __builtin_fma(fabs(d1) + fabs(d2), fabs(rc), S);
        Q1 += fabs(a1);
        Q2 += fabs(a2);
    }
    return stage_a_decide(a, x1, x2, a1, a2, S, sequential_bound(a.n_lens, S, Q1),
                          sequential_bound(a.n_lens, S, Q2), tiny, code);
}

// Stage A's sums over steps [it0, it1) of 64 U lenses each by a whole wave, for R rays: lanes
// take every 64th lens, U of them per step; every L steps (blocks of 64 U L lenses in lens
// order) the lanes' running sums are added over the wave to give the partial sum at the block's
// end, whose magnitudes add up to Q1, Q2 (for block_bound); the totals meet in the same
// butterfly. Every lane returns the same result.
struct FastSums {
    double a1, a2, S, Q1, Q2;
    bool tiny;
};
__device__ __forceinline__ int64_t fast_steps(const RecheckArgs &a, int U) {
    return (a.n_lens + 64 * U - 1) / (64 * U);
}
// Steps per block. (A block's butterfly takes as long as its 16 lenses per lane; where there
// are many lenses, blocks of 4096 add little to the bound.)
__device__ __forceinline__ int fast_block(const RecheckArgs &a, int U) { return (a.n_lens < (1 << 18) ? 16 : 64) / U; }

// AHEAD: as written above; without it a step's lenses are loaded at its start, for kernels short
// of registers.
template <bool UNIT, int R, int U, bool AHEAD = true>
__device__ inline void fast_sums(const RecheckArgs &a, const double (&x1)[R], const double (&x2)[R], int64_t it0,
                                 int64_t it1, FastSums (&out)[R]) {
    double a1[R], a2[R], S[R], Q1[R], Q2[R];
    int tiny[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        a1[r] = a2[r] = S[r] = Q1[r] = Q2[r] = 0.0;
        tiny[r] = 0;
    }
    // Lane l takes lenses l, l + 64, ...; U of them per step, whose positions were
    // loaded during the previous step, so the memory latency is not waited for. In the
    // last, partial step loads past the last lens read the last lens and their terms are
    // dropped, so the loop has no branches per lane and the compiler can count the loads
    // in flight. Four lenses share one reciprocal (v_rcp_f64 issues like four
    // FMAs, and its Newton steps are four more; sharing takes nine products).
    const int L = fast_block(a, U);
    double LX[U], LY[U], LM[U];
    const int lane = __lane_id();
    const int64_t last = a.n_lens - 1;
    const int64_t full = a.n_lens / (64 * U);                   // steps without a remainder
    auto load = [&](int64_t it) {
        const int64_t k0 = 64 * U * it + lane;
        if (it < full) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                LX[u] = lens_x(a, k0 + 64 * u);
                LY[u] = lens_y(a, k0 + 64 * u);
                LM[u] = UNIT ? 1.0 : lens_mass(a, k0 + 64 * u);
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t k = k0 + 64 * u < a.n_lens ? k0 + 64 * u : last;
                LX[u] = lens_x(a, k);
                LY[u] = lens_y(a, k);
                LM[u] = UNIT ? 1.0 : lens_mass(a, k);
            }
        }
    };
    auto wave_sum = [](double v) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        return v;
    };
    if (AHEAD && it0 < it1) load(it0);
    for (int64_t it = it0; it < it1; ++it) {
        if (!AHEAD) load(it);
        double X[U], Y[U], M[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            X[u] = LX[u];
            Y[u] = LY[u];
            M[u] = LM[u];
        }
        if (AHEAD && it + 1 < it1) load(it + 1);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            double d1[U], d2[U], r2[U], rc[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                d1[u] = x1[r] - X[u];
                d2[u] = x2[r] - Y[u];
                r2[u] = __builtin_fma(d1[u], d1[u], d2[u] * d2[u]);
            }
#pragma unroll
            for (int q = 0; q < U; q += 4) {
                const double pab = r2[q] * r2[q + 1], pcd = r2[q + 2] * r2[q + 3], P = pab * pcd;
                tiny[r] |= !(P > 1e-290);   // (and a product that overflows makes S NaN: not decided either)
                double rp = __builtin_amdgcn_rcp(P);
                double e = __builtin_fma(-P, rp, 1.0);
                rp = __builtin_fma(rp, e, rp);
                e = __builtin_fma(-P, rp, 1.0);
                rp = __builtin_fma(rp, e, rp);
                const double qab = rp * pcd, qcd = rp * pab;
                rc[q] = r2[q + 1] * qab;
                rc[q + 1] = r2[q] * qab;
                rc[q + 2] = r2[q + 3] * qcd;
                rc[q + 3] = r2[q + 2] * qcd;
            }
            if (it >= full) {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (64 * U * it + 64 * u + lane >= a.n_lens) rc[u] = 0.0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (!UNIT) rc[u] = rc[u] * M[u];
                a1[r] = __builtin_fma(d1[u], rc[u], a1[r]);
                a2[r] = __builtin_fma(d2[u], rc[u], a2[r]);
                S[r] = __builtin_fma(fabs(d1[u]) + fabs(d2[u]), fabs(rc[u]), S[r]);
            }
        }
        if (((it - it0) & (L - 1)) == L - 1 || it == it1 - 1) {   // a block's end: its partial sums
#pragma unroll
            for (int r = 0; r < R; ++r) {
                Q1[r] += fabs(wave_sum(a1[r]));
                Q2[r] += fabs(wave_sum(a2[r]));
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        out[r] = FastSums{wave_sum(a1[r]), wave_sum(a2[r]), wave_sum(S[r]), Q1[r], Q2[r], __ballot(tiny[r]) != 0};
}

// Stage A by a whole wave for R rays, ray r at (i[r], j[r]) (wave-uniform).
template <bool UNIT, int R, int U, bool AHEAD = true>
__device__ inline void fast_rays_wave(const RecheckArgs &a, const int64_t (&i)[R], const int64_t (&j)[R],
                                      bool (&decided)[R], int (&code)[R]) {
    double x1[R], x2[R];
#pragma unroll
    for (int r = 0; r < R; ++r) ray_xy(a, i[r], j[r], x1[r], x2[r]);
    const int64_t steps = fast_steps(a, U);
    FastSums f[R];
    fast_sums<UNIT, R, U, AHEAD>(a, x1, x2, 0, steps, f);
    // a partial sum's depth: a lane's running sum plus the six butterfly levels
    const double depth = (double)steps * U + 6.0, B = 64.0 * U * fast_block(a, U);
#pragma unroll
    for (int r = 0; r < R; ++r)
        decided[r] = stage_a_decide(a, x1[r], x2[r], f[r].a1, f[r].a2, f[r].S,
                                    block_bound(a.n_lens, f[r].S, f[r].Q1, B, depth),
                                    block_bound(a.n_lens, f[r].S, f[r].Q2, B, depth), f[r].tiny, code[r]);
}

// Stage A by a block of WAVES waves for one ray (i, j block-uniform), each wave over one range
// of the lenses: a partial sum is the total of the ranges before plus the range's own, and its
// magnitude at most the sum of theirs. part: WAVES entries of shared memory, free on entry.
template <bool UNIT, int U, int WAVES>
__device__ inline bool fast_ray_block(const RecheckArgs &a, int64_t i, int64_t j, FastSums *part, int &code) {
    double x1[1], x2[1];
    ray_xy(a, i, j, x1[0], x2[0]);
    const int wave = threadIdx.x >> 6;
    const int64_t steps = fast_steps(a, U), per = (steps + WAVES - 1) / WAVES;
    const int L = fast_block(a, U);
    auto bound = [&](int w) { return w * per < steps ? w * per : steps; };
    FastSums f[1];
    fast_sums<UNIT, 1, U>(a, x1, x2, bound(wave), bound(wave + 1), f);
    if (__lane_id() == 0) part[wave] = f[0];
    __syncthreads();
    FastSums t{0.0, 0.0, 0.0, 0.0, 0.0, false};
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const FastSums p = part[w];
        const double blocks = (double)((bound(w + 1) - bound(w) + L - 1) / L);
        t.Q1 += blocks * fabs(t.a1) + p.Q1;
        t.Q2 += blocks * fabs(t.a2) + p.Q2;
        t.a1 += p.a1;
        t.a2 += p.a2;
        t.S += p.S;
        t.tiny |= p.tiny;
    }
    __syncthreads();
    const double depth = (double)per * U + 6.0 + WAVES, B = 64.0 * U * L;
    return stage_a_decide(a, x1[0], x2[0], t.a1, t.a2, t.S, block_bound(a.n_lens, t.S, t.Q1, B, depth),
                          block_bound(a.n_lens, t.S, t.Q2, B, depth), t.tiny, code);
}

// U: 8 where a kernel has the registers (a lone wave waits less for its lenses), 4 elsewhere.
template <bool UNIT, int U, bool AHEAD = true>
__device__ inline bool fast_ray_wave(const RecheckArgs &a, int64_t i, int64_t j, int &code) {
    const int64_t ri[1] = {i}, rj[1] = {j};
    bool decided[1];
    int c[1] = {code};
    fast_rays_wave<UNIT, 1, U, AHEAD>(a, ri, rj, decided, c);
    code = c[0];
    return decided[0];
}

// Bin one re-checked ray (or write its pixel) and count it in the map's counters.
__device__ inline void emit_ray(const RecheckArgs &a, int64_t i, int64_t j, int code) {
    if (a.pix_out) {
        a.pix_out[(j - a.j0) * (a.i1 - a.i0) + (i - a.i0)] = code;
    } else if (code >= 0) {
        atomicAdd(a.map + code, 1u);
    }
    atomicAdd(a.counters + (code >= 0 ? C_IN : (code == CODE_OUT ? C_OUT : C_SING)), 1ull);
}

}  // namespace rs
