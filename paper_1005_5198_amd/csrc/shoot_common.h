// Device helpers shared by the deflection kernels (regular grid, random rays,
// far field): error-bound constants, ray positions, binning by way of LDS,
// re-check sinks, lens staging with the per-lens FP32 bound, and the per-ray
// classification against a pixel edge.
#pragma once

#include "recheck_ray.h"

namespace rs {
namespace {


constexpr double U32 = 5.9604644775390625e-08;  // 2^-24, FP32 unit roundoff

// Per-lens FP32 error constants (derivation in the design notes):
//   |t_hat - t| <= u m (K_TERM |dx| + K_H h) / r^2 for one term t = m dx / r^2,
//   the FP32 group sum adds u (GROUP - pos) |t_hat| for the lens at position pos.
// Unit masses: K_TERM covers dx (2.04u), r^2 (6.08u + 4.08u h/r) and the reciprocal,
// shared by two terms (two rays of one lens on the grid, two lenses of one ray for
// random rays): b * rcp(a * b) is within 4u of 1/a (the product, v_rcp_f32's 1 ulp,
// the final multiply); with masses the FP32 mass rounding and the mass multiply
// add 2u.
constexpr double K_TERM_UNIT = 12.5;
constexpr double K_TERM_MASS = 15.0;
// Regular-grid unit-mass loop: one reciprocal for four rays (two rows of two
// columns) through the product of their r^2; b * (rcp(P) * cd) with
// P = (a b)(c d) is within 6u of 1/a (three products, the reciprocal, two
// multiplies; the rounding of c d cancels), so the term constant grows by 2.
constexpr double K_TERM_QUAD = 14.5;
constexpr double K_TERM_MASS_QUAD = 17.0;   // the same with masses (+2u)
// Range of the four-ray product P = r_a^2 r_b^2 r_c^2 r_d^2 in FP32: a tile whose
// lenses all lie within QUAD_RANGE of the patch centre on both axes, in a patch
// of half-diagonal h in [QUAD_H_MIN, QUAD_H_MAX], keeps P below 2^110 (no
// overflow); lenses outside the near list are at least 2h from every ray, so P
// stays above 256 h^8 >= 2^-100 (normal, with room); near lenses are checked per
// ray. Other tiles and patches use the two-ray form.
constexpr double QUAD_RANGE = 8192.0;
constexpr double QUAD_H_MIN = 1.0e-4;
constexpr double QUAD_H_MAX = 1024.0;
constexpr double QUAD_P_MIN = 7.888609052210118e-31;   // 2^-100
constexpr double K_GROUP = 1.01;
constexpr double K_H = 6.5;

constexpr double PAD_OFFSET = 1.0e9;   // exactly representable in FP32

constexpr int OUT = -1;
constexpr int SINGULAR = -2;
constexpr int FLAGGED = -3;

struct NearLens {
    float x, y, m;
    float wgt;   // k_term + K_GROUP (GROUP - the lens's position in its group)
};

__device__ __forceinline__ double ray_coord(double origin, int64_t idx, double spacing) {
    // The definition's own operations: origin + ((double)idx + 0.5) * spacing.
    // The library is built without floating-point contraction.
    return origin + ((double)idx + 0.5) * spacing;
}

// Reciprocals of every R, back to back and at a raised wave priority.
// v_rcp_f32 takes a quarter of the FMA rate. Beside that, gfx950 issues two waves' FP32
// instructions together (2.1 cycles each at four waves per SIMD instead of 4.1), and a
// reciprocal of one wave among them ends that pairing: with one per 26 instructions every
// instruction takes 4.1 cycles; issued at priority 1, 2.4 (the reciprocal's own 8 cycles
// included). The deflection of the 19200 x 3840-ray, 17240-lens map: 158.5 -> 134.4 ms.
// (The s_setprio after the last reciprocal is also the wait state that its result needs.)
template <int N>
__device__ __forceinline__ void rcp_all(float (&R)[N]) {
    static_assert(N % 2 == 0 || N == 1, "reciprocals come in twos");
    if (N == 1) asm volatile("s_setprio 1\n\tv_rcp_f32 %0, %0\n\ts_setprio 0" : "+v"(R[0]));
#pragma unroll
    for (int i = 0; i + 2 < N; i += 4)
        asm volatile("s_setprio 1\n\tv_rcp_f32 %0, %0\n\tv_rcp_f32 %1, %1\n\tv_rcp_f32 %2, %2\n\tv_rcp_f32 %3, %3\n\t"
                     "s_setprio 0"
                     : "+v"(R[i]), "+v"(R[i + 1]), "+v"(R[i + 2]), "+v"(R[i + 3]));
    if (N % 4 == 2)
        asm volatile("s_setprio 1\n\tv_rcp_f32 %0, %0\n\tv_rcp_f32 %1, %1\n\ts_setprio 0"
                     : "+v"(R[N - 2]), "+v"(R[N - 1]));
}

__device__ __forceinline__ int lane_id() { return __lane_id(); }

// A block's counts per pixel in LDS, by lines of 16 consecutive pixels (64 bytes of the
// map; open addressing on the line index): rays add with LDS atomics, and the block then
// adds each used line's counts to the map, 16 lanes per line, so that a line costs one
// memory transaction instead of one per pixel (atomics bound the far-field map of 19200 x
// 3840 rays: of its 1.61 ms, 0.70 ms went with a table of single pixels flushed in hash
// order). A ray whose line finds no free slot within PT_PROBES probes adds to the map
// directly. Counts are integers, so the map does not depend on the order of the additions.
constexpr int PT_LINE = 16;
constexpr int PT_SLOTS = 256;
constexpr int PT_PROBES = 2;
struct PixelTable {
    uint32_t cnt[PT_SLOTS * PT_LINE];
    uint32_t key[PT_SLOTS];     // line + 1; 0 = empty
    uint8_t list[PT_SLOTS];     // used slots, in order of their first use
    uint32_t used[2];           // their number (of two counts, so that one can be reset while the other is in use)
};

template <int THREADS>
__device__ __forceinline__ void table_clear(PixelTable &t, int tid) {
    for (int s = tid; s < PT_SLOTS * PT_LINE; s += THREADS) t.cnt[s] = 0u;
    for (int s = tid; s < PT_SLOTS; s += THREADS) t.key[s] = 0u;
    if (tid < 2) t.used[tid] = 0u;
}

// Count n rays in pixel p >= 0.
__device__ __forceinline__ void table_add(PixelTable &t, uint32_t *map, int p, uint32_t n, int par = 0) {
    const uint32_t k = ((uint32_t)p / PT_LINE) + 1u;
    uint32_t s = (k * 2654435761u) >> 24;   // multiplicative hash onto 2^8 slots
    for (int probe = 0; probe < PT_PROBES; ++probe) {
        uint32_t old = __hip_atomic_load(&t.key[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (old == 0u) {
            old = atomicCAS(&t.key[s], 0u, k);
            if (old == 0u) {
                t.list[atomicAdd(&t.used[par], 1u)] = (uint8_t)s;   // at most once per slot
                old = k;
            }
        }
        if (old == k) {
            atomicAdd(&t.cnt[s * PT_LINE + (uint32_t)p % PT_LINE], n);
            return;
        }
        s = (s + 1u) % PT_SLOTS;
    }
    global_add(map + p, n);
}
static_assert(PT_SLOTS == 1 << 8, "the hash keeps 8 bits");


// Count each lane's ray in its pixel p (p < 0: nothing to count). Lanes of one pixel
// are added together while that takes AGG_MIN lanes or more off the wave; the others add
// one by one.
constexpr int AGG_MIN = 8;
__device__ __forceinline__ void wave_table_add(PixelTable &t, uint32_t *map, int p) {
    uint64_t pending = __ballot(p >= 0);
    while (pending) {
        const int leader = __builtin_ctzll(pending);
        const int lp = __builtin_amdgcn_readlane(p, leader);
        const uint64_t same = __ballot(p == lp) & pending;
        const int n = __builtin_popcountll(same);
        if (n < AGG_MIN) break;
        if (lane_id() == leader) table_add(t, map, lp, (uint32_t)n);
        pending &= ~same;
    }
    if ((pending >> lane_id()) & 1ull) table_add(t, map, p, 1u);
}

// Adds every used line's counts to the map and empties the table. The caller separates
// this from the table's last and next use by barriers, and resets used[par], which every
// thread reads here, between two further ones.
template <int THREADS>
__device__ __forceinline__ void table_flush_clear(PixelTable &t, uint32_t *map, int tid, int par = 0) {
    static_assert(THREADS % PT_LINE == 0, "whole lines");
    const uint32_t used = t.used[par];
    for (uint32_t e = (uint32_t)tid / PT_LINE; e < used; e += THREADS / PT_LINE) {
        const uint32_t s = t.list[e], at = s * PT_LINE + (uint32_t)tid % PT_LINE;
        const uint32_t c = t.cnt[at], k = t.key[s];
        if (c) {
            t.cnt[at] = 0u;
            global_add(map + ((k - 1u) * PT_LINE + (uint32_t)tid % PT_LINE), c);
        }
        if (tid % PT_LINE == 0) t.key[s] = 0u;   // (the line's lanes read it in the instruction above)
    }
}

constexpr int FLAG_LIST = 512;   // rays to re-check that a block holds before it appends them to the queue

struct ShootSmem {
    float4 tile[LENS_TILE];        // UNIT: two (x,y) pairs per float4; else (x,y,m,0)
    NearLens near_list[NEAR_MAX];
    int near_count;
    int far_tile;                  // last tile (index) with a lens beyond QUAD_RANGE of the patch centre
    double red_bx[16], red_by[16];
    PixelTable table;              // the patch's counts per pixel (map output)
    uint32_t count[3];             // its rays in the map, out and singular
    uint32_t n_flagged;            // its rays to re-check (the first FLAG_LIST of them in flagged)
    uint32_t flagged[FLAG_LIST];
};

// Queue sink of a single-map launch: uint32 chunk-relative ray indices; the
// queue holds every ray of the launch, so it cannot overflow. A block collects its rays
// in LDS and takes its part of the queue once, at its end: one atomic on the queue's
// length per block instead of one per wave and ray of a lane.
struct SingleSink {
    __device__ void append(const ShootArgs &a, ShootSmem &sm, uint64_t fl, int lane, bool mine, int64_t i, int64_t j) const {
        const int first = __builtin_ctzll(fl);
        uint32_t base = 0;
        if (lane == first) base = atomicAdd(&sm.n_flagged, (uint32_t)__builtin_popcountll(fl));
        base = (uint32_t)__builtin_amdgcn_readlane((int)base, first);
        if (mine) {
            const uint32_t at = base + (uint32_t)__builtin_popcountll(fl & ((1ull << lane) - 1ull));
            const uint32_t ray = (uint32_t)((j - a.jc0) * (a.i1 - a.i0) + (i - a.i0));
            if (at < (uint32_t)FLAG_LIST) sm.flagged[at] = ray;
            else a.queue[atomicAdd(a.qcount, 1u)] = ray;   // the list is full
        }
    }
    // By one wave, after every append (and a barrier).
    __device__ void flush(const ShootArgs &a, const ShootSmem &sm, int lane) const {
        const uint32_t n = sm.n_flagged < (uint32_t)FLAG_LIST ? sm.n_flagged : (uint32_t)FLAG_LIST;
        if (n == 0) return;
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(a.qcount, n);
        base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
        for (uint32_t k = lane; k < n; k += 64) a.queue[base + k] = sm.flagged[k];
    }
};

// Re-check sink of a batch launch: one bit per flagged ray in the map's flag
// bitmap (two bits per ray of workspace in all, whatever the flagged fraction).
struct BatchSink {
    unsigned long long *counters;
    uint32_t *flag_bits;
    __device__ void append(const ShootArgs &a, ShootSmem &sm, uint64_t fl, int lane, bool mine, int64_t i, int64_t j) const {
        if (lane == __builtin_ctzll(fl)) atomicAdd(&sm.n_flagged, (uint32_t)__builtin_popcountll(fl));
        if (mine) {
            const uint32_t ray = (uint32_t)((j - a.j0) * (a.i1 - a.i0) + (i - a.i0));
            atomicOr(flag_bits + (ray >> 5), 1u << (ray & 31u));
        }
    }
    __device__ void flush(const ShootArgs &a, const ShootSmem &sm, int lane) const {
        if (lane == 0 && sm.n_flagged) global_add(counters + C_RECHECK, (unsigned long long)sm.n_flagged);
    }
};

// A block's bookkeeping for one patch (or bin chunk): cleared before its first barrier,
// added to after it.
__device__ __forceinline__ void smem_begin(ShootSmem &sm, int tid) {
    if (tid == 0) {
        sm.near_count = 0;
        sm.far_tile = -1;
        sm.n_flagged = 0u;
        sm.table.used[0] = 0u;   // flushed at the previous patch's end
    }
    if (tid < 3) sm.count[tid] = 0u;
}

// The patch's results leave the block: its pixels' counts (the table is empty after it),
// its counters and the rays to re-check.
template <int THREADS, int MODE, bool PIX, class Sink>
__device__ __forceinline__ void smem_end(const ShootArgs &a, ShootSmem &sm, const Sink &sink, int tid, uint32_t n_in,
                                         uint32_t n_out, uint32_t n_sing) {
    static_assert(C_IN == 0 && C_OUT == 1 && C_SING == 2, "order of sm.count");
    if ((tid & 63) == 0) {
        if (n_in) atomicAdd(&sm.count[C_IN], n_in);
        if (n_out) atomicAdd(&sm.count[C_OUT], n_out);
        if (n_sing) atomicAdd(&sm.count[C_SING], n_sing);
    }
    __syncthreads();
    if (MODE == 1 && tid < 64) sink.flush(a, sm, tid);
    if (!PIX) table_flush_clear<THREADS>(sm.table, a.map, tid);
    if (tid < 3 && sm.count[tid]) global_add(a.counters + tid, (unsigned long long)sm.count[tid]);
}

// Stage lenses t0 .. t0+cnt of the lens array into the LDS tile as FP32 offsets
// from the block origin (ox, oy), padded to whole half groups with lenses at
// offset (PAD_OFFSET, 0): massless where masses are stored; with unit masses
// each adds at most 1/(PAD_OFFSET - hx) to a ray's deflection, which mixed mode
// adds to the bound (far enough to be negligible, near enough that a product
// of two r^2 stays finite). Mixed mode: lenses within 2h of the block's box go to the near list
// (bounded per ray later); the others add their rigorous FP32 error weight for
// any ray in the box [ox +- hx] x [oy +- hy] to this thread's share (bx, by).
template <bool UNIT, int MODE, int BLOCK_THREADS>
__device__ __forceinline__ void stage_tile(const ShootArgs &a, int64_t t0, int cnt, int cnt_pad, double ox, double oy,
                                           double hx, double hy, double h, double near_r2, double k_term,
                                           ShootSmem &sm, int tid, double &bx, double &by) {
    float4 *tile = sm.tile;
        for (int s = tid; s < cnt_pad; s += BLOCK_THREADS) {
            float fx = (float)PAD_OFFSET, fy = 0.0f, fm = 0.0f;  // padding lens
            if (s < cnt) {
                const int64_t k = t0 + s;
                // global-address-space reads (a batch descriptor's pointers are generic)
                const double X = ((global_double *)a.lens_xy)[2 * k];
                const double Y = ((global_double *)a.lens_xy)[2 * k + 1];
                const double m = (UNIT || a.lens_m == nullptr) ? 1.0 : ((global_double *)a.lens_m)[k];
                const double Lx = X - ox, Ly = Y - oy;
                fx = (float)Lx;
                fy = (float)Ly;
                fm = (float)m;
                // (every thread that finds one writes the same value)
                if (!(fmax(fabs(Lx), fabs(Ly)) <= QUAD_RANGE)) sm.far_tile = (int)(t0 / LENS_TILE);
                if (MODE == 1) {
                    const double alx = fabs(Lx), aly = fabs(Ly);
                    const double ex = fmax(alx - hx, 0.0), ey = fmax(aly - hy, 0.0);
                    const double dmin2 = ex * ex + ey * ey;
                    const int pos = s % GROUP;
                    // A lens beyond 1e9 could overflow the paired products of r^2: the
                    // block's rays all go to the FP64 re-check instead.
                    if (fmax(alx, aly) > 1.0e9) atomicAdd(&sm.near_count, NEAR_MAX + 1);
                    const double wgt = k_term + K_GROUP * (double)(GROUP - pos);
                    if (dmin2 < near_r2) {
                        const int q = atomicAdd(&sm.near_count, 1);
                        if (q < NEAR_MAX) sm.near_list[q] = NearLens{fx, fy, (float)fabs(m), (float)wgt};
                    } else {
                        const double im = fabs(m) / dmin2;
                        bx += im * (wgt * (alx + hx) + K_H * h);
                        by += im * (wgt * (aly + hy) + K_H * h);
                    }
                }
            } else if (MODE == 1 && UNIT) {
                // a unit-mass padding lens's whole term, in units of u
                const double d = PAD_OFFSET - hx;
                bx += 1.0 / (d * U32);
                by += hy / (d * d * U32);
            }
            if (UNIT) {
                float *t2 = reinterpret_cast<float *>(tile);
                t2[2 * s] = fx;
                t2[2 * s + 1] = fy;
            } else {
                tile[s] = make_float4(fx, fy, fm, 0.0f);
            }
        }
}

// Pixel code of one ray from its FP64 position x, its folded deflection A and
// its source position (u, v) in pixel units. Mixed mode: the ray's error
// bound is the block's (Bx, By) plus the near lenses' per-ray terms, and a ray
// within it of a pixel edge is FLAGGED for the FP64 re-check. (rxp, ryp) is the
// ray whose reciprocals this one's share: a near lens almost on either of the
// two flags it (their product of r^2 could underflow). With quad set, the ray
// also shares reciprocals with the two rays of column rxq (rows ry and ryp), and
// a near lens whose four r^2, or either pair of them, multiply to less than
// QUAD_P_MIN flags it too. A ray with a non-finite position is never counted
// out, only flagged.
template <int MODE>
__device__ __forceinline__ int classify_ray(const ShootArgs &a, double x1, double x2, double Axv, double Ayv, double u,
                                            double v, float rx, float ry, float rxp, float ryp, float rxq, bool quad,
                                            double Bx, double By, int n_near,
                                            bool all_flagged, const NearLens *near_list, float h_f, float tiny_r2) {
    int code;
    if (MODE == 0) {
        if (!(isfinite(u) && isfinite(v))) code = SINGULAR;
        else if (u >= 0.0 && u < (double)a.npx && v >= 0.0 && v < (double)a.npy)
            code = (int)((int64_t)floor(v) * a.npx + (int64_t)floor(u));
        else code = OUT;
    } else {
        // Per-ray bound from the lenses next to the block.
        float cx = 0.0f, cy = 0.0f;
        bool bad = false;
#pragma unroll 2
        for (int q = 0; q < n_near; ++q) {
            const NearLens nl = near_list[q];
            const float dxn = rx - nl.x, dyn = ry - nl.y;
            const float r2n = dxn * dxn + dyn * dyn;
            const float dxp = rxp - nl.x, dyp = ryp - nl.y;
            const float r2p = dxp * dxp + dyp * dyp;
            bad |= !(r2n > tiny_r2) || !(r2p > tiny_r2);
            if (quad) {
                const float dxq = rxq - nl.x;
                const float r2q = dxq * dxq + dyn * dyn, r2qp = dxq * dxq + dyp * dyp;
                // (four factors above 2^-25 have products above 2^-100)
                if (!(fminf(fminf(r2n, r2p), fminf(r2q, r2qp)) > 0x1p-25f)) {
                    const double pa = (double)r2n * (double)r2p, pc = (double)r2q * (double)r2qp;
                    bad |= !(pa > QUAD_P_MIN && pc > QUAD_P_MIN && pa * pc > QUAD_P_MIN);
                }
            }
            // (v_rcp_f32 is within 1 ulp; the factor also covers r2n's rounding)
            const float im = nl.m * __builtin_amdgcn_rcpf(0.9985f * r2n);
            cx += im * (nl.wgt * (1.001f * fabsf(dxn) + 1e-6f * h_f) + (float)K_H * h_f);
            cy += im * (nl.wgt * (1.001f * fabsf(dyn) + 1e-6f * h_f) + (float)K_H * h_f);
        }
        if (bad) {
            cx = __builtin_inff();
            cy = __builtin_inff();
        }
        const double ea = 1e-15 + 8.9e-16 * (fabs(a.c1 * x1) + fabs(Axv) + fabs(a.tx0));
        const double eb = 1e-15 + 8.9e-16 * (fabs(a.c2 * x2) + fabs(Ayv) + fabs(a.ty0));
        const double Eu = (U32 * (Bx + (double)cx) * a.bound_scale + ea) * a.inv_pixw * 1.000001;
        const double Ev = (U32 * (By + (double)cy) * a.bound_scale + eb) * a.inv_pixh * 1.000001;
        const double fu = floor(u), fv = floor(v);
        const bool ok_u = (fmin(u - fu, fu + 1.0 - u) > Eu) && (fu >= 0.0) && (fu < (double)a.npx);
        const bool ok_v = (fmin(v - fv, fv + 1.0 - v) > Ev) && (fv >= 0.0) && (fv < (double)a.npy);
        const bool fin = isfinite(u) && isfinite(v);
        const bool out_u = (u < -Eu) || (u > (double)a.npx + Eu);
        const bool out_v = (v < -Ev) || (v > (double)a.npy + Ev);
        if (all_flagged) code = FLAGGED;
        else if (ok_u && ok_v) code = (int)((int64_t)fv * a.npx + (int64_t)fu);
        else if (fin && (out_u || out_v)) code = OUT;
        else code = FLAGGED;
    }
    return code;
}

}  // namespace
}  // namespace rs
