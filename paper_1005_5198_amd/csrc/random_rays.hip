// Random ray positions (RS_RANDOM_RAYS): count the launch's rays into square bins
// of the shooting rectangle, scan, scatter them into bin order, deflect bin by bin.
#include "shoot_common.h"

namespace rs {
namespace {

// ---------------------------------------------------------------------------
// Random rays (RS_RANDOM_RAYS). The launch's rays are counted into square bins
// of the shooting rectangle, the bins' offsets are scanned, and the rays are
// scattered into bin order (index and FP64 position); then one block deflects
// the rays of one bin, relative to the bin's centre, with the same lens tiles,
// FP32 sum, FP64 folding, error bound and binning as a grid patch (the shared
// reciprocal pairs two lenses of a ray rather than two rays). A ray's
// arithmetic depends only on its position and its bin, not on its slot.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int64_t bin_of(const ShootArgs &a, double x1, double x2) {
    int64_t bx = (int64_t)floor((x1 - a.sx0) * a.inv_bw);
    int64_t by = (int64_t)floor((x2 - a.sy0) * a.inv_bh);
    bx = bx < 0 ? 0 : (bx >= a.nbx_r ? a.nbx_r - 1 : bx);
    by = by < 0 ? 0 : (by >= a.nby_r ? a.nby_r - 1 : by);
    return by * a.nbx_r + bx;
}

// Counting and scattering by blocks, each over one range of the launch's rays, with the
// bins' counts in LDS: a block adds its count of a bin to the bin at once, and reserves its
// slots of the bin at once; bins past the LDS counts' number (a launch of RAND_CHUNK_RAYS has
// fewer, but a launch is at least 32 rows: 2^27 rays and 70600 bins of a window 2^22 wide) take
// further rounds over the block's rays. One atomic per ray on the
// bins bound both kernels: 4.9 million rays in 2600 bins took 0.48 ms each, now 0.05 and 0.2
// (the scatter makes the positions twice); 60000 rays a map of 0.26 ms, now 0.06; launches of
// 64 million rays a map of 9.1 ms, now 5.8 (6.2 with 1024 blocks, 8.5 with 512).
constexpr int RAND_THREADS = 1024;
constexpr int RAND_BLOCKS = 2048;
constexpr uint32_t RAND_LDS_BINS = 36864;
constexpr int64_t RAND_BLOCK_RAYS = 1024;   // at least, so that small launches make few atomics

// f(rel, x1, x2, bin) for every ray of the block's range.
template <class F>
__device__ __forceinline__ void block_rays(const ShootArgs &a, F f) {
    const uint32_t W = (uint32_t)(a.i1 - a.i0);                     // at most 2^22
    const uint32_t n = (uint32_t)((a.jc1 - a.jc0) * (a.i1 - a.i0));   // at most 2 RAND_CHUNK_RAYS (32 rows)
    const uint32_t per = (n + gridDim.x - 1) / gridDim.x;
    const uint32_t lo = min(n, blockIdx.x * per), hi = min(n, lo + per);
    for (uint32_t rel = lo + threadIdx.x; rel < hi; rel += RAND_THREADS) {
        const int64_t i = a.i0 + rel % W, j = a.jc0 + rel / W;
        double x1, x2;
        random_ray_xy(a.sx0, a.sy0, a.sw, a.sh, a.nx, a.seed, i, j, x1, x2);
        f(rel, x1, x2, (uint32_t)bin_of(a, x1, x2));
    }
}

// The block's rays of bins [first, first + RAND_LDS_BINS) counted into LDS.
__device__ __forceinline__ uint32_t block_count(const ShootArgs &a, uint32_t first, uint32_t nb, uint32_t *count) {
    const uint32_t bins = min(RAND_LDS_BINS, nb - first);
    for (uint32_t b = threadIdx.x; b < bins; b += RAND_THREADS) count[b] = 0u;
    __syncthreads();
    block_rays(a, [&](uint32_t, double, double, uint32_t bin) {
        if (bin - first < bins) atomicAdd(&count[bin - first], 1u);
    });
    __syncthreads();
    return bins;
}

__global__ __launch_bounds__(RAND_THREADS) void rand_count_kernel(const ShootArgs a) {
    extern __shared__ uint32_t count[];   // RAND_LDS_BINS, or one per bin
    const uint32_t nb = (uint32_t)(a.nbx_r * a.nby_r);
    for (uint32_t first = 0; first < nb; first += RAND_LDS_BINS) {
        const uint32_t bins = block_count(a, first, nb, count);
        for (uint32_t b = threadIdx.x; b < bins; b += RAND_THREADS)
            if (count[b]) atomicAdd(a.bin_count + first + b, count[b]);
        __syncthreads();
    }
}

__global__ __launch_bounds__(1024) void rand_scan_kernel(const uint32_t *count, int64_t nb, uint32_t *offset,
                                                         uint32_t *cursor) {
    __shared__ uint32_t wsum[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t carry = 0;
    for (int64_t base = 0; base < nb; base += 1024) {
        const int64_t k = base + threadIdx.x;
        const uint32_t v = k < nb ? count[k] : 0u;
        uint32_t x = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)x, o);
            if (lane >= o) x += y;
        }
        if (lane == 63) wsum[wave] = x;
        __syncthreads();
        if (wave == 0) {
            uint32_t y = lane < 16 ? wsum[lane] : 0u;
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) {
                const uint32_t z = (uint32_t)__shfl_up((int)y, o);
                if (lane >= o) y += z;
            }
            if (lane < 16) wsum[lane] = y;
        }
        __syncthreads();
        const uint32_t excl = carry + (wave ? wsum[wave - 1] : 0u) + x - v;
        if (k < nb) {
            offset[k] = excl;
            cursor[k] = excl;
        }
        carry += wsum[15];
        __syncthreads();
    }
    if (threadIdx.x == 0) offset[nb] = carry;
}

__global__ __launch_bounds__(RAND_THREADS) void rand_scatter_kernel(const ShootArgs a) {
    extern __shared__ uint32_t count[];
    uint32_t *const cursor = count;   // the block's counts, then its next slots
    const uint32_t nb = (uint32_t)(a.nbx_r * a.nby_r);
    for (uint32_t first = 0; first < nb; first += RAND_LDS_BINS) {
        const uint32_t bins = block_count(a, first, nb, cursor);
        for (uint32_t b = threadIdx.x; b < bins; b += RAND_THREADS)
            if (cursor[b]) cursor[b] = atomicAdd(a.bin_cursor + first + b, cursor[b]);
        __syncthreads();
        block_rays(a, [&](uint32_t rel, double x1, double x2, uint32_t bin) {
            if (bin - first >= bins) return;
            const uint32_t slot = atomicAdd(&cursor[bin - first], 1u);
            a.ray_rel[slot] = rel;
            a.ray_x[slot] = x1;
            a.ray_y[slot] = x2;
        });
        __syncthreads();
    }
}

// FP32 sums over the n lenses of tile entries g .. g+n-1 for RR rays with no
// shared rows or columns (per ray dx, dy, dy^2, r^2, reciprocal, two FMAs),
// folded into the FP64 accumulators. Two lenses share one v_rcp_f32 per ray, of
// the product of the ray's two r^2 (a ray's arithmetic must not depend on its
// slot, which the scatter's atomics set).
template <int RR, bool UNIT>
__device__ __forceinline__ void free_group_sums(const float4 *tile, int g, int n, const float (&rx)[RR],
                                                const float (&ry)[RR], double (&Ax)[RR], double (&Ay)[RR]) {
    constexpr int READS = 4;   // pairs of lenses per round (GROUP / 2 is a multiple of two rounds' lenses)
    static_assert((GROUP / 2) % (2 * READS) == 0, "whole rounds");
    float sx[RR], sy[RR];
#pragma unroll
    for (int q = 0; q < RR; ++q) {
        sx[q] = 0.0f;
        sy[q] = 0.0f;
    }
#pragma unroll 1
    for (int kk = 0; kk < n; kk += 2 * READS)
#pragma unroll
        for (int k = 0; k < READS; ++k) {
            // lenses a and b: of one read (unit masses) or two
            const float4 la = UNIT ? tile[((g + kk) >> 1) + k] : tile[g + kk + 2 * k];
            const float4 lb = UNIT ? make_float4(la.z, la.w, 1.0f, 0.0f) : tile[g + kk + 2 * k + 1];
#pragma unroll
            for (int q0 = 0; q0 < RR; q0 += 4) {   // four rays' reciprocals at a time
                float dxa[4], dya[4], dxb[4], dyb[4], ra[4], rb[4], R[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int q = q0 + e;
                    dxa[e] = rx[q] - la.x;
                    dya[e] = ry[q] - la.y;
                    dxb[e] = rx[q] - lb.x;
                    dyb[e] = ry[q] - lb.y;
                    ra[e] = __builtin_fmaf(dxa[e], dxa[e], dya[e] * dya[e]);
                    rb[e] = __builtin_fmaf(dxb[e], dxb[e], dyb[e] * dyb[e]);
                    R[e] = ra[e] * rb[e];
                }
                rcp_all(R);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int q = q0 + e;
                    float ia = rb[e] * R[e], ib = ra[e] * R[e];
                    if (!UNIT) {
                        ia = la.z * ia;
                        ib = lb.z * ib;
                    }
                    sx[q] = __builtin_fmaf(dxa[e], ia, sx[q]);
                    sy[q] = __builtin_fmaf(dya[e], ia, sy[q]);
                    sx[q] = __builtin_fmaf(dxb[e], ib, sx[q]);
                    sy[q] = __builtin_fmaf(dyb[e], ib, sy[q]);
                }
            }
        }
#pragma unroll
    for (int q = 0; q < RR; ++q) {
        Ax[q] += (double)sx[q];
        Ay[q] += (double)sy[q];
    }
}

// Up to 64 * WAVES * RR rays of one bin, slots [base, end) of the sorted list;
// (ox, oy) is the bin centre and [ox +- hx] x [oy +- hy] holds every ray of the bin.
template <int RR, int WAVES, bool UNIT, int MODE, bool PIX>
__device__ __forceinline__ void shoot_free_chunk(const ShootArgs &a, uint32_t base, uint32_t end, double ox,
                                                 double oy, double hx, double hy, ShootSmem &sm) {
    constexpr int BLOCK_THREADS = 64 * WAVES;
    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const int lane = tid & 63;
    __syncthreads();  // the previous chunk of this block is done with the shared buffers
    const double h = sqrt(hx * hx + hy * hy);
    const double near_r2 = 4.0 * h * h;

    float rx[RR], ry[RR];
    double Ax[RR], Ay[RR];
#pragma unroll
    for (int q = 0; q < RR; ++q) {
        const uint32_t slot = base + (uint32_t)(q * BLOCK_THREADS + tid);
        const bool ok = slot < end;
        rx[q] = ok ? (float)(a.ray_x[slot] - ox) : 0.0f;
        ry[q] = ok ? (float)(a.ray_y[slot] - oy) : 0.0f;
        Ax[q] = 0.0;
        Ay[q] = 0.0;
    }

    smem_begin(sm, tid);
    double bx = 0.0, by = 0.0;
    const double k_term = UNIT ? K_TERM_UNIT : K_TERM_MASS;
    float4 *tile = sm.tile;

    for (int64_t t0 = 0; t0 < a.n_lens; t0 += LENS_TILE) {
        const int cnt = (int)((a.n_lens - t0) < LENS_TILE ? (a.n_lens - t0) : LENS_TILE);
        const int cnt_pad = (cnt + GROUP / 2 - 1) / (GROUP / 2) * (GROUP / 2);
        __syncthreads();
        stage_tile<UNIT, MODE, BLOCK_THREADS>(a, t0, cnt, cnt_pad, ox, oy, hx, hy, h, near_r2, k_term, sm, tid, bx,
                                              by);
        __syncthreads();
        // the last tile may end with half a group
#pragma unroll 1
        for (int g = 0; g < cnt_pad; g += GROUP)
            free_group_sums<RR, UNIT>(tile, g, cnt_pad - g < GROUP ? cnt_pad - g : GROUP, rx, ry, Ax, Ay);
    }

    double Bx = 0.0, By = 0.0;
    int n_near = 0;
    bool all_flagged = false;
    if (MODE == 1) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            bx += __shfl_xor(bx, off);
            by += __shfl_xor(by, off);
        }
        __syncthreads();
        if (lane == 0) {
            sm.red_bx[wave] = bx;
            sm.red_by[wave] = by;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            Bx += sm.red_bx[w];
            By += sm.red_by[w];
        }
        n_near = sm.near_count;
        // (a bin under 1e-6 across could underflow the paired products of r^2)
        all_flagged = n_near > NEAR_MAX || h < 1.0e-6;
        if (all_flagged) n_near = 0;
    }

    // One ray of each lane at a time, the deflections through the tile's LDS (each wave's
    // own part, half of its rays at a time), so that the loop is not unrolled over registers.
    const float h_f = (float)h;
    const float tiny_r2 = 1.0e-6f * h_f * h_f;
    uint32_t n_in = 0, n_out = 0, n_sing = 0;
    const int64_t W = a.i1 - a.i0;
    constexpr int HELD = RR / 2;
    static_assert(sizeof(double2) * HELD * BLOCK_THREADS <= sizeof(sm.tile), "half of the rays fit the tile");
    double2 *const held = reinterpret_cast<double2 *>(sm.tile) + wave * (HELD * 64) + lane;
    __syncthreads();   // every wave is done with the tile
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int k = 0; k < HELD; ++k)
            held[64 * k] = half ? make_double2(Ax[HELD + k], Ay[HELD + k]) : make_double2(Ax[k], Ay[k]);
        wave_lds_fence();
#pragma unroll 1
        for (int k = 0; k < HELD; ++k) {
            const double2 A = held[64 * k];
            const uint32_t slot = base + (uint32_t)((half * HELD + k) * BLOCK_THREADS + tid);
            const bool valid = slot < end;
            const int64_t rel = valid ? (int64_t)a.ray_rel[slot] : 0;
            const int64_t i = a.i0 + rel % W, j = a.jc0 + rel / W;
            const double x1 = valid ? a.ray_x[slot] : ox;
            const double x2 = valid ? a.ray_y[slot] : oy;
            const float fx = valid ? (float)(x1 - ox) : 0.0f, fy = valid ? (float)(x2 - oy) : 0.0f;
            const double y1 = a.c1 * x1 - A.x;
            const double y2 = a.c2 * x2 - A.y;
            const double u = (y1 - a.tx0) * a.inv_pixw;
            const double v = (y2 - a.ty0) * a.inv_pixh;
            // reciprocals are shared between two lenses of one ray, not between rays
            int code = classify_ray<MODE>(a, x1, x2, A.x, A.y, u, v, fx, fy, fx, fy, fx, false, Bx, By, n_near,
                                          all_flagged, sm.near_list, h_f, tiny_r2);
            if (!valid) code = INT32_MIN;

            n_in += __builtin_popcountll(__ballot(code >= 0));
            n_out += __builtin_popcountll(__ballot(code == OUT));
            n_sing += __builtin_popcountll(__ballot(code == SINGULAR));

            if (PIX) {
                if (valid && code != FLAGGED) a.pix_out[(j - a.j0) * W + (i - a.i0)] = code;
            } else {
                wave_table_add(sm.table, a.map, code);
            }
            if (MODE == 1) {
                const uint64_t fl = __ballot(code == FLAGGED);
                if (fl) SingleSink{}.append(a, sm, fl, lane, code == FLAGGED, i, j);
            }
        }
        wave_lds_fence();
    }
    smem_end<BLOCK_THREADS, MODE, PIX>(a, sm, SingleSink{}, tid, n_in, n_out, n_sing);
}

constexpr int FREE_RR = 8;
constexpr int FREE_WAVES = 4;
constexpr int FREE_CAP = 64 * FREE_WAVES * FREE_RR;

// One block per bin; a bin with more rays than one chunk holds takes several passes. Four waves
// per SIMD: the mixed forms hold 128 registers by spilling 22 to 26 (92 to 108 bytes a lane; with
// masses FP32 spills 2). 4950 x 990 rays, 17240 lenses, mixed: 14.97 ms; 15.14 with three waves,
// which spill nothing.
template <bool UNIT, int MODE, bool PIX>
__global__ __launch_bounds__(64 * FREE_WAVES, 4) void shoot_free_kernel(const ShootArgs a) {
    __shared__ ShootSmem sm;
    if (!PIX) table_clear<64 * FREE_WAVES>(sm.table, threadIdx.x);
    const int64_t bin = blockIdx.x;
    const uint32_t beg = a.bin_offset[bin], end = a.bin_offset[bin + 1];
    const int64_t bxi = bin % a.nbx_r, byi = bin / a.nbx_r;
    const double ox = a.sx0 + ((double)bxi + 0.5) * a.bw;
    const double oy = a.sy0 + ((double)byi + 0.5) * a.bh;
    // Half-extents with slack for the rounding of positions, bin indices and centres.
    const double hx = 0.5 * a.bw * (1.0 + 1e-6) + 1e-14 * (fabs(a.sx0) + a.sw);
    const double hy = 0.5 * a.bh * (1.0 + 1e-6) + 1e-14 * (fabs(a.sy0) + a.sh);
    for (uint32_t base = beg; base < end; base += (uint32_t)FREE_CAP)
        shoot_free_chunk<FREE_RR, FREE_WAVES, UNIT, MODE, PIX>(a, base, end, ox, oy, hx, hy, sm);
}

}  // namespace

hipError_t launch_shoot_random(const ShootArgs &a, int mode, hipStream_t stream) {
    const int64_t n = (a.jc1 - a.jc0) * (a.i1 - a.i0);
    const int64_t nb = a.nbx_r * a.nby_r;
    if (n <= 0) return hipSuccess;
    hipError_t e = launch_zero(a.bin_count, nb, stream);
    if (e != hipSuccess) return e;
    const int64_t want = (n + RAND_BLOCK_RAYS - 1) / RAND_BLOCK_RAYS;
    const int blocks = (int)(want < RAND_BLOCKS ? want : RAND_BLOCKS);
    const size_t lds = sizeof(uint32_t) * (size_t)(nb < RAND_LDS_BINS ? nb : RAND_LDS_BINS);
    hipLaunchKernelGGL(rand_count_kernel, dim3(blocks), dim3(RAND_THREADS), lds, stream, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(rand_scan_kernel, dim3(1), dim3(1024), 0, stream, (const uint32_t *)a.bin_count, nb,
                       a.bin_offset, a.bin_cursor);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(rand_scatter_kernel, dim3(blocks), dim3(RAND_THREADS), lds, stream, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const bool unit = a.lens_m == nullptr;
    const bool pix = a.pix_out != nullptr;
    const dim3 grid((unsigned)nb), block(64 * FREE_WAVES);
#define RS_FREE(U, M, P) hipLaunchKernelGGL((shoot_free_kernel<U, M, P>), grid, block, 0, stream, a)
    if (mode == RS_MIXED) {
        if (unit) { if (pix) RS_FREE(true, 1, true); else RS_FREE(true, 1, false); }
        else { if (pix) RS_FREE(false, 1, true); else RS_FREE(false, 1, false); }
    } else {
        if (unit) { if (pix) RS_FREE(true, 0, true); else RS_FREE(true, 0, false); }
        else { if (pix) RS_FREE(false, 0, true); else RS_FREE(false, 0, false); }
    }
#undef RS_FREE
    return hipGetLastError();
}

}  // namespace rs
