// Map statistics of the accuracy assessment (Section 3.1, Accuracy; Eq. deltam; Eq. mu):
// per-pixel change in magnitude, the RMS of its difference between two maps,
// the two-sample Kolmogorov-Smirnov statistic of the two dm distributions and
// its probability, and the histogram of ray counts.
//
// Plan for a pair of maps (one stream, six launches):
//   zero      clear the globals and both histograms (by a kernel, so that the
//             sequence stays valid under stream capture);
//   pass      one streaming read of both maps (16-byte loads): per-block LDS
//             histograms of the counts (counts >= LDS_BINS go straight to the
//             global histogram), FP64 sums for the RMS and the means, maxima;
//             per-block partial sums are stored, not atomically added, so the
//             result does not depend on block timing;
//   scan      inclusive prefix sums of both histograms, in runs of tiles: the runs' sums,
//             then each run from the sums of the runs before it (two launches);
//   ks        the histogram bins of either map: D is the largest
//             |G_a(x) - G_b(x)| over the sample values x, G the empirical CDF
//             of mu (dm is a decreasing function of mu, so the statistic is the
//             same); the other map's CDF is read at the bin of the same value;
//   final     one block: fixed-order sum of the partials, P(KS), the result.
// The histograms hold 32-bit counts (a map has fewer than 2^31 pixels) at the start of a
// workspace of 8 bytes per bin, whose size is part of the interface. A map's caustic
// pixels reach 10^6 rays and more, so that the histograms are as long as a map: zero, scan
// and ks are bound by memory. The pass is bound by LDS (two atomics and two reads of the dm
// tables per pair of pixels; it reads the maps at 1.9 TB/s). Atomics on one address
// (12 ns each) are kept to one per block or fewer. A call for two 4096^2 maps with counts up to 1.5e6 and
// 3e6 takes 145 us; it took 323 with 64-bit histograms, 8 waves per CU in the pass, a
// binary search per bin and an atomic maximum per wave in ks, and a third scan launch.
#include "rs_internal.h"
#include "rayshoot.h"

#include <cmath>

namespace rs {
int fail(int code, const char *fmt, ...);
int hip_fail(hipError_t e, const char *what);
int validate(const rs_map_params *p, int64_t n_lens);
}  // namespace rs

using namespace rs;

namespace {

// One block of 16 waves per CU: the pair's LDS histograms and dm tables take 96 KiB.
constexpr int PASS_THREADS = 1024;
constexpr int PASS_WAVES = PASS_THREADS / 64;
constexpr int LDS_BINS = 4096;          // per map; also the counts whose dm comes from an LDS table
constexpr int PASS_BLOCKS = 256;
constexpr int MAX_PASS_BLOCKS = 1024;   // (the workspace's partial records)
constexpr int SCAN_THREADS = 1024;
constexpr int SCAN_ITEMS = 4;
constexpr int KS_THREADS = 256;
constexpr int FINAL_THREADS = 256;
constexpr int64_t MAX_PIX = int64_t(1) << 31;

struct Partial {               // one block's sums over its pixels
    double rms_sum;
    unsigned long long n_both, sum_a, sum_b, zero_a, zero_b;
    unsigned int max_a, max_b;
    unsigned long long pad;
};
static_assert(sizeof(Partial) == 64, "partial record is one 64-byte line");

struct Globals {               // head of the compare workspace
    unsigned long long d_bits; // D as the bit pattern of a non-negative double (ordered like the value)
    unsigned long long overflow;
    unsigned long long pad[6];
    rs_compare_result result;
};
static_assert(sizeof(Globals) <= 256, "globals fit the 256-byte head");

constexpr size_t WS_PARTIALS = 256;
constexpr size_t WS_HIST = WS_PARTIALS + sizeof(Partial) * MAX_PASS_BLOCKS;

size_t hist_bytes(uint32_t max_count) { return align256(((size_t)max_count + 2) * sizeof(unsigned long long)); }

template <class Count>
struct PassArgs {
    const uint32_t *map_a, *map_b;   // map_b == nullptr: histogram of map_a only
    int64_t npix;
    double nr_a, nr_b;
    uint32_t max_a, max_b;           // histogram bounds; larger counts go to bin max + 1
    Count *hist_a, *hist_b;
    Partial *partials;               // nullptr: no sums
    int vec4;                        // both maps 16-byte aligned
};

__global__ void zero_u64_kernel(unsigned long long *p, int64_t n) {
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x)
        p[k] = 0ull;
}

// The globals and two arrays of n_a and n_b 16-byte words.
__global__ void zero_compare_kernel(Globals *g, uint4 *a, int64_t n_a, uint4 *b, int64_t n_b) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    const uint4 z = make_uint4(0u, 0u, 0u, 0u);
    if (t < (int64_t)(sizeof(Globals) / sizeof(unsigned long long))) reinterpret_cast<unsigned long long *>(g)[t] = 0ull;
    for (int64_t k = t; k < n_a; k += stride) a[k] = z;
    for (int64_t k = t; k < n_b; k += stride) b[k] = z;
}

__global__ void zero_u32_kernel(uint32_t *p) { *p = 0u; }

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
__device__ __forceinline__ unsigned int wave_max(unsigned int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, (unsigned int)__shfl_xor((int)v, o));
    return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    return v;
}

// dm of one pixel, the definition's operations: mu = N / N_rays, dm = -2.5 log10(mu).
__device__ __forceinline__ double delta_m_of(uint32_t c, double n_rays) {
    const double mu = (double)c / n_rays;
    return -2.5 * log10(mu);
}

template <bool PAIR>
struct PassState {
    double rms = 0.0;
    unsigned long long n_both = 0, sum_a = 0, sum_b = 0, zero_a = 0, zero_b = 0;
    unsigned int mx_a = 0, mx_b = 0;
};

template <class Count>
__device__ __forceinline__ void bin_count(uint32_t c, uint32_t max_c, uint32_t *lds, Count *hist) {
    if (c < (uint32_t)LDS_BINS && c <= max_c)
        atomicAdd(&lds[c], 1u);
    else
        atomicAdd(&hist[c <= max_c ? (size_t)c : (size_t)max_c + 1], (Count)1);
}

template <bool PAIR, class Count>
__device__ __forceinline__ void visit(const PassArgs<Count> &a, PassState<PAIR> &s, uint32_t ca, uint32_t cb,
                                      uint32_t *lds_a, uint32_t *lds_b, const double *tbl) {
    bin_count(ca, a.max_a, lds_a, a.hist_a);
    if (PAIR) {
        s.mx_a = max(s.mx_a, ca);
        s.sum_a += ca;
        s.zero_a += (ca == 0u);
        bin_count(cb, a.max_b, lds_b, a.hist_b);
        s.mx_b = max(s.mx_b, cb);
        s.sum_b += cb;
        s.zero_b += (cb == 0u);
        if (ca != 0u && cb != 0u) {
            // the table holds delta_m_of(c, N_rays) itself, so both branches give the same value
            const double da = ca < (uint32_t)LDS_BINS && ca <= a.max_a ? tbl[ca] : delta_m_of(ca, a.nr_a);
            const double db = cb < (uint32_t)LDS_BINS && cb <= a.max_b ? tbl[LDS_BINS + cb] : delta_m_of(cb, a.nr_b);
            const double d = da - db;
            s.rms += d * d;
            s.n_both += 1;
        }
    }
}

template <bool PAIR, class Count>
__global__ __launch_bounds__(PASS_THREADS) void pass_kernel(const PassArgs<Count> a) {
    __shared__ uint32_t lds[PAIR ? 2 * LDS_BINS : LDS_BINS];
    __shared__ double tbl[PAIR ? 2 * LDS_BINS : 1];
    __shared__ double red_d[PASS_WAVES];
    __shared__ unsigned long long red_u[5][PASS_WAVES];
    __shared__ unsigned int red_m[2][PASS_WAVES];
    uint32_t *lds_a = lds;
    uint32_t *lds_b = PAIR ? lds + LDS_BINS : lds;
    const int lim_a = (int)min((uint32_t)LDS_BINS, a.max_a + 1u);   // max < 2^32 - 1
    const int lim_b = PAIR ? (int)min((uint32_t)LDS_BINS, a.max_b + 1u) : 0;
    for (int k = threadIdx.x; k < lim_a; k += PASS_THREADS) {
        lds_a[k] = 0u;
        if (PAIR) tbl[k] = delta_m_of((uint32_t)k, a.nr_a);
    }
    for (int k = threadIdx.x; k < lim_b; k += PASS_THREADS) {
        lds_b[k] = 0u;
        tbl[LDS_BINS + k] = delta_m_of((uint32_t)k, a.nr_b);
    }
    __syncthreads();

    PassState<PAIR> s;
    const int64_t gid = blockIdx.x * (int64_t)PASS_THREADS + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * PASS_THREADS;
    int64_t tail = 0;
    if (a.vec4) {
        const int64_t n4 = a.npix / 4;
        const uint4 *va = reinterpret_cast<const uint4 *>(a.map_a);
        const uint4 *vb = reinterpret_cast<const uint4 *>(a.map_b);
        const uint4 none = make_uint4(0u, 0u, 0u, 0u);
        uint4 x = none, y = none;   // the next pixels, loaded while these are counted
        if (gid < n4) {
            x = va[gid];
            if (PAIR) y = vb[gid];
        }
        for (int64_t q = gid; q < n4; q += stride) {
            const uint4 cx = x, cy = y;
            if (q + stride < n4) {
                x = va[q + stride];
                if (PAIR) y = vb[q + stride];
            }
            visit<PAIR>(a, s, cx.x, cy.x, lds_a, lds_b, tbl);
            visit<PAIR>(a, s, cx.y, cy.y, lds_a, lds_b, tbl);
            visit<PAIR>(a, s, cx.z, cy.z, lds_a, lds_b, tbl);
            visit<PAIR>(a, s, cx.w, cy.w, lds_a, lds_b, tbl);
        }
        tail = n4 * 4;
    }
    for (int64_t p = tail + gid; p < a.npix; p += stride)
        visit<PAIR>(a, s, a.map_a[p], PAIR ? a.map_b[p] : 0u, lds_a, lds_b, tbl);

    if (PAIR) {
        // Block sums in a fixed order: lanes (butterfly), then waves in index order.
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const double r = wave_sum(s.rms);
        const unsigned long long u0 = wave_sum(s.n_both), u1 = wave_sum(s.sum_a), u2 = wave_sum(s.sum_b),
                                 u3 = wave_sum(s.zero_a), u4 = wave_sum(s.zero_b);
        const unsigned int m0 = wave_max(s.mx_a), m1 = wave_max(s.mx_b);
        if (lane == 0) {
            red_d[wave] = r;
            red_u[0][wave] = u0;
            red_u[1][wave] = u1;
            red_u[2][wave] = u2;
            red_u[3][wave] = u3;
            red_u[4][wave] = u4;
            red_m[0][wave] = m0;
            red_m[1][wave] = m1;
        }
    }
    __syncthreads();
    if (PAIR && threadIdx.x == 0) {
        Partial pt{};
        for (int w = 0; w < PASS_WAVES; ++w) {
            pt.rms_sum += red_d[w];
            pt.n_both += red_u[0][w];
            pt.sum_a += red_u[1][w];
            pt.sum_b += red_u[2][w];
            pt.zero_a += red_u[3][w];
            pt.zero_b += red_u[4][w];
            pt.max_a = max(pt.max_a, red_m[0][w]);
            pt.max_b = max(pt.max_b, red_m[1][w]);
        }
        a.partials[blockIdx.x] = pt;
    }
    // Flush the LDS histograms: only bins that can hold counts, only non-zero ones.
    for (int k = threadIdx.x; k < lim_a; k += PASS_THREADS)
        if (lds_a[k]) atomicAdd(&a.hist_a[k], (Count)lds_a[k]);
    for (int k = threadIdx.x; k < lim_b; k += PASS_THREADS)
        if (lds_b[k]) atomicAdd(&a.hist_b[k], (Count)lds_b[k]);
}

constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;   // histogram bins per block of the tiled scan

int64_t scan_tiles(uint32_t max_count) { return ((int64_t)max_count + 1 + SCAN_TILE - 1) / SCAN_TILE; }

// Blocks per histogram: each takes a run of consecutive tiles, one as long as there are
// no more tiles than this (counts below 4 million), so that a block sums few run totals.
constexpr int64_t SCAN_RUNS = 1024;
int64_t run_tiles(uint32_t max_count) { return (scan_tiles(max_count) + SCAN_RUNS - 1) / SCAN_RUNS; }
int64_t scan_runs(uint32_t max_count) {
    const int64_t per = run_tiles(max_count);
    return (scan_tiles(max_count) + per - 1) / per;
}

struct ScanArgs {
    uint32_t *ha, *hb;      // na and nb bins
    int64_t na, nb;
    int64_t runs_a;         // blocks [0, runs_a) take map a's runs, the rest map b's
    int64_t per_a, per_b;   // tiles per run
    uint32_t *sums;         // one per block
};
struct Run {                // a block's run
    uint32_t *h;
    int64_t n, index, begin, end;   // bins [begin, end) of n
    const uint32_t *sums;           // its histogram's run totals
};
__device__ __forceinline__ Run run_of(const ScanArgs &s) {
    const bool side_a = (int64_t)blockIdx.x < s.runs_a;
    Run r;
    r.h = side_a ? s.ha : s.hb;
    r.n = side_a ? s.na : s.nb;
    r.index = (int64_t)blockIdx.x - (side_a ? 0 : s.runs_a);
    const int64_t bins = (side_a ? s.per_a : s.per_b) * SCAN_TILE;
    r.begin = r.index * bins;
    r.end = r.begin + bins < r.n ? r.begin + bins : r.n;
    r.sums = side_a ? s.sums : s.sums + s.runs_a;
    return r;
}

// Four bins from bin i on (zeros past the end).
__device__ __forceinline__ uint4 load_bins(const uint32_t *h, int64_t i, int64_t n) {
    static_assert(SCAN_ITEMS == 4, "a thread takes one uint4 of a tile");
    if (i + 4 <= n) return *reinterpret_cast<const uint4 *>(h + i);
    return make_uint4(i < n ? h[i] : 0u, i + 1 < n ? h[i + 1] : 0u, i + 2 < n ? h[i + 2] : 0u, 0u);
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += (uint32_t)__shfl_xor((int)v, o);
    return v;
}

// The block's sum of v, in every thread.
__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t *wsum) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = v;
    __syncthreads();
    uint32_t total = 0;
    for (int w = 0; w < SCAN_THREADS / 64; ++w) total += wsum[w];
    __syncthreads();
    return total;
}

__global__ __launch_bounds__(SCAN_THREADS) void run_sum_kernel(const ScanArgs s) {
    __shared__ uint32_t wsum[SCAN_THREADS / 64];
    const Run r = run_of(s);
    uint32_t sum = 0;
    for (int64_t i = r.begin + (int64_t)threadIdx.x * SCAN_ITEMS; i < r.end; i += SCAN_TILE) {
        const uint4 v = load_bins(r.h, i, r.n);
        sum += v.x + v.y + v.z + v.w;
    }
    const uint32_t total = block_sum(sum, wsum);
    if (threadIdx.x == 0) s.sums[blockIdx.x] = total;
}

// Inclusive prefix sums of each run in place, from the total of the runs before it.
__global__ __launch_bounds__(SCAN_THREADS) void run_scan_kernel(const ScanArgs s) {
    __shared__ uint32_t wsum[SCAN_THREADS / 64];
    const Run r = run_of(s);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t carry = 0;
    for (int64_t k = threadIdx.x; k < r.index; k += SCAN_THREADS) carry += r.sums[k];
    carry = block_sum(carry, wsum);
    for (int64_t base = r.begin; base < r.end; base += SCAN_TILE) {
        const int64_t i = base + (int64_t)threadIdx.x * SCAN_ITEMS;
        uint4 v = load_bins(r.h, i, r.n);
        v.y += v.x;
        v.z += v.y;
        v.w += v.z;
        uint32_t x = v.w;   // inclusive scan of the thread totals within the wave
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)x, o);
            if (lane >= o) x += y;
        }
        if (lane == 63) wsum[wave] = x;
        __syncthreads();
        uint32_t before = carry + x - v.w;
        for (int w = 0; w < SCAN_THREADS / 64; ++w) {
            const uint32_t t = wsum[w];
            if (w < wave) before += t;
            carry += t;
        }
        __syncthreads();
        if (i + 4 <= r.n) {
            *reinterpret_cast<uint4 *>(r.h + i) = make_uint4(v.x + before, v.y + before, v.z + before, v.w + before);
        } else {
            if (i < r.n) r.h[i] = v.x + before;
            if (i + 1 < r.n) r.h[i + 1] = v.y + before;
            if (i + 2 < r.n) r.h[i + 2] = v.z + before;
        }
    }
}

struct KsArgs {
    const uint32_t *cum_a, *cum_b;   // inclusive prefix sums of the histograms
    uint32_t max_a, max_b;
    double nr_a, nr_b;
    double npix;
    Globals *g;
};

// Four bins of either histogram per thread and step. A bin with pixels is a sample value
// x = c / N_rays of its map; both CDFs are evaluated there, the other map's by
// the largest of its bins whose value does not exceed x (next to x N_rays: the comparison
// itself decides, so that the bin is the one a search would find).
__global__ __launch_bounds__(KS_THREADS) void ks_kernel(const KsArgs a) {
    const int64_t q_a = ((int64_t)a.max_a + 4) / 4, q_all = q_a + ((int64_t)a.max_b + 4) / 4;
    double diff = 0.0;
    for (int64_t q = blockIdx.x * (int64_t)KS_THREADS + threadIdx.x; q < q_all; q += (int64_t)gridDim.x * KS_THREADS) {
        const bool own_a = q < q_a;
        const uint32_t *own = own_a ? a.cum_a : a.cum_b;
        const uint32_t *oth = own_a ? a.cum_b : a.cum_a;
        const uint32_t c0 = (uint32_t)(4 * (own_a ? q : q - q_a));
        const uint32_t m_own = own_a ? a.max_a : a.max_b, m_oth = own_a ? a.max_b : a.max_a;
        const double nr_own = own_a ? a.nr_a : a.nr_b, nr_oth = own_a ? a.nr_b : a.nr_a;
        uint32_t cum[5];
        cum[0] = c0 ? own[c0 - 1] : 0u;
#pragma unroll
        for (int k = 0; k < 4; ++k) cum[k + 1] = c0 + (uint32_t)k <= m_own ? own[c0 + k] : cum[k];
        if (cum[4] == cum[0]) continue;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (cum[k + 1] == cum[k]) continue;
            const double x = (double)(c0 + (uint32_t)k) / nr_own;
            const double guess = x * nr_oth;
            uint32_t lo = guess < (double)m_oth ? (uint32_t)guess : m_oth;
            while (lo < m_oth && (double)(lo + 1u) / nr_oth <= x) ++lo;
            while (lo > 0u && !((double)lo / nr_oth <= x)) --lo;   // 0 / nr_oth <= x always holds
            const double f_own = (double)cum[k + 1] / a.npix;
            const double f_oth = (double)oth[lo] / a.npix;
            diff = fmax(diff, fabs(f_own - f_oth));
        }
    }
    __shared__ double wave_d[KS_THREADS / 64];
    const double m = wave_max(diff);
    if ((threadIdx.x & 63) == 0) wave_d[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        double d = 0.0;
        for (int w = 0; w < KS_THREADS / 64; ++w) d = fmax(d, wave_d[w]);
        const unsigned long long bits = (unsigned long long)__double_as_longlong(d);
        if (bits > __hip_atomic_load(&a.g->d_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(&a.g->d_bits, bits);
    }
}

// Kolmogorov survival function Q(l) = P(K > l): the alternating series for
// l >= 1.18, else one minus the theta-transformed series of the CDF,
// sqrt(2 pi)/l sum_j exp(-(2j-1)^2 pi^2 / (8 l^2)).
__device__ double kolmogorov_q(double l) {
    if (!(l > 0.0)) return 1.0;
    const double pi = 3.14159265358979323846;
    double s = 0.0;
    if (l < 1.18) {
        for (int j = 1; j <= 7; ++j) {
            const double k = 2.0 * j - 1.0;
            s += exp(-(k * k) * (pi * pi) / (8.0 * l * l));
        }
        return 1.0 - sqrt(2.0 * pi) / l * s;
    }
    for (int j = 1; j <= 11; ++j) {
        const double t = exp(-2.0 * j * j * l * l);
        s += (j & 1) ? t : -t;
    }
    return 2.0 * s;
}

struct FinalArgs {
    const Partial *partials;
    int n_blocks;
    int64_t npix;
    double nr_a, nr_b;
    const uint32_t *hist_a, *hist_b;   // after the scan: overflow bins are untouched
    uint32_t max_a, max_b;
    Globals *g;
};

__global__ __launch_bounds__(FINAL_THREADS) void final_kernel(const FinalArgs a) {
    __shared__ double sd[FINAL_THREADS];
    __shared__ unsigned long long su[5][FINAL_THREADS];
    __shared__ unsigned int sm[2][FINAL_THREADS];
    double r = 0.0;
    unsigned int mx_a = 0, mx_b = 0;
    unsigned long long u[5] = {0, 0, 0, 0, 0};
    for (int b = threadIdx.x; b < a.n_blocks; b += FINAL_THREADS) {
        const Partial &p = a.partials[b];
        r += p.rms_sum;
        u[0] += p.n_both;
        u[1] += p.sum_a;
        u[2] += p.sum_b;
        u[3] += p.zero_a;
        u[4] += p.zero_b;
        mx_a = max(mx_a, p.max_a);
        mx_b = max(mx_b, p.max_b);
    }
    sd[threadIdx.x] = r;
    sm[0][threadIdx.x] = mx_a;
    sm[1][threadIdx.x] = mx_b;
    for (int k = 0; k < 5; ++k) su[k][threadIdx.x] = u[k];
    __syncthreads();
    for (int h = FINAL_THREADS / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            sd[threadIdx.x] += sd[threadIdx.x + h];
            for (int k = 0; k < 5; ++k) su[k][threadIdx.x] += su[k][threadIdx.x + h];
            for (int k = 0; k < 2; ++k) sm[k][threadIdx.x] = max(sm[k][threadIdx.x], sm[k][threadIdx.x + h]);
        }
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    rs_compare_result &res = a.g->result;
    const double npix = (double)a.npix;
    res.n_pix = a.npix;
    res.n_both = (int64_t)su[0][0];
    res.n_zero_a = (int64_t)su[3][0];
    res.n_zero_b = (int64_t)su[4][0];
    res.mean_mu_a = (double)su[1][0] / (npix * a.nr_a);
    res.mean_mu_b = (double)su[2][0] / (npix * a.nr_b);
    res.rms_dm = su[0][0] ? sqrt(sd[0] / (double)su[0][0]) : __longlong_as_double(0x7ff8000000000000ll);
    const double d = __longlong_as_double((long long)a.g->d_bits);
    const double ne = 0.5 * npix;                 // n_a n_b / (n_a + n_b) with n_a = n_b = npix
    const double sq = sqrt(ne);
    res.ks_d = d;
    res.ks_p = kolmogorov_q((sq + 0.12 + 0.11 / sq) * d);
    res.max_a = sm[0][0];
    res.max_b = sm[1][0];
    a.g->overflow = (unsigned long long)a.hist_a[(size_t)a.max_a + 1] + a.hist_b[(size_t)a.max_b + 1];
}

constexpr int MAX_THREADS = 1024;
__global__ __launch_bounds__(MAX_THREADS) void max_kernel(const uint32_t *map, int64_t npix, int vec4, uint32_t *out) {
    const int64_t gid = blockIdx.x * (int64_t)MAX_THREADS + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * MAX_THREADS;
    unsigned int m = 0;
    int64_t tail = 0;
    if (vec4) {
        const int64_t n4 = npix / 4;
        const uint4 *v = reinterpret_cast<const uint4 *>(map);
#pragma unroll 4
        for (int64_t q = gid; q < n4; q += stride) {
            const uint4 x = v[q];
            m = max(m, max(max(x.x, x.y), max(x.z, x.w)));
        }
        tail = n4 * 4;
    }
    for (int64_t p = tail + gid; p < npix; p += stride) m = max(m, map[p]);
    __shared__ unsigned int wmax[MAX_THREADS / 64];
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned int b = 0;
        for (int w = 0; w < MAX_THREADS / 64; ++w) b = max(b, wmax[w]);
        // (most blocks find a larger maximum there: atomics on one address take 12 ns each)
        if (b > __hip_atomic_load(out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(out, b);
    }
}

// Four pixels per thread and step where both arrays are aligned for it. TABLE: dm of the
// counts below LDS_BINS from an LDS table of the same values (each block makes its own, so
// only where a block has many more pixels than that): a logarithm takes some 100 FP64
// instructions, which bound the plain form on large maps. One count beyond the table costs its
// wave a logarithm, so that a block makes a table only if at least half of DM_THREADS / 64 runs of
// 64 pixels, spread over the map, hold none (16.8 million pixels of 5000 and
// more: 61 us; 76 with tables for nothing, 59 by the plain form; below 700: 36).
template <bool TABLE>
constexpr int DM_THREADS = TABLE ? 512 : 256;
template <bool TABLE>
__global__ __launch_bounds__(DM_THREADS<TABLE>) void delta_m_kernel(const uint32_t *map, int64_t npix, double n_rays, double *dm, int vec4) {
    constexpr int THREADS = DM_THREADS<TABLE>;
    __shared__ double tbl[TABLE ? LDS_BINS : 1];
    const int64_t gid = blockIdx.x * (int64_t)THREADS + threadIdx.x, stride = (int64_t)gridDim.x * THREADS;
    uint32_t bins = 0;   // counts whose dm is in the table
    if (TABLE) {
        const int64_t wave = gid / 64, n_waves = stride / 64;
        const uint32_t sample = map[wave * (npix / n_waves) + (gid & 63)];   // (npix >= DM_TABLE_MIN: 64 n_waves at least)
        if (2 * __syncthreads_count(__all(sample < (uint32_t)LDS_BINS)) >= THREADS) {
            bins = LDS_BINS;
            for (int k = threadIdx.x; k < LDS_BINS; k += THREADS) tbl[k] = delta_m_of((uint32_t)k, n_rays);
            __syncthreads();
        }
    }
    auto value = [&](uint32_t c) { return TABLE && c < bins ? tbl[c] : delta_m_of(c, n_rays); };
    int64_t tail = 0;
    if (vec4) {
        const int64_t n4 = npix / 4;
        const uint4 *v = reinterpret_cast<const uint4 *>(map);
        double2 *o = reinterpret_cast<double2 *>(dm);
        for (int64_t q = gid; q < n4; q += stride) {
            const uint4 x = v[q];
            o[2 * q] = make_double2(value(x.x), value(x.y));
            o[2 * q + 1] = make_double2(value(x.z), value(x.w));
        }
        tail = n4 * 4;
    }
    for (int64_t p = tail + gid; p < npix; p += stride) dm[p] = value(map[p]);
}

// Pixels from which delta_m's tables pay: 1024 blocks make one of LDS_BINS values each
// (6.3 million pixels of counts below 700: 22 us a call with them, 27 without).
constexpr int64_t DM_TABLE_MIN = int64_t(3) * 1024 * LDS_BINS / 2;

// Four pixels per thread until every CU has a block (16 per thread: 252 us instead of 230
// for 256^2 pixels, 514 instead of 506 for 1024^2, with counts to 3e7 and 7e7).
int pass_blocks(int64_t npix) {
    const int64_t b = (npix + (int64_t)PASS_THREADS * 4 - 1) / ((int64_t)PASS_THREADS * 4);
    return (int)(b < 1 ? 1 : (b > PASS_BLOCKS ? PASS_BLOCKS : b));
}

int stream_blocks(int64_t n, int threads, int cap) {
    const int64_t b = (n + threads - 1) / threads;
    return (int)(b < 1 ? 1 : (b > cap ? cap : b));
}

bool aligned(const void *p, size_t k) { return (reinterpret_cast<uintptr_t>(p) % k) == 0; }

int check_map(const uint32_t *map, int64_t npix, const char *name) {
    if (!map) return fail(RS_EINVAL, "%s is NULL", name);
    if (!aligned(map, 4)) return fail(RS_EINVAL, "%s must be 4-byte aligned", name);
    if (npix < 1 || npix >= MAX_PIX) return fail(RS_EINVAL, "npix must be in [1, 2^31), got %lld", (long long)npix);
    return RS_OK;
}

int check_n_rays(double n, const char *name) {
    if (!std::isfinite(n) || !(n > 0.0)) return fail(RS_EINVAL, "%s must be finite and > 0", name);
    return RS_OK;
}

}  // namespace

extern "C" {

double rs_rays_per_pixel(const rs_map_params *params) {
    if (validate(params, 0) != RS_OK) return NAN;
    const double density = ((double)params->nx / params->sw) * ((double)params->ny / params->sh);
    const double pixel_area = (params->tw / (double)params->npx) * (params->th / (double)params->npy);
    return density * pixel_area;
}

size_t rs_compare_workspace_bytes(uint32_t max_a, uint32_t max_b) {
    return WS_HIST + hist_bytes(max_a) + hist_bytes(max_b) +
           align256(sizeof(unsigned long long) * (size_t)(scan_tiles(max_a) + scan_tiles(max_b)));
}

int rs_map_max(const uint32_t *map, int64_t npix, uint32_t *max_dev, void *stream) {
    int rc = check_map(map, npix, "map");
    if (rc) return rc;
    if (!max_dev || !aligned(max_dev, 4)) return fail(RS_EINVAL, "max_dev must be a 4-byte aligned device pointer");
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(zero_u32_kernel, dim3(1), dim3(1), 0, s, max_dev);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "zeroing the maximum");
    hipLaunchKernelGGL(max_kernel, dim3(stream_blocks(npix, MAX_THREADS * 8, 512)), dim3(MAX_THREADS), 0, s, map, npix,
                       aligned(map, 16) ? 1 : 0, max_dev);
    e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "map maximum kernel");
}

int rs_map_histogram(const uint32_t *map, int64_t npix, uint32_t max_count, uint64_t *hist, void *stream) {
    int rc = check_map(map, npix, "map");
    if (rc) return rc;
    if (!hist || !aligned(hist, 8)) return fail(RS_EINVAL, "hist must be an 8-byte aligned device pointer");
    if (max_count == 0xffffffffu) return fail(RS_EINVAL, "max_count must be below 2^32 - 1");
    hipStream_t s = static_cast<hipStream_t>(stream);
    auto *h = reinterpret_cast<unsigned long long *>(hist);
    const int64_t n = (int64_t)max_count + 2;
    hipLaunchKernelGGL(zero_u64_kernel, dim3(stream_blocks(n, 256, 1024)), dim3(256), 0, s, h, n);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "zeroing the histogram");
    PassArgs<unsigned long long> a{};
    a.map_a = map;
    a.npix = npix;
    a.max_a = max_count;
    a.hist_a = h;
    a.vec4 = aligned(map, 16) ? 1 : 0;
    hipLaunchKernelGGL((pass_kernel<false, unsigned long long>), dim3(pass_blocks(npix)), dim3(PASS_THREADS), 0, s, a);
    e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "histogram kernel");
}

int rs_delta_m(const uint32_t *map, int64_t npix, double n_rays, double *dm, void *stream) {
    int rc = check_map(map, npix, "map");
    if (rc) return rc;
    if ((rc = check_n_rays(n_rays, "n_rays"))) return rc;
    if (!dm || !aligned(dm, 8)) return fail(RS_EINVAL, "dm must be an 8-byte aligned device pointer");
    const int vec4 = aligned(map, 16) && aligned(dm, 16) ? 1 : 0;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (npix >= DM_TABLE_MIN)
        hipLaunchKernelGGL(delta_m_kernel<true>, dim3(1024), dim3(DM_THREADS<true>), 0, s, map, npix, n_rays, dm, vec4);
    else
        hipLaunchKernelGGL(delta_m_kernel<false>, dim3(stream_blocks(npix, 256 * 4, 4096)), dim3(256), 0, s, map, npix,
                           n_rays, dm, vec4);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? RS_OK : hip_fail(e, "dm kernel");
}

int rs_compare_maps(const uint32_t *map_a, const uint32_t *map_b, int64_t npix, double n_rays_a, double n_rays_b,
                    uint32_t max_a, uint32_t max_b, void *workspace, size_t workspace_bytes,
                    rs_compare_result *result_host, void *stream) {
    int rc = check_map(map_a, npix, "map_a");
    if (rc) return rc;
    if ((rc = check_map(map_b, npix, "map_b"))) return rc;
    if ((rc = check_n_rays(n_rays_a, "n_rays_a"))) return rc;
    if ((rc = check_n_rays(n_rays_b, "n_rays_b"))) return rc;
    if (!result_host) return fail(RS_EINVAL, "result_host is NULL");
    if (max_a == 0xffffffffu || max_b == 0xffffffffu) return fail(RS_EINVAL, "count bounds must be below 2^32 - 1");
    if (!workspace || !aligned(workspace, 256)) return fail(RS_EINVAL, "workspace must be a 256-byte aligned device pointer");
    const size_t need = rs_compare_workspace_bytes(max_a, max_b);
    if (workspace_bytes < need) return fail(RS_ENOMEM, "workspace has %zu bytes, needs %zu", workspace_bytes, need);

    char *ws = static_cast<char *>(workspace);
    auto *g = reinterpret_cast<Globals *>(ws);
    auto *partials = reinterpret_cast<Partial *>(ws + WS_PARTIALS);
    auto *hist_a = reinterpret_cast<uint32_t *>(ws + WS_HIST);
    auto *hist_b = reinterpret_cast<uint32_t *>(ws + WS_HIST + hist_bytes(max_a));
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e;

    // (max + 2 bins in whole 16-byte words: within hist_bytes, which counts 8 bytes per bin)
    const int64_t z_a = ((int64_t)max_a + 2 + 3) / 4, z_b = ((int64_t)max_b + 2 + 3) / 4;
    hipLaunchKernelGGL(zero_compare_kernel, dim3(stream_blocks(z_a > z_b ? z_a : z_b, 256, 1024)), dim3(256), 0, s, g,
                       reinterpret_cast<uint4 *>(hist_a), z_a, reinterpret_cast<uint4 *>(hist_b), z_b);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "zeroing the compare workspace");

    PassArgs<uint32_t> pa{};
    pa.map_a = map_a;
    pa.map_b = map_b;
    pa.npix = npix;
    pa.nr_a = n_rays_a;
    pa.nr_b = n_rays_b;
    pa.max_a = max_a;
    pa.max_b = max_b;
    pa.hist_a = hist_a;
    pa.hist_b = hist_b;
    pa.partials = partials;
    pa.vec4 = (aligned(map_a, 16) && aligned(map_b, 16)) ? 1 : 0;
    const int blocks = pass_blocks(npix);
    hipLaunchKernelGGL((pass_kernel<true, uint32_t>), dim3(blocks), dim3(PASS_THREADS), 0, s, pa);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "compare pass kernel");

    // scan of both histograms: the runs' sums, then the runs
    ScanArgs sa{};
    sa.ha = hist_a;
    sa.hb = hist_b;
    sa.na = (int64_t)max_a + 1;
    sa.nb = (int64_t)max_b + 1;
    sa.runs_a = scan_runs(max_a);
    sa.per_a = run_tiles(max_a);
    sa.per_b = run_tiles(max_b);
    sa.sums = reinterpret_cast<uint32_t *>(ws + WS_HIST + hist_bytes(max_a) + hist_bytes(max_b));
    const dim3 runs((unsigned)(sa.runs_a + scan_runs(max_b)));
    hipLaunchKernelGGL(run_sum_kernel, runs, dim3(SCAN_THREADS), 0, s, sa);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "histogram sums");
    hipLaunchKernelGGL(run_scan_kernel, runs, dim3(SCAN_THREADS), 0, s, sa);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "histogram scan");

    KsArgs ka{};
    ka.cum_a = hist_a;
    ka.cum_b = hist_b;
    ka.max_a = max_a;
    ka.max_b = max_b;
    ka.nr_a = n_rays_a;
    ka.nr_b = n_rays_b;
    ka.npix = (double)npix;
    ka.g = g;
    const int64_t quads = (int64_t)max_a / 4 + (int64_t)max_b / 4 + 2;
    hipLaunchKernelGGL(ks_kernel, dim3(stream_blocks(quads, KS_THREADS, 2048)), dim3(KS_THREADS), 0, s, ka);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "K-S kernel");

    FinalArgs fa{};
    fa.partials = partials;
    fa.n_blocks = blocks;
    fa.npix = npix;
    fa.nr_a = n_rays_a;
    fa.nr_b = n_rays_b;
    fa.hist_a = hist_a;
    fa.hist_b = hist_b;
    fa.max_a = max_a;
    fa.max_b = max_b;
    fa.g = g;
    hipLaunchKernelGGL(final_kernel, dim3(1), dim3(FINAL_THREADS), 0, s, fa);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "compare final kernel");

    Globals host{};
    e = hipMemcpyAsync(&host, g, sizeof(Globals), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "reading the comparison");
    *result_host = host.result;
    if (host.overflow)
        return fail(RS_EINVAL, "a ray count exceeds its bound (max_a=%u max_b=%u, found %u and %u)", max_a, max_b,
                    host.result.max_a, host.result.max_b);
    return RS_OK;
}

}  // extern "C"
