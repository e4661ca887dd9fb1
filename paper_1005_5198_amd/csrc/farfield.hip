// Far-field expansion (RS_FARFIELD): levels of FP64 local expansions of the
// distant lenses, near lenses summed directly, a rigorous per-ray bound.
#include "far_ray.h"
#include "rs_decide.h"
#include "rs_launch.h"

namespace rs {
namespace {

// ---------------------------------------------------------------------------
// Far-field expansion (RS_FARFIELD). The paper's tree codes group distant
// lenses into pseudo-lenses with higher multipoles (Section 2, Eq.
// (hierarchical)); here distant lenses enter local expansions of the
// deflection, to order FAR_P, on three levels, four from FF_TOP_MIN_LENSES lenses
// on. The last two (tops of groups and groups of super-patches are alike):
//   * super-patch (FF_SP_X x FF_SP_Y patches, centre zS, half-diagonal H):
//     lenses farther than FAR_RATIO H give C_n = sum_k m_k tS_k^(n+1),
//     tS_k = 1 / (zS - z_k); nearer lenses go to the super-patch's list;
//   * patch (64 x 32 rays, centre z0, half-diagonal h): the super expansion
//     is re-centred exactly on z0 (a polynomial translation), and the listed
//     lenses farther than FAR_RATIO h from z0 add c_n = sum_k m_k t_k^(n+1),
//     t_k = 1 / (z0 - z_k); the rest are summed directly.
// With z = x1 + i x2 and w = z - z0, sum_k m_k / (z - z_k) = sum_n (-w)^n T_n,
// and the deflection (a1, a2) is (Re, -Im) of that sum. All of it is FP64; each
// ray carries a rigorous bound (series truncation on every level, rounding of
// the coefficients, the translation and the evaluation, the near sum) plus the
// definition's own rounding, and rays within it of a pixel edge go to the FP64
// re-check, so the map equals the definition's.
// ---------------------------------------------------------------------------
constexpr int FAR_THREADS = 256;
constexpr int FAR_ROWS = PATCH_X * PATCH_Y / FAR_THREADS;     // rays per thread (8)
static_assert(FAR_ROWS * (FAR_THREADS / 64) == (PATCH_X / 8) * (PATCH_Y / 8), "8 x 8 blocks cover the patch");
constexpr int NEAR_EXP = 512;

// binom(n, m) for n, m < FAR_P (Pascal's triangle; integers below 2^13, exact in FP64).
struct BinomTable {
    double v[FAR_P][FAR_P];
    constexpr BinomTable() : v() {
        for (int n = 0; n < FAR_P; ++n) {
            v[n][0] = 1.0;
            for (int m = 1; m <= n; ++m) v[n][m] = v[n - 1][m - 1] + (m < n ? v[n - 1][m] : 0.0);
        }
    }
};
__constant__ constexpr BinomTable BINOM_TABLE{};
#define BINOM BINOM_TABLE.v
// n! and 1 / n! for n < FAR_P (n! below 2^41, exact in FP64).
struct FactorialTable {
    double f[FAR_P], inv[FAR_P];
    constexpr FactorialTable() : f(), inv() {
        f[0] = inv[0] = 1.0;
        for (int n = 1; n < FAR_P; ++n) {
            f[n] = f[n - 1] * n;
            inv[n] = 1.0 / f[n];
        }
    }
};
__constant__ constexpr FactorialTable FACTORIAL{};
// Steps of a reduction over the wave's lanes that leaves each lane with part of the
// values: of its N values a lane keeps the first (N + 1) / 2 if its bit BIT is 0, the
// others if it is 1, and adds its partner's partial sums of them. at and end follow
// which values of the whole list a lane holds.
template <int BIT, int N>
__device__ __forceinline__ void scatter_range(int lane, int &at, int &end) {
    constexpr int H = (N + 1) / 2;
    if (lane & BIT) at += H;
    else if (end > at + H) end = at + H;
}

// BIT 32 or 16: v_permlane32_swap / v_permlane16_swap exchange the upper lanes (odd
// rows) of one register with the lower lanes (even rows) of another.
template <int BIT, int N, int M>
__device__ __forceinline__ void scatter_swap(double (&v)[M], int lane, int &at, int &end) {
    static_assert(N % 2 == 0, "halves");
    constexpr int H = N / 2;
#pragma unroll
    for (int k = 0; k < H; ++k) {
        const uint64_t a = (uint64_t)__double_as_longlong(v[k]), b = (uint64_t)__double_as_longlong(v[k + H]);
        uint64_t x, y;
        if constexpr (BIT == 32) {
            const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
            const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
            x = ((uint64_t)hi[0] << 32) | lo[0];
            y = ((uint64_t)hi[1] << 32) | lo[1];
        } else {
            const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)a, (uint32_t)b, false, false);
            const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
            x = ((uint64_t)hi[0] << 32) | lo[0];
            y = ((uint64_t)hi[1] << 32) | lo[1];
        }
        v[k] = __longlong_as_double((long long)x) + __longlong_as_double((long long)y);
    }
    scatter_range<BIT, N>(lane, at, end);
}

// Smaller BIT: the partner (the lane that differs in BIT, and maybe in lower bits) by DPP.
template <int BIT, int N, int CTRL, int M>
__device__ __forceinline__ void scatter_dpp(double (&v)[M], int lane, int &at, int &end) {
    constexpr int H = (N + 1) / 2;
    const bool up = (lane & BIT) != 0;
#pragma unroll
    for (int k = 0; k < H; ++k) {
        const double lo = v[k], hi = k + H < N ? v[k + H] : 0.0;
        const double keep = up ? hi : lo, send = up ? lo : hi;
        const uint64_t w = (uint64_t)__double_as_longlong(send);
        const uint32_t w0 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)w, CTRL, 0xf, 0xf, false);
        const uint32_t w1 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(w >> 32), CTRL, 0xf, 0xf, false);
        v[k] = keep + __longlong_as_double((long long)(((uint64_t)w1 << 32) | w0));
    }
    scatter_range<BIT, N>(lane, at, end);
}

// One lens's contribution to an expansion about (ox, oy) with half-diagonal h
// (the lens is at least FAR_RATIO h away): the powers m t^(n+1) and the bound
// terms m/|d|, m/|d| rho^P / (1 - rho) and m / (|d| - h).
struct FarAcc {
    double c1[FAR_P], c2[FAR_P];
    double sfar, trunc, sdef;
    __device__ void zero() {
#pragma unroll
        for (int n = 0; n < FAR_P; ++n) {
            c1[n] = 0.0;
            c2[n] = 0.0;
        }
        sfar = trunc = sdef = 0.0;
    }
    __device__ __forceinline__ void add(double d1, double d2, double r2, double m, double h) {
        const double inv = rcp64(r2);
        const double t1 = d1 * inv, t2 = -d2 * inv;   // t = 1 / d, d = centre - lens
        double p1 = m * t1, p2 = m * t2;
        c1[0] += p1;
        c2[0] += p2;
#pragma unroll
        for (int n = 1; n < FAR_P; ++n) {
            const double q1 = __builtin_fma(p1, t1, -p2 * t2);
            const double q2 = __builtin_fma(p1, t2, p2 * t1);
            p1 = q1;
            p2 = q2;
            c1[n] += p1;
            c2[n] += p2;
        }
        // Bound terms from 1/|d| and 1/(1 - rho) (Newton-refined, within a few units of
        // 2^-53 relative; the decision's final factor 1.001 covers that): |m|/(|d| - h)
        // is |m|/|d| / (1 - rho).
        const double inv_ad = rsq64(r2);
        const double s = fabs(m) * inv_ad;
        const double rho = h * inv_ad;
        const double rho2 = rho * rho, rho4 = rho2 * rho2, rho8 = rho4 * rho4, rho16 = rho8 * rho8;
        const double sg = s * rcp64(1.0 - rho);
        sfar += s;
        trunc = __builtin_fma(sg, rho16, trunc);
        sdef += sg;
    }
    // The wave's totals into tot[FAR_REC] (shared): a reduction that scatters as it goes
    // (each step halves the number of values a lane holds), 38 exchanges of a double in all
    // and none of them through LDS. (A butterfly of the 36 values takes 216, through LDS:
    // a third of the patch record kernel's time.)
    __device__ __forceinline__ void wave_totals(double *tot) {
        double v[FAR_REC];
#pragma unroll
        for (int n = 0; n < FAR_P; ++n) {
            v[n] = c1[n];
            v[FAR_P + n] = c2[n];
        }
        v[2 * FAR_P] = sfar;
        v[2 * FAR_P + 1] = trunc;
        v[2 * FAR_P + 2] = sdef;
        v[2 * FAR_P + 3] = 0.0;   // (CHAIN is the builder's)
        const int lane = threadIdx.x & 63;
        int at = 0, end = FAR_REC;   // this lane's values are at .. end - 1 of the 36
        scatter_swap<32, 36>(v, lane, at, end);
        scatter_swap<16, 18>(v, lane, at, end);
        scatter_dpp<8, 9, 0x128>(v, lane, at, end);   // row_ror:8
        scatter_dpp<4, 5, 0x141>(v, lane, at, end);   // row_half_mirror: the lane's three low bits flipped
        scatter_dpp<2, 3, 0x4e>(v, lane, at, end);    // quad_perm [2,3,0,1]
        scatter_dpp<1, 2, 0xb1>(v, lane, at, end);    // quad_perm [1,0,3,2]
        if (at < end) tot[at] = v[0];
    }
    // Block sum into out[FAR_REC] (shared); lanes first, then waves in index order.
    template <int THREADS = FAR_THREADS>
    __device__ void reduce(double (*part)[FAR_REC], double *out) {
        wave_totals(part[threadIdx.x >> 6]);
        __syncthreads();
        if (threadIdx.x < FAR_REC) {
            double v = 0.0;
            for (int w = 0; w < THREADS / 64; ++w) v += part[w][threadIdx.x];
            out[threadIdx.x] = v;
        }
        __syncthreads();
    }
};

// Shared memory of a level builder with THREADS threads.
template <int THREADS = FAR_THREADS>
struct FarLevelSmem {
    double part[THREADS / 64][FAR_REC];
    double out[FAR_REC];
    int count;
};
using FarSuperSmem = FarLevelSmem<FAR_THREADS>;
// Groups hold 2^19 rays and there are few of them: two blocks' worth of threads each.
constexpr int FAR_GROUP_THREADS = 2 * FAR_THREADS;

// Record of one level about (cx, cy) with half-diagonal H: of the candidates
// (cand(q, k, X, Y) gives candidate q's lens, or false when q is none), those
// farther than FAR_RATIO H add to the expansion C_n = sum m t^(n+1) and to the
// bound sums; the others go to list (count in list[0]; a count above cap means
// the list is incomplete and the level below scans every lens instead). With a
// parent record about (pcx, pcy) (a level above, whose own candidates these
// are; held as n_parts records to be added in order), the parent's expansion is
// re-centred exactly on (cx, cy),
//   E_m = sum_{n>=m} binom(n, m) e^(n-m) C_n, e = z_parent - z,
// and added, and its bound sums are added to this level's. The sums stay valid
// bounds below: their rounding constants allow for several translations.
template <bool UNIT, int THREADS = FAR_THREADS, class Cand>
__device__ __forceinline__ void build_level(const ShootArgs &a, double cx, double cy, double H, int64_t n_cand, Cand cand,
                                   int32_t *list, int cap, double *rec, const double *parent, int n_parts,
                                   double pcx, double pcy, FarLevelSmem<THREADS> &sm) {
    const double near_r2 = (FAR_RATIO * H) * (FAR_RATIO * H);
    if (threadIdx.x == 0) sm.count = 0;
    __syncthreads();
    FarAcc acc;
    acc.zero();
    // The next candidate's lens is loaded before this one is expanded, so its
    // memory latency overlaps the expansion.
    int64_t kn = 0;
    double Xn = 0.0, Yn = 0.0;
    bool vn = (int64_t)threadIdx.x < n_cand && cand(threadIdx.x, kn, Xn, Yn);
#pragma unroll 1
    for (int64_t q = threadIdx.x; q < n_cand; q += THREADS) {
        const int64_t k = kn;
        const double X = Xn, Y = Yn;
        const bool v = vn;
        vn = q + THREADS < n_cand && cand(q + THREADS, kn, Xn, Yn);
        if (!v) continue;
        const double d1 = cx - X, d2 = cy - Y;
        const double r2 = d1 * d1 + d2 * d2;
        if (!(r2 >= near_r2)) {
            const int j = atomicAdd(&sm.count, 1);
            if (j < cap) list[1 + j] = (int32_t)k;
            continue;
        }
        const double m = (UNIT || a.lens_m == nullptr) ? 1.0 : ((global_double *)a.lens_m)[k];
        acc.add(d1, d2, r2, m, H);
    }
    acc.template reduce<THREADS>(sm.part, sm.out);
    // The most additions any term of this level's sums went through: its thread's own, the
    // lanes', the waves'. (With the number of lenses in its place, 10^6 at the top, this
    // rounding was half of the bound.)
    const double chain = (double)((n_cand + THREADS - 1) / THREADS + 6 + THREADS / 64);
    const int t = threadIdx.x;
    if (parent == nullptr) {
        if (t < FAR_REC) rec[t] = t == FAR_REC - 1 ? chain : sm.out[t];
    } else {
        const global_double *Pp = (const global_double *)parent;
        auto P = [&](int n) {
            double v = Pp[n];
            for (int part = 1; part < n_parts; ++part) v += Pp[part * FAR_REC + n];
            return v;
        };
        if (t < FAR_P) {
            const double e1 = pcx - cx, e2 = pcy - cy;
            double s1 = 0.0, s2 = 0.0;
            double g1 = 1.0, g2 = 0.0;   // e^(n-m)
            for (int n = t; n < FAR_P; ++n) {
                const double binom = BINOM[n][t];   // exact in FP64 for n < 16
                const double C1 = P(n), C2 = P(FAR_P + n);
                s1 = __builtin_fma(binom, g1 * C1 - g2 * C2, s1);
                s2 = __builtin_fma(binom, g1 * C2 + g2 * C1, s2);
                const double q1 = g1 * e1 - g2 * e2, q2 = g1 * e2 + g2 * e1;
                g1 = q1;
                g2 = q2;
            }
            rec[t] = s1 + sm.out[t];
            rec[FAR_P + t] = s2 + sm.out[FAR_P + t];
        } else if (t < FAR_P + FAR_EXTRA) {
            const int k = FAR_P + t;   // the bound terms (the parts' chains add up to more than the longest and the joining)
            rec[k] = P(k) + (k == FAR_REC - 1 ? chain : sm.out[k]);
        }
    }
    if (t == 0) list[0] = sm.count;
}

// Every lens from index first on is a candidate.
struct AllLenses {
    const double *xy;
    int64_t first;
    __device__ bool operator()(int64_t q, int64_t &k, double &X, double &Y) const {
        k = first + q;
        X = ((global_double *)xy)[2 * k];
        Y = ((global_double *)xy)[2 * k + 1];
        return true;
    }
};

// Records of super-patch sp from every lens (the mixed mode's re-check stage,
// random rays and batches): far lenses -> coefficients about zS; the others ->
// the super-patch's lens list.
template <bool UNIT>
__device__ __forceinline__ void build_super(const ShootArgs &a, int64_t sp, FarSuperSmem &sm) {
    double cx, cy, H;
    super_geometry(a, sp, cx, cy, H);
    build_level<UNIT>(a, cx, cy, H, a.n_lens, AllLenses{a.lens_xy, 0}, a.ff_near + sp * (int64_t)(1 + a.ff_cap), a.ff_cap,
                      a.ff_super + sp * (int64_t)FAR_REC, nullptr, 0, 0.0, 0.0, sm);
}

// Level 1 of one launch (or, for random rays, of the whole rectangle): one block
// per super-patch. RECHECK: the grid re-check stage needs the records only when
// the deflection launch queued rays.
template <bool UNIT, bool RECHECK>
__global__ __launch_bounds__(FAR_THREADS) void farfield_super_kernel(const ShootArgs a) {
    __shared__ FarSuperSmem sm;
    if (RECHECK && *a.qcount == 0) return;
    build_super<UNIT>(a, blockIdx.x, sm);
}

// Records and the map's zeroing in one launch: the first n_super blocks build the records,
// the others clear the map and the workspace's words.
template <bool UNIT>
__global__ __launch_bounds__(FAR_THREADS) void fill_records_kernel(const ShootArgs a, uint32_t n_super, uint32_t *map,
                                                                   int64_t n_pix, uint32_t *ws_words, int64_t n_ws_words) {
    __shared__ FarSuperSmem sm;
    if (blockIdx.x < n_super) {
        build_super<UNIT>(a, blockIdx.x, sm);
        return;
    }
    const int64_t t0 = (int64_t)(blockIdx.x - n_super) * FAR_THREADS + threadIdx.x;
    const int64_t stride = (int64_t)(gridDim.x - n_super) * FAR_THREADS;
    for (int64_t t = t0; t < n_pix; t += stride) map[t] = 0u;
    for (int64_t t = t0; t < n_ws_words; t += stride) ws_words[t] = 0u;
}

// Blocks that scan one group's lenses: one per 8192 lenses, at most FF_GROUP_PARTS.
__host__ __device__ inline int group_parts(int64_t n_lens) {
    return n_lens / 8192 + 1 < FF_GROUP_PARTS ? (int)(n_lens / 8192 + 1) : FF_GROUP_PARTS;
}

// Far-field mode, level 0: groups of FF_GROUP x FF_GROUP super-patches (centre
// zG, half-diagonal HG, one ray spacing of slack on each side, of the full box).
__device__ __forceinline__ void group_geometry(const ShootArgs &a, int64_t g, double &cx, double &cy, double &H) {
    constexpr int GX = FF_GROUP * FF_SP_X * PATCH_X, GY = FF_GROUP * FF_SP_Y * PATCH_Y;
    const int64_t gx = g % a.ff_gbx, gy = g / a.ff_gbx;
    const int64_t i_g = a.ff_i0 + gx * GX;
    const int64_t j_g = a.ff_j0 + gy * GY;
    cx = a.sx0 + ((double)i_g + 0.5 * GX) * a.spx;
    cy = a.sy0 + ((double)j_g + 0.5 * GY) * a.spy;
    const double hx = (0.5 * GX + 1.0) * a.spx;
    const double hy = (0.5 * GY + 1.0) * a.spy;
    H = sqrt(hx * hx + hy * hy) * (1.0 + 1e-12);
}

__device__ __forceinline__ int64_t group_of(const ShootArgs &a, int64_t sp) {
    return ((sp / a.ff_sbx) / FF_GROUP) * a.ff_gbx + (sp % a.ff_sbx) / FF_GROUP;
}

// Far-field mode with tops: top t of FF_TOP x FF_TOP groups, the same construction one
// level up (its box holds its groups' boxes).
__device__ __forceinline__ void top_geometry(const ShootArgs &a, int64_t t, double &cx, double &cy, double &H) {
    constexpr int TX = FF_TOP * FF_GROUP * FF_SP_X * PATCH_X, TY = FF_TOP * FF_GROUP * FF_SP_Y * PATCH_Y;
    const int64_t tx = t % a.ff_tbx, ty = t / a.ff_tbx;
    const int64_t i_t = a.ff_i0 + tx * TX;
    const int64_t j_t = a.ff_j0 + ty * TY;
    cx = a.sx0 + ((double)i_t + 0.5 * TX) * a.spx;
    cy = a.sy0 + ((double)j_t + 0.5 * TY) * a.spy;
    const double hx = (0.5 * TX + 1.0) * a.spx;
    const double hy = (0.5 * TY + 1.0) * a.spy;
    H = sqrt(hx * hx + hy * hy) * (1.0 + 1e-12);
}

__device__ __forceinline__ int64_t top_of(const ShootArgs &a, int64_t g) {
    return ((g / a.ff_gbx) / FF_TOP) * a.ff_tbx + (g % a.ff_gbx) / FF_TOP;
}

// A level's candidates: the lists of the level above (one per part, in part order), or,
// when one of them overflowed, every lens that level did not expand (the same test it
// made).
template <int P>
struct ListCandidates {
    const double *xy;
    const global_i32 *lists;   // the parts' lists, stride apart
    int64_t stride;
    int64_t e[P - 1];          // candidates before the end of parts 0 .. P - 2 (non-decreasing)
    bool scan_all;
    double cx, cy, r2;
    __device__ bool operator()(int64_t q, int64_t &k, double &X, double &Y) const {
        if (scan_all) {
            k = q;
        } else {
            // q's part is the number of part ends at or below q; its offset counts from the
            // last of them (unrolled, so e stays in registers)
            int64_t part = 0, before = 0;
#pragma unroll
            for (int i = 0; i < P - 1; ++i) {
                const bool past = q >= e[i];
                part += past;
                before = past ? e[i] : before;
            }
            k = (int64_t)lists[part * stride + 1 + (q - before)];
        }
        X = ((global_double *)xy)[2 * k];
        Y = ((global_double *)xy)[2 * k + 1];
        if (scan_all) {
            const double f1 = cx - X, f2 = cy - Y;
            if (f1 * f1 + f2 * f2 >= r2) return false;
        }
        return true;
    }
};

// Candidates from `used` lists of capacity cap, stride apart, of the level about (cx, cy)
// with half-diagonal H.
template <int P>
__device__ __forceinline__ ListCandidates<P> list_candidates(const ShootArgs &a, const int32_t *lists, int64_t stride,
                                                             int32_t cap, int used, double cx, double cy, double H,
                                                             int64_t &n) {
    ListCandidates<P> c;
    c.xy = a.lens_xy;
    c.cx = cx;
    c.cy = cy;
    c.r2 = (FAR_RATIO * H) * (FAR_RATIO * H);
    c.lists = (const global_i32 *)lists;
    c.stride = stride;
    c.scan_all = false;
    int64_t total = 0;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int32_t np = p < used ? c.lists[p * stride] : 0;   // the lists past `used` were not written
        c.scan_all = c.scan_all || np > cap;
        total += np;
        if (p < P - 1) c.e[p] = total;
    }
    n = c.scan_all ? a.n_lens : total;
    return c;
}

// A super-patch's candidates: its group's lists (one per part), or with tops the
// group's one list.
__device__ __forceinline__ ListCandidates<FF_GROUP_PARTS> group_candidates(const ShootArgs &a, int64_t g, int64_t &n) {
    double cx, cy, H;
    group_geometry(a, g, cx, cy, H);
    const int32_t *lists = a.ff_glist + g * FF_GROUP_PARTS * (int64_t)(1 + FF_PART_CAP);
    if (a.ff_top) return list_candidates<FF_GROUP_PARTS>(a, lists, 0, FF_GROUP_ONE_CAP, 1, cx, cy, H, n);
    return list_candidates<FF_GROUP_PARTS>(a, lists, 1 + FF_PART_CAP, FF_PART_CAP, group_parts(a.n_lens), cx, cy,
                                           H, n);
}

// Far-field mode, level 0: group_parts(N) blocks per group, each over its range of
// lens indices.
template <bool UNIT>
__global__ __launch_bounds__(FAR_GROUP_THREADS) __attribute__((amdgpu_waves_per_eu(4))) void farfield_group_kernel(const ShootArgs a) {
    __shared__ FarLevelSmem<FAR_GROUP_THREADS> sm;
    const int used = group_parts(a.n_lens);
    const int64_t g = blockIdx.x / used;
    const int part = (int)(blockIdx.x % used);
    const int64_t first = a.n_lens * part / used;
    const int64_t last = a.n_lens * (part + 1) / used;
    double cx, cy, H;
    group_geometry(a, g, cx, cy, H);
    const int64_t slot = g * FF_GROUP_PARTS + part;
    build_level<UNIT, FAR_GROUP_THREADS>(a, cx, cy, H, last - first, AllLenses{a.lens_xy, first},
                                         a.ff_glist + slot * (int64_t)(1 + FF_PART_CAP), FF_PART_CAP,
                                         a.ff_group + slot * (int64_t)FAR_REC, nullptr, 0, 0.0, 0.0, sm);
}

// Far-field mode with tops, level 0: FF_TOP_PARTS blocks per top, each over its range of
// lens indices (the group kernel's scan one level up). A launch has few tops (a band of
// 2^27 rays holds about 30), so the blocks are as large as they can be.
constexpr int FAR_TOP_THREADS = 1024;
template <bool UNIT>
__global__ __launch_bounds__(FAR_TOP_THREADS) __attribute__((amdgpu_waves_per_eu(4))) void farfield_top_kernel(const ShootArgs a) {
    __shared__ FarLevelSmem<FAR_TOP_THREADS> sm;
    const int64_t t = blockIdx.x / FF_TOP_PARTS;
    const int part = (int)(blockIdx.x % FF_TOP_PARTS);
    const int64_t first = a.n_lens * part / FF_TOP_PARTS;
    const int64_t last = a.n_lens * (part + 1) / FF_TOP_PARTS;
    double cx, cy, H;
    top_geometry(a, t, cx, cy, H);
    const int64_t slot = t * FF_TOP_PARTS + part;
    build_level<UNIT, FAR_TOP_THREADS>(a, cx, cy, H, last - first, AllLenses{a.lens_xy, first},
                                         a.ff_tlist + slot * (int64_t)(1 + FF_TOP_PART_CAP), FF_TOP_PART_CAP,
                                         a.ff_top + slot * (int64_t)FAR_REC, nullptr, 0, 0.0, 0.0, sm);
}

// Far-field mode with tops, level 1: one block per group, candidates from its top's
// lists, the top's expansion re-centred and added; one record (part 0) and one list.
template <bool UNIT>
__global__ __launch_bounds__(FAR_GROUP_THREADS) __attribute__((amdgpu_waves_per_eu(4))) void farfield_group_top_kernel(const ShootArgs a) {
    __shared__ FarLevelSmem<FAR_GROUP_THREADS> sm;
    const int64_t g = blockIdx.x;
    const int64_t t = top_of(a, g);
    double tcx, tcy, tH;
    top_geometry(a, t, tcx, tcy, tH);
    int64_t n;
    const ListCandidates<FF_TOP_PARTS> c =
        list_candidates<FF_TOP_PARTS>(a, a.ff_tlist + t * FF_TOP_PARTS * (int64_t)(1 + FF_TOP_PART_CAP),
                                      1 + FF_TOP_PART_CAP, FF_TOP_PART_CAP, FF_TOP_PARTS, tcx, tcy, tH, n);
    double cx, cy, H;
    group_geometry(a, g, cx, cy, H);
    build_level<UNIT, FAR_GROUP_THREADS>(a, cx, cy, H, n, c, a.ff_glist + g * FF_GROUP_PARTS * (int64_t)(1 + FF_PART_CAP),
                                         FF_GROUP_ONE_CAP, a.ff_group + g * FF_GROUP_PARTS * (int64_t)FAR_REC,
                                         a.ff_top + t * FF_TOP_PARTS * (int64_t)FAR_REC, FF_TOP_PARTS, tcx, tcy, sm);
}

// Far-field mode, level 1: one block per super-patch, candidates from its group,
// the group's expansion re-centred and added.
template <bool UNIT>
__global__ __launch_bounds__(FAR_THREADS) void farfield_super_group_kernel(const ShootArgs a) {
    __shared__ FarSuperSmem sm;
    const int64_t sp = blockIdx.x;
    const int64_t g = group_of(a, sp);
    int64_t n;
    const ListCandidates<FF_GROUP_PARTS> c = group_candidates(a, g, n);
    double cx, cy, H;
    super_geometry(a, sp, cx, cy, H);
    build_level<UNIT>(a, cx, cy, H, n, c, a.ff_near + sp * (int64_t)(1 + a.ff_cap), a.ff_cap,
                      a.ff_super + sp * (int64_t)FAR_REC, a.ff_group + g * FF_GROUP_PARTS * (int64_t)FAR_REC,
                      a.ff_top ? 1 : group_parts(a.n_lens), c.cx, c.cy, sm);
}

// Level 1 of every map of a mixed batch that flagged rays: one block per
// (map, super-patch), maps found by binary search on their first record.
template <bool UNIT>
__global__ __launch_bounds__(FAR_THREADS) void batch_super_kernel(const BatchArgs b) {
    __shared__ FarSuperSmem sm;
    const int64_t t = blockIdx.x;
    int lo = 0, hi = b.n_maps - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (b.maps[mid].super_begin <= t) lo = mid;
        else hi = mid - 1;
    }
    const BatchMap &m = b.maps[lo];
    if (t - m.super_begin >= m.n_super || m.counters[C_RECHECK] == 0ull) return;
    const ShootArgs a = make_uniform(batch_far_args(m));
    build_super<UNIT>(a, t - m.super_begin, sm);
}

// One patch of a far-field launch: first ray (ib, jb), centre (ox, oy), half-
// diagonal h (one ray spacing of slack on each side), the radius inside which
// lenses are summed directly, and the super-patch that holds it. Window widths
// stay below 2^22 rays and launches below 2^31 patches, so 32-bit indices hold.
struct PatchFrame {
    int64_t ib, jb, sp;
    double ox, oy, h, near_r2;
};

__device__ __forceinline__ PatchFrame patch_frame(const ShootArgs &a, int64_t patch) {
    PatchFrame f;
    const int32_t nbx = (int32_t)a.nbx, p = (int32_t)patch;
    const int32_t pbx = p % nbx, pby = p / nbx;
    f.ib = a.i0 + (int64_t)pbx * PATCH_X;
    f.jb = a.jc0 + (int64_t)pby * PATCH_Y;
    f.sp = (int64_t)(pby / FF_SP_Y) * a.ff_sbx + pbx / FF_SP_X;
    f.ox = a.sx0 + ((double)f.ib + 0.5 * PATCH_X) * a.spx;
    f.oy = a.sy0 + ((double)f.jb + 0.5 * PATCH_Y) * a.spy;
    const double hx = (0.5 * PATCH_X + 1.0) * a.spx;
    const double hy = (0.5 * PATCH_Y + 1.0) * a.spy;
    f.h = sqrt(hx * hx + hy * hy) * (1.0 + 1e-12);
    f.near_r2 = (FAR_RATIO * f.h) * (FAR_RATIO * f.h);
    return f;
}

// The candidates of a patch: the super-patch's list, or, when that list
// overflowed, every lens that neither its group nor the super-patch expanded
// (the same tests those levels made).
struct Candidates {
    const global_i32 *list;
    int64_t n;
    bool scan_all;
    double cx, cy, super_r2;
    double gx, gy, group_r2;
};

__device__ __forceinline__ Candidates candidates(const ShootArgs &a, int64_t sp) {
    Candidates c;
    double H;
    super_geometry(a, sp, c.cx, c.cy, H);
    c.super_r2 = (FAR_RATIO * H) * (FAR_RATIO * H);
    c.list = (const global_i32 *)(a.ff_near + sp * (int64_t)(1 + a.ff_cap));
    const int32_t listed = c.list[0];
    c.scan_all = listed > a.ff_cap;
    c.n = c.scan_all ? a.n_lens : listed;
    group_geometry(a, group_of(a, sp), c.gx, c.gy, H);
    c.group_r2 = (FAR_RATIO * H) * (FAR_RATIO * H);
    return c;
}

// Candidate q: its lens index and position; false when an overflowed list's
// scan meets a lens a level above expanded.
__device__ __forceinline__ bool candidate(const ShootArgs &a, const Candidates &c, int64_t q, int64_t &k, double &X,
                                          double &Y) {
    k = c.scan_all ? q : (int64_t)c.list[1 + q];
    X = ((global_double *)a.lens_xy)[2 * k];
    Y = ((global_double *)a.lens_xy)[2 * k + 1];
    if (c.scan_all) {
        const double f1 = c.gx - X, f2 = c.gy - Y;
        if (f1 * f1 + f2 * f2 >= c.group_r2) return false;
        const double e1 = c.cx - X, e2 = c.cy - Y;
        if (e1 * e1 + e2 * e2 >= c.super_r2) return false;
    }
    return true;
}

// Level 2, part 1: the record of each patch, one wave per patch. The candidates
// farther than FAR_RATIO h from the patch centre add their own expansion about
// it; the super-patch expansion is re-centred exactly on it,
//   sum_n C_n (e + v)^n = sum_m v^m sum_{n>=m} binom(n, m) e^(n-m) C_n,
// v = -w = z0 - z, e = zS - z0; the record holds the sum of both, the bound terms
// of both levels (truncation, and rounding of the coefficients, the translation
// and the evaluation, with per-level factors and generous constants), and the
// nearer candidates, in candidate order, for the ray kernel's direct sum. Block 0
// also resets the ray kernel's patch counter.
template <bool UNIT>
__global__ __launch_bounds__(FAR_THREADS) void farfield_patch_kernel(const ShootArgs a, int64_t patches) {
    constexpr double U64 = 1.1102230246251565e-16;  // 2^-53
    __shared__ double totals[FAR_THREADS / 64][FAR_REC];
    double *const own = totals[threadIdx.x >> 6];   // the expansion of the patch's own lenses
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.ff_work = 0u;
    const int lane = threadIdx.x & 63;
    const int64_t patch = (int64_t)blockIdx.x * (FAR_THREADS / 64) + (threadIdx.x >> 6);
    if (patch >= patches) return;   // the whole wave
    const PatchFrame f = patch_frame(a, patch);
    const Candidates c = candidates(a, f.sp);
    double *rec = a.ff_patch + patch * (int64_t)FF_PATCH_DOUBLES;
    FarAcc acc;
    acc.zero();
    int n_near = 0;
    for (int64_t q0 = 0; q0 < c.n; q0 += 64) {
        const int64_t q = q0 + lane;
        int64_t k = 0;
        double X = 0.0, Y = 0.0, m = 1.0, d1 = 0.0, d2 = 0.0, r2 = 0.0;
        bool is_far = false, is_near = false;
        if (q < c.n && candidate(a, c, q, k, X, Y)) {
            d1 = f.ox - X;
            d2 = f.oy - Y;
            r2 = d1 * d1 + d2 * d2;
            m = (UNIT || a.lens_m == nullptr) ? 1.0 : ((global_double *)a.lens_m)[k];
            is_far = r2 >= f.near_r2;
            is_near = !is_far;
        }
        if (is_far) acc.add(d1, d2, r2, m, f.h);
        const uint64_t nb = __ballot(is_near);
        if (is_near) {
            const int pos = n_near + __builtin_popcountll(nb & ((1ull << lane) - 1ull));
            if (pos < FF_PATCH_NEAR) {
                rec[FF_PATCH_HEAD + pos] = X;
                rec[FF_PATCH_HEAD + FF_PATCH_NEAR + pos] = Y;
                rec[FF_PATCH_HEAD + 2 * FF_PATCH_NEAR + pos] = m;
            }
        }
        n_near += __builtin_popcountll(nb);
    }
    acc.wave_totals(own);
    wave_lds_fence();
    const global_double *sc = (const global_double *)(a.ff_super + f.sp * (int64_t)FAR_REC);
    if (lane < FAR_P) {
        const int mm = lane;
        const double e1 = c.cx - f.ox, e2 = c.cy - f.oy;
        double s1 = 0.0, s2 = 0.0;
        double g1 = 1.0, g2 = 0.0;   // e^(n-m)
        for (int n = mm; n < FAR_P; ++n) {
            const double binom = BINOM[n][mm];   // exact in FP64 for n < 16
            const double C1 = sc[n], C2 = sc[FAR_P + n];
            s1 = __builtin_fma(binom, g1 * C1 - g2 * C2, s1);
            s2 = __builtin_fma(binom, g1 * C2 + g2 * C1, s2);
            const double q1 = g1 * e1 - g2 * e2, q2 = g1 * e2 + g2 * e1;
            g1 = q1;
            g2 = q2;
        }
        // (n! T_n, real and imaginary part: the ray kernel's form of the series)
        rec[2 * mm] = FACTORIAL.f[mm] * (s1 + own[mm]);
        rec[2 * mm + 1] = FACTORIAL.f[mm] * (s2 + own[FAR_P + mm]);
    } else if (lane == FAR_P) {
        const double SFAR_S = sc[2 * FAR_P], TRUNC_S = sc[2 * FAR_P + 1], SDEF_S = sc[2 * FAR_P + 2];
        const double CHAIN_S = sc[2 * FAR_P + 3], chain = (double)((c.n + 63) / 64 + 6);
        const double sfar = own[2 * FAR_P];
        rec[2 * FAR_P] = SFAR_S + sfar;
        rec[2 * FAR_P + 1] = TRUNC_S + own[2 * FAR_P + 1] + (CHAIN_S + 24.0 * FAR_P + 64.0) * U64 * 1.34 * SFAR_S +
                             (chain + 16.0 * FAR_P + 64.0) * U64 * 1.34 * sfar;
        rec[2 * FAR_P + 2] = SDEF_S + own[2 * FAR_P + 2];
        rec[2 * FAR_P + 3] = (double)n_near;
    } else if (lane <= FAR_P + FF_PATCH_HEAD - (2 * FAR_P + 4)) {
        rec[2 * FAR_P + 4 + (lane - FAR_P - 1)] = 0.0;   // the spare doubles
    }
}

// A patch's part of the pixel decision: the terms of far_decide that do not depend on the
// ray, in pixels. The bound on an axis is e + s snear (|x| on the patch and the size of the
// deflection, at most 1.35 SFAR + snear, are bounded for the whole patch), and the position
// is x c + o - a w.
struct PatchBound {
    double eu, ev, su, sv;
};

__device__ __forceinline__ PatchBound patch_bound(const ShootArgs &a, const PatchFrame &f, double far_err, double SFAR,
                                                  double SDEF, int n_near, bool all_flagged) {
    constexpr double U64 = 1.1102230246251565e-16;  // 2^-53
    const double kN = ((double)a.n_lens + 10.0) * U64 * 1.001;
    const double e = all_flagged ? __builtin_inf()
                                 : far_err + ((double)n_near * 1.34 + 16.0 * 1.35) * U64 * SFAR + kN * SDEF;
    const double s = ((double)n_near + NEAR_ROUNDINGS) * U64 * 1.001 + kN + 16.0 * U64;
    const double wu = 1.0011 * a.inv_pixw, wv = 1.0011 * a.inv_pixh;   // (0.0001 for the terms' own rounding)
    PatchBound b;
    b.eu = wu * (e + 16.0 * U64 * (fabs(a.c1) * (fabs(f.ox) + f.h) + fabs(a.tx0)));
    b.ev = wv * (e + 16.0 * U64 * (fabs(a.c2) * (fabs(f.oy) + f.h) + fabs(a.ty0)));
    b.su = wu * s;
    b.sv = wv * s;
    return b;
}

// The pixel decision of far_decide for the ray at (u, v) pixels; a position or bound that
// is not finite compares false: FLAGGED (a position that overflowed within its bound is
// out of the map in the definition too).
__device__ __forceinline__ int patch_decide(const ShootArgs &a, const PatchBound &b, double u, double v, double snear) {
    const double Mu = __builtin_fma(b.su, snear, b.eu);
    const double Mv = __builtin_fma(b.sv, snear, b.ev);
    int code = pixel_inside(u, v, Mu, Mv, a.npx, a.npy);
    if (__ballot(code < 0)) {
        const bool out = u < -Mu || u - (double)a.npx > Mu || v < -Mv || v - (double)a.npy > Mv;
        code = code >= 0 ? code : (out ? OUT : FLAGGED);
    }
    return code;
}

// A wave's rays to re-check (lanes fl) appended to the launch's queue, which holds every
// ray of the launch. The far-field mode leaves a handful of rays per map.
__device__ __forceinline__ void queue_append(const ShootArgs &a, uint64_t fl, int lane, bool mine, int64_t i, int64_t j) {
    const int first = __builtin_ctzll(fl);
    uint32_t base = 0;
    if (lane == first) base = atomicAdd(a.qcount, (uint32_t)__builtin_popcountll(fl));
    base = __builtin_amdgcn_readlane(base, first);
    if (mine) {
        const uint32_t below = (uint32_t)__builtin_popcountll(fl & ((1ull << lane) - 1ull));
        a.queue[base + below] = (uint32_t)((j - a.jc0) * (a.i1 - a.i0) + (i - a.i0));
    }
}

constexpr int ROW_STRIDE = FAR_P + 1;   // (rows of a wave start on different LDS banks)
struct FarSmem {
    PixelTable table;                    // the patch's counts per pixel (map mode)
    // this patch's record and the next one's: the series, followed by zeros, and the rest
    double2 series[2][2 * FAR_P - 1];
    double rest[2][FF_PATCH_DOUBLES - 2 * FAR_P];
    double2 row[FAR_THREADS / 64][8][ROW_STRIDE];   // per wave: its 8 rows' series in the column offset
    double near_x[NEAR_EXP], near_y[NEAR_EXP], near_m[NEAR_EXP];   // near lenses a record could not hold
    int near_count;
    int next;                            // the patch after the next one
};
static_assert(FAR_THREADS / 64 * 8 == PATCH_Y && FF_PATCH_DOUBLES <= FAR_THREADS, "a wave takes eight rows");

// Level 2, part 2: the rays. Persistent blocks take patches from a counter, `take` of
// them at a time (an atomic on one address takes 12 ns, 0.43 of the 1.61 ms of the
// 36000-patch map when each patch took one). The next patch's record is loaded while
// this one's rays are evaluated. A patch's near lenses come from its record, or, when the
// record could not hold them all, from the candidates with the record kernel's test
// (beyond NEAR_EXP of them the patch is re-checked whole).
//
// A lane takes 8 rays of one row (a wave eight rows, 8 x 8 rays at a time). The series
// in w' = z0 - z = p + i q, p the column's offset and q the row's, is re-centred on the
// row once for its 64 rays,
//   sum_n T_n (p + i q)^n = sum_m p^m / m! sum_k (n! T_n) (i q)^k / k!,  n = m + k,
// two values of m by each of the row's 8 lanes, so that a ray costs 30 FMAs (a real
// variable) instead of 60. Then the near lenses directly, four rays sharing a reciprocal,
// the pixel decision against the bound, and the count in the block's pixel table, which is
// added to the map and cleared after every patch. Rounding of the evaluation: every
// product of |p| and |q| sums to at most sum |T_n| (|p| + |q|)^n <= 1.55 sum m/|d|, with
// at most 95 roundings (1 for n!, 3 k for q^k / k!, 16 additions, 2 for 1 / m!, 2 m + 1 in
// p): within the record's terms, which allow 448 (super-patch and above) and 320 units of
// 1.34 sum m/|d| where the coefficients take at most 245 and 143.
template <bool UNIT, bool PIX>
__global__ __launch_bounds__(FAR_THREADS, 3) void farfield_kernel(const ShootArgs a, int64_t patches, int take) {
    __shared__ FarSmem sm;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    if (!PIX) table_clear<FAR_THREADS>(sm.table, tid);
    // Every block has its first two patches by its index. thread 0's share of the counter for
    // the others: tickets share .. share + left - 1 are this block's.
    uint32_t share = 0;
    int left = 0;
    auto fetch = [&]() {
        if (left == 0) {
            share = atomicAdd(a.ff_work, (uint32_t)take);
            left = take;
        }
        --left;
        return (int)ticket_patch(share++, gridDim.x);
    };
    int64_t patch = first_patch(blockIdx.x, gridDim.x, 0), next = first_patch(blockIdx.x, gridDim.x, 1);
    if (tid == 0) sm.near_count = 0;
    auto hold = [&](int par, double v) {   // a record's double tid into its place
        if (tid < 2 * FAR_P) reinterpret_cast<double *>(sm.series[par])[tid] = v;
        else if (tid < FF_PATCH_DOUBLES) sm.rest[par][tid - 2 * FAR_P] = v;
    };
    if (tid < 2 * (FAR_P - 1))
        for (int par = 0; par < 2; ++par) reinterpret_cast<double *>(sm.series[par])[2 * FAR_P + tid] = 0.0;
    if (patch < patches && tid < FF_PATCH_DOUBLES)
        hold(0, ((const global_double *)a.ff_patch)[patch * FF_PATCH_DOUBLES + tid]);
    const int m0 = lane & 7, m1 = 15 - m0;   // the coefficients this lane makes for its row
    const double inv0 = FACTORIAL.inv[m0], inv1 = FACTORIAL.inv[m1];
    double2 *const my_row = sm.row[wave][lane >> 3];
    const double oc1 = a.c1 * a.inv_pixw, oc2 = a.c2 * a.inv_pixh;   // position: x c + o - a w
    const double ou = -a.tx0 * a.inv_pixw, ov = -a.ty0 * a.inv_pixh;
    uint32_t n_in = 0, n_out = 0;   // (of a block's patches: below 2^32)
    const int64_t W = a.i1 - a.i0;
    __syncthreads();
    for (int par = 0; patch < patches; par ^= 1) {
        double ahead = 0.0;   // the next patch's record, one double per thread
        if (next < patches && tid < FF_PATCH_DOUBLES)
            ahead = ((const global_double *)a.ff_patch)[next * FF_PATCH_DOUBLES + tid];
        int after = 0;
        if (tid == 0) after = fetch();   // used after the rays: the atomic's latency is hidden
        const PatchFrame f = patch_frame(a, patch);
        const double *const rest = sm.rest[par];
        const int stored = (int)rest[3];
        const double *near_x = rest + FF_PATCH_HEAD - 2 * FAR_P, *near_y = near_x + FF_PATCH_NEAR, *near_m = near_y + FF_PATCH_NEAR;
        int n_near = stored;
        if (stored > FF_PATCH_NEAR) {
            const Candidates c = candidates(a, f.sp);
            for (int64_t q = tid; q < c.n; q += FAR_THREADS) {
                int64_t k;
                double X, Y;
                if (!candidate(a, c, q, k, X, Y)) continue;
                const double d1 = f.ox - X, d2 = f.oy - Y;
                const double r2 = d1 * d1 + d2 * d2;
                if (r2 >= f.near_r2) continue;   // in the patch's expansion
                const double m = (UNIT || a.lens_m == nullptr) ? 1.0 : ((global_double *)a.lens_m)[k];
                const int j = atomicAdd(&sm.near_count, 1);
                if (j < NEAR_EXP) {
                    sm.near_x[j] = X;
                    sm.near_y[j] = Y;
                    sm.near_m[j] = m;
                }
            }
            __syncthreads();
            n_near = sm.near_count;
            __syncthreads();
            if (tid == 0) sm.near_count = 0;   // (the next patch's first use follows two barriers)
            near_x = sm.near_x;
            near_y = sm.near_y;
            near_m = sm.near_m;
        }
        const bool all_flagged = n_near > NEAR_EXP;
        if (all_flagged) n_near = 0;
        const PatchBound bound =
            patch_bound(a, f, rest[1], rest[0], rest[2], n_near, all_flagged);

        // This lane's row, and two coefficients of its series.
        const int64_t j = f.jb + 8 * wave + (lane >> 3);
        const double x2 = ray_coord(a.sy0, j, a.spy);
        const double q = f.oy - x2;
        {
            const double2 *const T0 = sm.series[par] + m0, *const T1 = sm.series[par] + m1;   // n! T_n, n = m + k
            double2 r0 = make_double2(0.0, 0.0), r1 = r0;
#pragma unroll
            for (int k = FAR_P - 1; k >= 0; --k) {
                const double s = q * (1.0 / (k + 1));
                const double2 t = T0[k];
                r0 = make_double2(__builtin_fma(-s, r0.y, t.x), __builtin_fma(s, r0.x, t.y));
                if (k < FAR_P / 2) {   // (m1 is at least 8)
                    const double2 t1 = T1[k];
                    r1 = make_double2(__builtin_fma(-s, r1.y, t1.x), __builtin_fma(s, r1.x, t1.y));
                }
            }
            my_row[m0] = make_double2(r0.x * inv0, r0.y * inv0);
            my_row[m1] = make_double2(r1.x * inv1, r1.y * inv1);
            wave_lds_fence();
        }
        const double vrow = __builtin_fma(x2, oc2, ov);
        // The row's rays in two passes of RPASS columns.
        constexpr int RPASS = FAR_ROWS / 2;
        const double i_base = (double)(f.ib + (lane & 7)) + 0.5;
#pragma unroll 1
        for (int pass = 0; pass < FAR_ROWS / RPASS; ++pass) {
            double X1[RPASS], A1[RPASS], A2[RPASS], SN[RPASS];
            {
                double p[RPASS];
#pragma unroll
                for (int k = 0; k < RPASS; ++k) {
                    X1[k] = a.sx0 + (i_base + (double)(8 * (pass * RPASS + k))) * a.spx;   // ray_coord's operations
                    p[k] = f.ox - X1[k];
                    SN[k] = 0.0;
                }
                const double2 t = my_row[FAR_P - 1];
#pragma unroll
                for (int k = 0; k < RPASS; ++k) {
                    A1[k] = t.x;
                    A2[k] = -t.y;
                }
#pragma unroll
                for (int m = FAR_P - 2; m >= 0; --m) {
                    const double2 c = my_row[m];
#pragma unroll
                    for (int k = 0; k < RPASS; ++k) {
                        A1[k] = __builtin_fma(A1[k], p[k], c.x);
                        A2[k] = __builtin_fma(A2[k], p[k], -c.y);
                    }
                }
            }
            bool tiny = false;
            for (int l = 0; l < n_near; ++l) {
                const double e2 = x2 - near_y[l], e2sq = e2 * e2;
                double e1[RPASS], r2[RPASS], g[RPASS];
#pragma unroll
                for (int k = 0; k < RPASS; ++k) {
                    e1[k] = X1[k] - near_x[l];
                    r2[k] = __builtin_fma(e1[k], e1[k], e2sq);
                }
                // one reciprocal for the four (v_rcp_f64 takes four times an FMA's issue, and
                // its two Newton steps four FMAs)
                const double pab = r2[0] * r2[1], pcd = r2[2] * r2[3], P = pab * pcd;
                tiny |= !(P > 1e-290);
                const double R = rcp64(P);
                double qab = R * pcd, qcd = R * pab;
                if (!UNIT) {
                    const double M = near_m[l];
                    qab = M * qab;
                    qcd = M * qcd;
                }
                g[0] = r2[1] * qab;
                g[1] = r2[0] * qab;
                g[2] = r2[3] * qcd;
                g[3] = r2[2] * qcd;
#pragma unroll
                for (int k = 0; k < RPASS; ++k) {
                    A1[k] = __builtin_fma(g[k], e1[k], A1[k]);
                    A2[k] = __builtin_fma(g[k], e2, A2[k]);
                    SN[k] = __builtin_fma(fabs(e1[k]) + fabs(e2), UNIT ? g[k] : fabs(g[k]), SN[k]);
                }
            }
            if (pass == 0) {
                __syncthreads();   // the previous patch has left the pixel table
                if (tid == 0) sm.table.used[par ^ 1] = 0u;
            }
#pragma unroll
            for (int k = 0; k < RPASS; ++k) {
                const int64_t i = f.ib + (lane & 7) + 8 * (pass * RPASS + k);
                const bool valid = (i < a.i1) && (j < a.jc1);
                const double u = __builtin_fma(-A1[k], a.inv_pixw, __builtin_fma(X1[k], oc1, ou));
                const double v = __builtin_fma(-A2[k], a.inv_pixh, vrow);
                int code = patch_decide(a, bound, u, v, SN[k]);
                if (tiny) code = FLAGGED;
                if (!valid) code = INT32_MIN;

                n_in += __builtin_popcountll(__ballot(code >= 0));
                n_out += __builtin_popcountll(__ballot(code == OUT));
                if (PIX) {
                    if (valid && code != FLAGGED) a.pix_out[(j - a.j0) * W + (i - a.i0)] = code;
                } else {
                    if (code >= 0) table_add(sm.table, a.map, code, 1u, par);
                }
                const uint64_t fl = __ballot(code == FLAGGED);
                if (fl) queue_append(a, fl, lane, code == FLAGGED, i, j);
            }
        }
        hold(par ^ 1, ahead);
        if (tid == 0) sm.next = after;
        __syncthreads();   // every ray of the patch is in the table
        if (!PIX) table_flush_clear<FAR_THREADS>(sm.table, a.map, tid, par);
        patch = next;
        next = sm.next;
    }
    if (lane == 0) {
        if (n_in) global_add(a.counters + C_IN, (unsigned long long)n_in);
        if (n_out) global_add(a.counters + C_OUT, (unsigned long long)n_out);
    }
}

// At most this many queued rays take stage F one wave per ray (a short queue leaves
// most of the chip idle otherwise: the 1219 rays of the 1024^2-ray, 462-lens map, whose
// super-patches list almost every lens, took 84 us one thread per ray).
constexpr uint32_t FAR_WAVE_MAX = 32768;
// From this many of a wave's 64 rays left by stage F on, stage A takes them one per lane (a
// pass over the lenses for all of them); below it one after another, each by the whole wave.
constexpr int LANE_STAGE_MIN = 32;

// Re-check stage F of the mixed mode (far_recheck_ray), one thread or one wave per
// queued ray. A ray it places is binned. STAGE_A (recheck_in_one): the others take stage A at
// once, and are marked UNRESOLVED when that cannot place them either (or, with
// few lenses, take stage B at once: its kernel, which mostly finds nothing to do, costs 5 us
// of the 108 of the 1024^2-ray, 462-lens map); otherwise a ray it places is marked RESOLVED,
// and the others are counted in *qlive and left for the stages over every lens. Queue entries
// of one deflection block are adjacent and share a super-patch, so a wave that takes adjacent
// entries walks one list (dealt one by one to the waves, which spreads the rays stage F
// leaves more evenly, 5000-lens maps with every ray queued took 1.7 times as long).
// With stage A it takes the registers of three waves per SIMD, which leaves none for loading its
// wave form's lenses a step ahead (two waves that do: 700^2 rays, 900 lenses in clusters, 338 us
// a call; three that don't: 319).
constexpr int64_t STAGE_A_BLOCKS = 768;   // three waves per SIMD
constexpr uint32_t RUN_WAVES = 1024;      // one per SIMD
template <bool UNIT, bool STAGE_A>
__global__ __launch_bounds__(256, STAGE_A ? 3 : 4) void recheck_far_kernel(const ShootArgs a, const RecheckArgs r, uint32_t *qlive) {
    __shared__ uint32_t sums[3];   // rays in the map, out, left
    const uint32_t n = *a.qcount;
    if (n == 0) return;
    if (threadIdx.x < 3) sums[threadIdx.x] = 0u;
    __syncthreads();
    const uint32_t W = (uint32_t)(a.i1 - a.i0);   // at most 2^22
    const int lane = lane_id();
    const uint32_t wave_id = (uint32_t)__builtin_amdgcn_readfirstlane((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6));
    const uint32_t n_waves = (gridDim.x * blockDim.x) >> 6;
    uint32_t n_in = 0, n_out = 0, left = 0;   // this lane's
    const bool wave_form = n <= FAR_WAVE_MAX;
    if (STAGE_A && wave_id == 0 && lane == 0) atomicAdd(a.counters + C_RECHECK, (unsigned long long)n);
    const uint32_t run = wave_form ? 1u : entry_run(n, RUN_WAVES);   // entries a wave takes at a time
    for (uint64_t first = (uint64_t)run * wave_id; first < n; first += (uint64_t)run * n_waves) {
        const uint64_t idx = wave_form ? first : first + (uint32_t)lane;
        const bool mine = wave_form ? lane == 0 : (uint32_t)lane < run && idx < n;   // this lane records the entry's result
        const uint32_t q = a.queue[mine ? idx : first];   // (an entry of this wave's: others mark theirs)
        const int64_t i = a.i0 + (int64_t)(q % W);
        const int64_t j = a.jc0 + (int64_t)(q / W);
        int code = wave_form ? far_recheck_ray<UNIT, true>(a, i, j) : far_recheck_ray<UNIT, false>(a, i, j);
        uint64_t todo = __ballot(mine && code == FLAGGED);
        if (mine && code == FLAGGED) ++left;
        if (STAGE_A && todo) {
            uint64_t undecided = 0;
            if (__builtin_popcountll(todo) >= LANE_STAGE_MIN) {
                bool decided = true;
                if ((todo >> lane) & 1ull) {
                    int c = 0;
                    decided = fast_ray<UNIT>(r, i, j, c);
                    if (decided) code = c;
                }
                undecided = __ballot(!decided);
            } else {
                while (todo) {
                    const int src = __builtin_ctzll(todo);
                    todo &= todo - 1;
                    const uint32_t qs = (uint32_t)__builtin_amdgcn_readlane((int)q, src);
                    int c = 0;
                    if (!fast_ray_wave<UNIT, 4, false>(r, a.i0 + (int64_t)(qs % W), a.jc0 + (int64_t)(qs / W), c)) undecided |= 1ull << src;
                    else if (lane == src) code = c;
                }
            }
            if (r.n_lens > EXACT_INLINE_LENSES) {
                if ((undecided >> lane) & 1ull) {
                    a.queue[idx] = q | UNRESOLVED;
                    atomicAdd(r.qunres, 1u);
                }
            } else {
                while (undecided) {
                    const int src = __builtin_ctzll(undecided);
                    undecided &= undecided - 1;
                    const uint32_t qs = (uint32_t)__builtin_amdgcn_readlane((int)q, src);
                    const int64_t is = a.i0 + (int64_t)(qs % W), js = a.jc0 + (int64_t)(qs / W);
                    const int c = exact_ray_chain<UNIT, 2, 4>(r, is, js);
                    if (lane == 0) emit_ray(r, is, js, c);
                }
            }
        }
        if (mine && code != FLAGGED) {
            if (!STAGE_A) a.queue[idx] = q | RESOLVED;
            if (code >= 0) ++n_in;
            else ++n_out;
            if (a.pix_out) a.pix_out[(j - a.j0) * (int64_t)W + (i - a.i0)] = code;
            else if (code >= 0) global_add(a.map + code, 1u);
        }
    }
    // one atomic per block and counter: atomics on one address take about 12 ns each
    if (n_in) atomicAdd(&sums[0], n_in);
    if (n_out) atomicAdd(&sums[1], n_out);
    if (left) atomicAdd(&sums[2], left);
    __syncthreads();
    if (threadIdx.x < 2 && sums[threadIdx.x])
        global_add(a.counters + (threadIdx.x ? C_OUT : C_IN), (unsigned long long)sums[threadIdx.x]);
    if (threadIdx.x == 2 && sums[2]) {
        if (STAGE_A) global_add(a.counters + C_DIRECT, (unsigned long long)sums[2]);
        else atomicAdd(qlive, sums[2]);
    }
}

}  // namespace

static int64_t super_patches(const ShootArgs &a) {
    const int64_t nby = (a.jc1 - a.jc0 + PATCH_Y - 1) / PATCH_Y;
    return a.ff_sbx * ((nby + FF_SP_Y - 1) / FF_SP_Y);
}

hipError_t launch_fill_records(const ShootArgs &a, uint32_t *map, int64_t n_pix, void *workspace, int64_t n_qcount,
                               hipStream_t stream) {
    const int64_t n_super = super_patches(a);
    const int64_t n_ws_words = (int64_t)(WS_QCOUNT / 4) + n_qcount;
    const int64_t work = map && n_pix > n_ws_words ? n_pix : n_ws_words;
    int64_t blocks = (work + FAR_THREADS - 1) / FAR_THREADS;
    if (blocks > 4096) blocks = 4096;
    const dim3 grid((unsigned)(n_super + blocks));
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(FAR_THREADS), 0, stream, a, (uint32_t)n_super, map, map ? n_pix : 0,
                           static_cast<uint32_t *>(workspace), n_ws_words);
    };
    if (a.lens_m == nullptr) launch(fill_records_kernel<true>);
    else launch(fill_records_kernel<false>);
    return hipGetLastError();
}

hipError_t launch_recheck_far(const ShootArgs &a, const RecheckArgs &r, uint32_t *qlive, bool stage_a, bool records,
                              int64_t max_rays, hipStream_t stream) {
    if (max_rays <= 0) return hipSuccess;
    const bool unit = a.lens_m == nullptr;
    if (records) {
        const int64_t n_super = super_patches(a);
        if (n_super <= 0) return hipSuccess;
        if (unit) hipLaunchKernelGGL((farfield_super_kernel<true, true>), dim3((unsigned)n_super), dim3(FAR_THREADS), 0, stream, a);
        else hipLaunchKernelGGL((farfield_super_kernel<false, true>), dim3((unsigned)n_super), dim3(FAR_THREADS), 0, stream, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const dim3 grid((unsigned)queue_blocks(max_rays, 4, stage_a ? STAGE_A_BLOCKS : 1024)), block(256);   // (a wave per ray of a short queue)
    if (unit) {
        if (stage_a) hipLaunchKernelGGL((recheck_far_kernel<true, true>), grid, block, 0, stream, a, r, qlive);
        else hipLaunchKernelGGL((recheck_far_kernel<true, false>), grid, block, 0, stream, a, r, qlive);
    } else {
        if (stage_a) hipLaunchKernelGGL((recheck_far_kernel<false, true>), grid, block, 0, stream, a, r, qlive);
        else hipLaunchKernelGGL((recheck_far_kernel<false, false>), grid, block, 0, stream, a, r, qlive);
    }
    return hipGetLastError();
}

hipError_t launch_super_records(const ShootArgs &a, int64_t n_super, hipStream_t stream) {
    if (n_super <= 0) return hipSuccess;
    if (a.lens_m == nullptr) hipLaunchKernelGGL((farfield_super_kernel<true, false>), dim3((unsigned)n_super), dim3(FAR_THREADS), 0, stream, a);
    else hipLaunchKernelGGL((farfield_super_kernel<false, false>), dim3((unsigned)n_super), dim3(FAR_THREADS), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_batch_super(const BatchArgs &b, hipStream_t stream) {
    if (b.total_super <= 0) return hipSuccess;
    if (b.unit_masses) hipLaunchKernelGGL((batch_super_kernel<true>), dim3((unsigned)b.total_super), dim3(FAR_THREADS), 0, stream, b);
    else hipLaunchKernelGGL((batch_super_kernel<false>), dim3((unsigned)b.total_super), dim3(FAR_THREADS), 0, stream, b);
    return hipGetLastError();
}

hipError_t launch_farfield(const ShootArgs &a, hipStream_t stream) {
    const int64_t rows = a.jc1 - a.jc0;
    const int64_t nby = (rows + PATCH_Y - 1) / PATCH_Y;
    const int64_t patches = a.nbx * nby;
    if (patches <= 0) return hipSuccess;
    const int64_t n_super = a.ff_sbx * ((nby + FF_SP_Y - 1) / FF_SP_Y);
    const bool unit = a.lens_m == nullptr;
    const bool pix = a.pix_out != nullptr;
    const dim3 block(FAR_THREADS);
    const int64_t n_group = a.ff_gbx * ((((nby + FF_SP_Y - 1) / FF_SP_Y) + FF_GROUP - 1) / FF_GROUP);
    const dim3 group_block(FAR_GROUP_THREADS);
    if (a.ff_top) {
        const int64_t n_gy = (((nby + FF_SP_Y - 1) / FF_SP_Y) + FF_GROUP - 1) / FF_GROUP;
        const int64_t n_top = a.ff_tbx * ((n_gy + FF_TOP - 1) / FF_TOP);
        const dim3 top_grid((unsigned)(n_top * FF_TOP_PARTS));
        if (unit) hipLaunchKernelGGL((farfield_top_kernel<true>), top_grid, dim3(FAR_TOP_THREADS), 0, stream, a);
        else hipLaunchKernelGGL((farfield_top_kernel<false>), top_grid, dim3(FAR_TOP_THREADS), 0, stream, a);
        if (unit) hipLaunchKernelGGL((farfield_group_top_kernel<true>), dim3((unsigned)n_group), group_block, 0, stream, a);
        else hipLaunchKernelGGL((farfield_group_top_kernel<false>), dim3((unsigned)n_group), group_block, 0, stream, a);
    } else {
        const dim3 group_grid((unsigned)(n_group * group_parts(a.n_lens)));
        if (unit) hipLaunchKernelGGL((farfield_group_kernel<true>), group_grid, group_block, 0, stream, a);
        else hipLaunchKernelGGL((farfield_group_kernel<false>), group_grid, group_block, 0, stream, a);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (unit) hipLaunchKernelGGL((farfield_super_group_kernel<true>), dim3((unsigned)n_super), block, 0, stream, a);
    else hipLaunchKernelGGL((farfield_super_group_kernel<false>), dim3((unsigned)n_super), block, 0, stream, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 rec_grid((unsigned)((patches + FAR_THREADS / 64 - 1) / (FAR_THREADS / 64)));
    if (unit) hipLaunchKernelGGL((farfield_patch_kernel<true>), rec_grid, block, 0, stream, a, patches);
    else hipLaunchKernelGGL((farfield_patch_kernel<false>), rec_grid, block, 0, stream, a, patches);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    auto launch_rays = [&](auto kernel) {
        int64_t blocks = persistent_blocks(kernel, FAR_THREADS, 0);
        if (blocks > patches) blocks = patches;
        // few enough at a time for the blocks to end together
        const int take = patches >= 64 * blocks ? 4 : (patches >= 16 * blocks ? 2 : 1);
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), block, 0, stream, a, patches, take);
    };
    if (unit) {
        if (pix) launch_rays(farfield_kernel<true, true>);
        else launch_rays(farfield_kernel<true, false>);
    } else {
        if (pix) launch_rays(farfield_kernel<false, true>);
        else launch_rays(farfield_kernel<false, false>);
    }
    return hipGetLastError();
}

}  // namespace rs
