// FP64 re-evaluation of rays whose FP32 source position is within its error
// bound of a pixel edge (the arithmetic lives in recheck_ray.h).
//
// Three stages keep the work per queued ray small and the exact evaluation rare:
//   stage F (far_ray.h, farfield.hip): the ray's super-patch FP64 expansion
//     plus the lenses listed near the super-patch, under a rigorous bound; it
//     places all but a few queued rays;
//   stage A (fast_ray, fast_rays_wave, fast_ray_block): FP64 over every lens with
//     fused multiply-adds and a
//     bound that also covers the definition's own FP64 rounding; it decides
//     almost every ray stage F left, identically to the definition, and marks
//     the rest;
//   stage B (exact_ray_wave): the marked rays, one wave per ray, with the
//     definition's operations and the roundings of its order, in the form that suits the
//     number of lenses (ExactForm).
// RS_EXACT_RECHECK runs the exact sequence for every queued ray instead (one
// thread per ray).
//
// Single map: the queue holds uint32 chunk-relative ray indices. Unless the
// caller asked for the exact sequence only (or a random-ray window holds few of
// its map's rays), the far-field stage (farfield.hip) runs first. In a small map of
// one launch (recheck_in_one) its kernel takes its rays through stage A as well; otherwise it
// marks the entries it decided RESOLVED, and stage A skips them and picks its form from the
// number left (*qlive).
// Batch: the deflection kernel sets one bit per flagged ray in each map's
// bitmap; a persistent scan compacts the set bits per wave and the map's
// descriptor supplies its parameters and its super-patch records (stage F).
#include "far_ray.h"
#include "rs_launch.h"

namespace rs {
namespace {

__device__ inline void count_wave(unsigned long long *counters, unsigned long long n_in,
                                  unsigned long long n_out, unsigned long long n_sing) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        n_in += __shfl_xor(n_in, off);
        n_out += __shfl_xor(n_out, off);
        n_sing += __shfl_xor(n_sing, off);
    }
    if (__lane_id() == 0) {
        if (n_in) atomicAdd(counters + C_IN, n_in);
        if (n_out) atomicAdd(counters + C_OUT, n_out);
        if (n_sing) atomicAdd(counters + C_SING, n_sing);
    }
}

__device__ inline void tally(int code, unsigned long long &n_in, unsigned long long &n_out,
                             unsigned long long &n_sing) {
    if (code >= 0) ++n_in;
    else if (code == CODE_OUT) ++n_out;
    else ++n_sing;
}

__device__ inline void place(const RecheckArgs &a, int64_t i, int64_t j, int code) {
    if (a.pix_out) a.pix_out[(j - a.j0) * (a.i1 - a.i0) + (i - a.i0)] = code;
    else if (code >= 0) atomicAdd(a.map + code, 1u);
}

// ----------------------------- single map ---------------------------------

// Below this many queued rays stage A runs one block per ray (latency: a few
// rays must not each take a thread through every lens); above it, one thread
// per ray (throughput). The kernel checks the count on the device.
constexpr uint32_t BLOCK_STAGE_MAX = 32768;
enum StageAForm { FORM_EITHER, FORM_THREADS, FORM_BLOCKS };

template <bool UNIT>
__global__ __launch_bounds__(256) void recheck_exact_kernel(const RecheckArgs a) {
    const uint32_t n = *a.qcount;
    const int64_t W = a.i1 - a.i0;
    unsigned long long n_in = 0, n_out = 0, n_sing = 0;
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += stride) {
        const uint32_t q = a.queue[idx];
        const int64_t i = a.i0 + (int64_t)(q % (uint64_t)W);
        const int64_t j = a.jc0 + (int64_t)(q / (uint64_t)W);
        const int code = exact_ray_thread<UNIT>(a, i, j);
        tally(code, n_in, n_out, n_sing);
        place(a, i, j, code);
    }
    count_wave(a.counters, n_in, n_out, n_sing);
    if (blockIdx.x == 0 && threadIdx.x == 0 && n) {
        atomicAdd(a.counters + C_RECHECK, (unsigned long long)n);
        atomicAdd(a.counters + C_DIRECT, (unsigned long long)n);
    }
}

// Stage A over a launch's queue. Few live entries: entries are dealt to the blocks 64 at a
// time (lane l of each wave of block k reads entry k + (t + l) n_blocks), so a
// long queue whose entries the far-field stage mostly decided costs each block
// a few vector loads, and neighbouring live rays go to different blocks. (One wave per ray
// took 27 us for the 14 rays of the 19200 x 3840-ray, 17240-lens far-field map, and a kernel
// for each form 4.6 us more. But both forms in one kernel hold three waves per SIMD instead of
// the thread form's four: crowded maps, whose rays mostly come here, have a kernel for each.
// 3000^2 rays and 300000 lenses, far field: 1.72 s in one kernel, 1.62 in one for each.)
template <bool UNIT, StageAForm FORM>
__global__ __launch_bounds__(256) void recheck_fast_kernel(const RecheckArgs a) {
    constexpr int WAVES = 4;
    __shared__ FastSums part[WAVES];
    const uint32_t n = *a.qcount;
    const uint32_t live = a.qlive ? *a.qlive : n;
    if (FORM != FORM_BLOCKS && blockIdx.x == 0 && threadIdx.x == 0) {
        if (n) atomicAdd(a.counters + C_RECHECK, (unsigned long long)n);
        if (live) atomicAdd(a.counters + C_DIRECT, (unsigned long long)live);
    }
    const bool by_thread = live >= BLOCK_STAGE_MAX;
    if (live == 0 || (FORM == FORM_THREADS && !by_thread) || (FORM == FORM_BLOCKS && by_thread)) return;
    const uint32_t W = (uint32_t)(a.i1 - a.i0);   // at most 2^22
    uint32_t n_in = 0, n_out = 0;   // (stage A never yields a singular ray)
    auto record = [&](uint32_t idx, uint32_t q, bool decided, int code) __attribute__((always_inline)) {
        if (decided) {
            if (code >= 0) ++n_in;
            else ++n_out;
            place(a, a.i0 + (int64_t)(q % W), a.jc0 + (int64_t)(q / W), code);
        } else {
            a.queue[idx] = q | UNRESOLVED;
            if (a.qunres) atomicAdd(a.qunres, 1u);
        }
    };
    if (FORM == FORM_THREADS || (FORM == FORM_EITHER && by_thread)) {
        const uint32_t stride = gridDim.x * blockDim.x;
        for (uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += stride) {
            const uint32_t q = a.queue[idx];
            if (q & RESOLVED) continue;
            int code;
            const bool decided = fast_ray<UNIT>(a, a.i0 + (int64_t)(q % W), a.jc0 + (int64_t)(q / W), code);
            record(idx, q, decided, code);
        }
    } else {
        const int lane = __lane_id();
        for (uint64_t t0 = 0; blockIdx.x + t0 * gridDim.x < n; t0 += 64) {
            const uint64_t idx = blockIdx.x + (t0 + (uint64_t)lane) * gridDim.x;
            const uint32_t q_lane = idx < n ? a.queue[idx] : RESOLVED;
            uint64_t todo = __ballot(!(q_lane & (RESOLVED | UNRESOLVED)));   // the same in every wave
            __syncthreads();   // every wave has read the entries that thread `src` marks
            while (todo) {
                const int src = __builtin_ctzll(todo);
                todo &= todo - 1;
                const uint32_t q = (uint32_t)__builtin_amdgcn_readlane((int)q_lane, src);
                int code = 0;
                const bool decided = fast_ray_block<UNIT, 4, WAVES>(a, a.i0 + (int64_t)(q % W),
                                                                    a.jc0 + (int64_t)(q / W), part, code);
                if ((int)threadIdx.x == src) record((uint32_t)idx, q, decided, code);
            }
        }
    }
    count_wave(a.counters, n_in, n_out, 0ull);
}

template <bool UNIT, ExactForm FORM>
__global__ __launch_bounds__(256) void recheck_exact_wave_kernel(const RecheckArgs a) {
    if (a.qunres && *a.qunres == 0u) return;   // stage A decided every entry
    const uint32_t n = *a.qcount;
    const int64_t W = a.i1 - a.i0;
    const int lane = __lane_id();
    const uint32_t wave_id = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const uint32_t n_waves = (gridDim.x * blockDim.x) >> 6;
    // Entries are dealt to the waves one at a time (entry wave_id + t * n_waves), so
    // neighbouring marked rays go to different waves instead of queueing in one.
    for (uint64_t t0 = 0; (uint64_t)wave_id + t0 * n_waves < n; t0 += 64) {
        const uint64_t idx64 = (uint64_t)wave_id + (t0 + (uint64_t)lane) * n_waves;
        const uint32_t idx = (uint32_t)(idx64 < n ? idx64 : 0);
        const uint32_t q_lane = idx64 < n ? a.queue[idx] : 0u;
        uint64_t todo = __ballot(idx64 < n && (q_lane & UNRESOLVED));
        while (todo) {
            const int src = __builtin_ctzll(todo);
            todo &= todo - 1;
            const uint32_t q = (uint32_t)__builtin_amdgcn_readlane((int)q_lane, src) & ~UNRESOLVED;
            const int64_t i = a.i0 + (int64_t)(q % (uint64_t)W);
            const int64_t j = a.jc0 + (int64_t)(q / (uint64_t)W);
            const int code = exact_ray_wave<UNIT, FORM>(a, i, j);
            if (lane == 0) emit_ray(a, i, j, code);
        }
    }
}

// Maps of several launches: before stage A, the entries the far-field stage left
// (every entry, in the far-field mode) go to the map's gathered list and are
// marked placed in the launch's queue; the rest (past the list's capacity) are
// counted in *qleft, which stage A of this launch then reads as its live count.
// The stages over every lens cost about one pass over the lenses per wave whatever
// the number of rays, so running them once per map instead of once per launch
// saves a pass per launch.
__global__ __launch_bounds__(256) void recheck_defer_kernel(const RecheckArgs a) {
    const uint32_t n = *a.qcount;
    const int64_t W = a.i1 - a.i0;
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += stride) {
        const uint32_t q = a.queue[idx];
        if (q & RESOLVED) continue;
        // Once the list is full the count stops growing (by more than a grid's
        // worth), so it cannot wrap however many launches feed it.
        const uint32_t d = __hip_atomic_load(a.dcount, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >=
                                   (uint32_t)DEFER_CAP
                               ? (uint32_t)DEFER_CAP
                               : atomicAdd(a.dcount, 1u);
        if (d >= (uint32_t)DEFER_CAP) {
            atomicAdd(a.qleft, 1u);
            continue;
        }
        a.defer[2 * (int64_t)d] = a.i0 + (int64_t)(q % (uint64_t)W);
        a.defer[2 * (int64_t)d + 1] = a.jc0 + (int64_t)(q / (uint64_t)W);
        a.queue[idx] = q | RESOLVED;
    }
}

// Stage A over a map's gathered list, a wave per STAGE_A_RAYS rays once there are more than
// waves: each wave reads every lens (16 MB of the 10^6-lens map), and two rays a wave halve
// that (6626 rays: 4.7 ms; one ray a wave 6.2, three, which leaves the chip half empty, 6.3).
// The rays it cannot place go to a list of their own, so that the exact stage deals
// them out one per wave (marked in place, two of them could fall to one wave and its time
// would double).
constexpr int STAGE_A_RAYS = 2;
template <bool UNIT, int R, int U>
__device__ __forceinline__ void fast_deferred(const RecheckArgs &a, uint32_t n, uint32_t wave_id, uint32_t n_waves) {
    for (uint32_t e = wave_id * R; e < n; e += n_waves * R) {
        int64_t i[R], j[R];
        int code[R];
        bool decided[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t k = e + r < n ? e + r : n - 1;   // (the last one again: not counted)
            i[r] = a.defer[2 * k];
            j[r] = a.defer[2 * k + 1];
        }
        fast_rays_wave<UNIT, R, U>(a, i, j, decided, code);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (__lane_id() != 0 || e + r >= n) continue;
            if (decided[r]) {
                emit_ray(a, i[r], j[r], code[r]);
            } else {
                const uint32_t u = atomicAdd(a.ucount, 1u);   // u < n <= DEFER_CAP
                a.udefer[2 * (int64_t)u] = i[r];
                a.udefer[2 * (int64_t)u + 1] = j[r];
            }
        }
    }
}
template <bool UNIT>
__global__ __launch_bounds__(256) void recheck_fast_deferred_kernel(const RecheckArgs a) {
    const uint32_t total = *a.dcount;
    const uint32_t n = total < (uint32_t)DEFER_CAP ? total : (uint32_t)DEFER_CAP;
    if (blockIdx.x == 0 && threadIdx.x == 0 && n) atomicAdd(a.counters + C_DIRECT, (unsigned long long)n);
    const uint32_t wave_id = (uint32_t)__builtin_amdgcn_readfirstlane((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6));
    const uint32_t n_waves = (gridDim.x * blockDim.x) >> 6;
    if (n <= n_waves) fast_deferred<UNIT, 1, 8>(a, n, wave_id, n_waves);
    else fast_deferred<UNIT, STAGE_A_RAYS, 4>(a, n, wave_id, n_waves);
}

// The exact stage over the gathered rays stage A left, one wave per ray.
template <bool UNIT, ExactForm FORM>
__global__ __launch_bounds__(256) void recheck_exact_deferred_kernel(const RecheckArgs a) {
    const uint32_t n = *a.ucount;
    const int lane = __lane_id();
    const uint32_t wave_id = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const uint32_t n_waves = (gridDim.x * blockDim.x) >> 6;
    for (uint32_t e = wave_id; e < n; e += n_waves) {
        const int64_t i = a.udefer[2 * (int64_t)e], j = a.udefer[2 * (int64_t)e + 1];
        const int code = exact_ray_wave<UNIT, FORM>(a, i, j);
        if (lane == 0) emit_ray(a, i, j, code);
    }
}

// ------------------------------- batch -------------------------------------

__device__ inline RecheckArgs batch_recheck_args(const BatchMap &m) {
    return recheck_args_of(m.p, m.lens_xy, m.lens_m, m.n_lens, m.map, m.counters);
}

__device__ __forceinline__ void wave_sync() {
    // LDS operations of one wave execute in order; keep the compiler from moving
    // them across this point.
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Stage A for the entries held one per lane (valid lanes only): lanes are
// grouped by map, and each group runs with its map's parameters in scalar
// registers. Rays are decided, or marked for the exact stage.
template <bool ALL_UNIT>
__device__ inline void batch_stage_a(const BatchArgs &b, QueueEntry e, bool valid) {
    uint64_t pending = __ballot(valid);
    while (pending) {
        const int leader = __builtin_ctzll(pending);
        const uint32_t mi = (uint32_t)__builtin_amdgcn_readlane((int)e.map, leader);
        const bool mine = valid && e.map == mi;
        pending &= ~__ballot(mine);
        const BatchMap &m = b.maps[mi];
        const RecheckArgs a = make_uniform(batch_recheck_args(m));
        uint32_t *const unres = make_uniform(m.unres_bits);
        int code = CODE_OUT;
        bool ok = false;
        if (mine) {
            const int64_t W = a.i1 - a.i0;
            const int64_t i = a.i0 + (int64_t)(e.ray % (uint64_t)W);
            const int64_t j = a.j0 + (int64_t)(e.ray / (uint64_t)W);
            if (ALL_UNIT || a.lens_m == nullptr) ok = fast_ray<true>(a, i, j, code);
            else ok = fast_ray<false>(a, i, j, code);
            if (ok) {
                if (code >= 0) atomicAdd(a.map + code, 1u);
            } else {
                atomicOr(unres + (e.ray >> 5), 1u << (e.ray & 31u));
            }
        }
        // one counter update per group (stage A never yields a singular ray)
        const unsigned n_in = (unsigned)__builtin_popcountll(__ballot(mine && ok && code >= 0));
        const unsigned n_out = (unsigned)__builtin_popcountll(__ballot(mine && ok && code < 0));
        const bool any_unres = __ballot(mine && !ok) != 0;
        if (__lane_id() == leader) {
            if (n_in) atomicAdd(a.counters + C_IN, (unsigned long long)n_in);
            if (n_out) atomicAdd(a.counters + C_OUT, (unsigned long long)n_out);
            if (any_unres) atomicOr(b.unresolved, 1u);
        }
    }
}

// Stage F for the entries held one per lane (valid lanes only), lanes grouped
// by map as in stage A: each ray from its map's super-patch record and lens
// list. Returns true in the lanes whose ray it placed; the others are counted
// in their map's C_DIRECT and go on to stage A.
template <bool ALL_UNIT>
__device__ inline bool batch_stage_f(const BatchArgs &b, QueueEntry e, bool valid) {
    bool placed = false;
    uint64_t pending = __ballot(valid);
    while (pending) {
        const int leader = __builtin_ctzll(pending);
        const uint32_t mi = (uint32_t)__builtin_amdgcn_readlane((int)e.map, leader);
        const bool mine = valid && e.map == mi;
        pending &= ~__ballot(mine);
        const ShootArgs a = make_uniform(batch_far_args(b.maps[mi]));
        int code = FLAGGED;
        if (mine) {
            const int64_t W = a.i1 - a.i0;
            const int64_t i = a.i0 + (int64_t)(e.ray % (uint64_t)W);
            const int64_t j = a.j0 + (int64_t)(e.ray / (uint64_t)W);
            code = (ALL_UNIT || a.lens_m == nullptr) ? far_recheck_ray<true, false>(a, i, j) : far_recheck_ray<false, false>(a, i, j);
            if (code >= 0) atomicAdd(a.map + code, 1u);
            placed = code != FLAGGED;
        }
        const unsigned n_in = (unsigned)__builtin_popcountll(__ballot(mine && code >= 0));
        const unsigned n_out = (unsigned)__builtin_popcountll(__ballot(mine && code == OUT));
        const unsigned n_left = (unsigned)__builtin_popcountll(__ballot(mine && code == FLAGGED));
        if (__lane_id() == leader) {
            if (n_in) atomicAdd(a.counters + C_IN, (unsigned long long)n_in);
            if (n_out) atomicAdd(a.counters + C_OUT, (unsigned long long)n_out);
            if (n_left) atomicAdd(a.counters + C_DIRECT, (unsigned long long)n_left);
        }
    }
    return placed;
}

// Stage A of one queued ray (wave-uniform entry) by the whole wave: lanes split the
// lenses. Used for a wave's last few rays, where one ray per lane would leave the
// GPU mostly idle while each lane walks every lens.
__device__ inline void batch_stage_a_wave(const BatchArgs &b, QueueEntry e) {
    const BatchMap &m = b.maps[e.map];
    const RecheckArgs a = make_uniform(batch_recheck_args(m));
    const int64_t W = a.i1 - a.i0;
    const int64_t i = a.i0 + (int64_t)(e.ray % (uint64_t)W);
    const int64_t j = a.j0 + (int64_t)(e.ray / (uint64_t)W);
    int code = CODE_OUT;
    const bool ok = a.lens_m == nullptr ? fast_ray_wave<true, 4>(a, i, j, code) : fast_ray_wave<false, 4>(a, i, j, code);
    if (__lane_id() == 0) {
        if (ok) {
            if (code >= 0) atomicAdd(a.map + code, 1u);
            atomicAdd(a.counters + (code >= 0 ? C_IN : C_OUT), 1ull);
        } else {
            uint32_t *const unres = m.unres_bits;
            atomicOr(unres + (e.ray >> 5), 1u << (e.ray & 31u));
            atomicOr(b.unresolved, 1u);
        }
    }
}

// Exact stage for up to 64 entries held one per lane: one wave per ray. CHAIN: no map has
// more than BATCH_CHAIN_LENSES lenses.
template <bool ALL_UNIT, bool CHAIN>
__device__ inline void batch_stage_b(const BatchArgs &b, QueueEntry e, int n_valid) {
    const int lane = __lane_id();
    for (int s = 0; s < n_valid; ++s) {
        const uint32_t mi = (uint32_t)__builtin_amdgcn_readlane((int)e.map, s);
        const uint32_t ray = (uint32_t)__builtin_amdgcn_readlane((int)e.ray, s);
        const BatchMap &m = b.maps[mi];
        const RecheckArgs a = make_uniform(batch_recheck_args(m));
        const int64_t W = a.i1 - a.i0;
        const int64_t i = a.i0 + (int64_t)(ray % (uint64_t)W);
        const int64_t j = a.j0 + (int64_t)(ray / (uint64_t)W);
        const bool unit = ALL_UNIT || a.lens_m == nullptr;
        int code;
        if (CHAIN || a.n_lens <= BATCH_CHAIN_LENSES)
            code = unit ? exact_ray_chain<true>(a, i, j) : exact_ray_chain<false>(a, i, j);
        else
            code = unit ? exact_ray_parallel<true, 4, false>(a, i, j) : exact_ray_parallel<false, 4, false>(a, i, j);
        if (lane == 0) emit_ray(a, i, j, code);
    }
}

// Persistent scan of the batch's bitmaps (STAGE 0: flag bits -> stage F, then
// stage A for the rays it leaves; STAGE 1: unresolved bits -> exact stage). The batch's words are dealt to the
// waves one at a time (lane l of wave k reads word k + (t + l) n_waves), so a
// dense run of flagged rays - a crowded lens region fills whole rows of them -
// is spread over many waves instead of queueing in one. Each wave compacts its
// set bits into its own ring buffer in LDS and evaluates them 64 at a time, one
// per lane. A wave leaves when its words are done and its buffer is empty.
template <int STAGE, bool ALL_UNIT, bool CHAIN>
__global__ __launch_bounds__(256) void recheck_scan_batch_kernel(const BatchArgs b) {
    if (STAGE == 1 && *b.unresolved == 0u) return;
    constexpr int RING = 128;
    __shared__ QueueEntry ring_all[4][RING];
    const int lane = __lane_id();
    QueueEntry *ring = ring_all[threadIdx.x >> 6];
    const uint64_t below = (1ull << lane) - 1ull;
    int head = 0, tail = 0;  // wave-uniform; tail - head < 64 between evaluations
    const int64_t wave_id = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int64_t n_waves = (int64_t)gridDim.x * (blockDim.x >> 6);
    for (int64_t t0 = 0; wave_id + t0 * n_waves < b.total_words; t0 += 64) {
        const int64_t word = wave_id + (t0 + lane) * n_waves;
        uint32_t bits = 0u;
        int lo = 0;
        int64_t w = 0;
        if (word < b.total_words) {
            int hi = b.n_maps - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (b.maps[mid].word_begin <= word) lo = mid;
                else hi = mid - 1;
            }
            const BatchMap &m = b.maps[lo];
            w = word - m.word_begin;
            bits = (STAGE == 0 ? m.flag_bits : m.unres_bits)[w];
        }
        for (;;) {
            const uint64_t hm = __ballot(bits != 0u);
            if (!hm) break;
            if (bits) {
                const int bit = __builtin_ctz(bits);
                bits &= bits - 1u;
                const int pos = (tail + __builtin_popcountll(hm & below)) % RING;
                ring[pos] = QueueEntry{(uint32_t)lo, (uint32_t)(w * 32 + bit)};
            }
            tail += __builtin_popcountll(hm);
            wave_sync();
            if (tail - head >= 64) {
                const QueueEntry e = ring[(head + lane) % RING];
                head += 64;
                wave_sync();
                if (STAGE == 0) {
                    const bool placed = batch_stage_f<ALL_UNIT>(b, e, true);
                    batch_stage_a<ALL_UNIT>(b, e, !placed);
                }
                else batch_stage_b<ALL_UNIT, CHAIN>(b, e, 64);
            }
        }
    }
    const int left = tail - head;
    if (left > 0) {
        QueueEntry e{0u, 0u};
        if (lane < left) e = ring[(head + lane) % RING];
        if (STAGE == 0) {
            // the last few rays: stage F one per lane, then stage A one wave per ray
            // (lenses split over the lanes) for those it could not place
            const bool placed = batch_stage_f<ALL_UNIT>(b, e, lane < left);
            uint64_t rest = __ballot(lane < left && !placed);
            while (rest) {
                const int s = __builtin_ctzll(rest);
                rest &= rest - 1;
                QueueEntry es;
                es.map = (uint32_t)__builtin_amdgcn_readlane((int)e.map, s);
                es.ray = (uint32_t)__builtin_amdgcn_readlane((int)e.ray, s);
                batch_stage_a_wave(b, es);
            }
        } else {
            batch_stage_b<ALL_UNIT, CHAIN>(b, e, left);
        }
    }
}

}  // namespace

// f with the exact stage's form for a map of n_lens lenses.
template <class F>
static void with_exact_form(int64_t n_lens, F f) {
    if (n_lens <= EXACT_CHAIN_LENSES) f(std::integral_constant<ExactForm, EXACT_CHAIN>{});
    else if (n_lens < EXACT_PAUSE_LENSES) f(std::integral_constant<ExactForm, EXACT_PAUSE>{});
    else f(std::integral_constant<ExactForm, EXACT_PARALLEL>{});
}

static void launch_exact_wave(const RecheckArgs &a, dim3 grid, hipStream_t stream) {
    with_exact_form(a.n_lens, [&](auto form) {
        constexpr ExactForm FORM = decltype(form)::value;
        if (a.lens_m == nullptr) hipLaunchKernelGGL((recheck_exact_wave_kernel<true, FORM>), grid, dim3(256), 0, stream, a);
        else hipLaunchKernelGGL((recheck_exact_wave_kernel<false, FORM>), grid, dim3(256), 0, stream, a);
    });
}

hipError_t launch_recheck(const RecheckArgs &a, int64_t max_rays, bool exact_only, bool stage_a_done, hipStream_t stream) {
    const dim3 block(256);
    const dim3 threads((unsigned)queue_blocks(max_rays, 256, 2048));   // a ray per thread
    const bool unit = a.lens_m == nullptr;
    if (exact_only) {
        if (unit) hipLaunchKernelGGL(recheck_exact_kernel<true>, threads, block, 0, stream, a);
        else hipLaunchKernelGGL(recheck_exact_kernel<false>, threads, block, 0, stream, a);
    } else if (stage_a_done) {
        if (a.n_lens <= EXACT_INLINE_LENSES) return hipSuccess;   // stage B as well
        launch_exact_wave(a, dim3((unsigned)queue_blocks(max_rays, 4, 512)), stream);   // it mostly finds nothing to do
    } else {
        RecheckArgs b = a;
        if (a.defer) {
            hipLaunchKernelGGL(recheck_defer_kernel, threads, block, 0, stream, a);
            b.qlive = a.qleft;   // stage A of this launch takes what was not gathered
        }
        const dim3 grid((unsigned)queue_blocks(max_rays, 1, 2048));   // (a block per ray of a short queue)
        auto launch = [&](auto u) {
            constexpr bool U = decltype(u)::value;
            if (crowded(a.nx, a.ny, a.n_lens)) {
                hipLaunchKernelGGL((recheck_fast_kernel<U, FORM_THREADS>), threads, block, 0, stream, b);
                hipLaunchKernelGGL((recheck_fast_kernel<U, FORM_BLOCKS>), grid, block, 0, stream, b);
            } else {
                hipLaunchKernelGGL((recheck_fast_kernel<U, FORM_EITHER>), grid, block, 0, stream, b);
            }
        };
        if (unit) launch(std::true_type{});
        else launch(std::false_type{});
        launch_exact_wave(b, dim3((unsigned)queue_blocks(max_rays, 4, 2048)), stream);
    }
    return hipGetLastError();
}

hipError_t launch_recheck_deferred(const RecheckArgs &a, hipStream_t stream) {
    const dim3 grid(1024), block(256);
    auto launch = [&](auto unit) {
        constexpr bool U = decltype(unit)::value;
        hipLaunchKernelGGL(recheck_fast_deferred_kernel<U>, grid, block, 0, stream, a);
        with_exact_form(a.n_lens, [&](auto form) {
            hipLaunchKernelGGL((recheck_exact_deferred_kernel<U, decltype(form)::value>), grid, block, 0, stream, a);
        });
    };
    if (a.lens_m == nullptr) launch(std::true_type{});
    else launch(std::false_type{});
    return hipGetLastError();
}

hipError_t launch_recheck_batch(const BatchArgs &b, hipStream_t stream) {
    if (b.total_words <= 0) return hipSuccess;
    const dim3 grid(2048), block(256);
    // kernels of their own for batches of unit-mass maps only, and for batches whose maps all
    // take the exact stage's chain (fewer registers)
    const bool chain = b.max_lenses <= BATCH_CHAIN_LENSES;
    auto launch = [&](auto unit) {
        constexpr bool U = decltype(unit)::value;
        hipLaunchKernelGGL((recheck_scan_batch_kernel<0, U, true>), grid, block, 0, stream, b);
        if (chain) hipLaunchKernelGGL((recheck_scan_batch_kernel<1, U, true>), grid, block, 0, stream, b);
        else hipLaunchKernelGGL((recheck_scan_batch_kernel<1, U, false>), grid, block, 0, stream, b);
    };
    if (b.unit_masses) launch(std::true_type{});
    else launch(std::false_type{});
    return hipGetLastError();
}

}  // namespace rs
