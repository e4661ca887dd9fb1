// How launches are sized and queues dealt out: plain rules (no device calls), shared by the
// launch code, the kernels and their CPU tests.
#pragma once

#include <cstdint>

#include "rs_layout.h"

namespace rs {

// Thread shapes of the deflection kernel beside the N_SHAPES that can be forced and tuned:
// SHAPE_AUTO stands for the built-in choice, which is shape 0 (4 x 2 rays per lane, four waves) or,
// in launches of few patches, SHAPE_WIDE (2 x 2 rays per lane, eight waves).
constexpr int SHAPE_AUTO = -1;
constexpr int SHAPE_WIDE = N_SHAPES;

// At most two patches per CU (in FP32 mode one) are deflected by the wide shape: shape 0 would
// leave SIMDs with one or two waves. us a call, wide against shape 0, 2000 lenses: 256 patches 224
// / 347 (mixed), 150 / 222 (FP32); 512 patches 338 / 344 (mixed; with masses 379 / 371), 279 / 260
// (FP32). 300 lenses: 58 / 81, 33 / 46; 79 / 87 (with masses 90 / 94), 54 / 54.
inline int default_shape(bool mixed, int64_t patches, int64_t compute_units) {
    return patches <= (mixed ? 2 : 1) * compute_units ? SHAPE_WIDE : 0;
}

// The tuner's sample of a W x H window: whole bands of 32 rows and some of the lenses, with as
// many ray-lens pairs as about sample_rays rays with every lens have. Of 2048 lenses or more it
// takes up to a quarter, 1024 at least, and as many more rays: a launch's last blocks, which leave
// SIMDs with few waves, weigh on the shapes differently, and 4 million rays are under two rounds of
// blocks. (19200 x 3840 rays, 17240 lenses, 4 x 2 rays per lane 132 ms, 4 x 4 137: 4 million rays
// with every lens put 4 x 4 6% ahead, in 141 ms of tuning; 16 million 2% behind, in 533; 16 million
// with a quarter of the lenses 2% behind, in 141.)
struct TuneSample {
    int64_t rows, lenses;
};
inline TuneSample tune_sample(int64_t W, int64_t H, int64_t n_lens, int64_t sample_rays) {
    if (sample_rays / W >= H) return TuneSample{H, n_lens};   // the whole window
    const int64_t spread = n_lens < 2048 ? 1 : (n_lens < 4096 ? n_lens / 1024 : 4);
    TuneSample s{sample_rays / W * spread / PATCH_Y * PATCH_Y, n_lens};
    if (s.rows < PATCH_Y) s.rows = PATCH_Y;
    if (s.rows > H) s.rows = H;
    const double share = (double)sample_rays / ((double)s.rows * (double)W);   // of the lenses
    if (share < 1.0) s.lenses = (int64_t)((double)n_lens * (share * spread > 1.0 ? share : 1.0 / spread));
    return s;
}

// Blocks for a queue of at most max_entries rays, per_block of which a block takes at once in
// the kernel's form for short queues (one per wave, one per block or one per thread): one for
// each until the chip is full, at least one, at most cap. (Sized for the form for long queues, a
// small map's rays went one after another: the 2048 rays of a one-patch map of 300 lenses, all
// of them queued, took 64 turns of eight blocks' waves, 235 us a call; 45 now.)
inline int64_t queue_blocks(int64_t max_entries, int64_t per_block, int64_t cap) {
    const int64_t blocks = (max_entries + per_block - 1) / per_block;
    return blocks < 1 ? 1 : (blocks > cap ? cap : blocks);
}

// Adjacent entries of a long queue that a wave takes at a time: as many as give n_waves waves some,
// at most one per lane. (Shorter runs for more waves leave lanes idle that would walk the same
// list: 1024^2 rays, 900 lenses in clusters, 301 us with runs for a wave per SIMD, 340 for three.)
RS_HOST_DEVICE inline uint32_t entry_run(uint32_t entries, uint32_t n_waves) {
    const uint32_t share = (uint32_t)(((uint64_t)entries + n_waves - 1) / n_waves);
    return share < 64u ? share : 64u;
}

// Patches of the far-field ray kernel's persistent blocks, which load a patch's record while they
// evaluate the one before: the first two of each block by its index, the others by tickets from a
// counter. (With tickets for the first two as well, a block took two before others had any: 32
// patches of a map with a block for each took 69 us in most calls and 39 in the rest.)
RS_HOST_DEVICE inline int64_t first_patch(uint32_t block, uint32_t n_blocks, int turn) { return block + (int64_t)turn * n_blocks; }
RS_HOST_DEVICE inline int64_t ticket_patch(uint32_t ticket, uint32_t n_blocks) { return 2ll * n_blocks + ticket; }

// Ray grids (whole, whatever the window and launch) with fewer rays than this per lens have more
// lenses near a patch (a super-patch) than the deflection's near-lens list (the lens lists of
// stage F and of the far-field mode) holds, if the lenses are spread evenly over the grid: a patch
// has 2048 rays and lists at most 64 lenses of 16000 rays' area about it, a super-patch at most
// 4096 of 10^6 rays'. Most of their rays come to stage A.
inline bool crowded(int64_t nx, int64_t ny, int64_t n_lens) { return (double)nx * (double)ny < 256.0 * (double)n_lens; }

// Mixed maps of one launch and at most this many ray-lens pairs take the re-check's stages F and A
// in one kernel: a launch or two less, 4 us each, in a call of up to about 150 us. In larger maps
// stage A follows in kernels of its own, in the form that suits the number of rays stage F left
// and with those rays dealt out (in one kernel they stay with the waves that had them, and stage
// F has fewer registers: 1024 x 512 rays, 20000 lenses 7.43 ms in kernels of their own, 7.73 in
// one; 5000 lenses 755 and 750 us). Of crowded maps stage A takes
// most rays, so that they are large at fewer pairs (512^2 rays, 1500 lenses 506 us in kernels of
// their own, 574 in one; 256^2 and 3000 lenses 667 and 664).
constexpr double RECHECK_ONE_PAIRS = 1.0e9, RECHECK_ONE_CROWDED = 2.0e8;
inline bool recheck_in_one(int64_t rays, int64_t n_lens, bool several_launches, bool is_crowded) {
    return !several_launches && (double)rays * (double)n_lens <= (is_crowded ? RECHECK_ONE_CROWDED : RECHECK_ONE_PAIRS);
}

}  // namespace rs
