// How launches are sized: plain host rules (no device calls), shared by the launch
// code and its CPU tests.
#pragma once

#include <cstdint>

namespace rs {

// Blocks for a queue of at most max_entries rays, per_block of which a block takes at once in
// the kernel's form for short queues (one per wave, one per block or one per thread): one for
// each until the chip is full, at least one, at most cap. (Sized for the form for long queues, a
// small map's rays went one after another: the 2048 rays of a one-patch map of 300 lenses, all
// of them queued, took 64 turns of eight blocks' waves, 235 us a call; 45 now.)
inline int64_t queue_blocks(int64_t max_entries, int64_t per_block, int64_t cap) {
    const int64_t blocks = (max_entries + per_block - 1) / per_block;
    return blocks < 1 ? 1 : (blocks > cap ? cap : blocks);
}

}  // namespace rs
