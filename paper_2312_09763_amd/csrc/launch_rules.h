// Rules of the launches that depend on sizes alone, in plain C++ (so that they can be
// checked without a GPU).
#pragma once

#include <cstdint>

#if defined(__HIPCC__)
#define MV_RULE __host__ __device__ inline
#else
#define MV_RULE inline
#endif

namespace mv {

// HIP refuses a launch of 2^32 threads or more along x; y and z hold at most 65535 blocks.
constexpr int64_t kMaxThreadsX = (int64_t)1 << 32;
constexpr int64_t kMaxGridYZ = 65535;

// ---- beam step on the interleaved grid (kernels_beam.hip) -------------------
constexpr int kBeamGroup = 4;  // beams that one block evaluates its sources on

// Blocks of `spb` sources that one XCD may have to do of a time slot with up to max_m.
MV_RULE int64_t tf_blocks_per_xcd(int64_t max_m, int spb) { return ((max_m + spb - 1) / spb + 7) / 8; }

// Grid of the beam step: x the source blocks (8 XCDs), y the time slots, z the (channel
// group, beam group) pairs, of which one launch takes up to kMaxGridYZ.  As a single x
// dimension the product of the three passed 2^32 threads at sizes that fit the memory
// (128 beams, 3.1 million sources, 11 times of one channel).
struct TfGrid {
    int64_t x, y, z;
};
MV_RULE TfGrid tf_grid(int64_t max_m, int spb, int n_slot, int n_freq, int fg, int n_beam) {
    return TfGrid{8 * tf_blocks_per_xcd(max_m, spb), n_slot,
                  (int64_t)((n_freq + fg - 1) / fg) * ((n_beam + kBeamGroup - 1) / kBeamGroup)};
}

}  // namespace mv
