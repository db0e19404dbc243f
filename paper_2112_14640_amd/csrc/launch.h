// Sizes of a launch (host arithmetic only).
#pragma once

#include <cstdint>

namespace dirac {

// HIP takes fewer than 2^32 work-items in one grid dimension; of a larger launch it does a part, without an error.  A
// kernel with many threads per site gets there on lattices that fit the card (64 N_c threads per site of
// links_backward_kernel: 64^3 x 96 with N_c = 3, 174 GB), so its work-groups are launched in slices of at most
// max_blocks().
constexpr int64_t kMaxWorkItems = (int64_t(1) << 32) - 1;

// Most work-groups of `threads` threads in a launch, in eights (logical_block).
constexpr int64_t max_blocks(int threads) { return kMaxWorkItems / threads / 8 * 8; }

inline bool fits_launch(int64_t blocks, int threads) { return blocks <= max_blocks(threads); }

// launch(first, blocks) for each slice: `blocks` work-groups (a multiple of eight), numbered from `first` on.  The last
// slice is rounded up, so a kernel leaves where its number is past the work.
template <class F>
void launch_slices(int64_t blocks, int threads, F&& launch) {
    const int64_t most = max_blocks(threads);
    for (int64_t first = 0; first < blocks; first += most) {
        const int64_t n = blocks - first < most ? blocks - first : most;
        launch(first, static_cast<unsigned>((n + 7) / 8 * 8));
    }
}

}  // namespace dirac
