// Which samples a workgroup of the cost model's tile kernel takes: tiles of
// kMlpTile samples, workgroup g of `groups` taking tiles g, g + groups, ...
// Samples are counted in 64 bits: one step past the last of 2^30 and more
// samples does not fit an int.
#pragma once
#include <stdint.h>

namespace jk {

constexpr int kMlpTile = 16;
constexpr int kMlpThreads = 256;  // of a workgroup

// Workgroups of a forward pass: one a tile up to 2^20, whose threads stay far
// below the 2^32 that a launch may have (2^28 samples have 2^24 tiles).
constexpr int64_t kMlpMaxForward = 1 << 20;

constexpr int64_t mlp_tiles(int n) { return ((int64_t)n + kMlpTile - 1) / kMlpTile; }
constexpr unsigned mlp_groups(int n, int64_t most) { return (unsigned)(mlp_tiles(n) < most ? mlp_tiles(n) : most); }
constexpr int64_t mlp_first(unsigned group) { return (int64_t)group * kMlpTile; }
constexpr int64_t mlp_next(int64_t base, unsigned groups) { return base + (int64_t)groups * kMlpTile; }

}  // namespace jk
