// Which keys the single-sweep scoring kernel moves into its reference tiles.
// Plain C++ (no HIP header), so that the rule can be checked on the host.
#pragma once

#include <cstdint>

namespace kara {

// Keys that change places, at most: the reference tiles hold as many.
constexpr int kSwapMax = 64;
// Ranks lie in [0, 2^kSwapRankBits).  The bound on them is searched over that
// many bits, which makes fewer than kSwapMax keys rank above it.
constexpr int kSwapRankBits = 15;

// A key's rank: the upper half of its squared norm's fp32 bits, less the
// sign.  Squares have none, but a NaN keeps the sign it came with, and with
// the sign such a key would rank above any bound.
constexpr uint32_t swap_rank(uint32_t norm_bits) { return (norm_bits >> 16) & ((1u << kSwapRankBits) - 1); }

}  // namespace kara
