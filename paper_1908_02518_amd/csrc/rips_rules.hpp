// rips_rules.hpp -- the arithmetic of the rules that choose a method, in plain
// C++: no HIP, so that a host program can include it by itself.
#pragma once

#include <cstdint>

namespace rips {

// Triangles of which the chunked sweep of dimension 1 holds the places (12
// bytes each, 3 GiB in all). The number of edges says little about theirs: one
// cluster of 2955 points has more than 2^32 of them with 100 edges a point in
// a cloud of 44,000 points, so they are counted in 64 bits.
constexpr uint64_t kMostOwned = 1ull << 28;
constexpr bool owned_fit(uint64_t triangles) { return triangles <= kMostOwned; }

// Cofacets of a chunk of dimension 2 that do not cancel, of which the sweep
// holds this many. A wave ends with its first append (64 at most) past that.
constexpr int kMostPairs = 1 << 21;
constexpr int64_t most_pairs(int64_t cap, int64_t waves) { return cap + waves * 64; }

} // namespace rips
