// rips_rules.hpp -- the arithmetic of the rules that choose a method, in plain
// C++: no HIP, so that a host program can include it by itself.
#pragma once

#include <cstdint>

namespace rips {

// Points up to which one workgroup sweeps a cloud whole, distances to bars in
// one launch (0: never). The staged path's launches, waits and scalar reads
// cost 0.3 to 0.5 ms whatever the size, which the one workgroup's passes over
// n^2 pairs reach at about 256 points with a threshold (milliseconds swept and
// staged, 25 edges a point: torus 0.71 and 0.84, rotations 1.1 and 1.7, uniform
// in the cube of R^5 0.94 and 0.82, normal in R^3 0.71 and 0.59; 100 edges a
// point: 1.6 and 11.5, 3.1 and 14.0, 1.07 and 1.54, 0.92 and 1.15).
// Without a threshold the complex is dense and the reduction itself decides,
// for the sweep up to about 1000 points (700 points: sphere 5.3 and 46, torus
// 34 and 112, uniform in R^3 5.5 and 32, normal in R^5 8.3 and 23; 1000 points:
// 9.9 and 30, normal in R^3 12.2 and 12.1, in R^5 19.1 and 17.1; 2048 points:
// sphere 43 and 101, uniform in R^3 55 and 79, normal in R^2 39 and 31, in R^3
// 61 and 40, in R^5 191 and 67).
// Over another field a sum costs products and remainders for every class it
// has: half the points with a threshold, 200 without (whole_classes has the
// rest of that rule).
// Dimension 0 alone needs no cofacets, which the sweep looks for all the same:
// 100 points on the sphere 0.13 and 0.18 ms, uniform in R^10 0.15 and 0.18; 200
// points 0.24 and 0.26, 0.33 and 0.22; 1000 points 4.2 and 3.4, 6.5 and 2.2.
constexpr int kWholeN = 256, kWholeDenseN = 1024, kWholeOddN = 128, kWholeOddDenseN = 200, kWholeForestN = 128;
constexpr int whole_most(int max_dim, bool dense, uint32_t p) {
    const int most = dense ? (p == 2 ? kWholeDenseN : kWholeOddDenseN) : (p == 2 ? kWholeN : kWholeOddN);
    return max_dim == 0 ? (most < kWholeForestN ? most : kWholeForestN) : max_dim == 1 ? most : 0;
}

// Classes that it opens at most; with more the staged path takes over (after
// the distances, the scan and the forest, which are a small part). The vectors
// are as long as there are classes: over Z/2 the sweep loses above two a point
// (uniform in R^64: 128 points, 230 classes, 1.4 ms and 1.1; 200 points, 444,
// 3.5 and 1.5; 400 points, 1233, 33 and 16; lattices: 256 points, 495, 12 and
// 29; 400 points, 778, 74 and 110), over another field above some 220 (200
// points: uniform in R^5, 140 classes, 1.63 and 1.55, in R^10, 224, 2.6 and
// 1.6, orthogonal matrices, 274, 5.7 and 3.8, lattice, 299, 22 and 6.0).
constexpr int whole_classes(int n, uint32_t p) { return p != 2 ? 220 : n < 128 ? 256 : 2 * n; }

// Coordinates up to which that workgroup computes the distances itself. A
// lane's row of coordinates is as many cache lines apart from the next lane's
// as it is long, so their cost grows with n^2 times them; beyond, the whole
// chip does it in a launch before (100 uniform points, dimension 1, without and
// with it: R^4 0.32 ms and the same, R^64 2.0 and 0.73, R^1024 10.8 and 0.93;
// 128 points, dimension 0: R^8 0.21 and 0.15).
constexpr int kWholeCoords = 4;

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
