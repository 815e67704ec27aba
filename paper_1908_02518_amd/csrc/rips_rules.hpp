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

// Whether a batch over Z/2 is swept. Milliseconds swept and by columns, 16
// clouds of 300, 1000 and 2048 points on noisy circles at 0.3: 0.68 and 1.4,
// 7.3 and 25, 57 and 172; dimension 0 alone: 0.46 and 0.92, 4.5 and 9.8, 21 and
// 46; uniform points: 100 of R^64 0.89 and 3.2, of R^1024 1.9 and 5.9, 256 of
// R^64 8.8 and 21. It loses where points and coordinates are many, hence also
// the classes: 256 of R^256 38 and 27, of R^1024 57 and 44.
constexpr int kBatchManyN = 128, kBatchManyCoords = 128;
constexpr bool batch_swept(int n_max, int m, uint32_t p) {
    return p == 2 && (n_max <= kBatchManyN || m <= kBatchManyCoords);
}

// Whether dimension 1 of a larger cloud is swept in chunks, by its edges per
// point and by how evenly they lie. What the columns cost depends on how long
// the classes live, which nobody knows before; the sweep costs some 1.8 ns a
// triangle and 2.2 us a class whatever they do (milliseconds swept and reduced,
// 80 edges a point, 2000 points: rotations 5.6 and 78, torus 4.9 and 50,
// orthogonal matrices 5.7 and 66, uniform in R^5 7.9 and 29, in R^3 5.3 and 6.1,
// in R^2 4.6 and 4.2; 195 edges: 15 and 520, 17 and 427, 22 and 874, 17 and 51,
// 16 and 11, 16 and 7.2). Below 32 edges a point the columns are few and short
// (2500 points of the torus, 25 edges a point: 4.0 and 2.8; 35: 4.4 and 9.0).
// Above 200 the sweep's one workgroup looks at too many triangles (1000 points
// on the sphere: 200 edges a point 7.7 and 9.1, 300: 15 and 13, 1000: 290 and
// 36). And where the points crowd, the triangles do, in the crowd, whose
// classes are short: the mean degree seen from an edge is 1.03 times the mean
// at most on the manifolds above, 1.06 to 1.2 in cubes, and from about 1.22 on
// the sweep loses more than it wins (normal points of R^2, 4000, 80 edges: 1.3,
// 10.5 and 4.6; of R^5: 1.7, 18 and 8.8; 300 of 3000 points in one ball: 2.4,
// 17 and 6.0; 500 of them: 3.1, 57 and 14).
// Over another field sums cost more (p = 3, 104 edges a point: torus4-2000 8.2
// and 92, rotations 1000 4.7 and 8.4, sphere 2000 7.2 and 4.9; sphere-1500 at
// 136 7.9 and 4.9), and with more columns than kChunkOddColumns too many classes
// are open at once for its tables (1137 of 4000 points on the sphere fit, 1161
// of 2000 orthogonal matrices do not).
constexpr int64_t kChunkDegMin = 32, kChunkDegMax = 200, kChunkOddDegMax = 110, kChunkOddColumns = 1150;
constexpr double kUneven = 1.22;
constexpr bool lie_evenly(int64_t n, int64_t edges, uint64_t deg2) {
    return (double)n * (double)deg2 <= kUneven * 4.0 * (double)edges * (double)edges;
}
constexpr bool chunks_pay(int64_t n, int64_t edges, uint64_t deg2, uint32_t p) {
    return edges >= kChunkDegMin * n / 2 && edges <= (p == 2 ? kChunkDegMax : kChunkOddDegMax) * n / 2 &&
           lie_evenly(n, edges, deg2);
}

// Whether dimension 2 is swept by blocks: by its triangles, and by how many an
// edge has. Few triangles cost the sweep's launches what they cost the columns
// (12 points on the sphere 0.58 and 0.55 ms, 24 points 0.57 and 0.48, 357
// rotations at 1.3, 8000 triangles, 1.31 and 1.24; 64 points on the sphere,
// 37,000 triangles, 1.4 and 9.7). And with few an edge the columns are short
// while the sweep still looks at every edge's lune: over 107 clouds that the
// rule sends to the columns they took 0.80 of the sweep's time in the mean
// (1200 points, 25 edges a point, triangles an edge 3 to 5: rotations 0.8,
// uniform in R^5 0.5, in R^10 0.3, torus 1.0, sphere 1.0), over 145 that it
// has swept, 1.5 times (45 edges a point: 0.9 to 1.9 times on all of these but
// R^10; 80 edges a point: torus 2.5 to 8, rotations 5 to 9, sphere 3 to 10,
// uniform in R^3 1 to 3; dense clouds: sphere 5 to 67, uniform in R^5 0.5 to
// 0.8, normal in R^3 0.3 to 1.3, which nothing known by then tells apart).
// The same evenness as for dimension 1: above it clusters 0.4 to 0.75, normal
// points of R^3 and R^5 0.5 to 1.2, of R^2 0.9 to 2.3.
constexpr int64_t kBlockTriangles = 12288, kBlockRatio = 5;
constexpr bool blocks_pay(int64_t n, int64_t edges, uint64_t deg2, int64_t triangles) {
    return triangles >= kBlockTriangles && triangles >= kBlockRatio * edges && lie_evenly(n, edges, deg2);
}

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
