// rips_sweep_dim.hpp -- the sweep of dimension 1 or 2 of a single cloud over
// Z/p: buffers and launchers.
#pragma once

#include "rips_kernels.hpp"
#include "rips_rules.hpp"

namespace rips {

constexpr int kDimBins = 1 << 16;    // most diameter bins of the partition
constexpr int kDimMaxChunks = 16384;
constexpr int kDimWords = 64;        // words of a row: 2048 classes open at once
constexpr int kDimOddWords = 16;     // of its bits over a field other than Z/2: 512 classes open at once
constexpr int kDimSlots = kDimWords * 32;
constexpr int kDimRows = 1 << 14;    // rows
constexpr int kTiedMax = 1024, kTiedPairs = 1 << 14;
constexpr int kDimMaxVert = 65535;   // vertices are packed 16 bits each

// What the sweep reports.
struct DimOut {
    int full;                 // 1: a table was too small, the caller reduces columns instead; 2: broken
    int nch;                  // chunks
    int npair;                // dimension 2: cofacets of the chunk that do not cancel
    int ntied, npairs_tied;
    int nclasses;             // dimension 2: columns that no cofacet of their own block pairs
    unsigned long long owned; // dimension 1: triangles counted
    unsigned long long adds, rows;
    int64_t nbars, nonzero, essential, emergent, reduced;
    int64_t loc_emergent, loc_reduced; // dimension 2: columns paired within their block
};

struct DimArgs {
    Ctx<DistFull> c;
    SimplexList in;       // dimension 1: the edges <= t, in no order
    int64_t N;            // K-simplices
    const int *zj;        // dimension 1, per edge: third vertex of its zero apparent cofacet, -1 a column, -2 neither
    Columns cols;         // the columns, youngest first
    int S;
    u32 p;
    int nbins;            // a power of two from 2048 to kDimBins
    float scale;          // bins per unit of diameter
    float chunk_n;        // dimension 2: simplices of a chunk
    // per diameter bin: simplices, owned cofacets and columns (counts, then
    // first places), nbins + 1 each in one buffer; per chunk the same
    u32 *bin_n, *bin_t, *bin_s;
    u32 *ch_n, *ch_t, *ch_s;    // kDimMaxChunks + 1 each
    // in order of bin
    float *qdiam;         // N
    u64 *qverts;          // N: vertices, 16 bits each (edges: decreasing; triangles: see k_lune)
    int *qzj;             // N, dimension 1
    u32 *qdep;            // (K + 1) x N: the facets whose vectors a simplex's vector is the sum of
    u32 *ids;             // N: row of the simplex's vector (0: zero)
    // place of a simplex by index: a direct table, or the hash when it is null
    u32 *direct;
    PivotHash ph;
    // dimension 1: the cofacets whose youngest facet is q: q and the places of the other two
    u32 *tau;             // ntau x 3, entry-major
    u32 ntau;
    // dimension 2: a block is the triangles of one longest edge, at consecutive places
    EdgeList E;           // the edges <= t
    int64_t nE;
    u32 *bstart, *bcnt;   // nE: first place and size of an edge's block
    u32 *tlist;           // kTiedMax: edges with their bit in tied
    u32 *tplace;          // kTiedPairs: the pairs within their blocks: place, index of the tetrahedron
    int64_t *ttet;
    u32 *qblk, *qpar, *qkill; // N: block; parent in its forest, ~0 a root; the two ends of the edge a root fell to
    u32 *rhead, *rnext;   // N, 3 N: the triangles whose sum a triangle is part of, as lists of 3 N entries of qdep
    u32 *need;            // N bits: the sum may not be zero
    u32 *fl, *tied;       // n x fw words: edges of triangles with a nonzero vector; edges tied for longest in a simplex
    int fw;               // words of a vertex's bits, even
    u64 *pairs;           // paircap: cofacets of the chunk that do not cancel, as (place, vertex)
    int paircap;
    int strict;           // a dimension follows, which has to know every pair
    void *state;          // dimension 2: the sweep's LDS between two launches, dim_state_bytes()
    Columns all;          // every column, youngest first (cols: the classes among them)
    int nall;
    // the sweep
    u32 *bq;              // S: place of the k-th oldest column
    int64_t *kidx;        // S: index of the simplex that closes class k, -1 none
    float *kdiam;
    u32 *pool;            // kDimRows x W
    u64 *rsum;            // kDimRows: which words of a row are nonzero
    u32 *rfree, *rdead, *ract; // kDimRows each: free rows, replaced rows, rows in use
    u32 *nzl;             // N: simplices with a nonzero row
    int W;
    DimOut *out;
};

// dimension 1: edges by bin, owned triangles counted (out->owned; the bins'
// counts are good only if that is owned_fit); then written out
void launch_dim_partition(const DimArgs &A, hipStream_t st);
void launch_dim_fill(const DimArgs &A, hipStream_t st);
// dimension 2: triangles by block and bin, the blocks' forests, the pairs
// within blocks into `piv`, the other columns into cols; then their chunks
void launch_lune_partition(const DimArgs &A, PivotHash piv, hipStream_t st);
void launch_lune_chunks(const DimArgs &A, hipStream_t st);
hipError_t launch_dim_sweep(const DimArgs &A, hipStream_t st);
// dimension 2: at most `chunks` chunks, two launches each
hipError_t launch_lune_sweep(const DimArgs &A, int chunks, hipStream_t st);
size_t dim_state_bytes();
size_t dim_pool_bytes(u32 p, int W);
// the bars in column order, the counters, and the closing simplices as the
// next dimension's pivot table
void launch_dim_bars(int K, const DimArgs &A, BarBuf bars, PivotHash piv, hipStream_t st);

} // namespace rips
