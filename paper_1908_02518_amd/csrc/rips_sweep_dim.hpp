// rips_sweep_dim.hpp -- the sweep of one dimension K (1 or 2) of a single
// cloud over Z/2: buffers and launchers.
#pragma once

#include "rips_kernels.hpp"

namespace rips {

constexpr int kDimBins = 1 << 16;    // most diameter bins of the partition
constexpr int kDimMaxChunks = 16384;
constexpr int kDimWords = 64;        // words of a row: 2048 classes open at once
constexpr int kDimSlots = kDimWords * 32;
constexpr int kDimRows = 1 << 14;    // rows
constexpr int kDimMaxVert = 65535;   // vertices are packed 16 bits each

// What the sweep reports.
struct DimOut {
    int full;                 // 1: a table was too small, the caller reduces columns instead; 2: broken
    int nch;                  // chunks
    unsigned long long total; // owned cofacets
    unsigned long long adds, rows;
    int64_t nbars, nonzero, essential, emergent, reduced;
};

struct DimArgs {
    Ctx<DistFull> c;
    SimplexList in;       // the K-simplices <= t, in no order
    int64_t N;
    const int *zj;        // per simplex: third vertex of its zero apparent cofacet, -1 a column, -2 neither
    Columns cols;         // the columns, youngest first
    int S;
    int nbins;            // a power of two from 2048 to kDimBins
    float scale;          // bins per unit of diameter
    // per diameter bin: simplices, owned cofacets and columns (counts, then
    // first places), nbins + 1 each in one buffer; per chunk the same
    u32 *bin_n, *bin_t, *bin_s;
    u32 *ch_n, *ch_t, *ch_s;    // kDimMaxChunks + 1 each
    // in order of bin
    float *qdiam;         // N
    u64 *qverts;          // N: decreasing vertices, 16 bits each
    int *qzj;             // N
    u32 *qdep;            // (K + 1) x N: the other facets of the zero apparent cofacet, where there is one
    u32 *ids;             // N: row of the simplex's vector (0: zero)
    // place of a simplex by index: a direct table, or the hash when it is null
    u32 *direct;
    PivotHash ph;
    // the cofacets whose youngest facet is q: q and the places of the other K + 1 facets
    u32 *tau;             // total x (K + 2), entry-major
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

void launch_dim_partition(int K, const DimArgs &A, hipStream_t st);
void launch_dim_fill(int K, const DimArgs &A, hipStream_t st);
hipError_t launch_dim_sweep(int K, const DimArgs &A, hipStream_t st);
// the bars in column order, the counters, and the closing simplices as the
// next dimension's pivot table
void launch_dim_bars(int K, const DimArgs &A, BarBuf bars, PivotHash piv, hipStream_t st);

} // namespace rips
