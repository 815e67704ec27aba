// rips_sweep.hpp -- arguments of the sweep: dimensions 0 and 1 of one cloud
// over Z/p by one workgroup, in one pass over its edges in order of length.
#pragma once

#include "../../include/rips.h"
#include "rips_device.hpp"

namespace rips {

constexpr int kSweepT = 1024;        // threads of a sweep workgroup
constexpr int kSweepMaxN = 2048;     // largest cloud (a bar's triangle index fits 32 bits)
constexpr int kSweepBins = 2048;     // length bins of the edge partition
constexpr int kSweepCand = 1024;     // triangles eliminated together
constexpr int kSweepCandWords = 8192; // and their vectors, in words
constexpr int kSweepMaxClasses = 2048;
constexpr int kSweepOddClasses = 512; // over a field other than Z/2: half a word a class more
constexpr int kSweepMaskBytes = 48 << 10; // nonzero-edge bits kept in LDS up to this size

// status bit: a cloud exceeds the sweep's tables (too many loops or rows);
// its bars are not written and the caller takes the column reduction
constexpr int kSweepFull = 512;

// What the sweep of one cloud reports, in pinned host memory.
struct SweepSingle {
    int status; // kSweepFull (the staged path decides), else 0
    float t, renc;
    int64_t count[2];
    rips_dim_stats stats[2];
};

struct SweepArgs {
    const float *X;         // points (m > 0), or the n x n distances of one cloud (m == 0)
    const int64_t *offsets; // B + 1, or null: one cloud of nmax points
    int B, m, max_dim, nmax;
    u32 p;
    float threshold;
    int most_classes;       // more than these: kSweepFull
    const int *order;       // clouds by decreasing size, or null
    unsigned long long *queue;
    // per workgroup (blockIdx.x)
    float *D;               // n x n distances, +inf on the diagonal
    int64_t d_stride;
    u32 *ids;               // n x n: row of an edge's vector (0: zero); [a][b], a > b, of every edge,
                            // and [b][a] of the nonzero ones
    uint16_t *zc;           // per pair: third vertex of its zero apparent cofacet
    u64 *list;              // edges by length bin: (a << 16 | b) | c << 32
    u32 *aux;               // edges whose scan goes on, later the nonzero edges
    int64_t e_stride;       // C(nmax, 2)
    u64 *sv;                // edges in no zero apparent pair, by (length, ~index)
    u64 *ckey, *kkey;       // per class: its edge's key, its triangle's key
    int sv_cap;             // power of two
    u32 *pool;              // rows
    int64_t pool_stride;
    u64 *mask;              // nonzero-edge bits, when they exceed the LDS part
    int64_t mask_stride;
    // results
    float *ub, *ud;         // unordered bars
    int64_t *ubs, *uds;
    int64_t ucap;
    unsigned long long *ucount;
    int64_t *seg_start, *seg_count; // B * (max_dim + 1)
    rips_dim_stats *stats;          // B * (max_dim + 1)
    float *t_used;                  // B
    int *status;
    // one cloud (res not null, one workgroup, no queue): the bars of dimension
    // d go to [d * ucap, d * ucap + count) of ub .. uds, if every dimension fits
    SweepSingle *res;
    int64_t *col_idx; // the columns of dimension 1, youngest first, or null
    float *col_diam;
};

// words of one vertex's nonzero-edge bits
__host__ __device__ inline int sweep_mask_words(int n) { return (n + 63) / 64; }
size_t sweep_lds_bytes(int nmax, int sv_cap);
int sweep_sv_cap(int nmax);
int64_t sweep_pool_words(int nmax, u32 p);
hipError_t sweep_prepare(int nmax, int sv_cap, u32 p);
void launch_sweep_order(const int64_t *offsets, int B, int nmax, int *order, unsigned long long *queue,
                        unsigned long long *ucount, int *status, hipStream_t st);
void launch_sweep(const SweepArgs &A, int grid, hipStream_t st);

} // namespace rips
