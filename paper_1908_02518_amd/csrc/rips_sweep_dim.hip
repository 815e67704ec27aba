// rips_sweep_dim.hip -- the sweep of dimension 1 or 2 of a single cloud (the
// method of rips_sweep.hip, for any number of points and for triangles).
//
// Every K-simplex carries the vector of the open K-classes; a simplex that
// dimension K-1 has paired has the vector zero (a reduced boundary's pivot is
// never such a simplex), a class's own simplex its unit vector. A
// (K+1)-simplex whose facets do not sum to zero closes the youngest class of
// the sum.
//
// Dimension 1: an edge of a zero apparent pair (e, t) has the sum over the
// other two edges of t; the columns of the reduction (section "Assembling
// column indices") are the classes.
//
// Dimension 2: that would open thousands of classes of zero persistence and
// close them one by one (so3-1000: 31 ms, columns 5.3). But a pair of zero
// persistence lies in one block, the simplices with the same longest edge e:
// the triangles e + c stand for the points c of e's lune, the tetrahedra
// e + {c, d} for the lune's edges shorter than e, and the pairs are those of
// a spanning forest of that graph, its edges taken in the order of the
// tetrahedra: an edge that joins two trees pairs with the younger tree's
// oldest triangle. Only the oldest triangle of a tree without the block's
// oldest is a class (or closes one of dimension 1), and every other triangle
// has the sum over the other facets of the tetrahedron that joins it to its
// parent (so3-1000: 211 classes of 19,000 columns). Ties: edges of equal length are put in
// order by index, which moves simplices of equal diameter among themselves;
// that cannot change a pair unless one of the two is in a block that shares
// a simplex with another of the same length (and that simplex joins trees);
// a class opened or closed in such a block is left to the columns, and the
// pairs within it, which dimension 3 has to know, are found by k_lune_groups.
//
// All passes over simplices are data-parallel over the chip: the simplices by
// diameter bin, the place of each by index, and the places that the sweep
// will look at, so that the sweep itself, one workgroup, only follows places.
// It takes whole bins in chunks: opens the chunk's classes, resolves its
// vectors, gathers the cofacets that do not cancel, eliminates them in order
// and substitutes the closed classes. Few vectors are nonzero and most of
// those are shared, so a chunk is a few microseconds of one workgroup.
#include "rips_sweep_dim.hpp"

#include <algorithm>
#include <type_traits>

namespace rips {

namespace {

constexpr int kT = 1024;
constexpr int kWaves = kT / kWave;
constexpr u32 kPending = ~0u;
constexpr u32 kNeg = 1u << 31;      // of a place: less its vector
constexpr int kOddWords = 20480;     // kCandWords over a field other than Z/2
constexpr int kOddRows = 1 << 13;   // rows over a field other than Z/2
constexpr int kDimBroken = 2;       // a place or row number out of range: a mistake, not a full table
constexpr int kCand = 512;          // cofacets eliminated together
constexpr int kCandWords = 16384;   // and their vectors, in words
constexpr int kPurge = 32;          // eliminations between two purges
constexpr int kTaus = 4;            // cofacets a lane has in flight
constexpr int kLune = 1024;         // points of a lune
constexpr int kMostBlocks = 16384;  // of a grid

__device__ __forceinline__ int dim_bin(const DimArgs &A, float d) {
    return min(A.nbins - 1, (int)(d * A.scale)); // monotone; equal diameters share a bin
}

template <int K>
__device__ __forceinline__ void unpack(u64 p, int (&v)[K + 1]) {
#pragma unroll
    for (int i = 0; i <= K; ++i) v[i] = (int)((p >> (16 * i)) & 0xffff);
}

// index of a K-simplex given by decreasing vertices
template <int K>
__device__ __forceinline__ int64_t index_of(const int (&v)[K + 1]) {
    if constexpr (K == 1) {
        return (int64_t)v[0] * (v[0] - 1) / 2 + v[1];
    } else {
        const int64_t a = v[0], b = v[1];
        return a * (a - 1) * (a - 2) / 6 + b * (b - 1) / 2 + v[2];
    }
}

template <int K>
__device__ __forceinline__ u32 place_of(const DimArgs &A, const int (&v)[K + 1]) {
    const int64_t idx = index_of<K>(v);
    if (A.direct) return A.direct[idx];
    return (u32)ph_find(A.ph, idx);
}

// facet i of s u {c}: s without v[i], with c, decreasing
template <int K>
__device__ __forceinline__ void facet_of(const int (&v)[K + 1], int i, int c, int (&f)[K + 1]) {
    int q = 0;
    bool placed = false;
#pragma unroll
    for (int j = 0; j <= K; ++j) {
        if (j == i) continue;
        if (!placed && c > v[j]) {
            f[q++] = c;
            placed = true;
        }
        f[q++] = v[j];
    }
    if (!placed) f[q] = c;
}

// ---- the simplices by diameter bin
template <int K>
__global__ void __launch_bounds__(256) k_dim_hist(DimArgs A) {
    const int64_t stride = (int64_t)gridDim.x * 256, t0 = blockIdx.x * 256ll + threadIdx.x;
    if (K == 1)
        for (int64_t i = t0; i < A.N; i += stride) atomicAdd(&A.bin_n[dim_bin(A, A.in.diam[i])], 1u);
    for (int64_t i = t0; i < A.S; i += stride) atomicAdd(&A.bin_s[dim_bin(A, A.cols.diam[i])], 1u);
}

// exclusive scan of the bins of one array, in place; one workgroup an array,
// a multiple of 1024 bins. total (or null): the sum in 64 bits, all ones if it
// says that a bin has wrapped.
__global__ void __launch_bounds__(1024) k_dim_scan(u32 *a0, u32 *a1, int nbins, unsigned long long *total) {
    __shared__ u32 s_w[kWaves];
    __shared__ unsigned long long s_total;
    u32 *a = blockIdx.x == 0 ? a0 : a1;
    const int per = nbins / kT;
    const int lane = lane_id(), w = threadIdx.x / kWave;
    u32 sum = 0;
    unsigned long long all = 0;
    if (threadIdx.x == 0) s_total = 0;
#pragma unroll 8
    for (int i = 0; i < per; ++i) {
        const u32 x = a[threadIdx.x * per + i];
        sum += x;
        all += x;
    }
    u32 inc = sum;
    for (int o = 1; o < kWave; o <<= 1) {
        const u32 x = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += x;
    }
    if (lane == kWave - 1) s_w[w] = inc;
    __syncthreads();
    if (total) {
        for (int o = 32; o >= 1; o >>= 1) all += __shfl_xor(all, o, kWave);
        if (lane == 0) atomicAdd(&s_total, all);
    }
    u32 base = inc - sum;
    for (int q = 0; q < w; ++q) base += s_w[q];
#pragma unroll 8
    for (int i = 0; i < per; ++i) {
        const u32 x = a[threadIdx.x * per + i];
        a[threadIdx.x * per + i] = base;
        base += x;
    }
    if (threadIdx.x == kT - 1) a[nbins] = base;
    __syncthreads();
    if (total && threadIdx.x == 0) *total |= s_total;
}

__global__ void __launch_bounds__(256) k_dim_place(DimArgs A) {
    constexpr int K = 1;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = blockIdx.x * 256ll + threadIdx.x; i < A.N; i += stride) {
        const int64_t idx = A.in.idx[i];
        const float d = A.in.diam[i];
        const u32 q = atomicAdd(&A.bin_n[dim_bin(A, d)], 1u); // the bins' first places move up to their ends
        int v[K + 1];
        decode(idx, K, A.c.n, A.c.B, v);
        u64 p = 0;
#pragma unroll
        for (int j = 0; j <= K; ++j) p |= (u64)(u32)v[j] << (16 * j);
        const int z = A.zj[i];
        A.qdiam[q] = d;
        A.qverts[q] = p;
        A.qzj[q] = z;
        A.ids[q] = z >= 0 ? kPending : 0u;
        if (A.direct) A.direct[idx] = q;
        else (void)ph_insert(A.ph, idx, (int32_t)q); // room for twice the simplices: it cannot fail
    }
}

// ---- the triangles an edge owns: third vertices c with every new edge at
// most its diameter long and every other facet older (a facet of the same
// diameter is older when its index is larger, that is when c is larger than
// the vertex it replaces). A group of G lanes a simplex.
template <int G, bool kFill>
__global__ void __launch_bounds__(256) k_dim_own(DimArgs A) {
    constexpr int K = 1;
    const int lane = lane_id(), lg = lane & (G - 1), g0 = lane & ~(G - 1);
    const u64 gmask = G == 64 ? ~0ull : ((1ull << (G & 63)) - 1) << g0;
    const int64_t groups = (int64_t)gridDim.x * (256 / G);
    const int n = A.c.n;
    const float *D = A.c.d.D;
    const int64_t per_wave = kWave / G;
    const int64_t w0 = (blockIdx.x * 256ll + threadIdx.x) / kWave * per_wave;
    for (int64_t base = w0; base < A.N; base += groups) {
        const int64_t q = base + lane / G;
        const bool live = q < A.N;
        int v[K + 1];
        unpack<K>(live ? A.qverts[q] : 0, v);
        const float dm = live ? A.qdiam[q] : -1.0f;
        const int *nb = nullptr;
        int cnt = live ? n : 0;
        if (live && A.c.nb.off) {
            cnt = 0x7fffffff;
#pragma unroll
            for (int i = 0; i <= K; ++i) {
                const int o = A.c.nb.off[v[i]], l = A.c.nb.off[v[i] + 1] - o;
                if (l < cnt) {
                    cnt = l;
                    nb = A.c.nb.idx + o;
                }
            }
        }
        const int bin = live ? dim_bin(A, dm) : 0;
        u32 at = 0;
        int total = 0;
        const int zj = kFill && live ? A.qzj[q] : -2;
        // counting: every lane its own hits, added up at the end. Filling:
        // first the count again (to take the bin's next places), then the entries
        for (int pass = 0; pass < (kFill ? 2 : 1); ++pass) {
            int mine = 0;
            u32 put = at;
            for (int s = 0; __any(s < cnt); s += G) {
                const int k = s + lg;
                bool ok = k < cnt;
                int c = 0;
                float x[K + 1];
                if (ok) {
                    c = nb ? nb[k] : k;
                    float mx = 0.0f;
#pragma unroll
                    for (int i = 0; i <= K; ++i) {
                        ok = ok && c != v[i];
                        x[i] = D[(int64_t)v[i] * n + c];
                        mx = fmaxf(mx, x[i]);
                    }
                    ok = ok && mx <= dm;
                    if (ok) {
#pragma unroll
                        for (int i = 0; i <= K; ++i) {
                            float fd = 0.0f;
#pragma unroll
                            for (int j = 0; j <= K; ++j)
                                if (j != i) fd = fmaxf(fd, x[j]);
                            ok = ok && (fd < dm || c > v[i]);
                        }
                    }
                }
                const u64 hit = __ballot(ok) & gmask;
                const u32 e = put + (u32)__popcll(hit & ((1ull << lane) - 1));
                if (kFill && pass == 1 && ok && e >= A.ntau) {
                    A.out->full = kDimBroken;
                } else if (kFill && pass == 1 && ok) {
                    u32 *o = A.tau + (int64_t)e * (K + 2);
                    // over a field other than Z/2 a place has a sign, on the
                    // edge between the triangle's ends
                    const bool odd = A.p != 2;
                    const bool neg_q = odd && c < v[0] && c > v[1];
                    o[0] = (u32)q | (neg_q ? kNeg : 0u);
#pragma unroll
                    for (int i = 0; i <= K; ++i) {
                        int f[K + 1];
                        facet_of<K>(v, i, c, f);
                        const u32 pl = place_of<K>(A, f);
                        const bool neg = odd && (i == 0 ? c > v[0] : c < v[1]);
                        o[1 + i] = pl | (neg ? kNeg : 0u);
                        if (c == zj) A.qdep[(int64_t)i * A.N + q] = pl | (odd && neg == neg_q ? kNeg : 0u);
                    }
                }
                mine += __popcll(hit);
                put += (u32)__popcll(hit);
            }
            if (pass == 0) {
                total = mine; // the same in every lane of the group
                if (live && lg == 0 && total > 0) {
                    at = atomicAdd(&A.bin_t[bin], (u32)total);
                    if (!kFill && at + (u32)total < at) A.out->owned = ~0ull; // the bin has wrapped
                }
                at = __shfl(at, g0, kWave);
            }
        }
    }
}

// The chunks: bins taken together until a chunk holds about as many
// simplices, owned cofacets or columns as the targets say. bin_n and bin_t
// hold the bins' ends here (the placing passes moved them up), bin_s starts.
__global__ void __launch_bounds__(1024) k_dim_chunks(DimArgs A) {
    __shared__ int s_n;
    const u32 total = A.bin_t[A.nbins];
    const float n32 = (float)A.N / 32.0f, t32 = (float)total / 32.0f; // at least 32 chunks, but not tiny ones
    const float wn = A.chunk_n > 0.0f ? 1.0f / A.chunk_n
                                      : 1.0f / fmaxf(fminf(fmaxf(n32, 256.0f), 2048.0f), (float)A.N / 3000.0f);
    const float ws = 1.0f / 192.0f;
    const float wt = 1.0f / fmaxf(fminf(fmaxf(t32, 4096.0f), 16384.0f), (float)total / 3000.0f);
    auto first_n = [&](int b) { return b == 0 ? 0u : A.bin_n[b - 1]; };
    auto first_t = [&](int b) { return b == 0 ? 0u : A.bin_t[b - 1]; };
    auto chunk_of = [&](int b) { // monotone in b: every term is
        const float w = (float)first_n(b) * wn + (float)first_t(b) * wt + (float)A.bin_s[b] * ws;
        return (int)fminf(w, (float)(kDimMaxChunks - 2));
    };
    for (int q = threadIdx.x; q <= kDimMaxChunks; q += kT) A.ch_n[q] = A.ch_t[q] = A.ch_s[q] = ~0u;
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    const int per = A.nbins / kT, b0 = threadIdx.x * per;
    int last = b0 == 0 ? -1 : chunk_of(b0 - 1);
    for (int b = b0; b < b0 + per; ++b) {
        const int c = chunk_of(b);
        if (c != last) { // the chunk's first bin
            A.ch_n[c] = first_n(b);
            A.ch_t[c] = first_t(b);
            A.ch_s[c] = A.bin_s[b];
            atomicMax(&s_n, c + 1);
        }
        last = c;
    }
    __syncthreads();
    if (threadIdx.x < kWave) {
        // close the gaps (chunk numbers no bin fell to)
        const int lane = lane_id();
        int at = 0;
        for (int base = 0; base < s_n; base += kWave) {
            const int c = base + lane;
            const u32 xn = c < s_n ? A.ch_n[c] : ~0u, xt = c < s_n ? A.ch_t[c] : 0, xs = c < s_n ? A.ch_s[c] : 0;
            const u64 bal = __ballot(xn != ~0u);
            const int to = at + __popcll(bal & ((1ull << lane) - 1)); // at most c
            if (xn != ~0u) {
                A.ch_n[to] = xn;
                A.ch_t[to] = xt;
                A.ch_s[to] = xs;
            }
            at += __popcll(bal);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        if (lane == 0) {
            A.ch_n[at] = (u32)A.N;
            A.ch_t[at] = total;
            A.ch_s[at] = (u32)A.S;
            A.out->nch = at;
        }
    }
}

// ---- dimension 2: blocks and their forests

// index of a triangle, of a tetrahedron given in any order
__device__ __forceinline__ int64_t tri_index(int a, int b, int c) {
    const int hi = max(a, max(b, c)), lo = min(a, min(b, c));
    const int v[3] = {hi, a + b + c - hi - lo, lo};
    return index_of<2>(v);
}

__device__ __forceinline__ u32 tri_place(const DimArgs &A, int a, int b, int c) {
    const int64_t idx = tri_index(a, b, c);
    if (A.direct) return A.direct[idx];
    return (u32)ph_find(A.ph, idx);
}

__device__ __forceinline__ u64 tet_index(const DimArgs &A, int a, int b, int c, int d) {
    const int h0 = max(a, b), l0 = min(a, b), h1 = max(c, d), l1 = min(c, d);
    const int x = min(h0, h1), y = max(l0, l1);
    const int v[4] = {max(h0, h1), max(x, y), min(x, y), min(l0, l1)};
    return (u64)simplex_index(v, 3, A.c.B);
}

__device__ __forceinline__ int64_t pair_idx(int a, int b) {
    const int64_t x = max(a, b);
    return x * (x - 1) / 2 + min(a, b);
}

__device__ __forceinline__ bool bit_of(const DimArgs &A, const u32 *t, int a, int b) {
    return (t[(int64_t)a * A.fw + (b >> 5)] >> (b & 31)) & 1u;
}

__device__ __forceinline__ void set_bit(const DimArgs &A, u32 *t, int a, int b) {
    atomicOr(&t[(int64_t)a * A.fw + (b >> 5)], 1u << (b & 31));
    atomicOr(&t[(int64_t)b * A.fw + (a >> 5)], 1u << (a & 31));
}

// vertices of the triangle at a place: the longest edge's two (a > b), and the third
__device__ __forceinline__ void tri_verts(u64 p, int &a, int &b, int &c) {
    c = (int)(p & 0xffff);
    a = (int)((p >> 16) & 0xffff);
    b = (int)((p >> 32) & 0xffff);
}

// the facet of tetrahedron {a, b, c, d} without its vertex x has the minus
// sign in the coboundary: an odd number of the others is below x
__device__ __forceinline__ bool minus_facet(int x, int a, int b, int c, int d) {
    return ((a < x) + (b < x) + (c < x) + (d < x)) & 1;
}

// edge (x, y) of length d comes before edge e of length len and index ei
__device__ __forceinline__ bool edge_before(float d, int x, int y, float len, int64_t ei) {
    return d < len || (d == len && pair_idx(x, y) < ei);
}

struct LuneLds {
    uint16_t c[kLune];   // third vertices, largest first: oldest triangle first
    uint16_t lab[kLune]; // oldest point of the tree; bit 15: the point has an edge
    uint16_t par[kLune];
    u32 kill[kLune];
};

// One wave an edge: its lune counted, or (kPlace) written out, and its forest.
// The edges of the lune in the order of the tetrahedra are all (i, j), i < j,
// by i and then by j: a point with no edge yet joins point i's tree at once, a
// tree is joined by itself (rare) and turned so that its path to point i or j
// leads up. Bound by the distances' gathers, a row of D for a point.
template <bool kPlace>
__global__ void __launch_bounds__(256) k_lune(DimArgs A) {
    __shared__ LuneLds Ls[kPlace ? 4 : 1];
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    const int n = A.c.n;
    const float *D = A.c.d.D;
    const int64_t waves = (int64_t)gridDim.x * 4;
    for (int64_t e = blockIdx.x * 4ll + wave; e < A.nE; e += waves) {
        const int a = __builtin_amdgcn_readfirstlane(A.E.a[e]), b = __builtin_amdgcn_readfirstlane(A.E.b[e]);
        const float len = A.E.diam[e];
        const int64_t ei = pair_idx(a, b);
        const int bin = dim_bin(A, len);
        const int *nb = nullptr;
        int cnt = n;
        if (A.c.nb.off) {
            const int oa = A.c.nb.off[a], ob = A.c.nb.off[b];
            const int la = A.c.nb.off[a + 1] - oa, lb = A.c.nb.off[b + 1] - ob;
            nb = A.c.nb.idx + (la <= lb ? oa : ob);
            cnt = min(la, lb);
        }
        u32 base = 0;
        int size = 0;
        if (kPlace) {
            size = __builtin_amdgcn_readfirstlane((int)A.bcnt[e]);
            if (lane == 0) {
                base = atomicAdd(&A.bin_n[bin], (u32)size); // the bins' first places move up to their ends
                A.bstart[e] = base;
            }
            base = __builtin_amdgcn_readfirstlane(base);
            if (size == 0) continue;
            if (size > kLune || base + (u32)size > (u32)A.N) {
                if (lane == 0) A.out->full = 1;
                continue;
            }
        }
        LuneLds &L = Ls[kPlace ? wave : 0];
        int k = 0;
        for (int s = 0; s < cnt; s += kWave) {
            const int i = s + lane;
            const int c = i < cnt ? (nb ? nb[cnt - 1 - i] : n - 1 - i) : a;
            const float x = D[(int64_t)a * n + c], y = D[(int64_t)b * n + c];
            const bool in = c != a && c != b && x <= len && y <= len;
            if (kPlace && in && (x == len || y == len)) {
                set_bit(A, A.tied, a, b);
                if (x == len) set_bit(A, A.tied, a, c);
                if (y == len) set_bit(A, A.tied, b, c);
            }
            const bool ok = in && edge_before(x, a, c, len, ei) && edge_before(y, b, c, len, ei);
            const u64 hit = __ballot(ok);
            if (kPlace && ok) {
                const int at = k + __popcll(hit & ((1ull << lane) - 1));
                if (at < size) {
                    const u32 q = base + (u32)at;
                    L.c[at] = (uint16_t)c;
                    A.qdiam[q] = len;
                    A.qverts[q] = (u64)c | ((u64)a << 16) | ((u64)b << 32);
                    A.qblk[q] = (u32)e;
                    const int64_t idx = tri_index(a, b, c);
                    if (A.direct) A.direct[idx] = q;
                    else (void)ph_insert(A.ph, idx, (int32_t)q); // room for twice the triangles: it cannot fail
                }
            }
            k += __popcll(hit);
        }
        if (!kPlace) {
            if (lane == 0) {
                A.bcnt[e] = (u32)k;
                atomicAdd(&A.bin_n[bin], (u32)k);
            }
            continue;
        }
        for (int i = lane; i < size; i += kWave) {
            L.lab[i] = (uint16_t)i;
            L.par[i] = 0xffff;
            L.kill[i] = ~0u;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (int i = 0; i + 1 < size; ++i) {
            const int c = __builtin_amdgcn_readfirstlane((int)L.c[i]);
            int li = __builtin_amdgcn_readfirstlane((int)L.lab[i] & 0x7fff);
            for (int s = i + 1; s < size; s += kWave) {
                const int j = s + lane;
                const int d = j < size ? (int)L.c[j] : c;
                const float z = D[(int64_t)c * n + d];
                const bool adj = j < size && edge_before(z, c, d, len, ei);
                const int lj = j < size ? (int)L.lab[j] : li;
                // a tetrahedron of two blocks: no matter, unless it joins trees
                if (j < size && z == len && (lj & 0x7fff) != li) {
                    set_bit(A, A.tied, a, b);
                    set_bit(A, A.tied, c, d);
                }
                const bool single = adj && lj == j; // bit 15 clear, and its own label
                if (single) {
                    L.lab[j] = (uint16_t)(li | 0x8000);
                    L.par[j] = (uint16_t)i;
                    L.kill[j] = ((u32)i << 16) | (u32)j;
                }
                if (__any(single) && lane == 0) L.lab[i] = (uint16_t)(li | 0x8000);
                u64 m = __ballot(adj && !single && (lj & 0x7fff) != li);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                for (; m; m &= m - 1) {
                    const int jj = s + __ffsll((unsigned long long)m) - 1;
                    const int l2 = __builtin_amdgcn_readfirstlane((int)L.lab[jj] & 0x7fff);
                    if (l2 == li) continue;
                    const int young = max(li, l2), old = min(li, l2);
                    if (lane == 0) {
                        int q = l2 == young ? jj : i, up = l2 == young ? i : jj;
                        for (int hops = 0; q != 0xffff && hops < kLune; ++hops) { // the path to the root, turned
                            const int next = L.par[q];
                            L.par[q] = (uint16_t)up;
                            up = q;
                            q = next;
                        }
                        L.kill[young] = ((u32)i << 16) | (u32)jj;
                    }
                    for (int v = lane; v < size; v += kWave)
                        if ((L.lab[v] & 0x7fff) == young) L.lab[v] = (uint16_t)(old | 0x8000);
                    li = old;
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                }
            }
        }
        for (int i = lane; i < size; i += kWave) {
            const u32 up = L.par[i];
            A.qpar[base + i] = up == 0xffff ? ~0u : base + up;
            A.qkill[base + i] = L.kill[i];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

// the facets a triangle's vector is the sum of: its parent, and the two older
// ones of the tetrahedron that joins them; and the lists the other way round
__global__ void __launch_bounds__(256) k_lune_deps(DimArgs A) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    if (A.out->full) return; // places are missing
    for (int64_t q = blockIdx.x * 256ll + threadIdx.x; q < A.N; q += stride) {
        const u32 up = A.qpar[q];
        int a, b, c, a1, b1, d;
        tri_verts(A.qverts[q], a, b, c);
        A.ids[q] = 0;
        if (up >= (u32)A.N) {
            // not the block's oldest: a class, or one of dimension 1 closes
            if (A.bstart[A.qblk[q]] != (u32)q && bit_of(A, A.tied, a, b)) A.out->full = 1;
            continue;
        }
        tri_verts(A.qverts[up], a1, b1, d);
        const u32 dep[3] = {up, tri_place(A, a, c, d), tri_place(A, b, c, d)};
        const int out[3] = {c, b, a}; // the vertex of the tetrahedron that each is without
        for (int i = 0; i < 3; ++i) {
            if (dep[i] >= (u32)A.N) {
                A.out->full = kDimBroken;
                break;
            }
            const u32 o = (u32)(i * A.N + q);
            const bool neg = A.p != 2 && minus_facet(out[i], a, b, c, d) == minus_facet(d, a, b, c, d);
            A.qdep[o] = dep[i] | (neg ? kNeg : 0u);
            A.rnext[o] = atomicExch(&A.rhead[dep[i]], o);
        }
    }
}

// ---- the pairs within blocks that share a simplex with another block of the
// same length (a handful in a cloud of millions of triangles), for dimension
// 3: those of the relative boundary matrix of the blocks together, reduced in
// the filtration's own order. One workgroup a length; the tetrahedra's columns
// are bits over the triangles.
constexpr int kGroupEdges = 8, kGroupTri = 256, kGroupTet = 3072;

__global__ void __launch_bounds__(256) k_lune_ties(DimArgs A) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t e = blockIdx.x * 256ll + threadIdx.x; e < A.nE; e += stride) {
        if (!bit_of(A, A.tied, A.E.a[e], A.E.b[e])) continue;
        if (A.p != 2) A.out->full = 1; // the groups are reduced over Z/2
        const int at = atomicAdd(&A.out->ntied, 1);
        if (at < kTiedMax) A.tlist[at] = (u32)e;
        else A.out->full = 1;
    }
}

__global__ void __launch_bounds__(256) k_lune_groups(DimArgs A) {
    __shared__ int ga[kGroupEdges], gb[kGroupEdges];
    __shared__ int ng, ntri, ntet, lead, bad;
    __shared__ int64_t tri[kGroupTri], row[kGroupTri];  // indices: as found, oldest first
    __shared__ u32 tplace[kGroupTri];
    __shared__ int64_t tet[kGroupTet];
    __shared__ uint16_t order[kGroupTet];
    __shared__ u32 facet[kGroupTet]; // oldest first: the rows of its facets, a byte each, 255 none
    __shared__ u64 stored[kGroupTri][kGroupTri / 64];
    __shared__ int16_t owner[kGroupTri];
    static_assert(kGroupTri == 256, "four words of rows");
    const int n = A.c.n, tid = threadIdx.x;
    const float *D = A.c.d.D;
    const int nt = min(A.out->ntied, kTiedMax);
    for (int t = blockIdx.x; t < nt; t += gridDim.x) {
        const u32 e = A.tlist[t];
        const float len = A.E.diam[e];
        if (tid == 0) {
            ng = ntri = ntet = bad = 0;
            lead = 1;
            for (int q = 0; q < nt; ++q) {
                const u32 f = A.tlist[q];
                if (A.E.diam[f] != len) continue;
                if (f < e) lead = 0; // the group is another workgroup's
                if (ng < kGroupEdges) {
                    ga[ng] = A.E.a[f];
                    gb[ng] = A.E.b[f];
                }
                ++ng;
            }
        }
        __syncthreads();
        const bool mine = lead != 0, few = ng <= kGroupEdges;
        if (mine && !few && tid == 0) A.out->full = 1;
        __syncthreads();
        if (!mine || !few) continue;
        // the triangles on the group's edges, each once
        for (int g = 0; g < ng; ++g) {
            const int a = ga[g], b = gb[g];
            for (int c = tid; c < n; c += 256) {
                if (c == a || c == b || D[(int64_t)a * n + c] > len || D[(int64_t)b * n + c] > len) continue;
                bool seen = false;
                for (int h = 0; h < g; ++h) {
                    const bool x = ga[h] == a || ga[h] == b || ga[h] == c, y = gb[h] == a || gb[h] == b || gb[h] == c;
                    seen = seen || (x && y);
                }
                if (seen) continue;
                const int at = atomicAdd(&ntri, 1);
                if (at < kGroupTri) tri[at] = tri_index(a, b, c);
            }
        }
        __syncthreads();
        const int M = min(ntri, kGroupTri);
        for (int i = tid; i < M; i += 256) {
            int r = 0;
            for (int j = 0; j < M; ++j) r += tri[j] > tri[i] ? 1 : 0;
            row[r] = tri[i];
            owner[i] = -1;
        }
        __syncthreads();
        for (int i = tid; i < M; i += 256) {
            int v[3];
            decode(row[i], 2, n, A.c.B, v);
            tplace[i] = tri_place(A, v[0], v[1], v[2]);
        }
        // the tetrahedra: a triangle and a vertex, each found from the oldest of its triangles
        for (int i = 0; i < M; ++i) {
            int v[3];
            decode(row[i], 2, n, A.c.B, v);
            for (int d = tid; d < n; d += 256) {
                if (d == v[0] || d == v[1] || d == v[2] || D[(int64_t)v[0] * n + d] > len ||
                    D[(int64_t)v[1] * n + d] > len || D[(int64_t)v[2] * n + d] > len)
                    continue;
                bool first = true;
                for (int q = 0; q < 3; ++q) {
                    const int64_t f = tri_index(d, v[q == 0 ? 1 : 0], v[q == 2 ? 1 : 2]);
                    for (int j = 0; j < i; ++j) first = first && row[j] != f;
                }
                if (!first) continue;
                const int at = atomicAdd(&ntet, 1);
                if (at < kGroupTet) tet[at] = (int64_t)tet_index(A, v[0], v[1], v[2], d);
            }
        }
        __syncthreads();
        const int T = min(ntet, kGroupTet);
        if (tid == 0 && (ntri >= kGroupTri || ntet > kGroupTet)) {
            A.out->full = 1;
            bad = 1;
        }
        for (int i = tid; i < T; i += 256) {
            int r = 0;
            for (int j = 0; j < T; ++j) r += tet[j] > tet[i] ? 1 : 0;
            order[r] = (uint16_t)i;
            int w[4];
            decode(tet[i], 3, n, A.c.B, w);
            u32 fs = 0;
            for (int q = 0; q < 4; ++q) {
                const int64_t f = tri_index(w[q == 0 ? 1 : 0], w[q <= 1 ? 2 : 1], w[q == 3 ? 2 : 3]);
                int lo = 0, hi = M; // row is descending
                while (lo < hi) {
                    const int mid = (lo + hi) / 2;
                    if (row[mid] > f) lo = mid + 1;
                    else hi = mid;
                }
                fs |= (lo < M && row[lo] == f ? (u32)lo : 255u) << (8 * q);
            }
            facet[r] = fs;
        }
        __syncthreads();
        if (tid == 0 && !bad) {
            for (int k = 0; k < T; ++k) {
                u64 x[kGroupTri / 64] = {};
                for (int q = 0; q < 4; ++q) {
                    const u32 f = (facet[k] >> (8 * q)) & 255u;
                    for (int y = 0; y < kGroupTri / 64; ++y)
                        if (f != 255u && (int)(f >> 6) == y) x[y] |= 1ull << (f & 63);
                }
                for (;;) {
                    const int pv = x[3] ? 255 - __clzll((long long)x[3])
                                 : x[2] ? 191 - __clzll((long long)x[2])
                                 : x[1] ? 127 - __clzll((long long)x[1])
                                 : x[0] ? 63 - __clzll((long long)x[0]) : -1;
                    if (pv < 0) break;
                    if (owner[pv] < 0) {
                        owner[pv] = (int16_t)order[k];
                        for (int y = 0; y < kGroupTri / 64; ++y) stored[pv][y] = x[y];
                        const int at = atomicAdd(&A.out->npairs_tied, 1);
                        if (at < kTiedPairs) {
                            A.tplace[at] = tplace[pv];
                            A.ttet[at] = tet[order[k]];
                        } else {
                            A.out->full = 1;
                        }
                        break;
                    }
                    for (int y = 0; y < kGroupTri / 64; ++y) x[y] ^= stored[pv][y];
                }
            }
        }
        __syncthreads();
    }
}

// The columns that are roots of their block's forest, in column order; the
// others pair with the tetrahedron at which their tree was joined to an older
// one. One workgroup.
__global__ void __launch_bounds__(1024) k_lune_classes(DimArgs A, PivotHash piv) {
    __shared__ int s_w[kWaves];
    __shared__ int s_red, s_emg, s_full;
    const int lane = lane_id(), w = threadIdx.x / kWave;
    if (threadIdx.x == 0) {
        s_red = s_emg = 0;
        s_full = A.out->full;
    }
    __syncthreads();
    if (s_full) return; // places are missing
    int at = 0, red = 0, emg = 0;
    for (int c0 = 0; c0 < A.nall; c0 += kT) {
        const int col = c0 + (int)threadIdx.x;
        bool root = false;
        if (col < A.nall) {
            int v[3];
            decode(A.all.idx[col], 2, A.c.n, A.c.B, v);
            const u32 q = min(tri_place(A, v[0], v[1], v[2]), (u32)A.N - 1);
            const u32 start = A.bstart[A.qblk[q]], k = A.qkill[q];
            int a, b, c, d, a1, b1, own;
            tri_verts(A.qverts[q], a, b, own);
            root = A.qpar[q] >= (u32)A.N;
            const u32 q1 = start + (k >> 16), q2 = start + (k & 0xffff);
            const bool tied = bit_of(A, A.tied, a, b);
            int64_t t = -1;
            if (root && start != q) {
                // a class
            } else if (tied) {
                root = false;
                if (A.strict) { // the forest's pair may not be the filtration's
                    const int nt = min(A.out->npairs_tied, kTiedPairs);
                    for (int i = 0; i < nt; ++i)
                        if (A.tplace[i] == q) t = A.ttet[i];
                    if (t < 0) A.out->full = 1;
                }
            } else if (root) { // the block's oldest triangle pairs with the edge: no column
                root = false;
                A.out->full = kDimBroken;
            } else if (k == ~0u || q1 >= (u32)A.N || q2 >= (u32)A.N) {
                A.out->full = kDimBroken;
            } else {
                tri_verts(A.qverts[q1], a1, b1, c);
                tri_verts(A.qverts[q2], a1, b1, d);
                t = (int64_t)tet_index(A, a, b, c, d);
            }
            if (t >= 0) (void)ph_insert(piv, t, col);
            if (!root) {
                const int j = A.all.j[col];
                if (j >= 0 && t == (int64_t)tet_index(A, a, b, own, j)) ++emg;
                else ++red;
            }
        }
        const u64 bal = __ballot(root);
        if (lane == 0) s_w[w] = __popcll(bal);
        __syncthreads();
        int base = at, tot = 0;
        for (int q = 0; q < kWaves; ++q) {
            if (q < w) base += s_w[q];
            tot += s_w[q];
        }
        if (root) {
            const int o = base + __popcll(bal & ((1ull << lane) - 1));
            A.cols.idx[o] = A.all.idx[col];
            A.cols.diam[o] = A.all.diam[col];
            A.cols.j[o] = A.all.j[col];
        }
        at += tot;
        __syncthreads();
    }
    if (red) atomicAdd(&s_red, red);
    if (emg) atomicAdd(&s_emg, emg);
    __syncthreads();
    if (threadIdx.x == 0) {
        A.out->nclasses = at;
        A.out->loc_reduced = s_red;
        A.out->loc_emergent = s_emg;
        if (A.bin_n[A.nbins] != (u32)A.N) A.out->full = kDimBroken; // every triangle has one block
    }
}

// place of every column, oldest first
template <int K>
__global__ void __launch_bounds__(256) k_dim_births(DimArgs A) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t c = blockIdx.x * 256ll + threadIdx.x; c < A.S; c += stride) {
        int v[K + 1];
        decode(A.cols.idx[c], K, A.c.n, A.c.B, v);
        A.bq[A.S - 1 - c] = place_of<K>(A, v);
        A.kidx[c] = -1;
    }
}

// ---- the sweep
struct DimShared {
    int nrows, nact, nfree, ndead, nnz, ncand, nkill, fail, since;
    int sfree;                       // free slots
    int again;
    unsigned long long adds, rows;
    u32 hi_d;
    u64 hi_i;
    int kp[kCand], ki[kCand];
    u64 kz[kCand];                   // nonzero words of a kill's vector
    u32 kinv[kCand];                 // kOdd: the inverse of its coefficient
    uint16_t ord[kCand];             // oldest first
    u32 cd[kCand];                   // candidates: diameter bits (~0: done)
    u64 ci[kCand], cz[kCand];        // ~index, nonzero words
    u32 sage[kDimSlots];             // class of a slot
    uint16_t urow[kDimSlots];        // an open class's unit row, by slot
    uint16_t sl[kDimSlots];          // free slots
};

__device__ __forceinline__ bool key_less(u32 d0, u64 i0, u32 d1, u64 i1) { return d0 < d1 || (d0 == d1 && i0 < i1); }

// place of candidate i among the first n by age; their keys are distinct, and
// were they not, every place would still have one candidate
__device__ __forceinline__ int rank_of(const DimShared &Sh, int n, int i) {
    const u32 d = Sh.cd[i];
    const u64 x = Sh.ci[i];
    int at = 0;
    for (int q = 0; q < n; ++q) {
        const u32 dq = Sh.cd[q];
        const u64 xq = Sh.ci[q];
        at += key_less(dq, xq, d, x) || (dq == d && xq == x && q < i) ? 1 : 0;
    }
    return at;
}

__device__ __forceinline__ u64 lane_u64(u64 x, int l) {
    const u32 lo = __builtin_amdgcn_readlane((u32)x, l), hi = __builtin_amdgcn_readlane((u32)(x >> 32), l);
    return ((u64)hi << 32) | lo;
}

// nonzero and pairwise different rows among r[0..M): equal ones cancel
template <int M>
__device__ __forceinline__ int cancel(u32 (&r)[M]) {
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
        for (int j = i + 1; j < M; ++j)
            if (r[i] == r[j]) r[i] = r[j] = 0;
    int k = 0;
#pragma unroll
    for (int i = 0; i < M; ++i) k += r[i] != 0 ? 1 : 0;
    return k;
}

// one nonzero word, with one bit?
__device__ __forceinline__ bool is_unit(u64 z, u32 word) {
    return z != 0 && (z & (z - 1)) == 0 && (word & (word - 1)) == 0;
}

template <int M>
__device__ __forceinline__ u64 sum_words(const DimArgs &A, const u32 (&r)[M]) {
    u64 z = 0;
#pragma unroll
    for (int i = 0; i < M; ++i)
        if (r[i]) z |= A.rsum[r[i]];
    return z;
}

template <int M>
__device__ __forceinline__ u32 sum_word(const DimArgs &A, const u32 (&r)[M], int w) {
    u32 x = 0;
#pragma unroll
    for (int i = 0; i < M; ++i)
        if (r[i]) x ^= A.pool[(int64_t)r[i] * A.W + w];
    return x;
}

// the three edges of the triangle at place q have one with a nonzero vector
__device__ __forceinline__ void mark(const DimArgs &A, u32 q) {
    int a, b, c;
    tri_verts(A.qverts[q], a, b, c);
    set_bit(A, A.fl, a, b);
    set_bit(A, A.fl, a, c);
    set_bit(A, A.fl, b, c);
}

// the triangles whose sum the one at place q is part of have to be looked at
__device__ __forceinline__ void call_on(const DimArgs &A, u32 q) {
    u32 o = A.rhead[q];
    for (int hops = 0; o < 3u * (u32)A.N && hops < 3 * kDimMaxVert; ++hops) {
        const u32 s = o % (u32)A.N;
        atomicOr(&A.need[s >> 5], 1u << (s & 31));
        o = A.rnext[o];
    }
}

// ---- kOdd, a field other than Z/2: a simplex's id is a row (low half) and a
// coefficient in [1, p), or 0. A row is its W words of bits, set where the
// residue is not zero, and then a 16-bit residue for every slot.
constexpr int kOddStride = 17; // words of a row for each word of bits

__device__ __forceinline__ u32 odd_neg(u32 id, bool neg, u32 p) {
    return id && neg ? (id & 0xffffu) | ((p - (id >> 16)) << 16) : id;
}

// what the row map makes of an id
template <class Map>
__device__ __forceinline__ u32 odd_resolve(Map rmap, u32 id, u32 p) {
    if (!id) return 0;
    const u32 to = rmap[id & (kOddRows - 1)];
    return to ? (to & 0xffffu) | (odd_mul(to >> 16, id >> 16, p) << 16) : 0u;
}

// multiples of one row are added up; the number of nonzero ids left
template <int M>
__device__ __forceinline__ int odd_cancel(u32 (&r)[M], u32 p) {
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
        for (int j = i + 1; j < M; ++j)
            if (r[i] && r[j] && ((r[i] ^ r[j]) & 0xffffu) == 0) {
                const u32 c = ((r[i] >> 16) + (r[j] >> 16)) % p;
                r[i] = c ? (r[i] & 0xffffu) | (c << 16) : 0u;
                r[j] = 0;
            }
    int k = 0;
#pragma unroll
    for (int i = 0; i < M; ++i) k += r[i] != 0 ? 1 : 0;
    return k;
}

__device__ __forceinline__ const u32 *odd_row(const DimArgs &A, u32 id) {
    return A.pool + (int64_t)(id & 0xffffu) * (A.W * kOddStride);
}

template <int M>
__device__ __forceinline__ u64 odd_words(const DimArgs &A, const u32 (&r)[M]) {
    u64 z = 0;
#pragma unroll
    for (int i = 0; i < M; ++i)
        if (r[i]) z |= A.rsum[r[i] & 0xffffu];
    return z;
}

// put(slot, residue) for every nonzero residue of the sum, bits(word, bits) for every word with one
template <int M, class Put, class Bits>
__device__ __forceinline__ void odd_sum(const DimArgs &A, const u32 (&r)[M], Put put, Bits bits) {
    for (u64 zz = odd_words<M>(A, r); zz; zz &= zz - 1) {
        const int w = __ffsll((unsigned long long)zz) - 1;
        u32 has[M], all = 0, out = 0;
#pragma unroll
        for (int i = 0; i < M; ++i) all |= has[i] = r[i] ? odd_row(A, r[i])[w] : 0u;
        for (u32 m = all; m; m &= m - 1) {
            const u32 bit = m & (0u - m);
            const int slot = w * 32 + __ffs((int)m) - 1;
            u64 t = 0;
#pragma unroll
            for (int i = 0; i < M; ++i)
                if (has[i] & bit) t += (u64)(r[i] >> 16) * ((const uint16_t *)(odd_row(A, r[i]) + A.W))[slot];
            const u32 x = (u32)(t % A.p);
            if (!x) continue;
            out |= bit;
            put(slot, x);
        }
        if (out) bits(w, out);
    }
}

template <int M>
__device__ __forceinline__ u32 odd_row_of_sum(const DimArgs &A, DimShared &Sh, LDS u32 *rmap, u32 (&r)[M]) {
    const int k = odd_cancel<M>(r, A.p);
    u32 x = 0;
#pragma unroll
    for (int i = 0; i < M; ++i) x |= r[i];
    if (k <= 1) return x;
    int cnt = 0, at = 0;
    u32 val = 0;
    u64 z = 0;
    odd_sum<M>(A, r, [&](int slot, u32 y) {
        ++cnt;
        at = slot;
        val = y;
    }, [&](int w, u32) { z |= 1ull << w; });
    if (cnt == 0) return 0;
    if (cnt == 1) return Sh.urow[at] | (val << 16);
    const int f = atomicSub(&Sh.nfree, 1);
    const u32 row = f > 0 ? A.rfree[f - 1] : (u32)atomicAdd(&Sh.nrows, 1);
    if (row >= (u32)kOddRows) {
        Sh.fail = 1;
        return 0;
    }
    u32 *o = A.pool + (int64_t)row * (A.W * kOddStride);
    for (int w = 0; w < A.W; ++w) o[w] = 0;
    odd_sum<M>(A, r, [&](int slot, u32 y) { ((uint16_t *)(o + A.W))[slot] = (uint16_t)y; },
               [&](int w, u32 b) { o[w] = b; });
    A.rsum[row] = z;
    rmap[row] = row | (1u << 16);
    A.ract[atomicAdd(&Sh.nact, 1)] = row;
    atomicAdd(&Sh.rows, 1ull);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    return row | (1u << 16);
}

// x less f times kv, both bits and residues, in the words z of kv; the
// nonzero words of x, which were zx
template <class Word, class Half>
__device__ __forceinline__ u64 odd_less(Word *x, Half *xr, u32 f, const LDS u32 *kv, int W, u64 z, u64 zx, u32 p) {
    const LDS uint16_t *kr = (const LDS uint16_t *)(kv + W);
    for (u64 m = z; m; m &= m - 1) {
        const int w = __ffsll((unsigned long long)m) - 1;
        u32 bits = x[w];
        for (u32 b = kv[w]; b; b &= b - 1) {
            const u32 bit = b & (0u - b);
            const int slot = w * 32 + __ffs((int)b) - 1;
            const u32 y = (u32)(((bits & bit ? (u32)xr[slot] : 0u) + (u64)(p - f) * kr[slot]) % p);
            if (y) xr[slot] = (uint16_t)y;
            bits = y ? bits | bit : bits & ~bit;
        }
        x[w] = bits;
        zx = bits ? zx | (1ull << w) : zx & ~(1ull << w);
    }
    return zx;
}

// the sweep's LDS in global memory: DimShared, then the row map
constexpr int kStateWords = sizeof(DimShared) / 4;
constexpr int kStateScalars = offsetof(DimShared, kp) / 4; // of them those before the arrays

// ---- dimension 2: the tetrahedra e + {c, d} of a chunk's blocks whose facets
// do not cancel. One wave a triangle e + c, its lanes the d's of the block;
// most have no nonzero triangle on the edges (a, c) and (b, c) and nothing to
// do. A facet (a, c, d) can be nonzero only if each of its edges has a
// nonzero triangle, which leaves few pairs to look up (of the 39 million
// tetrahedra of 192 points on the sphere 1 to 2 million). By the whole chip:
// one workgroup took 60 ms for that cloud, its lookups one line a clock.
template <bool kOdd>
__global__ void __launch_bounds__(256) k_lune_tests(DimArgs A, int chunk) {
    if (chunk >= A.out->nch || A.out->full) return;
    const DimShared *S = (const DimShared *)A.state;
    if (S->nnz == 0) return;
    using Map = typename std::conditional<kOdd, u32, uint16_t>::type;
    const Map *rmap = (const Map *)((const u32 *)A.state + kStateWords);
    auto resolve = [&](u32 id) -> u32 {
        if constexpr (kOdd) return odd_resolve(rmap, id, A.p);
        else return rmap[id & (kDimRows - 1)] & (kDimRows - 1);
    };
    const int lane = lane_id(), n = A.c.n;
    const float *D = A.c.d.D;
    const u32 n0 = A.ch_n[chunk], n1 = A.ch_n[chunk + 1], waves = gridDim.x * 4;
    for (u32 q = n0 + blockIdx.x * 4 + threadIdx.x / kWave; q < n1; q += waves) {
        int a, b, c;
        tri_verts(A.qverts[q], a, b, c);
        const u32 own = resolve(A.ids[q]);
        const bool fa = bit_of(A, A.fl, a, c), fb = bit_of(A, A.fl, b, c);
        if (!own && !fa && !fb) continue;
        const u32 blk = A.qblk[q], start = A.bstart[blk], size = A.bcnt[blk];
        const float len = A.qdiam[q];
        const int64_t ei = pair_idx(a, b);
        for (u32 s = 0; s < size; s += kWave) {
            const u32 j = s + (u32)lane, qd = min(start + min(j, size - 1), (u32)A.N - 1);
            const int d = (int)(A.qverts[qd] & 0xffff);
            bool ok = j < size && qd != q;
            const float z = D[(int64_t)c * n + d];
            const u32 other = resolve(A.ids[qd]);
            const bool fc = bit_of(A, A.fl, c, d);
            const bool ta = fc && fa && bit_of(A, A.fl, a, d), tb = fc && fb && bit_of(A, A.fl, b, d);
            ok = ok && edge_before(z, c, d, len, ei) && (own || ta || tb);
            // from d's side too, if that looks at it: only from the first
            ok = ok && !(qd < q && (other || ta || tb));
            if (!__any(ok)) continue;
            u32 r[4] = {own, other, 0, 0};
            if (ok && ta) r[2] = tri_place(A, a, c, d);
            if (ok && tb) r[3] = tri_place(A, b, c, d);
            if (ok && ((ta && r[2] >= (u32)A.N) || (tb && r[3] >= (u32)A.N))) A.out->full = kDimBroken;
            r[2] = ta ? resolve(A.ids[min(r[2], (u32)A.N - 1)]) : 0;
            r[3] = tb ? resolve(A.ids[min(r[3], (u32)A.N - 1)]) : 0;
            bool nonzero = false;
            if constexpr (kOdd) {
                const int out[4] = {d, c, b, a};
#pragma unroll
                for (int i = 0; i < 4; ++i) r[i] = odd_neg(r[i], minus_facet(out[i], a, b, c, d), A.p);
                if (ok && odd_cancel<4>(r, A.p) > 0) odd_sum<4>(A, r, [&](int, u32) { nonzero = true; }, [](int, u32) {});
            } else if (ok && cancel<4>(r) > 0)
                for (u64 m = sum_words<4>(A, r); m && !nonzero; m &= m - 1)
                    nonzero = sum_word<4>(A, r, __ffsll((unsigned long long)m) - 1) != 0;
            const int at = wave_place(nonzero, &A.out->npair);
            if (nonzero && at < A.paircap) A.pairs[at] = ((u64)q << 32) | (u32)d;
            // too many: the sweep ends after this, and the count goes no
            // further than one append of every wave takes it
            if (__any(nonzero && at >= A.paircap)) return;
        }
    }
}

// The lanes with `ok` hold cofacets that do not cancel (rows r, key (kd, ki),
// nonzero words z): of those with the same rows the oldest becomes a
// candidate. No cofacet is found twice: a triangle is owned by one edge, and a
// tetrahedron is listed from one side of its block's edge.
template <bool kOdd, int M>
__device__ __forceinline__ void candidates(const DimArgs &A, DimShared &Sh, LDS u32 *vec, int ccap, const u32 (&r)[M],
                                           bool ok, u32 kd, u64 ki, u64 z) {
    const int lane = lane_id();
    for (u64 todo = __ballot(ok); todo;) {
        int l = __ffsll((unsigned long long)todo) - 1;
        bool same = ok;
#pragma unroll
        for (int i = 0; i < M; ++i) same = same & (r[i] == (u32)__builtin_amdgcn_readlane(r[i], l));
        const u64 sm = __ballot(same);
        todo &= ~sm;
        for (u64 m = sm; m; m &= m - 1) { // the oldest of them
            const int j = __ffsll((unsigned long long)m) - 1;
            const u32 jd = __builtin_amdgcn_readlane(kd, j), bd = __builtin_amdgcn_readlane(kd, l);
            const u64 ji = lane_u64(ki, j), bi = lane_u64(ki, l);
            if (key_less(jd, ji, bd, bi)) l = j;
        }
        if (lane == l) {
            const int s = atomicAdd(&Sh.ncand, 1);
            if (s < ccap) {
                Sh.cd[s] = kd;
                Sh.ci[s] = ki;
                Sh.cz[s] = z;
                if constexpr (kOdd) {
                    LDS u32 *o = vec + s * A.W * kOddStride;
                    for (int w = 0; w < A.W; ++w) o[w] = 0;
                    odd_sum<M>(A, r, [&](int slot, u32 y) { ((LDS uint16_t *)(o + A.W))[slot] = (uint16_t)y; },
                               [&](int w, u32 b) { o[w] = b; });
                } else
                    for (int w = 0; w < A.W; ++w) vec[s * A.W + w] = (z >> w) & 1ull ? sum_word<M>(A, r, w) : 0u;
            }
        }
    }
}

// The row of the sum of the rows r: an old one where the sum is one of them,
// zero or a unit vector, else a new one.
template <int M>
__device__ __forceinline__ u32 row_of_sum(const DimArgs &A, DimShared &Sh, LDS uint16_t *rmap, u32 (&r)[M]) {
    const int W = A.W;
        const int k = cancel<M>(r);
        u32 x = 0;
#pragma unroll
        for (int i = 0; i < M; ++i) x |= r[i];
        if (k > 1) {
            u64 z = 0;
            u32 one = 0; // the only nonzero word
            for (u64 m = sum_words<M>(A, r); m; m &= m - 1) {
                const int w = __ffsll((unsigned long long)m) - 1;
                const u32 y = sum_word<M>(A, r, w);
                if (y) {
                    z |= 1ull << w;
                    one = y;
                }
            }
            x = 0;
            if (is_unit(z, one)) {
                x = Sh.urow[(__ffsll((unsigned long long)z) - 1) * 32 + __ffs((int)one) - 1];
            } else if (z) {
                const int f = atomicSub(&Sh.nfree, 1);
                if (f > 0) x = A.rfree[f - 1];
                else x = (u32)atomicAdd(&Sh.nrows, 1);
                if (x < (u32)kDimRows) {
                    for (int w = 0; w < W; ++w) A.pool[(int64_t)x * W + w] = sum_word<M>(A, r, w);
                    A.rsum[x] = z;
                    rmap[x] = (uint16_t)x;
                    A.ract[atomicAdd(&Sh.nact, 1)] = x;
                    atomicAdd(&Sh.rows, 1ull);
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                } else {
                    x = 0;
                    Sh.fail = 1;
                }
            }
        }
    return x;
}

// A row's vector is shared by all simplices that hold its number, and rows
// with equal unit vectors are one row: a row that becomes zero or a unit
// vector keeps its number on the simplices and is replaced on the way, by
// rmap (most sums that cancel are of two such rows, and then cost no look at
// the vectors). Every kPurge eliminations the simplices' numbers are brought
// up to date and the replaced rows are free again.
template <int K, bool kOdd>
__global__ void __launch_bounds__(kT) k_dim_sweep(DimArgs A, int chunk) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ DimShared Sh;
    LDS u32 *vec = (LDS u32 *)smem;                                // kWords
    using Map = typename std::conditional<kOdd, u32, uint16_t>::type;
    constexpr int kRows = kOdd ? kOddRows : kDimRows, kWords = kOdd ? kOddWords : kCandWords;
    LDS Map *rmap = (LDS Map *)(smem + kWords * 4);                // kRows
    const u32 p = A.p;
    // the id that an id stands for, and a row's own
    auto resolve = [&](u32 id) -> u32 {
        if constexpr (kOdd) return odd_resolve(rmap, id, p);
        else return rmap[id & (kDimRows - 1)] & (kDimRows - 1);
    };
    auto own_id = [&](u32 row) -> u32 { return kOdd ? row | (1u << 16) : row; };
    const int tid = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int W = A.W;
    [[maybe_unused]] const int n = A.c.n;
    const int PW = kOdd ? W * kOddStride : W; // words of a row
    const int nslots = W * 32, ccap = min(kCand, kWords / PW);
    const int nch = __builtin_amdgcn_readfirstlane(A.out->nch);
    const bool more = K == 2 && chunk > 0; // the tables as the launch before left them
    if (more) {
        if (chunk > nch || A.out->full) return;
        const DimShared *S = (const DimShared *)A.state;
        const u32 *from = (const u32 *)S, *rm = from + kStateWords;
        const int rows = S->nrows;
        for (int i = tid; i < kStateScalars; i += kT) ((LDS u32 *)&Sh)[i] = from[i];
        for (int i = tid; i < nslots; i += kT) {
            Sh.sage[i] = S->sage[i];
            Sh.urow[i] = S->urow[i];
            Sh.sl[i] = S->sl[i];
        }
        for (int i = tid; i * (kOdd ? 1 : 2) < rows; i += kT) ((LDS u32 *)rmap)[i] = rm[i];
    } else {
        if (tid == 0) {
            Sh.nact = Sh.nnz = Sh.nfree = Sh.ndead = Sh.since = 0;
            Sh.fail = A.out->full; // what the passes before found
            Sh.nrows = 1; // row 0: the zero vector
            rmap[0] = 0;
            Sh.sfree = nslots;
            Sh.adds = Sh.rows = 0;
        }
        for (int q = tid; q < nslots; q += kT) Sh.sl[q] = (uint16_t)(nslots - 1 - q);
    }
    __syncthreads();
    // dimension 2: the end of the chunk before, whose cofacets k_lune_tests has
    // looked at meanwhile, and the vectors of this one
    for (int ch = K == 2 ? max(chunk - 1, 0) : 0; ch < (K == 2 ? min(chunk + 1, nch) : nch); ++ch) {
        const bool vectors = K == 1 || ch == chunk;
        const u32 n0 = A.ch_n[ch], n1 = A.ch_n[ch + 1], t0 = A.ch_t[ch], t1 = A.ch_t[ch + 1];
        const int s0 = (int)A.ch_s[ch], s1 = (int)A.ch_s[ch + 1];
        // ---- the classes that open here
        if (vectors && s1 > s0) {
            const int ns = s1 - s0, nf = Sh.sfree, nr = Sh.nfree, top = Sh.nrows, na = Sh.nact, nz = Sh.nnz;
            const int fresh = max(0, ns - nr);
            if (ns > nf || top + fresh > kRows || (int64_t)nz + ns > A.N) { // (a triangle may be listed twice)
                __syncthreads();
                if (tid == 0) Sh.fail = 1;
                __syncthreads();
                break;
            }
            __syncthreads();
            for (int i = tid; i < ns; i += kT) {
                const int slot = Sh.sl[nf - 1 - i];
                const u32 r = i < nr ? A.rfree[nr - 1 - i] : (u32)(top + i - nr);
                Sh.sage[slot] = (u32)(s0 + i);
                for (int w = 0; w < W; ++w) A.pool[(int64_t)r * PW + w] = w == (slot >> 5) ? 1u << (slot & 31) : 0u;
                if constexpr (kOdd) ((uint16_t *)(A.pool + (int64_t)r * PW + W))[slot] = 1;
                A.rsum[r] = 1ull << (slot >> 5);
                rmap[r] = (Map)own_id(r);
                Sh.urow[slot] = (uint16_t)r;
                A.ract[na + i] = r;
                const u32 pl = A.bq[s0 + i];
                if (pl >= (u32)A.N) Sh.fail = kDimBroken;
                const u32 q = min(pl, (u32)A.N - 1);
                A.ids[q] = own_id(r);
                A.nzl[nz + i] = q;
                if constexpr (K == 2) {
                    mark(A, q);
                    call_on(A, q);
                }
            }
            if (tid == 0) {
                Sh.sfree = nf - ns;
                Sh.nfree = max(0, nr - ns);
                Sh.nrows = top + fresh;
                Sh.nact = na + ns;
                Sh.nnz = nz + ns;
                Sh.rows += ns;
            }
            __syncthreads();
        }
        // ---- the vectors of the chunk's simplices (see rips_sweep.hip)
        if constexpr (K == 1)
        for (int tries = 0;; ++tries) {
            bool left = false;
            for (u32 q = n0 + tid; q < n1; q += kT) {
                if (ld(&A.ids[q]) != kPending) continue;
                u32 r[K + 1];
#pragma unroll
                for (int i = 0; i <= K; ++i) {
                    const u32 part = A.qdep[(int64_t)i * A.N + q], pl = kOdd ? part & ~kNeg : part;
                    if (pl >= (u32)A.N) Sh.fail = kDimBroken;
                    r[i] = ld(&A.ids[min(pl, (u32)A.N - 1)]);
                    if (kOdd && r[i] != kPending) r[i] = odd_neg(r[i], (part & kNeg) != 0, p);
                }
                bool wait = false;
#pragma unroll
                for (int i = 0; i <= K; ++i) wait = wait || r[i] == kPending;
                if (wait) {
                    left = true;
                    continue;
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
#pragma unroll
                for (int i = 0; i <= K; ++i) {
                    if ((kOdd ? r[i] & 0xffffu : r[i]) >= (u32)kRows) Sh.fail = kDimBroken;
                    r[i] = resolve(r[i]);
                }
                u32 x;
                if constexpr (kOdd) x = odd_row_of_sum<K + 1>(A, Sh, rmap, r);
                else x = row_of_sum<K + 1>(A, Sh, rmap, r);
                if (x) A.nzl[atomicAdd(&Sh.nnz, 1)] = q;
                st(&A.ids[q], x);
            }
            if (!__any(left)) break;
            if (tries > (1 << 16)) { // cannot happen: the order is acyclic
                Sh.fail = 1;
                break;
            }
        }
        // dimension 2: only the triangles that a nonzero one calls on. A sum
        // taken too early is taken again: its last part calls once more.
        if constexpr (K == 2)
        if (vectors) {
            const u32 w0 = n0 >> 5, w1 = n1 > n0 ? ((n1 - 1) >> 5) + 1 : w0;
            for (int tries = 0;; ++tries) {
                if (tid == 0) Sh.again = 0;
                __syncthreads();
                for (u32 w = w0 + tid; w < w1; w += kT) {
                    const u32 from = w * 32 < n0 ? n0 & 31 : 0, to = n1 - w * 32 < 32 ? n1 & 31 : 32;
                    const u32 in = (to == 32 ? ~0u : (1u << to) - 1) & ~((1u << from) - 1);
                    u32 m = ld(&A.need[w]) & in;
                    if (!m) continue;
                    atomicAnd(&A.need[w], ~m);
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
                    Sh.again = 1;
                    for (; m; m &= m - 1) {
                        const u32 q = w * 32 + (u32)__ffs((int)m) - 1;
                        u32 r[3];
#pragma unroll
                        for (int i = 0; i < 3; ++i) {
                            const u32 part = A.qdep[(int64_t)i * A.N + q];
                            r[i] = ld(&A.ids[min(kOdd ? part & ~kNeg : part, (u32)A.N - 1)]);
                            if ((kOdd ? r[i] & 0xffffu : r[i]) >= (u32)kRows) Sh.fail = kDimBroken;
                            if constexpr (kOdd) r[i] = odd_neg(r[i], (part & kNeg) != 0, p);
                        }
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
#pragma unroll
                        for (int i = 0; i < 3; ++i) r[i] = resolve(r[i]);
                        const u32 was = ld(&A.ids[q]);
                        u32 x;
                        if constexpr (kOdd) x = odd_row_of_sum<3>(A, Sh, rmap, r);
                        else x = row_of_sum<3>(A, Sh, rmap, r);
                        if (x == was) continue;
                        st(&A.ids[q], x);
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                        if (!was) {
                            const int at = atomicAdd(&Sh.nnz, 1);
                            if (at < (int)A.N) A.nzl[at] = q;
                            else Sh.fail = 1;
                            mark(A, q);
                        }
                        call_on(A, q);
                    }
                }
                __syncthreads();
                const bool again = Sh.again != 0;
                __syncthreads();
                if (!again) break;
                if (tries > (1 << 16)) { // cannot happen: the order is acyclic
                    if (tid == 0) Sh.fail = 1;
                    break;
                }
            }
        }
        __syncthreads();
        const bool none = Sh.nnz == 0, failed = Sh.fail != 0;
        if (tid == 0 && Sh.nfree < 0) Sh.nfree = 0;
        __syncthreads();
        if (failed) break;
        if (K == 2 && vectors) break; // the last chunk of this launch
        if (none) continue;
        const int np = K == 2 ? __builtin_amdgcn_readfirstlane(A.out->npair) : 0;
        if (K == 2 && np > A.paircap) {
            if (tid == 0) Sh.fail = 1;
            __syncthreads();
            break;
        }
        if (K == 2 && np == 0) continue;
        // ---- the owned cofacets whose facets do not cancel
        u32 lo_d = 0, hi_d = ~0u;
        u64 lo_i = 0, hi_i = ~0ull;
        bool first = true;
        for (;;) {
            if (tid == 0) Sh.ncand = 0;
            __syncthreads();
            if constexpr (K == 1) {
            for (u32 b = t0 + (u32)wave * kWave; b < t1; b += kTaus * kT) {
                // kTaus of them a lane, so that their loads are in flight together
                u32 qs[kTaus], rs[kTaus][K + 2];
                bool some = false, broken = false;
#pragma unroll
                for (int u = 0; u < kTaus; ++u) {
                    const u32 t = min(b + u * kT + (u32)lane, t1 - 1);
                    const u32 *o = A.tau + (int64_t)t * (K + 2);
                    qs[u] = kOdd ? o[0] & ~kNeg : o[0];
#pragma unroll
                    for (int i = 0; i < K + 2; ++i) rs[u][i] = o[i];
                }
#pragma unroll
                for (int u = 0; u < kTaus; ++u)
#pragma unroll
                    for (int i = 0; i < K + 2; ++i) {
                        const u32 part = rs[u][i], pl = kOdd ? part & ~kNeg : part;
                        broken = broken | (pl >= (u32)A.N);
                        rs[u][i] = A.ids[min(pl, (u32)A.N - 1)];
                        if constexpr (kOdd) rs[u][i] = odd_neg(rs[u][i], (part & kNeg) != 0, p);
                    }
#pragma unroll
                for (int u = 0; u < kTaus; ++u) {
#pragma unroll
                    for (int i = 0; i < K + 2; ++i) {
                        broken = broken | ((kOdd ? rs[u][i] & 0xffffu : rs[u][i]) >= (u32)kRows);
                        rs[u][i] = resolve(rs[u][i]);
                    }
                    if constexpr (kOdd) some = some | (odd_cancel<K + 2>(rs[u], p) > 0);
                    else some = some | (cancel<K + 2>(rs[u]) > 0);
                }
                if (broken) Sh.fail = kDimBroken;
                if (!__any(some)) continue;
#pragma unroll
                for (int u = 0; u < kTaus; ++u) {
                const u32 t = b + u * kT + (u32)lane;
                u32 r[K + 2];
                bool ok = false;
#pragma unroll
                for (int i = 0; i < K + 2; ++i) {
                    r[i] = rs[u][i];
                    ok = ok || r[i] != 0;
                }
                const u32 q = min(qs[u], (u32)A.N - 1);
                ok = ok && t < t1;
                if (!__any(ok)) continue;
                u64 z = 0;
                if (ok) {
                    if constexpr (kOdd)
                        odd_sum<K + 2>(A, r, [](int, u32) {}, [&](int w, u32) { z |= 1ull << w; });
                    else
                        for (u64 m = sum_words<K + 2>(A, r); m; m &= m - 1) {
                            const int w = __ffsll((unsigned long long)m) - 1;
                            if (sum_word<K + 2>(A, r, w)) z |= 1ull << w;
                        }
                }
                ok = ok && z != 0;
                u32 kd = 0;
                u64 ki = 0;
                if (ok) {
                    // the cofacet's index, from its owner and the vertex that
                    // its facet opposite to the owner's first vertex adds
                    const u64 pv = A.qverts[q];
                    const u64 pf = A.qverts[min(A.tau[(int64_t)t * (K + 2) + 1] & (kOdd ? ~kNeg : ~0u), (u32)A.N - 1)];
                    int v[K + 1], f[K + 1];
                    unpack<K>(pv, v);
                    unpack<K>(pf, f);
                    int c = 0;
#pragma unroll
                    for (int i = 0; i <= K; ++i) {
                        bool in = false;
#pragma unroll
                        for (int j = 0; j <= K; ++j) in = in || f[i] == v[j];
                        if (!in) c = f[i];
                    }
                    kd = __float_as_uint(A.qdiam[q]);
                    int below;
                    ki = ~(u64)cofacet_index(v, K, c, A.c.B, &below);
                    ok = (first || key_less(lo_d, lo_i, kd, ki)) && !key_less(hi_d, hi_i, kd, ki);
                }
                candidates<kOdd, K + 2>(A, Sh, vec, ccap, r, ok, kd, ki, z);
                }
            }
            } else {
                // those that k_lune_tests has found; a lane has several in flight
                for (int b0 = wave * kWave; b0 < np; b0 += kTaus * kT) {
                    u32 rs[kTaus][4];
                    int va[kTaus], vb[kTaus], vc[kTaus], vd[kTaus];
                    float len[kTaus];
                    bool oks[kTaus], some = false, broken = false;
#pragma unroll
                    for (int u = 0; u < kTaus; ++u) {
                        const int i = b0 + u * kT + lane;
                        const u64 pr = A.pairs[min(i, np - 1)];
                        const u32 q = min((u32)(pr >> 32), (u32)A.N - 1);
                        vd[u] = (int)(pr & 0xffff);
                        tri_verts(A.qverts[q], va[u], vb[u], vc[u]);
                        len[u] = A.qdiam[q];
                        rs[u][0] = q;
                        oks[u] = i < np;
                    }
#pragma unroll
                    for (int u = 0; u < kTaus; ++u) {
                        const int64_t ei = pair_idx(va[u], vb[u]);
                        const float x = A.c.d.D[(int64_t)vd[u] * n + va[u]], y = A.c.d.D[(int64_t)vd[u] * n + vb[u]],
                                    w = A.c.d.D[(int64_t)vd[u] * n + vc[u]];
                        oks[u] = oks[u] && vd[u] != va[u] && vd[u] != vb[u] && vd[u] != vc[u] &&
                                 edge_before(x, vd[u], va[u], len[u], ei) && edge_before(y, vd[u], vb[u], len[u], ei) &&
                                 edge_before(w, vd[u], vc[u], len[u], ei);
                        rs[u][1] = rs[u][2] = rs[u][3] = 0;
                        if (oks[u]) {
                            rs[u][1] = tri_place(A, va[u], vb[u], vd[u]);
                            rs[u][2] = tri_place(A, va[u], vc[u], vd[u]);
                            rs[u][3] = tri_place(A, vb[u], vc[u], vd[u]);
                        }
                    }
#pragma unroll
                    for (int u = 0; u < kTaus; ++u)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            broken = broken | (rs[u][i] >= (u32)A.N);
                            rs[u][i] = A.ids[min(rs[u][i], (u32)A.N - 1)];
                        }
#pragma unroll
                    for (int u = 0; u < kTaus; ++u) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            broken = broken | ((kOdd ? rs[u][i] & 0xffffu : rs[u][i]) >= (u32)kRows);
                            rs[u][i] = resolve(rs[u][i]);
                            const int x = i == 0 ? vd[u] : i == 1 ? vc[u] : i == 2 ? vb[u] : va[u];
                            if constexpr (kOdd)
                                rs[u][i] = odd_neg(rs[u][i], minus_facet(x, va[u], vb[u], vc[u], vd[u]), p);
                        }
                        if constexpr (kOdd) oks[u] = oks[u] && odd_cancel<4>(rs[u], p) > 0;
                        else oks[u] = oks[u] && cancel<4>(rs[u]) > 0;
                        some = some | oks[u];
                    }
                    if (broken) Sh.fail = kDimBroken;
                    if (!__any(some)) continue;
#pragma unroll
                    for (int u = 0; u < kTaus; ++u) {
                        bool ok = oks[u];
                        if (!__any(ok)) continue;
                        u64 z = 0;
                        if (ok) {
                            if constexpr (kOdd)
                                odd_sum<4>(A, rs[u], [](int, u32) {}, [&](int w, u32) { z |= 1ull << w; });
                            else
                                for (u64 m = sum_words<4>(A, rs[u]); m; m &= m - 1) {
                                    const int w = __ffsll((unsigned long long)m) - 1;
                                    if (sum_word<4>(A, rs[u], w)) z |= 1ull << w;
                                }
                        }
                        ok = ok && z != 0;
                        u32 kd = 0;
                        u64 ki = 0;
                        if (ok) {
                            if (bit_of(A, A.tied, va[u], vb[u])) Sh.fail = 1;
                            kd = __float_as_uint(len[u]);
                            ki = ~tet_index(A, va[u], vb[u], vc[u], vd[u]);
                            ok = (first || key_less(lo_d, lo_i, kd, ki)) && !key_less(hi_d, hi_i, kd, ki);
                        }
                        candidates<kOdd, 4>(A, Sh, vec, ccap, rs[u], ok, kd, ki, z);
                    }
                }
            }
            __syncthreads();
            const int nc = __builtin_amdgcn_readfirstlane(Sh.ncand);
            if (Sh.fail) break; // set before the barrier, if at all
            const bool last = hi_d == ~0u;
            if (nc > ccap) {
                // too many at once: only those up to the quarter point of the stored ones
                if (tid < ccap && rank_of(Sh, ccap, tid) == ccap / 4) {
                    Sh.hi_d = Sh.cd[tid];
                    Sh.hi_i = Sh.ci[tid];
                }
                __syncthreads();
                hi_d = Sh.hi_d;
                hi_i = Sh.hi_i;
                continue;
            }
            if (nc > 0) {
                // ---- elimination in order, by one wave
                if (tid < nc) Sh.ord[rank_of(Sh, nc, tid)] = (uint16_t)tid;
                __syncthreads();
                if (wave == 0) {
                    int nk = 0;
                    unsigned long long adds = 0;
                    for (int i = 0; i < nc; ++i) {
                        const int bj = __builtin_amdgcn_readfirstlane((int)Sh.ord[i]);
                        const u32 bd = __builtin_amdgcn_readfirstlane(Sh.cd[bj]);
                        if (bd == ~0u) continue; // cancelled by older ones
                        const u64 bi = Sh.ci[bj];
                        // its youngest class: a lane a word, then the largest class number
                        const u32 wd = lane < W ? vec[bj * PW + lane] : 0u;
                        const u64 zw = __ballot(wd != 0u);
                        u64 top = 0; // class number + 1, slot
                        for (u32 m = wd; m; m &= m - 1) {
                            const int sl = lane * 32 + __ffs((int)m) - 1;
                            const u64 x = ((u64)(Sh.sage[sl] + 1) << 32) | (u32)sl;
                            top = x > top ? x : top;
                        }
                        // over the lanes with a nonzero word, few of them
                        u64 best = 0;
                        for (u64 m = zw; m; m &= m - 1) {
                            const u64 x = lane_u64(top, __ffsll((unsigned long long)m) - 1);
                            best = x > best ? x : best;
                        }
                        const int slot = __builtin_amdgcn_readfirstlane((int)(u32)best);
                        u32 inv = 1;
                        if constexpr (kOdd) inv = odd_inverse(((LDS uint16_t *)(vec + bj * PW + W))[slot], p);
                        if (lane == 0) {
                            Sh.kinv[nk] = inv;
                            const int cls = min((int)Sh.sage[slot], A.S - 1);
                            A.kidx[cls] = (int64_t)~bi;
                            A.kdiam[cls] = __uint_as_float(bd);
                            Sh.kp[nk] = slot;
                            Sh.ki[nk] = bj;
                            Sh.kz[nk] = zw;
                            Sh.cd[bj] = ~0u;
                        }
                        ++nk;
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                        for (int j = lane; j < nc; j += kWave) {
                            if (Sh.cd[j] == ~0u || !((vec[j * PW + (slot >> 5)] >> (slot & 31)) & 1u)) continue;
                            u64 z = Sh.cz[j];
                            if constexpr (kOdd) {
                                LDS uint16_t *xr = (LDS uint16_t *)(vec + j * PW + W);
                                z = odd_less(vec + j * PW, xr, odd_mul(xr[slot], inv, p), vec + bj * PW, W, zw, z, p);
                            } else
                                for (u64 m = zw; m; m &= m - 1) {
                                    const int w = __ffsll((unsigned long long)m) - 1;
                                    const u32 x = vec[j * W + w] ^ vec[bj * W + w];
                                    vec[j * W + w] = x;
                                    z = x ? z | (1ull << w) : z & ~(1ull << w);
                                }
                            Sh.cz[j] = z;
                            if (!z) Sh.cd[j] = ~0u;
                            ++adds;
                        }
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    }
                    if (lane == 0) {
                        Sh.nkill = nk;
                        ++Sh.since;
                    }
                    atomicAdd(&Sh.adds, adds);
                }
                __syncthreads();
                // ---- the closed classes replaced in every row in use
                const int nk = __builtin_amdgcn_readfirstlane(Sh.nkill);
                const int na = __builtin_amdgcn_readfirstlane(Sh.nact);
                unsigned long long adds = 0;
                for (int i = tid; i < na; i += kT) {
                    const u32 r = A.ract[i];
                    u32 *row = A.pool + (int64_t)r * PW;
                    u64 z = A.rsum[r];
                    bool changed = false;
                    for (int q = 0; q < nk; ++q) {
                        const int ks = Sh.kp[q];
                        if (!((z >> (ks >> 5)) & 1ull) || !((row[ks >> 5] >> (ks & 31)) & 1u)) continue;
                        const LDS u32 *kv = vec + Sh.ki[q] * PW;
                        if constexpr (kOdd) {
                            uint16_t *xr = (uint16_t *)(row + W);
                            z = odd_less(row, xr, odd_mul(xr[ks], Sh.kinv[q], p), kv, W, Sh.kz[q], z, p);
                        } else
                            for (u64 m = Sh.kz[q]; m; m &= m - 1) {
                                const int w = __ffsll((unsigned long long)m) - 1;
                                const u32 x = row[w] ^ kv[w];
                                row[w] = x;
                                z = x ? z | (1ull << w) : z & ~(1ull << w);
                            }
                        changed = true;
                        ++adds;
                    }
                    if (!changed) continue;
                    A.rsum[r] = z;
                    u32 one = 0;
                    if (z) one = row[__ffsll((unsigned long long)z) - 1];
                    if (!z) {
                        rmap[r] = 0;
                    } else if (is_unit(z, one)) {
                        const int slot = (__ffsll((unsigned long long)z) - 1) * 32 + __ffs((int)one) - 1;
                        if constexpr (kOdd) rmap[r] = Sh.urow[slot] | ((u32)((uint16_t *)(row + W))[slot] << 16);
                        else rmap[r] = Sh.urow[slot];
                    }
                }
                if (adds) atomicAdd(&Sh.adds, adds);
                // the closed classes' slots are free again
                for (int q = tid; q < nk; q += kT) Sh.sl[Sh.sfree + q] = (uint16_t)Sh.kp[q];
                __syncthreads();
                // replaced rows leave the rows in use; what pointed to them
                // points to what replaced them
                const int nr = Sh.nrows, nz = Sh.nnz;
                const bool purge = Sh.since >= kPurge || nr > kRows * 3 / 4;
                for (int r = tid; r < nr; r += kT) rmap[r] = (Map)resolve(rmap[r]);
                __syncthreads();
                if (tid == 0) {
                    Sh.sfree += nk;
                    Sh.nact = 0;
                    if (purge) Sh.nnz = Sh.since = 0;
                }
                for (int q0 = 0; q0 < na; q0 += kT) {
                    const int i = q0 + tid;
                    const u32 r = i < na ? A.ract[i] : 0;
                    __syncthreads();
                    const bool keep = i < na && rmap[r] == own_id(r);
                    const int at = wave_place(keep, &Sh.nact);
                    if (keep) A.ract[at] = r; // at most i: entries already read
                    const int de = wave_place(i < na && !keep, &Sh.ndead);
                    if (i < na && !keep) A.rdead[de] = r;
                    __syncthreads();
                }
                if (purge) {
                    // ---- the simplices' numbers brought up to date
                    if constexpr (K == 2) {
                        for (int i = tid; i < nz; i += kT) {
                            int v[3];
                            tri_verts(A.qverts[A.nzl[i]], v[0], v[1], v[2]);
                            for (int x = 0; x < 3; ++x)
                                for (int y = 0; y < 3; ++y)
                                    if (x != y) A.fl[(int64_t)v[x] * A.fw + (v[y] >> 5)] = 0;
                        }
                        __syncthreads();
                    }
                    for (int q0 = 0; q0 < nz; q0 += kT) {
                        const int i = q0 + tid;
                        const u32 q = i < nz ? A.nzl[i] : 0;
                        __syncthreads();
                        bool keep = false;
                        if (i < nz) {
                            const u32 r = resolve(A.ids[q]);
                            A.ids[q] = r;
                            keep = r != 0;
                            if constexpr (K == 2)
                                if (keep) mark(A, q);
                        }
                        const int at = wave_place(keep, &Sh.nnz);
                        if (keep) A.nzl[at] = q;
                        __syncthreads();
                    }
                    const int nd = Sh.ndead, nf = Sh.nfree;
                    for (int i = tid; i < nd; i += kT) A.rfree[nf + i] = A.rdead[i];
                    __syncthreads();
                    if (tid == 0) {
                        Sh.nfree = nf + nd;
                        Sh.ndead = 0;
                    }
                }
                __syncthreads();
            }
            if (last) break;
            lo_d = hi_d;
            lo_i = hi_i;
            first = false;
            hi_d = ~0u;
            hi_i = ~0ull;
            __syncthreads();
        }
        __syncthreads();
        if (Sh.fail) break;
    }
    __syncthreads();
    if (K == 2) {
        DimShared *S = (DimShared *)A.state;
        u32 *to = (u32 *)S, *rm = to + kStateWords;
        const int rows = min(Sh.nrows, kRows);
        for (int i = tid; i < kStateScalars; i += kT) to[i] = ((LDS u32 *)&Sh)[i];
        for (int i = tid; i < nslots; i += kT) {
            S->sage[i] = Sh.sage[i];
            S->urow[i] = Sh.urow[i];
            S->sl[i] = Sh.sl[i];
        }
        for (int i = tid; i * (kOdd ? 1 : 2) < rows; i += kT) rm[i] = ((LDS u32 *)rmap)[i];
        if (tid == 0) A.out->npair = 0;
    }
    if (tid == 0) {
        A.out->full = Sh.fail;
        A.out->adds = Sh.adds;
        A.out->rows = Sh.rows;
    }
}

// Bars in column order (youngest first), counters, and the closing simplices
// into the pivot table. One workgroup.
template <int K>
__global__ void __launch_bounds__(1024) k_dim_bars(DimArgs A, BarBuf out, PivotHash piv) {
    __shared__ int s_w[kWaves + 1];
    __shared__ int s_ess, s_red, s_emg;
    const int lane = lane_id(), w = threadIdx.x / kWave;
    if (threadIdx.x == 0) s_ess = s_red = s_emg = 0;
    __syncthreads();
    int at = 0, ess = 0, red = 0, emg = 0;
    for (int c0 = 0; c0 < A.S; c0 += kT) {
        const int c = c0 + (int)threadIdx.x;
        bool has = false;
        float birth = 0.0f, death = 0.0f;
        int64_t di = -1;
        if (c < A.S) {
            const int k = A.S - 1 - c;
            di = A.kidx[k];
            birth = A.cols.diam[c];
            death = di < 0 ? INFINITY : A.kdiam[k];
            has = death > birth;
            if (di < 0) ++ess;
            else {
                // an emergent pair: closed by the column's own zero pivot cofacet
                const int j = A.cols.j[c];
                bool own = false;
                if (j >= 0) {
                    int v[K + 1], tv[K + 2];
                    decode(A.cols.idx[c], K, A.c.n, A.c.B, v);
                    (void)insert_vertex(v, K, j, tv);
                    own = simplex_index(tv, K + 1, A.c.B) == di;
                }
                emg += own ? 1 : 0;
                red += own ? 0 : 1;
                (void)ph_insert(piv, di, c);
            }
        }
        int inc = has ? 1 : 0;
        for (int o = 1; o < kWave; o <<= 1) {
            const int x = __shfl_up(inc, o, kWave);
            if (lane >= o) inc += x;
        }
        if (lane == kWave - 1) s_w[w] = inc;
        __syncthreads();
        int base = at, tot = 0;
        for (int q = 0; q < kWaves; ++q) {
            if (q < w) base += s_w[q];
            tot += s_w[q];
        }
        if (has) {
            const int o = base + inc - 1;
            out.birth[o] = birth;
            out.death[o] = death;
            out.bs[o] = A.cols.idx[c];
            out.ds[o] = di;
        }
        at += tot;
        __syncthreads();
    }
    if (ess) atomicAdd(&s_ess, ess);
    if (red) atomicAdd(&s_red, red);
    if (emg) atomicAdd(&s_emg, emg);
    __syncthreads();
    if (threadIdx.x == 0) {
        A.out->nbars = at;
        A.out->essential = s_ess;
        A.out->nonzero = at - s_ess;
        A.out->emergent = s_emg;
        A.out->reduced = s_red;
    }
}

unsigned blocks_for(int64_t n, int per) {
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + per - 1) / per, kMostBlocks));
}

template <int K, bool kOdd>
hipError_t prepare_sweep(size_t *lds) {
    *lds = kOdd ? kOddWords * 4 + kOddRows * 4 : kCandWords * 4 + kDimRows * 2;
    return hipFuncSetAttribute((const void *)k_dim_sweep<K, kOdd>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)*lds);
}

} // namespace

void launch_dim_partition(const DimArgs &A, hipStream_t st) {
    launch_fill_u32(A.bin_n, 3 * (kDimBins + 64), 0u, st); // bin_n, bin_t and bin_s are one buffer
    launch_fill_u32((u32 *)A.out, sizeof(DimOut) / 4, 0u, st);
    hipLaunchKernelGGL((k_dim_hist<1>), dim3(blocks_for(A.N, 256)), dim3(256), 0, st, A);
    hipLaunchKernelGGL(k_dim_scan, dim3(2), dim3(kT), 0, st, A.bin_n, A.bin_s, A.nbins,
                       (unsigned long long *)nullptr);
    if (!A.direct) launch_fill_i64(A.ph.keys, (int64_t)A.ph.mask + 1, kEmpty, st);
    hipLaunchKernelGGL(k_dim_place, dim3(blocks_for(A.N, 256)), dim3(256), 0, st, A);
    if (A.c.nb.off) hipLaunchKernelGGL((k_dim_own<16, false>), dim3(blocks_for(A.N, 16)), dim3(256), 0, st, A);
    else hipLaunchKernelGGL((k_dim_own<64, false>), dim3(blocks_for(A.N, 4)), dim3(256), 0, st, A);
    hipLaunchKernelGGL(k_dim_scan, dim3(1), dim3(kT), 0, st, A.bin_t, A.bin_t, A.nbins, &A.out->owned);
}

void launch_dim_fill(const DimArgs &A, hipStream_t st) {
    if (A.c.nb.off) hipLaunchKernelGGL((k_dim_own<16, true>), dim3(blocks_for(A.N, 16)), dim3(256), 0, st, A);
    else hipLaunchKernelGGL((k_dim_own<64, true>), dim3(blocks_for(A.N, 4)), dim3(256), 0, st, A);
    hipLaunchKernelGGL((k_dim_births<1>), dim3(blocks_for(A.S, 256)), dim3(256), 0, st, A);
    hipLaunchKernelGGL(k_dim_chunks, dim3(1), dim3(kT), 0, st, A);
}

void launch_lune_partition(const DimArgs &A, PivotHash piv, hipStream_t st) {
    const int64_t words = (int64_t)A.c.n * A.fw;
    launch_fill_u32(A.bin_n, 3 * (kDimBins + 64), 0u, st);
    launch_fill_u32((u32 *)A.out, sizeof(DimOut) / 4, 0u, st);
    launch_fill_u32(A.fl, words, 0u, st);
    launch_fill_u32(A.tied, words, 0u, st);
    launch_fill_u32(A.rhead, A.N, ~0u, st);
    launch_fill_u32(A.need, A.N / 32 + 1, 0u, st);
    if (!A.direct) launch_fill_i64(A.ph.keys, (int64_t)A.ph.mask + 1, kEmpty, st);
    hipLaunchKernelGGL((k_lune<false>), dim3(blocks_for(A.nE, 4)), dim3(256), 0, st, A);
    hipLaunchKernelGGL(k_dim_scan, dim3(1), dim3(kT), 0, st, A.bin_n, A.bin_n, A.nbins, (unsigned long long *)nullptr);
    hipLaunchKernelGGL((k_lune<true>), dim3(blocks_for(A.nE, 4)), dim3(256), 0, st, A);
    hipLaunchKernelGGL(k_lune_deps, dim3(blocks_for(A.N, 256)), dim3(256), 0, st, A);
    if (A.strict) {
        hipLaunchKernelGGL(k_lune_ties, dim3(blocks_for(A.nE, 256)), dim3(256), 0, st, A);
        hipLaunchKernelGGL(k_lune_groups, dim3(32), dim3(256), 0, st, A);
    }
    hipLaunchKernelGGL(k_lune_classes, dim3(1), dim3(kT), 0, st, A, piv);
}

void launch_lune_chunks(const DimArgs &A, hipStream_t st) {
    hipLaunchKernelGGL((k_dim_hist<2>), dim3(blocks_for(A.S, 256)), dim3(256), 0, st, A);
    hipLaunchKernelGGL(k_dim_scan, dim3(1), dim3(kT), 0, st, A.bin_s, A.bin_s, A.nbins, (unsigned long long *)nullptr);
    hipLaunchKernelGGL((k_dim_births<2>), dim3(blocks_for(A.S, 256)), dim3(256), 0, st, A);
    hipLaunchKernelGGL(k_dim_chunks, dim3(1), dim3(kT), 0, st, A);
}

hipError_t launch_dim_sweep(const DimArgs &A, hipStream_t st) {
    size_t lds;
    const hipError_t e = A.p == 2 ? prepare_sweep<1, false>(&lds) : prepare_sweep<1, true>(&lds);
    if (e != hipSuccess) return e;
    if (A.p == 2) hipLaunchKernelGGL((k_dim_sweep<1, false>), dim3(1), dim3(kT), lds, st, A, 0);
    else hipLaunchKernelGGL((k_dim_sweep<1, true>), dim3(1), dim3(kT), lds, st, A, 0);
    return hipSuccess;
}

hipError_t launch_lune_sweep(const DimArgs &A, int chunks, hipStream_t st) {
    size_t lds;
    const hipError_t e = A.p == 2 ? prepare_sweep<2, false>(&lds) : prepare_sweep<2, true>(&lds);
    if (e != hipSuccess) return e;
    const auto sweep = A.p == 2 ? k_dim_sweep<2, false> : k_dim_sweep<2, true>;
    const auto tests = A.p == 2 ? k_lune_tests<false> : k_lune_tests<true>;
    const unsigned grid = blocks_for((int64_t)A.chunk_n, 4);
    static_assert(most_pairs(kMostPairs, kMostBlocks * 4) < 1ll << 31, "npair is an int");
    for (int c = 0; c <= chunks; ++c) { // those past the last chunk end at once
        hipLaunchKernelGGL(sweep, dim3(1), dim3(kT), lds, st, A, c);
        if (c < chunks) hipLaunchKernelGGL(tests, dim3(grid), dim3(256), 0, st, A, c);
    }
    return hipSuccess;
}

size_t dim_pool_bytes(u32 p, int W) {
    return p == 2 ? (size_t)kDimRows * W * 4 : (size_t)kOddRows * W * kOddStride * 4;
}

size_t dim_state_bytes() { return (size_t)kStateWords * 4 + (size_t)kDimRows * 2; }

void launch_dim_bars(int K, const DimArgs &A, BarBuf bars, PivotHash piv, hipStream_t st) {
    if (K == 1) hipLaunchKernelGGL(k_dim_bars<1>, dim3(1), dim3(kT), 0, st, A, bars, piv);
    else hipLaunchKernelGGL(k_dim_bars<2>, dim3(1), dim3(kT), 0, st, A, bars, piv);
}

} // namespace rips
