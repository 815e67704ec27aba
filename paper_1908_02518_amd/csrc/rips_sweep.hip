// rips_sweep.hip -- dimensions 0 and 1 of a cloud over Z/p in one sweep over
// its edges in order of length, one workgroup per cloud.
//
// The pairs of a filtration are those of its boundary matrix and of its
// coboundary matrix alike (section "Persistent cohomology"), and the zero
// apparent pairs are pairs of both (section "Apparent pairs"). So instead of
// reducing one coboundary column after another, the sweep carries, on every
// edge, the vector of the open classes it belongs to:
//   - an edge of a zero apparent pair (e, t) gets the sum of the vectors of
//     the other two edges of t, so that the boundary of t sums to zero;
//   - a forest edge (one that merges two components) gets zero;
//   - any other edge opens a class and gets its unit vector.
// A triangle whose three vectors do not sum to zero closes the youngest class
// of the sum: the oldest such triangle does it first, and the class is then
// replaced by the rest of the sum everywhere. These are the columns of the
// triangle boundaries over the edges in no zero apparent pair and no forest,
// reduced in the order of the filtration (Algorithm 1 on that matrix).
//
// Why it is fast: nearly every vector is zero and nearly every nonzero one is
// a copy of another edge's. Edges hold row numbers, a row is a vector shared
// by all edges with that sum, and only the edges at a vertex with a nonzero
// edge are looked at again. A 400-point noisy circle has 77,400 edges and 9.8
// million triangles, 74 classes, 94 rows ever, and 6,700 edges whose
// triangles are looked at. What is left is the distances and one scan per
// edge for its zero apparent cofacet.
//
// Over Z/2 a row is bits. Over another field (kOdd) it is those bits and
// residues, 16 bits a class, an edge holds a row and a coefficient, and the vectors are a cochain:
// its value on the coboundary's triangle of vertices x < y < z is that of
// (y, z) less that of (x, z) plus that of (x, y).
#include "rips_sweep.hpp"

#include <algorithm>

namespace rips {

namespace {

constexpr int kT = kSweepT;
constexpr int kWaves = kT / kWave;
constexpr u32 kPending = ~0u;      // an edge whose vector is not known yet
constexpr u32 kNone = 0xffffu;     // no zero apparent cofacet
constexpr u32 kNotEdge = 0xfffeu;  // longer than the threshold
constexpr int kProbe = 32;         // third vertices one lane tries before a whole wave takes over
constexpr int kMaxChunks = 1024;
constexpr int kPoolLdsWords = 4096;

struct SweepShared {
    int cloud, fin;
    u32 renc;
    int nlong, nsurv, ncls, nroot;
    int nch, nrows, nnz, nwork, ncand, nkill, act, fail;
    u64 hi;
    unsigned long long base, adds, entries;
    int nb0, nb1, ness;
    unsigned long long ncand0, nzap;
    int scan[kWaves + 1];
    u32 work[kT];
    u32 cstart[kMaxChunks + 1]; // first list entry of a chunk
    u32 cbin[kMaxChunks + 1];   // first bin after a chunk
    int kp[kSweepCand], ki[kSweepCand]; // kills: class, candidate
    u32 kinv[kSweepCand];               // and the inverse of its coefficient
};

// The dynamic LDS of a cloud of n points.
struct SweepLds {
    LDS u32 *hist;     // kSweepBins
    LDS int *parent;   // n
    LDS float *hdeath; // n
    LDS u32 *hde;      // n
    LDS u32 *vnz;      // n bits: vertices with a nonzero edge
    LDS u32 *pool;     // the first rows
    LDS u64 *keys;     // survivors while they are sorted, then the candidates' keys
    LDS u32 *vec;      // the candidates' vectors
};

__host__ __device__ inline size_t sweep_fixed_bytes(int nmax) {
    return kSweepBins * 4 + kPoolLdsWords * 4 + (size_t)nmax * 12 + (size_t)((nmax + 63) / 64) * 8;
}

__host__ __device__ inline size_t sweep_mask_lds(int nmax) {
    const size_t b = (size_t)nmax * sweep_mask_words(nmax) * 8;
    return b <= (size_t)kSweepMaskBytes ? b : 0;
}

__device__ __forceinline__ void edge_of(int64_t e, int *a, int *b) {
    int x = (int)((1.0f + sqrtf(1.0f + 8.0f * (float)e)) * 0.5f);
    while ((int64_t)x * (x - 1) / 2 > e) --x;
    while ((int64_t)(x + 1) * x / 2 <= e) ++x;
    *a = x;
    *b = (int)(e - (int64_t)x * (x - 1) / 2);
}

__device__ __forceinline__ u32 pair_index(int a, int b) {
    const u32 hi = (u32)max(a, b), lo = (u32)min(a, b);
    return hi * (hi - 1) / 2 + lo;
}

// key of an edge: ascending in the refined order (length, then larger index first)
__device__ __forceinline__ u64 edge_key(float len, u32 e) {
    return ((u64)__float_as_uint(len) << 32) | (u64)(0xffffffffu - e);
}

__device__ __forceinline__ u32 triangle_index(int a, int b, int c) { // a > b
    const u32 h = (u32)max(a, c), l = (u32)min(b, c);
    const u32 m = (u32)(a + b + c) - h - l;
    return (u32)((u64)h * (h - 1) * (h - 2) / 6) + m * (m - 1) / 2 + l;
}

// Is the facet {u, c} of length d older than the edge (len, e)?
__device__ __forceinline__ bool older(float d, int u, int c, float len, u32 e) {
    return d < len || (d == len && pair_index(u, c) > e);
}

__device__ __forceinline__ int bin_of(float len, float scale) {
    return min(kSweepBins - 1, (int)(len * scale)); // monotone in len; equal lengths share a bin
}

__device__ __forceinline__ u64 first_u64(u64 v) {
    const u32 lo = __builtin_amdgcn_readfirstlane((u32)v), hi = __builtin_amdgcn_readfirstlane((u32)(v >> 32));
    return ((u64)hi << 32) | lo;
}

__device__ __forceinline__ u64 wave_min_u64(u64 v) {
    for (int o = 32; o >= 1; o >>= 1) {
        const u32 lo = __shfl_xor((u32)v, o, kWave), hi = __shfl_xor((u32)(v >> 32), o, kWave);
        const u64 w = ((u64)hi << 32) | lo;
        v = w < v ? w : v;
    }
    return v;
}

// exclusive block scan of one int per thread
__device__ __forceinline__ int sweep_scan(int x, int *s_w, int *total) {
    const int lane = lane_id(), w = threadIdx.x / kWave;
    int inc = x;
    for (int o = 1; o < kWave; o <<= 1) {
        const int t = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += t;
    }
    if (lane == kWave - 1) s_w[w] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        int acc = 0;
        for (int q = 0; q < kWaves; ++q) {
            const int t = s_w[q];
            s_w[q] = acc;
            acc += t;
        }
        s_w[kWaves] = acc;
    }
    __syncthreads();
    const int ex = s_w[w] + inc - x;
    *total = s_w[kWaves];
    __syncthreads();
    return ex;
}

// One edge's scan result: its place in the partition, or a survivor.
__device__ __forceinline__ void scan_result(const SweepArgs &A, SweepShared &Sh, const SweepLds &L, const float *D,
                                            u32 *ids, int64_t wo, int n, bool live, int a, int b, float len,
                                            int c, float scale, u64 *sv, u32 *zapped) {
    const u32 e = live ? pair_index(a, b) : 0;
    bool zap = live && c >= 0;
    if (zap) {
        const float x = D[(int64_t)a * n + c], y = D[(int64_t)b * n + c];
        zap = fmaxf(x, y) < len || (older(x, a, c, len, e) && older(y, b, c, len, e));
    }
    if (live) {
        A.zc[wo + e] = (uint16_t)(zap ? (u32)c : kNone);
        ids[(int64_t)a * n + b] = kPending;
        atomicAdd((u32 *)&L.hist[bin_of(len, scale)], 1u);
        *zapped += zap ? 1u : 0u;
    }
    const int at = wave_place(live && !zap, &Sh.nsurv);
    if (live && !zap && at < A.sv_cap) sv[at] = edge_key(len, e);
}

// The rows: the first ones in LDS, the rest in the workgroup's global slice.
// (Separate accesses, not one pointer to either: a generic access waits for
// every outstanding load of the wave.)
struct Rows {
    LDS u32 *lds;
    u32 *glob;
    int nl, W; // rows below nl are in LDS
    __device__ __forceinline__ u32 get(u32 r, int w) const {
        const int o = (int)r * W + w;
        return (int)r < nl ? lds[o] : glob[o];
    }
    __device__ __forceinline__ void set(u32 r, int w, u32 x) const {
        const int o = (int)r * W + w;
        if ((int)r < nl) lds[o] = x;
        else glob[o] = x;
    }
    // half words, after the first nm words
    __device__ __forceinline__ u32 half(u32 r, int nm, int k) const {
        const int o = ((int)r * W + nm) * 2 + k;
        return (int)r < nl ? ((const LDS uint16_t *)lds)[o] : ((const uint16_t *)glob)[o];
    }
    __device__ __forceinline__ void set_half(u32 r, int nm, int k, u32 x) const {
        const int o = ((int)r * W + nm) * 2 + k;
        if ((int)r < nl) ((LDS uint16_t *)lds)[o] = (uint16_t)x;
        else ((uint16_t *)glob)[o] = (uint16_t)x;
    }
};

__device__ __forceinline__ u32 row_word(const Rows &P, u32 r, int w) { return r ? P.get(r, w) : 0u; }

// ---- kOdd: an edge's id is a row (low half) and a coefficient in [1, p), or 0
__device__ __forceinline__ u32 id_neg(u32 id, u32 p) { return id ? (id & 0xffffu) | ((p - (id >> 16)) << 16) : 0u; }
__device__ __forceinline__ u32 id_if_neg(u32 id, bool neg, u32 p) { return neg ? id_neg(id, p) : id; }

// A row of residues: first a bit for each class, set where it is not zero,
// then the residues, 16 bits each, of which those without a bit are not read.

// the bits of word mw of up to three of them
__device__ __forceinline__ u32 odd_bits(const Rows &P, u32 i0, u32 i1, u32 i2, int mw) {
    return (i0 ? P.get(i0 & 0xffffu, mw) : 0u) | (i1 ? P.get(i1 & 0xffffu, mw) : 0u) |
           (i2 ? P.get(i2 & 0xffffu, mw) : 0u);
}

// the residue at class k of their sum
__device__ __forceinline__ u32 odd_at(const Rows &P, u32 i0, u32 i1, u32 i2, int k, int nm, u32 p) {
    const u32 id[3] = {i0, i1, i2};
    u64 t = 0; // three products below 2^32
#pragma unroll
    for (int q = 0; q < 3; ++q)
        if (id[q] && ((P.get(id[q] & 0xffffu, k >> 5) >> (k & 31)) & 1u))
            t += (u64)(id[q] >> 16) * P.half(id[q] & 0xffffu, nm, k);
    return t < (1ull << 32) ? (u32)t % p : (u32)(t % p);
}

__device__ __forceinline__ bool odd_any(const Rows &P, u32 i0, u32 i1, u32 i2, int nm, u32 p) {
    for (int mw = 0; mw < nm; ++mw)
        for (u32 m = odd_bits(P, i0, i1, i2, mw); m; m &= m - 1)
            if (odd_at(P, i0, i1, i2, mw * 32 + __ffs((int)m) - 1, nm, p)) return true;
    return false;
}

// their sum, written by put(word, bits) and res(class, residue)
template <class Put, class Res>
__device__ __forceinline__ void odd_sum(const Rows &P, u32 i0, u32 i1, u32 i2, int nm, u32 p, Put put, Res res) {
    for (int mw = 0; mw < nm; ++mw) {
        u32 bits = 0;
        for (u32 m = odd_bits(P, i0, i1, i2, mw); m; m &= m - 1) {
            const int k = mw * 32 + __ffs((int)m) - 1;
            const u32 x = odd_at(P, i0, i1, i2, k, nm, p);
            if (!x) continue;
            bits |= m & (0u - m);
            res(k, x);
        }
        put(mw, bits);
    }
}

// x less f times the candidate kv, both as rows; is anything left?
template <class Get, class Put, class GetRes, class Res>
__device__ __forceinline__ bool odd_less(Get get, Put put, GetRes get_res, Res res, u32 f, const LDS u32 *kv, int nm,
                                         u32 p) {
    const LDS uint16_t *kr = (const LDS uint16_t *)(kv + nm);
    u32 any = 0;
    for (int mw = 0; mw < nm; ++mw) {
        u32 bits = get(mw);
        const u32 take = kv[mw];
        for (u32 m = take; m; m &= m - 1) {
            const u32 bit = m & (0u - m);
            const int k = mw * 32 + __ffs((int)m) - 1;
            const u32 x = (u32)(((bits & bit ? get_res(k) : 0u) + (u64)(p - f) * kr[k]) % p);
            if (x) res(k, x);
            bits = x ? bits | bit : bits & ~bit;
        }
        if (take) put(mw, bits);
        any |= bits;
    }
    return any != 0;
}

// The nonzero-edge bits: in LDS up to kSweepMaskBytes, else in global memory.
template <bool kMaskLds>
struct MaskPtr {
    typedef LDS u64 *T;
};
template <>
struct MaskPtr<false> {
    typedef u64 *T;
};

// Half a word of them. In global memory the other waves' updates are atomics,
// which execute in the L2, so a plain load could return a stale line of the L1.
__device__ __forceinline__ u32 mask_half(const LDS u64 *m, int i) { return ((const LDS u32 *)m)[i]; }
__device__ __forceinline__ u32 mask_half(const u64 *m, int i) { return ld((const u32 *)m + i); }

struct TestArgs {
    const float *D;
    const u32 *ids;
    int n, MW, nw, ccap;
    u64 lo, hi;
    u32 p;
    int nm; // kOdd: words of a row's bits
};

// The triangles of the listed edges whose vectors do not cancel, appended to
// the candidates: NE edges a wave at once, their third vertices over the
// lanes, NW words of 64 of them in flight. The pass is bound by instruction
// issue, so what an edge has in common is in scalar registers, every load is
// unconditional (from a clamped place) and all are issued before the first is
// used. (With one work item per edge and word, the setup of each cost more
// than its test: circles-64x400 5.8 ms, so 41,000 items a cloud at 440
// instructions each.)
template <bool kOdd, int NE, int NW, class Mask>
__device__ __forceinline__ void test_edges(const TestArgs &T, Mask mask, const Rows &P, SweepShared &Sh,
                                           const SweepLds &L, int wave, int lane) {
    constexpr int N = NE * NW;
    const int n = T.n, MW = T.MW, W = P.W, half = lane >> 5, bit = lane & 31;
    for (int q = wave * NE; q < T.nw; q += kWaves * NE)
        for (int w0 = 0; w0 < MW; w0 += NW) {
            int ea[NE], ev[NE];
            float len[NE], x[N], y[N];
            u32 r0[NE], r1[N], r2[N], fa[N], fv[N], fo[NE];
#pragma unroll
            for (int g = 0; g < NE; ++g) {
                const u32 ab = __builtin_amdgcn_readfirstlane(Sh.work[min(q + g, T.nw - 1)]);
                ea[g] = (int)(ab >> 16);
                ev[g] = (int)(ab & 0xffff);
                const float *Da = T.D + (int64_t)ea[g] * n, *Dv = T.D + (int64_t)ev[g] * n;
                const u32 *Ia = T.ids + (int64_t)ea[g] * n, *Iv = T.ids + (int64_t)ev[g] * n;
                len[g] = Da[ev[g]];
                r0[g] = Ia[ev[g]];
                fo[g] = mask_half(mask, ea[g] * MW * 2 + (ev[g] >> 5)) >> (ev[g] & 31);
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    const int u = g * NW + w, mw = min(w0 + w, MW - 1);
                    const int at = min(mw * 64 + lane, n - 1);
                    x[u] = Da[at];
                    y[u] = Dv[at];
                    r1[u] = Ia[at];
                    r2[u] = Iv[at];
                    fa[u] = mask_half(mask, ea[g] * MW * 2 + mw * 2 + half);
                    fv[u] = mask_half(mask, ev[g] * MW * 2 + mw * 2 + half);
                }
            }
            bool nz[N];
            bool some = false, tie = false;
#pragma unroll
            for (int g = 0; g < NE; ++g) {
                const bool own = fo[g] & 1u;
                r0[g] = own ? r0[g] : 0u;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    const int u = g * NW + w, c = (w0 + w) * 64 + lane;
                    const bool ba = (fa[u] >> bit) & 1u, bv = (fv[u] >> bit) & 1u;
                    const float far = fmaxf(x[u], y[u]);
                    r1[u] = ba ? r1[u] : 0u;
                    r2[u] = bv ? r2[u] : 0u;
                    // two equal rows and a zero one cancel
                    bool gone;
                    if constexpr (kOdd) {
                        // the edge between the triangle's ends has the minus sign
                        const u32 i0 = id_if_neg(r0[g], c < ea[g] && c > ev[g], T.p);
                        const u32 i1 = r1[u] = id_if_neg(r1[u], c < ev[g], T.p);
                        const u32 i2 = r2[u] = id_if_neg(r2[u], c > ea[g], T.p);
                        gone = (i0 == 0 && id_neg(i1, T.p) == i2) || (i1 == 0 && id_neg(i0, T.p) == i2) ||
                               (i2 == 0 && id_neg(i0, T.p) == i1);
                    } else {
                        const u32 sum = r0[g] ^ r1[u] ^ r2[u];
                        gone = sum == 0 && (r0[g] == 0 || r1[u] == 0 || r2[u] == 0);
                    }
                    nz[u] = far <= len[g] && !gone && c < n && q + g < T.nw;
                    some = some || nz[u];
                    tie = tie || (nz[u] && far == len[g]);
                }
            }
            if (!__any(some)) continue;
            if (__any(tie)) { // equal lengths: the larger index is older
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    const int g = u / NW, c = (w0 + u % NW) * 64 + lane;
                    const u32 e = pair_index(ea[g], ev[g]);
                    nz[u] = nz[u] && older(x[u], ea[g], c, len[g], e) && older(y[u], ev[g], c, len[g], e);
                }
            }
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int g = u / NW, a = ea[g], v = ev[g], c = (w0 + u % NW) * 64 + lane;
                if (!__any(nz[u])) continue;
                const u32 p0 = kOdd ? id_if_neg(r0[g], c < a && c > v, T.p) : r0[g], p1 = r1[u], p2 = r2[u];
                auto word = [&](int w) { return row_word(P, p0, w) ^ row_word(P, p1, w) ^ row_word(P, p2, w); };
                u32 any = 0;
                u64 key = 0;
                if (nz[u]) {
                    if constexpr (kOdd) any = odd_any(P, p0, p1, p2, T.nm, T.p) ? 1u : 0u;
                    else
                        for (int w = 0; w < W; ++w) any |= word(w);
                    key = ((u64)__float_as_uint(len[g]) << 32) | (u64)(0xffffffffu - triangle_index(a, v, c));
                }
                const bool open = nz[u] && any != 0 && key > T.lo && key <= T.hi;
                // one triangle of each sum is enough: the oldest, with the largest c
                u64 todo = __ballot(open);
                while (todo) {
                    const int l = 63 - __clzll((long long)todo);
                    const u32 q1 = __builtin_amdgcn_readlane(p1, l), q2 = __builtin_amdgcn_readlane(p2, l);
                    const u32 q0 = kOdd ? __builtin_amdgcn_readlane(p0, l) : p0;
                    todo &= ~__ballot(open && p0 == q0 && ((p1 == q1 && p2 == q2) || (p1 == q2 && p2 == q1)));
                    if (lane == l) {
                        const int s = atomicAdd(&Sh.ncand, 1);
                        if (s < T.ccap) {
                            L.keys[s] = key;
                            if constexpr (kOdd)
                                odd_sum(P, p0, p1, p2, T.nm, T.p, [&](int w, u32 x) { L.vec[s * W + w] = x; },
                                        [&](int k, u32 x) {
                                            ((LDS uint16_t *)(L.vec + s * W + T.nm))[k] = (uint16_t)x;
                                        });
                            else
                                for (int w = 0; w < W; ++w) L.vec[s * W + w] = word(w);
                        }
                    }
                }
            }
        }
}

// One cloud. Returns through the queue loop; every thread of the workgroup calls it.
// A cloud that gives no bars: its segments are empty and the status says why.
__device__ __forceinline__ void sweep_reject(const SweepArgs &A, int b, int D1, int why) {
    if (A.res) {
        if (threadIdx.x == 0) A.res->status = why;
        return;
    }
    if ((int)threadIdx.x < D1) {
        A.seg_start[(int64_t)b * D1 + threadIdx.x] = 0;
        A.seg_count[(int64_t)b * D1 + threadIdx.x] = 0;
    }
    if (threadIdx.x == 0 && why) atomicOr(A.status, why);
}

template <bool kMaskLds, bool kOdd>
__device__ void sweep_cloud(const SweepArgs &A, int b_cloud, unsigned char *smem, SweepShared &Sh) {
    const int tid = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int b = __builtin_amdgcn_readfirstlane(b_cloud);
    const int max_dim = __builtin_amdgcn_readfirstlane(A.max_dim);
    const int D1 = max_dim + 1;
    const int64_t o0 = A.offsets ? A.offsets[b] : 0;
    const int64_t nn = A.offsets ? A.offsets[b + 1] - o0 : A.nmax;
    if (nn < 1 || nn > A.nmax) { // the order pass has set status bit 16
        sweep_reject(A, b, D1, 0);
        return;
    }
    const int n = __builtin_amdgcn_readfirstlane((int)nn);
    const int m = A.m;
    const int64_t wg = blockIdx.x;
    float *D = A.D + wg * A.d_stride;
    u32 *ids = A.ids + wg * A.d_stride;
    const int64_t wo = wg * A.e_stride;
    const int MW = sweep_mask_words(n);
    SweepLds L;
    typename MaskPtr<kMaskLds>::T mask;
    {
        LDS unsigned char *q = (LDS unsigned char *)smem;
        L.keys = (LDS u64 *)q;
        const size_t kb = max((size_t)A.sv_cap * 8, (size_t)kSweepCand * 8 + (size_t)kSweepCandWords * 4);
        L.vec = (LDS u32 *)(q + (size_t)kSweepCand * 8);
        q += kb;
        if constexpr (kMaskLds) mask = (LDS u64 *)q;
        else mask = A.mask + wg * A.mask_stride;
        q += sweep_mask_lds(A.nmax);
        L.vnz = (LDS u32 *)q;
        q += (size_t)((A.nmax + 63) / 64) * 8;
        L.hist = (LDS u32 *)q;
        q += kSweepBins * 4;
        L.pool = (LDS u32 *)q;
        q += kPoolLdsWords * 4;
        L.parent = (LDS int *)q;
        L.hdeath = (LDS float *)(q + (size_t)A.nmax * 4);
        L.hde = (LDS u32 *)(q + (size_t)A.nmax * 8);
    }
    if (tid == 0) {
        Sh.fin = 1;
        Sh.renc = 0x7f800000u;
        Sh.nlong = Sh.nsurv = Sh.ncls = Sh.fail = 0;
        Sh.ncand0 = Sh.nzap = Sh.adds = Sh.entries = 0;
        Sh.nb0 = Sh.nb1 = Sh.ness = 0;
    }
    __syncthreads();
    // ---- distances: a row per wave; the row's maximum on the way
    {
        const float *X = A.X + (m > 0 ? o0 * m : 0);
        bool fin = true;
        // Of more than a few coordinates: each pair once, and kAhead of them
        // loaded before the first is used, so that a lane's cache line is read
        // while it is there (16 clouds of 100 points, dimension 0, both ways
        // and one coordinate at a time, and like this: of R^64 0.44 ms and
        // 0.22, of R^1024 4.8 and 1.04).
        constexpr int kAhead = 8;
        const bool once = m > kAhead;
        if (once) {
            for (int i = wave; i < n; i += kWaves)
                for (int j = lane; j <= i; j += kWave) {
                    const float *xi = X + (int64_t)i * m, *xj = X + (int64_t)j * m;
                    float s = 0.0f;
                    int c = 0;
                    for (; c + kAhead <= m; c += kAhead) {
                        float u[kAhead], v[kAhead];
#pragma unroll
                        for (int k = 0; k < kAhead; ++k) {
                            u[k] = xi[c + k];
                            v[k] = xj[c + k];
                        }
#pragma unroll
                        for (int k = 0; k < kAhead; ++k) {
                            const float t = u[k] - v[k];
                            const float sq = t * t;
                            s = s + sq;
                        }
                    }
                    for (; c < m; ++c) {
                        const float t = xi[c] - xj[c];
                        const float sq = t * t;
                        s = s + sq;
                    }
                    const float d = __builtin_sqrtf(s);
                    D[(int64_t)i * n + j] = d;
                    D[(int64_t)j * n + i] = d;
                }
            __syncthreads();
        }
        for (int i = wave; i < n; i += kWaves) {
            float mx = 0.0f;
            for (int j = lane; j < n; j += kWave) {
                float d;
                if (i == j) {
                    d = INFINITY;
                } else if (once) {
                    d = D[(int64_t)i * n + j];
                } else if (m > 0) {
                    float s = 0.0f;
                    const float *xi = X + (int64_t)i * m, *xj = X + (int64_t)j * m;
                    for (int c = 0; c < m; ++c) {
                        const float t = xi[c] - xj[c];
                        const float sq = t * t;
                        s = s + sq;
                    }
                    d = __builtin_sqrtf(s);
                } else {
                    d = X[(int64_t)max(i, j) * n + min(i, j)];
                }
                if (i != j) {
                    fin = fin && __float_as_uint(d) <= 0x7f7fffffu; // finite, the sign bit clear
                    mx = fmaxf(mx, d);
                }
                D[(int64_t)i * n + j] = d;
            }
            for (int o = 32; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, kWave));
            if (lane == 0) atomicMin(&Sh.renc, __float_as_uint(mx));
        }
        if (!fin) Sh.fin = 0;
    }
    for (int q = tid; q < kSweepBins; q += kT) L.hist[q] = 0;
    for (int q = tid; q < n; q += kT) {
        L.parent[q] = q;
        L.hdeath[q] = -1.0f;
    }
    for (int q = tid; q < n * MW; q += kT) mask[q] = 0;
    for (int q = tid; q < MW * 2; q += kT) L.vnz[q] = 0;
    __syncthreads();
    if (!Sh.fin) {
        // one cloud: the staged path says whether the input or only a
        // distance is out of range, and handles the latter
        sweep_reject(A, b, D1, A.res ? kSweepFull : 4);
        __syncthreads();
        return;
    }
    const float renc = n > 1 ? __uint_as_float(Sh.renc) : 0.0f;
    const float t = fminf(A.threshold, renc);
    const float scale = t > 0.0f ? (float)kSweepBins / t : 0.0f;
    u64 *sv = A.sv + wg * (int64_t)A.sv_cap;
    u32 *aux = A.aux + wo;
    // ---- the zero apparent cofacet of every edge: the oldest cofacet is the
    // one with the largest third vertex no farther from both ends than the
    // edge is long. One lane per edge tries the first kProbe vertices from the
    // top (a lane's row of distances to its vertex is read across the wave);
    // long edges find theirs at once, a short one goes to a list.
    u32 ncand = 0, nzap = 0;
    for (int a = wave; a < n; a += kWaves) {
        const float *Da = D + (int64_t)a * n;
        const int top = n - 1;
        const float xr = lane <= top ? Da[top - lane] : INFINITY;
        for (int b0 = 0; b0 < a; b0 += kWave) {
            const int v = b0 + lane;
            const float len = v < a ? Da[v] : INFINITY;
            const bool edge = v < a && len <= t;
            int c = -1;
            u64 open = __ballot(edge);
            const int col = v < a ? v : 0;
            const float *Dc = D + (int64_t)top * n;
            for (int p = 0; p < kProbe && p < n && open; p += 8, Dc -= 8 * (int64_t)n) {
                float yy[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) yy[u] = (p + u < n ? Dc - u * (int64_t)n : D)[col];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    // +inf past the last vertex
                    const float xx = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(xr), p + u));
                    const u64 hit = __ballot(fmaxf(xx, yy[u]) <= len) & open;
                    c = __builtin_amdgcn_inverse_ballot_w64(hit) ? top - p - u : c;
                    open &= ~hit;
                }
            }
            const bool more = edge && c < 0 && n > kProbe;
            ncand += edge ? 1u : 0u;
            if (v < a && !edge) A.zc[wo + pair_index(a, v)] = (uint16_t)kNotEdge;
            scan_result(A, Sh, L, D, ids, wo, n, edge && !more, a, v, len, c, scale, sv, &nzap);
            const int at = wave_place(more, &Sh.nlong);
            if (more) aux[at] = ((u32)a << 16) | (u32)v;
        }
    }
    __syncthreads();
    // the short edges: one wave per edge over the remaining vertices
    const int nlong = Sh.nlong;
    for (int base = wave * kWave; base < nlong; base += kWaves * kWave) {
        const u32 mine = base + lane < nlong ? aux[base + lane] : 0;
        const int cnt = min(kWave, nlong - base);
        int rc = -1;
        for (int q = 0; q < cnt; ++q) {
            const u32 ab = __builtin_amdgcn_readlane(mine, q);
            const int a = (int)(ab >> 16), v = (int)(ab & 0xffff);
            const float *Da = D + (int64_t)a * n, *Dv = D + (int64_t)v * n;
            const float len = Da[v];
            int c = -1;
            for (int top = n - 1 - kProbe; top >= 0 && c < 0; top -= 4 * kWave) {
                float far[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int w = top - u * kWave - lane;
                    const float d = fmaxf(Da[max(w, 0)], Dv[max(w, 0)]);
                    far[u] = w >= 0 ? d : INFINITY;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const u64 bal = __ballot(far[u] <= len);
                    if (c < 0 && bal) c = top - u * kWave - (__ffsll((unsigned long long)bal) - 1);
                }
            }
            if (lane == q) rc = c;
        }
        const int a = (int)(mine >> 16), v = (int)(mine & 0xffff);
        const float len = lane < cnt ? D[(int64_t)a * n + v] : 0.0f;
        scan_result(A, Sh, L, D, ids, wo, n, lane < cnt, a, v, len, rc, scale, sv, &nzap);
    }
    for (int o = 32; o >= 1; o >>= 1) {
        ncand += __shfl_xor(ncand, o, kWave);
        nzap += __shfl_xor(nzap, o, kWave);
    }
    if (lane == 0) {
        atomicAdd(&Sh.ncand0, (unsigned long long)ncand);
        atomicAdd(&Sh.nzap, (unsigned long long)nzap);
    }
    __syncthreads();
    const int ns = Sh.nsurv;
    if (ns > A.sv_cap) { // the caller runs the column reduction instead
        sweep_reject(A, b, D1, kSweepFull);
        __syncthreads();
        return;
    }
    // ---- the edges in no zero apparent pair, sorted (bitonic, in LDS)
    int np = 2;
    while (np < ns) np <<= 1;
    for (int q = tid; q < np; q += kT) L.keys[q] = q < ns ? sv[q] : ~0ull;
    __syncthreads();
    for (int k = 2; k <= np; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int q = tid; q < np / 2; q += kT) {
                const int i = ((q & ~(j - 1)) << 1) | (q & (j - 1)), l = i | j;
                const u64 x = L.keys[i], y = L.keys[l];
                if ((x > y) == ((i & k) == 0)) {
                    L.keys[i] = y;
                    L.keys[l] = x;
                }
            }
            __syncthreads();
        }
    // ---- dimension 0: Kruskal on them (a forest edge is in no zero apparent
    // pair), 64 at a time on wave 0. The root of a component is its largest,
    // its oldest, vertex: the younger component's root is the one that dies.
    // The other edges open the classes of dimension 1, in order.
    u64 *ckey = A.ckey + wg * (int64_t)A.sv_cap, *kkey = A.kkey + wg * (int64_t)A.sv_cap;
    if (wave == 0) {
        int ncls = 0;
        for (int base = 0; base < ns; base += kWave) {
            const bool valid = base + lane < ns;
            const u64 key = valid ? L.keys[base + lane] : 0;
            const u32 e = 0xffffffffu - (u32)key;
            int a = 0, v = 0, ra = 0, rb = 0;
            if (valid) {
                edge_of(e, &a, &v);
                ra = a;
                rb = v;
                while (L.parent[ra] != ra) ra = L.parent[ra];
                while (L.parent[rb] != rb) rb = L.parent[rb];
            }
            bool forest = false;
            int dies = 0;
            for (u64 todo = __ballot(valid && ra != rb); todo; todo &= todo - 1) {
                const int q = __ffsll((unsigned long long)todo) - 1;
                const int RA = __builtin_amdgcn_readlane(ra, q), RB = __builtin_amdgcn_readlane(rb, q);
                if (RA == RB) continue;
                const int win = max(RA, RB), los = min(RA, RB);
                if (lane == q) {
                    forest = true;
                    dies = los;
                }
                if (ra == los) ra = win;
                if (rb == los) rb = win;
                if (lane == 0) L.parent[los] = win;
            }
            if (forest) {
                const float len = __uint_as_float((u32)(key >> 32));
                L.hdeath[dies] = len > 0.0f ? len : -2.0f; // -2: a bar of length zero
                L.hde[dies] = e;
            }
            const u64 cls = __ballot(valid && !forest);
            if (valid) {
                u32 id = 0;
                if (!forest) {
                    const int k = ncls + __popcll(cls & ((1ull << lane) - 1));
                    ckey[k] = key;
                    kkey[k] = ~0ull;
                    id = (u32)k + 1 + (kOdd ? 1u << 16 : 0u);
                }
                ids[(int64_t)a * n + v] = id;
                ids[(int64_t)v * n + a] = id;
            }
            ncls += __popcll(cls);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        if (lane == 0) Sh.ncls = ncls;
    }
    __syncthreads();
    const int S = __builtin_amdgcn_readfirstlane(Sh.ncls);
    const int nm = (S + 31) / 32, W = kOdd ? nm + (S + 1) / 2 : nm;
    const u32 p = A.p;
    const Rows P{L.pool, A.pool + wg * A.pool_stride, W > 0 ? kPoolLdsWords / W : 0, W};
    const int rcap = W > 0 ? (int)min((int64_t)(kOdd ? 0xffff : 1 << 30), A.pool_stride / W) : 0;
    if (max_dim >= 1 && S > 0) {
        if (S > min(A.most_classes, kOdd ? kSweepOddClasses : kSweepMaxClasses) || S + 1 >= rcap) {
            sweep_reject(A, b, D1, kSweepFull);
            __syncthreads();
            return;
        }
        const int ccap = min(kSweepCand, kSweepCandWords / W);
        // ---- the edges by length bin, whole bins to a chunk of about as many
        // edges as there are threads (more, where a cloud has very many; fewer in
        // a small one: the triangles of a chunk that a class closed in it leaves
        // nonzero are all eliminated at once)
        const u32 E = (u32)Sh.ncand0;
        const u32 target = max(min(max(E / 32, 256u), (u32)kT), (E + kMaxChunks - 3) / (kMaxChunks - 2));
        for (int q = tid; q <= kMaxChunks; q += kT) {
            Sh.cstart[q] = ~0u;
            Sh.cbin[q] = 0;
        }
        static_assert(kSweepBins == 2 * kT, "two bins per thread");
        const u32 h0 = L.hist[2 * tid], h1 = L.hist[2 * tid + 1];
        int total;
        const u32 p0 = (u32)sweep_scan((int)(h0 + h1), Sh.scan, &total);
        L.hist[2 * tid] = p0;
        L.hist[2 * tid + 1] = p0 + h0;
        if (h0) {
            atomicMin(&Sh.cstart[p0 / target], p0);
            atomicMax(&Sh.cbin[p0 / target], (u32)(2 * tid + 1));
        }
        if (h1) {
            atomicMin(&Sh.cstart[(p0 + h0) / target], p0 + h0);
            atomicMax(&Sh.cbin[(p0 + h0) / target], (u32)(2 * tid + 2));
        }
        __syncthreads();
        if (wave == 0) { // the chunks that hold edges, in order
            const int nch0 = (int)(E / target) + 1;
            int at = 0;
            for (int base = 0; base < nch0; base += kWave) {
                const bool in = base + lane < nch0;
                const u32 s = in ? Sh.cstart[base + lane] : ~0u, bb = in ? Sh.cbin[base + lane] : 0;
                const u64 bal = __ballot(s != ~0u);
                const int pos = at + __popcll(bal & ((1ull << lane) - 1));
                if (s != ~0u) {
                    Sh.cstart[pos] = s; // pos is at most this entry's own place
                    Sh.cbin[pos] = bb;
                }
                at += __popcll(bal);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            }
            if (lane == 0) {
                Sh.cstart[at] = E;
                Sh.nch = at;
                Sh.nrows = S + 1;
                Sh.nnz = 0;
                Sh.act = 0;
            }
        }
        u64 *list = A.list + wo;
        for (int a = wave; a < n; a += kWaves)
            for (int v = lane; v < a; v += kWave) {
                const u32 c = A.zc[wo + pair_index(a, v)];
                if (c == kNotEdge) continue;
                const u32 at = atomicAdd((u32 *)&L.hist[bin_of(D[(int64_t)a * n + v], scale)], 1u);
                list[at] = ((u64)c << 32) | ((u32)a << 16) | (u32)v;
            }
        // the unit rows of the classes
        for (int q = tid; q < S * W; q += kT) {
            const int k = q / W, w = q - k * W;
            P.set((u32)k + 1, w, w < nm ? (w == (k >> 5) ? 1u << (k & 31) : 0u) : 0x10001u);
        }
        __syncthreads();
        const int nch = __builtin_amdgcn_readfirstlane(Sh.nch);
        int bp = 0; // classes opened so far
        for (int ch = 0; ch < nch; ++ch) {
            const int c0 = (int)Sh.cstart[ch], c1 = (int)Sh.cstart[ch + 1];
            const int b1 = (int)Sh.cbin[ch];
            // ---- the classes that open here: their edges become nonzero
            for (;;) {
                const int k = bp + tid;
                const u64 key = k < S ? ckey[k] : 0;
                const bool opens = k < S && bin_of(__uint_as_float((u32)(key >> 32)), scale) < b1;
                if (opens) {
                    int a, v;
                    edge_of(0xffffffffu - (u32)key, &a, &v);
                    atomicOr((unsigned long long *)&mask[a * MW + (v >> 6)], 1ull << (v & 63));
                    atomicOr((unsigned long long *)&mask[v * MW + (a >> 6)], 1ull << (a & 63));
                    atomicOr((u32 *)&L.vnz[a >> 5], 1u << (a & 31));
                    atomicOr((u32 *)&L.vnz[v >> 5], 1u << (v & 31));
                }
                const u64 bal = __ballot(opens);
                if (lane == 0 && bal) atomicAdd(&Sh.act, __popcll(bal));
                const int at = wave_place(opens, &Sh.nnz);
                if (opens) aux[at] = 0xffffffffu - (u32)key;
                __syncthreads();
                const int now = Sh.act;
                __syncthreads();
                if (now - bp < kT) {
                    bp = now;
                    break;
                }
                bp = now;
            }
            // ---- the vectors of the chunk's edges: the sum of the other two
            // edges of the zero apparent cofacet. Those are older, so some
            // edge of the chunk can always go on; an edge whose sums are not
            // there yet is tried again.
            for (int tries = 0;; ++tries) {
                bool left = false;
                for (int i = c0 + tid; i < c1; i += kT) {
                    const u64 en = list[i];
                    const u32 c = (u32)(en >> 32);
                    if (c == kNone) continue;
                    const int a = (int)((u32)en >> 16), v = (int)((u32)en & 0xffff);
                    u32 *mine = ids + ((int64_t)a * n + v);
                    if (ld(mine) != kPending) continue;
                    const u32 r1 = ld(&ids[(int64_t)max(a, (int)c) * n + min(a, (int)c)]);
                    const u32 r2 = ld(&ids[(int64_t)max(v, (int)c) * n + min(v, (int)c)]);
                    if (r1 == kPending || r2 == kPending) {
                        left = true;
                        continue;
                    }
                    u32 r;
                    if constexpr (kOdd) {
                        const u32 i1 = id_if_neg(r1, (int)c > a, p), i2 = id_if_neg(r2, (int)c < v, p);
                        if (i1 == 0 || i2 == 0) {
                            r = i1 | i2;
                        } else if (((i1 ^ i2) & 0xffffu) == 0) {
                            const u32 cf = ((i1 >> 16) + (i2 >> 16)) % p;
                            r = cf ? (i1 & 0xffffu) | (cf << 16) : 0u;
                        } else {
                            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                            r = 0;
                            if (odd_any(P, i1, i2, 0, nm, p)) {
                                const u32 at = (u32)atomicAdd(&Sh.nrows, 1);
                                if ((int)at < rcap) {
                                    odd_sum(P, i1, i2, 0, nm, p, [&](int w, u32 x) { P.set(at, w, x); },
                                            [&](int k, u32 x) { P.set_half(at, nm, k, x); });
                                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                                    r = at | (1u << 16);
                                } else {
                                    Sh.fail = 1;
                                }
                            }
                        }
                    } else
                        r = r1 == r2 ? 0u : (r1 ? (r2 ? kPending : r1) : r2);
                    if (!kOdd && r == kPending) {
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                        u32 any = 0;
                        for (int w = 0; w < W; ++w) any |= P.get(r1, w) ^ P.get(r2, w);
                        r = 0;
                        if (any) {
                            r = (u32)atomicAdd(&Sh.nrows, 1);
                            if ((int)r < rcap) {
                                for (int w = 0; w < W; ++w) P.set(r, w, P.get(r1, w) ^ P.get(r2, w));
                                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                            } else {
                                r = 0;
                                Sh.fail = 1;
                            }
                        }
                    }
                    if (r) {
                        atomicOr((unsigned long long *)&mask[a * MW + (v >> 6)], 1ull << (v & 63));
                        atomicOr((unsigned long long *)&mask[v * MW + (a >> 6)], 1ull << (a & 63));
                        atomicOr((u32 *)&L.vnz[a >> 5], 1u << (a & 31));
                        atomicOr((u32 *)&L.vnz[v >> 5], 1u << (v & 31));
                        aux[atomicAdd(&Sh.nnz, 1)] = pair_index(a, v);
                        ids[(int64_t)v * n + a] = r;
                    }
                    st(mine, r);
                }
                if (!__any(left)) break;
                if (tries > (1 << 16)) { // cannot happen: the order is acyclic
                    Sh.fail = 1;
                    break;
                }
            }
            __syncthreads();
            const bool none = Sh.nnz == 0, failed = Sh.fail != 0;
            __syncthreads(); // before the next chunk's classes change the count
            if (failed) break;
            if (none) continue;
            // ---- the triangles whose youngest edge is in the chunk and whose
            // vectors do not sum to zero, oldest first
            u64 lo = 0, hi = ~0ull;
            for (;;) {
                if (tid == 0) {
                    Sh.ncand = 0;
                    Sh.nwork = 0;
                }
                __syncthreads();
                for (int t0 = c0; t0 < c1; t0 += kT) {
                    // the edges with a nonzero edge at one of their vertices
                    const int i = t0 + tid;
                    u32 ab = 0;
                    bool look = false;
                    if (i < c1) {
                        ab = (u32)list[i];
                        const int a = (int)(ab >> 16), v = (int)(ab & 0xffff);
                        look = ((L.vnz[a >> 5] >> (a & 31)) & 1u) || ((L.vnz[v >> 5] >> (v & 31)) & 1u);
                    }
                    const int at = wave_place(look, &Sh.nwork);
                    if (look) Sh.work[at] = ab;
                    __syncthreads();
                    const int nw = Sh.nwork;
                    const TestArgs TA{D, ids, n, MW, nw, ccap, lo, hi, p, nm};
                    if (MW == 1) test_edges<kOdd, 4, 1>(TA, mask, P, Sh, L, wave, lane);
                    else if (MW == 2) test_edges<kOdd, 2, 2>(TA, mask, P, Sh, L, wave, lane);
                    else test_edges<kOdd, 1, 4>(TA, mask, P, Sh, L, wave, lane);
                    __syncthreads();
                    if (tid == 0) Sh.nwork = 0;
                    __syncthreads();
                }
                const int nc = __builtin_amdgcn_readfirstlane(Sh.ncand);
                if (nc == 0) {
                    if (hi == ~0ull) break;
                    lo = hi;
                    hi = ~0ull;
                    __syncthreads();
                    continue;
                }
                if (nc > ccap) {
                    // too many at once: only those up to the quarter point of
                    // the ones stored (keys are distinct)
                    if (tid < ccap) {
                        const u64 mine = L.keys[tid];
                        int less = 0;
                        for (int q = 0; q < ccap; ++q) less += L.keys[q] < mine ? 1 : 0;
                        if (less == ccap / 4) Sh.hi = mine;
                    }
                    __syncthreads();
                    hi = Sh.hi;
                    continue;
                }
                // ---- elimination in order, by one wave
                if (wave == 0) {
                    int nk = 0;
                    unsigned long long adds = 0;
                    for (;;) {
                        u64 best = ~0ull;
                        int bi = 0;
                        for (int j = lane; j < nc; j += kWave)
                            if (L.keys[j] < best) {
                                best = L.keys[j];
                                bi = j;
                            }
                        const u64 mn = wave_min_u64(best);
                        if (mn == ~0ull) break;
                        const int src = __ffsll((unsigned long long)__ballot(best == mn)) - 1;
                        bi = __builtin_amdgcn_readlane(bi, src);
                        // the youngest class
                        const u32 wd = lane < nm ? L.vec[bi * W + lane] : 0u;
                        const u64 nzw = __ballot(wd != 0u);
                        const int top = 63 - __clzll((long long)nzw);
                        const u32 tw = __builtin_amdgcn_readlane(wd, top);
                        const int cls = top * 32 + 31 - __clz((int)tw);
                        const u32 inv = kOdd ? odd_inverse(((LDS uint16_t *)(L.vec + bi * W + nm))[cls], p) : 1u;
                        if (lane == 0) {
                            kkey[cls] = mn;
                            Sh.kp[nk] = cls;
                            Sh.kinv[nk] = inv;
                            Sh.ki[nk] = bi;
                            L.keys[bi] = ~0ull;
                        }
                        ++nk;
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                        for (int j = lane; j < nc; j += kWave) {
                            if (L.keys[j] == ~0ull || !((L.vec[j * W + (cls >> 5)] >> (cls & 31)) & 1u)) continue;
                            u32 any = 0;
                            if constexpr (kOdd) {
                                LDS u32 *x = L.vec + j * W;
                                LDS uint16_t *xr = (LDS uint16_t *)(x + nm);
                                const u32 f = (u32)((u64)xr[cls] * inv % p);
                                any = odd_less([&](int w) { return x[w]; }, [&](int w, u32 y) { x[w] = y; },
                                               [&](int k) { return (u32)xr[k]; },
                                               [&](int k, u32 y) { xr[k] = (uint16_t)y; }, f, L.vec + bi * W, nm, p)
                                          ? 1u : 0u;
                            } else
                                for (int w = 0; w < W; ++w) {
                                    const u32 z = L.vec[j * W + w] ^ L.vec[bi * W + w];
                                    L.vec[j * W + w] = z;
                                    any |= z;
                                }
                            if (!any) L.keys[j] = ~0ull;
                            ++adds;
                        }
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    }
                    if (lane == 0) Sh.nkill = nk;
                    atomicAdd(&Sh.adds, adds);
                }
                __syncthreads();
                // ---- the closed classes replaced in every row
                const int nk = __builtin_amdgcn_readfirstlane(Sh.nkill);
                const int R = __builtin_amdgcn_readfirstlane(Sh.nrows);
                unsigned long long adds = 0;
                for (int r = 1 + tid; r < R; r += kT)
                    for (int q = 0; q < nk; ++q) {
                        const int cls = Sh.kp[q];
                        if (!((P.get((u32)r, cls >> 5) >> (cls & 31)) & 1u)) continue;
                        const LDS u32 *kv = L.vec + Sh.ki[q] * W;
                        if constexpr (kOdd) {
                            const u32 f = (u32)((u64)P.half((u32)r, nm, cls) * Sh.kinv[q] % p);
                            (void)odd_less([&](int w) { return P.get((u32)r, w); },
                                           [&](int w, u32 y) { P.set((u32)r, w, y); },
                                           [&](int k) { return P.half((u32)r, nm, k); },
                                           [&](int k, u32 y) { P.set_half((u32)r, nm, k, y); }, f, kv, nm, p);
                        } else
                            for (int w = 0; w < W; ++w) P.set((u32)r, w, P.get((u32)r, w) ^ kv[w]);
                        ++adds;
                    }
                if (adds) atomicAdd(&Sh.adds, adds);
                for (int q = tid; q < MW * 2; q += kT) L.vnz[q] = 0;
                const int nz = Sh.nnz;
                __syncthreads();
                if (tid == 0) Sh.nnz = 0;
                // ---- the edges whose row became zero leave the nonzero edges
                for (int q0 = 0; q0 < nz; q0 += kT) {
                    const int q = q0 + tid;
                    const u32 e = q < nz ? aux[q] : 0;
                    __syncthreads();
                    bool keep = false;
                    if (q < nz) {
                        int a, v;
                        edge_of(e, &a, &v);
                        u32 any = 0;
                        const u32 id = ids[(int64_t)a * n + v], r = kOdd ? id & 0xffffu : id;
                        for (int w = 0; w < nm; ++w) any |= P.get(r, w);
                        keep = any != 0;
                        if (keep) {
                            atomicOr((u32 *)&L.vnz[a >> 5], 1u << (a & 31));
                            atomicOr((u32 *)&L.vnz[v >> 5], 1u << (v & 31));
                        } else {
                            ids[(int64_t)a * n + v] = 0;
                            ids[(int64_t)v * n + a] = 0;
                            atomicAnd((unsigned long long *)&mask[a * MW + (v >> 6)], ~(1ull << (v & 63)));
                            atomicAnd((unsigned long long *)&mask[v * MW + (a >> 6)], ~(1ull << (a & 63)));
                        }
                    }
                    const int at = wave_place(keep, &Sh.nnz);
                    if (keep) aux[at] = e; // at most q0 + tid: entries already read
                    __syncthreads();
                }
                __syncthreads();
                if (hi == ~0ull) break;
                lo = hi;
                hi = ~0ull;
            }
            __syncthreads();
        }
        __syncthreads();
        if (Sh.fail) {
            sweep_reject(A, b, D1, kSweepFull);
            __syncthreads();
            return;
        }
    }
    // ---- the bars: dimension 0 by birth vertex descending, dimension 1 by
    // class; counted, then written to one segment each of the unordered buffer
    __syncthreads();
    int c0n = 0, c1n = 0;
    for (int q = tid; q < n; q += kT) {
        const bool root = L.parent[q] == q;
        c0n += (root || L.hdeath[q] > 0.0f) ? 1 : 0;
        if (root) atomicAdd(&Sh.nb1, 1); // essential classes of dimension 0, for now
    }
    if (max_dim >= 1)
        for (int k = tid; k < S; k += kT) {
            const u64 kk = kkey[k];
            const bool ess = kk == ~0ull;
            c1n += (ess || (u32)(kk >> 32) > (u32)(ckey[k] >> 32)) ? 1 : 0;
            if (ess) atomicAdd(&Sh.ness, 1);
        }
    for (int o = 32; o >= 1; o >>= 1) {
        c0n += __shfl_xor(c0n, o, kWave);
        c1n += __shfl_xor(c1n, o, kWave);
    }
    if (tid == 0) Sh.act = 0;
    __syncthreads();
    if (lane == 0) {
        atomicAdd(&Sh.nb0, c0n);
        atomicAdd(&Sh.act, c1n);
    }
    __syncthreads();
    const int nb0 = Sh.nb0, nb1 = Sh.act, ess0 = Sh.nb1, ess1 = Sh.ness;
    if (tid == 0) {
        Sh.base = A.res ? 0ull : atomicAdd(A.ucount, (unsigned long long)(nb0 + nb1));
        rips_dim_stats s0 = {}, s1 = {};
        s0.candidates = n;
        s0.columns = n;
        s0.bars_nonzero = nb0 - ess0;
        s0.essential = ess0;
        s1.candidates = (int64_t)Sh.ncand0;
        s1.cleared = ns - S;
        s1.apparent_col = (int64_t)Sh.nzap;
        s1.columns = S;
        s1.reduced = S - ess1;
        s1.additions = (int64_t)Sh.adds + (S > 0 && max_dim >= 1 ? Sh.nrows - S - 1 : 0);
        s1.bars_nonzero = nb1 - ess1;
        s1.essential = ess1;
        s1.entries_added = s1.additions * W;
        s1.entries_stored = S > 0 && max_dim >= 1 ? (int64_t)(Sh.nrows - 1) * W : 0;
        if (A.res) {
            A.res->status = 0;
            A.res->t = t;
            A.res->renc = renc;
            A.res->count[0] = nb0;
            A.res->count[1] = nb1;
            A.res->stats[0] = s0;
            A.res->stats[1] = s1;
        } else {
            A.stats[(int64_t)b * D1] = s0;
            A.t_used[b] = t;
            if (max_dim >= 1) A.stats[(int64_t)b * D1 + 1] = s1;
        }
    }
    __syncthreads();
    const int64_t base = (int64_t)Sh.base;
    const bool fits = A.res ? max(nb0, nb1) <= A.ucap : base + nb0 + nb1 <= A.ucap;
    int at = 0;
    for (int q0 = 0; q0 < n; q0 += kT) {
        const int v = n - 1 - (q0 + tid);
        const bool root = v >= 0 && L.parent[v] == v;
        const bool has = root || (v >= 0 && L.hdeath[v] > 0.0f);
        int tot;
        const int ex = sweep_scan(has ? 1 : 0, Sh.scan, &tot);
        if (has && fits) {
            const int64_t w = base + at + ex;
            A.ub[w] = 0.0f;
            A.ud[w] = root ? INFINITY : L.hdeath[v];
            A.ubs[w] = v;
            A.uds[w] = root ? -1 : (int64_t)L.hde[v];
        }
        at += tot;
    }
    if (A.res && A.col_idx && max_dim >= 1)
        for (int k = tid; k < S; k += kT) {
            A.col_idx[S - 1 - k] = (int64_t)(0xffffffffu - (u32)ckey[k]);
            A.col_diam[S - 1 - k] = __uint_as_float((u32)(ckey[k] >> 32));
        }
    if (max_dim >= 1)
        for (int q0 = 0, at1 = 0; q0 < S; q0 += kT) {
            const int k = q0 + tid;
            const u64 ck = k < S ? ckey[k] : 0, kk = k < S ? kkey[k] : 0;
            const bool ess = kk == ~0ull;
            const bool has = k < S && (ess || (u32)(kk >> 32) > (u32)(ck >> 32));
            int tot;
            const int ex = sweep_scan(has ? 1 : 0, Sh.scan, &tot);
            if (has && fits) {
                const int64_t w = A.res ? A.ucap + at1 + ex : base + nb0 + at1 + ex;
                A.ub[w] = __uint_as_float((u32)(ck >> 32));
                A.ud[w] = ess ? INFINITY : __uint_as_float((u32)(kk >> 32));
                A.ubs[w] = (int64_t)(0xffffffffu - (u32)ck);
                A.uds[w] = ess ? -1 : (int64_t)(0xffffffffu - (u32)kk);
            }
            at1 += tot;
        }
    if (tid == 0 && !A.res) {
        A.seg_start[(int64_t)b * D1] = base;
        A.seg_count[(int64_t)b * D1] = nb0;
        if (D1 > 1) {
            A.seg_start[(int64_t)b * D1 + 1] = base + nb0;
            A.seg_count[(int64_t)b * D1 + 1] = nb1;
        }
    }
    __syncthreads();
}

template <bool kMaskLds, bool kOdd>
__global__ void __launch_bounds__(kT) k_sweep(SweepArgs A) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ SweepShared Sh;
    if (A.res) {
        sweep_cloud<kMaskLds, kOdd>(A, 0, smem, Sh);
        return;
    }
    for (;;) {
        if (threadIdx.x == 0) Sh.cloud = (int)atomicAdd(A.queue, 1ull);
        __syncthreads();
        const int qi = Sh.cloud;
        __syncthreads();
        if (qi >= A.B) break;
        sweep_cloud<kMaskLds, kOdd>(A, A.order ? A.order[qi] : qi, smem, Sh);
    }
}

// Clouds by decreasing size (longest first), by counting; one workgroup.
__global__ void __launch_bounds__(1024) k_sweep_order(const int64_t *offsets, int B, int nmax, int *order,
                                                      unsigned long long *queue, unsigned long long *ucount,
                                                      int *status) {
    __shared__ int cnt[kSweepMaxN + 2];
    __shared__ int bad;
    for (int q = threadIdx.x; q < kSweepMaxN + 2; q += 1024) cnt[q] = 0;
    if (threadIdx.x == 0) bad = 0;
    __syncthreads();
    for (int b = threadIdx.x; b < B; b += 1024) {
        const int64_t n = offsets ? offsets[b + 1] - offsets[b] : nmax;
        if (n < 1 || n > nmax) bad = 1;
        const int s = kSweepMaxN - (int)(n < 0 ? 0 : (n > kSweepMaxN ? kSweepMaxN : n));
        atomicAdd(&cnt[s + 1], 1);
    }
    __syncthreads();
    if (threadIdx.x < kWave) {
        int carry = 0;
        for (int base = 0; base < kSweepMaxN + 2; base += kWave) {
            const int q = base + (int)threadIdx.x;
            int x = q < kSweepMaxN + 2 ? cnt[q] : 0;
            for (int o = 1; o < kWave; o <<= 1) {
                const int y = __shfl_up(x, o, kWave);
                if ((int)threadIdx.x >= o) x += y;
            }
            if (q < kSweepMaxN + 2) cnt[q] = carry + x;
            carry += __shfl(x, kWave - 1, kWave);
        }
    }
    __syncthreads();
    for (int b = threadIdx.x; b < B; b += 1024) {
        const int64_t n = offsets ? offsets[b + 1] - offsets[b] : nmax;
        const int s = kSweepMaxN - (int)(n < 0 ? 0 : (n > kSweepMaxN ? kSweepMaxN : n));
        order[atomicAdd(&cnt[s], 1)] = b;
    }
    if (threadIdx.x == 0) {
        *queue = 0;
        *ucount = 0;
        *status = bad ? 16 : 0;
    }
}

} // namespace

int sweep_sv_cap(int nmax) {
    int c = 1024;
    while (c < 4 * nmax && c < 8192) c <<= 1;
    return c;
}

int64_t sweep_pool_words(int nmax, u32 p) {
    const int64_t pairs2 = (int64_t)nmax * (nmax - 1);
    return p == 2 ? std::max<int64_t>(1 << 14, pairs2) : std::max<int64_t>(1 << 20, 8 * pairs2);
}

size_t sweep_lds_bytes(int nmax, int sv_cap) {
    const size_t keys = std::max((size_t)sv_cap * 8, (size_t)kSweepCand * 8 + (size_t)kSweepCandWords * 4);
    return keys + sweep_mask_lds(nmax) + sweep_fixed_bytes(nmax);
}

namespace {
using SweepKernel = void (*)(SweepArgs);
SweepKernel sweep_kernel(int nmax, u32 p) {
    if (sweep_mask_lds(nmax)) return p == 2 ? k_sweep<true, false> : k_sweep<true, true>;
    return p == 2 ? k_sweep<false, false> : k_sweep<false, true>;
}
} // namespace

hipError_t sweep_prepare(int nmax, int sv_cap, u32 p) {
    return hipFuncSetAttribute((const void *)sweep_kernel(nmax, p), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)sweep_lds_bytes(nmax, sv_cap));
}

void launch_sweep_order(const int64_t *offsets, int B, int nmax, int *order, unsigned long long *queue,
                        unsigned long long *ucount, int *status, hipStream_t st) {
    hipLaunchKernelGGL(k_sweep_order, dim3(1), dim3(1024), 0, st, offsets, B, nmax, order, queue, ucount, status);
}

void launch_sweep(const SweepArgs &A, int grid, hipStream_t st) {
    hipLaunchKernelGGL(sweep_kernel(A.nmax, A.p), dim3(grid), dim3(kT), sweep_lds_bytes(A.nmax, A.sv_cap), st, A);
}

} // namespace rips
