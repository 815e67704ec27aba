// rips_sweep_dim.hip -- the sweep of one dimension K (1 or 2) of a single
// cloud over Z/2 (the method of rips_sweep.hip, for any number of points and
// for triangles).
//
// Every K-simplex carries the vector of the open K-classes: the simplex of a
// zero apparent pair (s, t) the sum over the other facets of t, a column of
// the reduction (section "Assembling column indices") its unit vector, a
// simplex that dimension K-1 has paired zero (its row can be left out: a
// reduced boundary's pivot is never such a simplex). A (K+1)-simplex whose
// facets do not sum to zero closes the youngest class of the sum.
//
// All passes over simplices are data-parallel over the chip: the simplices by
// diameter bin, the place of each by index, and per simplex the cofacets it
// owns (whose youngest facet it is) as the places of their facets, so that
// the sweep itself, one workgroup, only follows places. It takes whole bins
// in chunks: opens the chunk's classes, resolves its vectors, gathers the
// cofacets that do not cancel, eliminates them in order and substitutes the
// closed classes. Few vectors are nonzero and most of those are shared, so a
// chunk is a few microseconds of one workgroup.
#include "rips_sweep_dim.hpp"

#include <algorithm>

namespace rips {

namespace {

constexpr int kT = 1024;
constexpr int kWaves = kT / kWave;
constexpr u32 kPending = ~0u;
constexpr int kDimBroken = 2;       // a place or row number out of range: a mistake, not a full table
constexpr int kCand = 512;          // cofacets eliminated together
constexpr int kCandWords = 16384;   // and their vectors, in words
constexpr int kPurge = 32;          // eliminations between two purges
constexpr int kTaus = 4;            // cofacets a lane has in flight

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
    for (int64_t i = t0; i < A.N; i += stride) atomicAdd(&A.bin_n[dim_bin(A, A.in.diam[i])], 1u);
    for (int64_t i = t0; i < A.S; i += stride) atomicAdd(&A.bin_s[dim_bin(A, A.cols.diam[i])], 1u);
}

// exclusive scan of the bins of one array, in place; one workgroup an array,
// a multiple of 1024 bins
__global__ void __launch_bounds__(1024) k_dim_scan(u32 *a0, u32 *a1, int nbins) {
    __shared__ u32 s_w[kWaves];
    u32 *a = blockIdx.x == 0 ? a0 : a1;
    const int per = nbins / kT;
    const int lane = lane_id(), w = threadIdx.x / kWave;
    u32 sum = 0;
#pragma unroll 8
    for (int i = 0; i < per; ++i) sum += a[threadIdx.x * per + i];
    u32 inc = sum;
    for (int o = 1; o < kWave; o <<= 1) {
        const u32 x = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += x;
    }
    if (lane == kWave - 1) s_w[w] = inc;
    __syncthreads();
    u32 base = inc - sum;
    for (int q = 0; q < w; ++q) base += s_w[q];
#pragma unroll 8
    for (int i = 0; i < per; ++i) {
        const u32 x = a[threadIdx.x * per + i];
        a[threadIdx.x * per + i] = base;
        base += x;
    }
    if (threadIdx.x == kT - 1) a[nbins] = base;
}

template <int K>
__global__ void __launch_bounds__(256) k_dim_place(DimArgs A) {
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

// ---- the cofacets a simplex owns: third vertices c with every new edge at
// most its diameter long and every other facet older (a facet of the same
// diameter is older when its index is larger, that is when c is larger than
// the vertex it replaces). A group of G lanes a simplex.
template <int K, int G, bool kFill>
__global__ void __launch_bounds__(256) k_dim_own(DimArgs A) {
    const int lane = lane_id(), lg = lane & (G - 1), g0 = lane & ~(G - 1);
    const u64 gmask = G == 64 ? ~0ull : ((1ull << G) - 1) << g0;
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
        float inner[3] = {0.0f, 0.0f, 0.0f}; // K == 2: the edge opposite to vertex i
        if constexpr (K == 2) {
            inner[0] = D[(int64_t)v[1] * n + v[2]];
            inner[1] = D[(int64_t)v[0] * n + v[2]];
            inner[2] = D[(int64_t)v[0] * n + v[1]];
        }
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
                            float fd = K == 2 ? inner[i] : 0.0f;
#pragma unroll
                            for (int j = 0; j <= K; ++j)
                                if (j != i) fd = fmaxf(fd, x[j]);
                            ok = ok && (fd < dm || c > v[i]);
                        }
                    }
                }
                const u64 hit = __ballot(ok) & gmask;
                if (kFill && pass == 1 && ok) {
                    const u32 e = put + (u32)__popcll(hit & ((1ull << lane) - 1));
                    u32 *o = A.tau + (int64_t)e * (K + 2);
                    o[0] = (u32)q;
#pragma unroll
                    for (int i = 0; i <= K; ++i) {
                        int f[K + 1];
                        facet_of<K>(v, i, c, f);
                        const u32 pl = place_of<K>(A, f);
                        o[1 + i] = pl;
                        if (c == zj) A.qdep[(int64_t)i * A.N + q] = pl;
                    }
                }
                mine += __popcll(hit);
                put += (u32)__popcll(hit);
            }
            if (pass == 0) {
                total = mine; // the same in every lane of the group
                if (live && lg == 0 && total > 0) at = atomicAdd(&A.bin_t[bin], (u32)total);
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
    const float wn = 1.0f / fmaxf(fminf(fmaxf(n32, 256.0f), 2048.0f), (float)A.N / 3000.0f), ws = 1.0f / 192.0f;
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
    unsigned long long adds, rows;
    u32 hi_d;
    u64 hi_i;
    int kp[kCand], ki[kCand];
    u64 kz[kCand];                   // nonzero words of a kill's vector
    u32 cd[kCand];                   // candidates: diameter bits (~0: done)
    u64 ci[kCand], cz[kCand];        // ~index, nonzero words
    u32 sage[kDimSlots];             // class of a slot
    uint16_t urow[kDimSlots];        // an open class's unit row, by slot
    uint16_t sl[kDimSlots];          // free slots
    int scan[kWaves + 1];
};

__device__ __forceinline__ bool key_less(u32 d0, u64 i0, u32 d1, u64 i1) { return d0 < d1 || (d0 == d1 && i0 < i1); }

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

__device__ __forceinline__ int dim_append(bool want, int *counter) {
    const u64 bal = __ballot(want);
    if (!bal) return -1;
    const int lane = lane_id(), lead = __ffsll((unsigned long long)bal) - 1;
    int base = 0;
    if (lane == lead) base = atomicAdd(counter, __popcll(bal));
    base = __shfl(base, lead, kWave);
    return base + __popcll(bal & ((1ull << lane) - 1));
}

// A row's vector is shared by all simplices that hold its number, and rows
// with equal unit vectors are one row: a row that becomes zero or a unit
// vector keeps its number on the simplices and is replaced on the way, by
// rmap (most sums that cancel are of two such rows, and then cost no look at
// the vectors). Every kPurge eliminations the simplices' numbers are brought
// up to date and the replaced rows are free again.
template <int K>
__global__ void __launch_bounds__(kT) k_dim_sweep(DimArgs A) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ DimShared Sh;
    LDS u32 *vec = (LDS u32 *)smem;                                // kCandWords
    LDS uint16_t *rmap = (LDS uint16_t *)(smem + kCandWords * 4);  // kDimRows
    const int tid = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int W = A.W;
    const int nslots = W * 32, ccap = min(kCand, kCandWords / W);
    if (tid == 0) {
        Sh.nact = Sh.nnz = Sh.fail = Sh.nfree = Sh.ndead = Sh.since = 0;
        Sh.nrows = 1; // row 0: the zero vector
        rmap[0] = 0;
        Sh.sfree = nslots;
        Sh.adds = Sh.rows = 0;
    }
    for (int q = tid; q < nslots; q += kT) Sh.sl[q] = (uint16_t)(nslots - 1 - q);
    __syncthreads();
    const int nch = __builtin_amdgcn_readfirstlane(A.out->nch);
    for (int ch = 0; ch < nch; ++ch) {
        const u32 n0 = A.ch_n[ch], n1 = A.ch_n[ch + 1], t0 = A.ch_t[ch], t1 = A.ch_t[ch + 1];
        const int s0 = (int)A.ch_s[ch], s1 = (int)A.ch_s[ch + 1];
        // ---- the classes that open here
        if (s1 > s0) {
            const int ns = s1 - s0, nf = Sh.sfree, nr = Sh.nfree, top = Sh.nrows, na = Sh.nact, nz = Sh.nnz;
            const int fresh = max(0, ns - nr);
            if (ns > nf || top + fresh > kDimRows) {
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
                for (int w = 0; w < W; ++w) A.pool[(int64_t)r * W + w] = w == (slot >> 5) ? 1u << (slot & 31) : 0u;
                A.rsum[r] = 1ull << (slot >> 5);
                rmap[r] = (uint16_t)r;
                Sh.urow[slot] = (uint16_t)r;
                A.ract[na + i] = r;
                const u32 pl = A.bq[s0 + i];
                if (pl >= (u32)A.N) Sh.fail = kDimBroken;
                const u32 q = min(pl, (u32)A.N - 1);
                A.ids[q] = r;
                A.nzl[nz + i] = q;
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
        for (int tries = 0;; ++tries) {
            bool left = false;
            for (u32 q = n0 + tid; q < n1; q += kT) {
                if (ld(&A.ids[q]) != kPending) continue;
                u32 r[K + 1];
#pragma unroll
                for (int i = 0; i <= K; ++i) {
                    const u32 pl = A.qdep[(int64_t)i * A.N + q];
                    if (pl >= (u32)A.N) Sh.fail = kDimBroken;
                    r[i] = ld(&A.ids[min(pl, (u32)A.N - 1)]);
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
                    if (r[i] >= (u32)kDimRows) Sh.fail = kDimBroken;
                    r[i] = rmap[r[i] & (kDimRows - 1)] & (kDimRows - 1);
                }
                const int k = cancel<K + 1>(r);
                u32 x = 0;
#pragma unroll
                for (int i = 0; i <= K; ++i) x |= r[i];
                if (k > 1) {
                    u64 z = 0;
                    u32 one = 0; // the only nonzero word
                    for (u64 m = sum_words<K + 1>(A, r); m; m &= m - 1) {
                        const int w = __ffsll((unsigned long long)m) - 1;
                        const u32 y = sum_word<K + 1>(A, r, w);
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
                            for (int w = 0; w < W; ++w) A.pool[(int64_t)x * W + w] = sum_word<K + 1>(A, r, w);
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
                if (x) A.nzl[atomicAdd(&Sh.nnz, 1)] = q;
                st(&A.ids[q], x);
            }
            if (!__any(left)) break;
            if (tries > (1 << 16)) { // cannot happen: the order is acyclic
                Sh.fail = 1;
                break;
            }
        }
        __syncthreads();
        const bool none = Sh.nnz == 0, failed = Sh.fail != 0;
        if (tid == 0 && Sh.nfree < 0) Sh.nfree = 0;
        __syncthreads();
        if (failed) break;
        if (none) continue;
        // ---- the owned cofacets whose facets do not cancel
        u32 lo_d = 0, hi_d = ~0u;
        u64 lo_i = 0, hi_i = ~0ull;
        bool first = true;
        for (;;) {
            if (tid == 0) Sh.ncand = 0;
            __syncthreads();
            for (u32 b = t0 + (u32)wave * kWave; b < t1; b += kTaus * kT) {
                // kTaus of them a lane, so that their loads are in flight together
                u32 qs[kTaus], rs[kTaus][K + 2];
                bool some = false, broken = false;
#pragma unroll
                for (int u = 0; u < kTaus; ++u) {
                    const u32 t = min(b + u * kT + (u32)lane, t1 - 1);
                    const u32 *o = A.tau + (int64_t)t * (K + 2);
                    qs[u] = o[0];
#pragma unroll
                    for (int i = 0; i < K + 2; ++i) rs[u][i] = o[i];
                }
#pragma unroll
                for (int u = 0; u < kTaus; ++u)
#pragma unroll
                    for (int i = 0; i < K + 2; ++i) {
                        broken = broken | (rs[u][i] >= (u32)A.N);
                        rs[u][i] = A.ids[min(rs[u][i], (u32)A.N - 1)];
                    }
#pragma unroll
                for (int u = 0; u < kTaus; ++u) {
#pragma unroll
                    for (int i = 0; i < K + 2; ++i) {
                        broken = broken | (rs[u][i] >= (u32)kDimRows);
                        rs[u][i] = rmap[rs[u][i] & (kDimRows - 1)] & (kDimRows - 1);
                    }
                    some = some | (cancel<K + 2>(rs[u]) > 0);
                }
                if (broken) Sh.fail = kDimBroken;
                if (!__any(some)) continue;
#pragma unroll
                for (int u = 0; u < kTaus; ++u) {
                const u32 t = b + u * kT + (u32)lane;
                u32 r[K + 2], id[K + 2];
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
                if (ok)
                    for (u64 m = sum_words<K + 2>(A, r); m; m &= m - 1) {
                        const int w = __ffsll((unsigned long long)m) - 1;
                        if (sum_word<K + 2>(A, r, w)) z |= 1ull << w;
                    }
                ok = ok && z != 0;
                u32 kd = 0;
                u64 ki = 0;
                if (ok) {
                    // the cofacet's index, from its owner and the vertex that
                    // its facet opposite to the owner's first vertex adds
                    const u64 pv = A.qverts[q];
                    const u64 pf = A.qverts[min(A.tau[(int64_t)t * (K + 2) + 1], (u32)A.N - 1)];
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
                // of the lanes with the same rows only the oldest cofacet
                for (int i = 0; i < K + 2; ++i) id[i] = r[i];
                for (u64 todo = __ballot(ok); todo;) {
                    int l = __ffsll((unsigned long long)todo) - 1;
                    bool same = ok;
#pragma unroll
                    for (int i = 0; i < K + 2; ++i) same = same & (id[i] == (u32)__builtin_amdgcn_readlane(id[i], l));
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
                            for (int w = 0; w < W; ++w) vec[s * W + w] = (z >> w) & 1ull ? sum_word<K + 2>(A, r, w) : 0u;
                        }
                    }
                }
                }
            }
            __syncthreads();
            const int nc = __builtin_amdgcn_readfirstlane(Sh.ncand);
            if (Sh.fail) break; // set before the barrier, if at all
            const bool last = hi_d == ~0u;
            if (nc > ccap) {
                // too many at once: only those up to the quarter point of the stored ones
                if (tid < ccap) {
                    int less = 0;
                    for (int q = 0; q < ccap; ++q) less += key_less(Sh.cd[q], Sh.ci[q], Sh.cd[tid], Sh.ci[tid]) ? 1 : 0;
                    if (less == ccap / 4) {
                        Sh.hi_d = Sh.cd[tid];
                        Sh.hi_i = Sh.ci[tid];
                    }
                }
                __syncthreads();
                hi_d = Sh.hi_d;
                hi_i = Sh.hi_i;
                continue;
            }
            if (nc > 0) {
                // ---- elimination in order, by one wave
                if (wave == 0) {
                    int nk = 0;
                    unsigned long long adds = 0;
                    for (;;) {
                        u32 bd = ~0u;
                        u64 bi = ~0ull;
                        int bj = 0;
                        for (int j = lane; j < nc; j += kWave)
                            if (Sh.cd[j] != ~0u && key_less(Sh.cd[j], Sh.ci[j], bd, bi)) {
                                bd = Sh.cd[j];
                                bi = Sh.ci[j];
                                bj = j;
                            }
                        for (int o = 32; o >= 1; o >>= 1) {
                            const u32 xd = __shfl_xor(bd, o, kWave);
                            const u64 xi = ((u64)__shfl_xor((u32)(bi >> 32), o, kWave) << 32) | __shfl_xor((u32)bi, o, kWave);
                            const int xj = __shfl_xor(bj, o, kWave);
                            if (key_less(xd, xi, bd, bi)) {
                                bd = xd;
                                bi = xi;
                                bj = xj;
                            }
                        }
                        if (bd == ~0u) break;
                        bj = __builtin_amdgcn_readfirstlane(bj);
                        // its youngest class: a lane a word, then the largest class number
                        const u32 wd = lane < W ? vec[bj * W + lane] : 0u;
                        const u64 zw = __ballot(wd != 0u);
                        u32 age = 0;
                        int slot = 0;
                        for (u32 m = wd; m; m &= m - 1) {
                            const int s = lane * 32 + __ffs((int)m) - 1;
                            if (Sh.sage[s] + 1 > age) {
                                age = Sh.sage[s] + 1;
                                slot = s;
                            }
                        }
                        for (int o = 32; o >= 1; o >>= 1) {
                            const u32 xa = __shfl_xor(age, o, kWave);
                            const int xs = __shfl_xor(slot, o, kWave);
                            if (xa > age) {
                                age = xa;
                                slot = xs;
                            }
                        }
                        slot = __builtin_amdgcn_readfirstlane(slot);
                        if (lane == 0) {
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
                            if (Sh.cd[j] == ~0u || !((vec[j * W + (slot >> 5)] >> (slot & 31)) & 1u)) continue;
                            u64 z = Sh.cz[j];
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
                    u32 *row = A.pool + (int64_t)r * W;
                    u64 z = A.rsum[r];
                    bool changed = false;
                    for (int q = 0; q < nk; ++q) {
                        const int p = Sh.kp[q];
                        if (!((z >> (p >> 5)) & 1ull) || !((row[p >> 5] >> (p & 31)) & 1u)) continue;
                        const LDS u32 *kv = vec + Sh.ki[q] * W;
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
                    if (!z) rmap[r] = 0;
                    else if (is_unit(z, one))
                        rmap[r] = Sh.urow[(__ffsll((unsigned long long)z) - 1) * 32 + __ffs((int)one) - 1];
                }
                if (adds) atomicAdd(&Sh.adds, adds);
                // the closed classes' slots are free again
                for (int q = tid; q < nk; q += kT) Sh.sl[Sh.sfree + q] = (uint16_t)Sh.kp[q];
                __syncthreads();
                // replaced rows leave the rows in use; what pointed to them
                // points to what replaced them
                const int nr = Sh.nrows, nz = Sh.nnz;
                const bool purge = Sh.since >= kPurge || nr > kDimRows * 3 / 4;
                for (int r = tid; r < nr; r += kT) rmap[r] = rmap[rmap[r]];
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
                    const bool keep = i < na && rmap[r] == r;
                    const int at = dim_append(keep, &Sh.nact);
                    if (keep) A.ract[at] = r; // at most i: entries already read
                    const int de = dim_append(i < na && !keep, &Sh.ndead);
                    if (i < na && !keep) A.rdead[de] = r;
                    __syncthreads();
                }
                if (purge) {
                    // ---- the simplices' numbers brought up to date
                    for (int q0 = 0; q0 < nz; q0 += kT) {
                        const int i = q0 + tid;
                        const u32 q = i < nz ? A.nzl[i] : 0;
                        __syncthreads();
                        bool keep = false;
                        if (i < nz) {
                            const u32 r = rmap[A.ids[q] & (kDimRows - 1)] & (kDimRows - 1);
                            A.ids[q] = r;
                            keep = r != 0;
                        }
                        const int at = dim_append(keep, &Sh.nnz);
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
        A.out->total = A.bin_t[A.nbins];
    }
}

unsigned blocks_for(int64_t n, int per) {
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + per - 1) / per, 16384));
}

template <int K>
void partition_k(const DimArgs &A, hipStream_t st) {
    launch_fill_u32(A.bin_n, 3 * (kDimBins + 64), 0u, st); // bin_n, bin_t and bin_s are one buffer
    hipLaunchKernelGGL((k_dim_hist<K>), dim3(blocks_for(A.N, 256)), dim3(256), 0, st, A);
    hipLaunchKernelGGL(k_dim_scan, dim3(2), dim3(kT), 0, st, A.bin_n, A.bin_s, A.nbins);
    if (!A.direct) launch_fill_i64(A.ph.keys, (int64_t)A.ph.mask + 1, kEmpty, st);
    hipLaunchKernelGGL((k_dim_place<K>), dim3(blocks_for(A.N, 256)), dim3(256), 0, st, A);
    if (A.c.nb.off) hipLaunchKernelGGL((k_dim_own<K, 16, false>), dim3(blocks_for(A.N, 16)), dim3(256), 0, st, A);
    else hipLaunchKernelGGL((k_dim_own<K, 64, false>), dim3(blocks_for(A.N, 4)), dim3(256), 0, st, A);
    hipLaunchKernelGGL(k_dim_scan, dim3(1), dim3(kT), 0, st, A.bin_t, A.bin_t, A.nbins);
}

template <int K>
void fill_k(const DimArgs &A, hipStream_t st) {
    if (A.c.nb.off) hipLaunchKernelGGL((k_dim_own<K, 16, true>), dim3(blocks_for(A.N, 16)), dim3(256), 0, st, A);
    else hipLaunchKernelGGL((k_dim_own<K, 64, true>), dim3(blocks_for(A.N, 4)), dim3(256), 0, st, A);
    hipLaunchKernelGGL((k_dim_births<K>), dim3(blocks_for(A.S, 256)), dim3(256), 0, st, A);
    hipLaunchKernelGGL(k_dim_chunks, dim3(1), dim3(kT), 0, st, A);
}

constexpr int kSweepLds = kCandWords * 4 + kDimRows * 2;

template <int K>
hipError_t sweep_k(const DimArgs &A, hipStream_t st) {
    hipError_t e = hipFuncSetAttribute((const void *)k_dim_sweep<K>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       kSweepLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_dim_sweep<K>), dim3(1), dim3(kT), kSweepLds, st, A);
    return hipSuccess;
}

} // namespace

void launch_dim_partition(int K, const DimArgs &A, hipStream_t st) {
    if (K == 1) partition_k<1>(A, st);
    else partition_k<2>(A, st);
}

void launch_dim_fill(int K, const DimArgs &A, hipStream_t st) {
    if (K == 1) fill_k<1>(A, st);
    else fill_k<2>(A, st);
}

hipError_t launch_dim_sweep(int K, const DimArgs &A, hipStream_t st) {
    return K == 1 ? sweep_k<1>(A, st) : sweep_k<2>(A, st);
}

void launch_dim_bars(int K, const DimArgs &A, BarBuf bars, PivotHash piv, hipStream_t st) {
    if (K == 1) hipLaunchKernelGGL(k_dim_bars<1>, dim3(1), dim3(kT), 0, st, A, bars, piv);
    else hipLaunchKernelGGL(k_dim_bars<2>, dim3(1), dim3(kT), 0, st, A, bars, piv);
}

} // namespace rips
