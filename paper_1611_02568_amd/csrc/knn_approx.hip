// Approximate k nearest neighbours on gfx950: the K-NNG construction the
// paper adopts from LargeVis to build P faster (Section 4.3).
//
// 1. Random-projection trees, built level by level for all ranges at once.
//    The points are a permutation; a range [a, b) of more than leaf_size
//    points splits by the hyperplane halfway between two of its points x_a
//    and x_b: a point goes right iff sum_d (x_d - (x_ad + x_bd) / 2)
//    (x_ad - x_bd) > 0, in FP64 with the terms in order of d and every
//    operation rounded on its own.  The split keeps the order inside each
//    side (a global exclusive scan of the side flags gives each point its new
//    place).  If a side would get fewer than k + 1 points, or from level 48
//    on, the range is cut in the middle instead, so every leaf (at most
//    leaf_size >= 2k + 2 points) offers each of its points k candidates.  The
//    two points come from SplitMix64 (Steele, Lea and Flood, 2014) keyed by
//    the seed, the tree, the level and the range's first position.
// 2. Each point's list keeps the best k of its leaf mates over all trees by
//    (squared distance, index), distinct, in FP64 (terms in order of d).
// 3. Rounds of neighbour exploring: each point's new list is the best k of
//    its list and its neighbours' lists, all read from the previous round.
//
// Every decision is taken in FP64 with a fixed operation order, so the result
// is a deterministic function of the data and the seed (the CPU reference
// takes the same steps).
#include "ctx.h"
#include "nearest.h"

namespace psne {

namespace {

constexpr int kBlock = 256;
constexpr int kRpMaxLevel = 48;
constexpr int kXcds = 8;
constexpr int kDeal = 64;                   // positions dealt to an XCD at a time

inline dim3 grid_for(int64_t n) { return dim3((unsigned)ceil_div(n > 0 ? n : 1, kBlock)); }

__device__ __forceinline__ uint64_t rp_draw(uint64_t seed, int tree, int level, int64_t a,
                                            int which) {
    uint64_t x = splitmix64(seed ^ (uint64_t)(uint32_t)tree);
    x = splitmix64(x ^ (uint64_t)(uint32_t)level);
    return splitmix64(x ^ (((uint64_t)a << 1) | (uint64_t)which));
}

__device__ __forceinline__ double as_f64(float v) { return (double)v; }
__device__ __forceinline__ double as_f64(double v) { return v; }
__device__ __forceinline__ double as_f64(uint8_t v) { return (double)v; }

__global__ __launch_bounds__(kBlock) void k_rp_init(uint32_t* __restrict__ perm,
                                                    uint32_t* __restrict__ sa,
                                                    uint32_t* __restrict__ sb, int64_t n) {
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p >= n) return;
    perm[p] = (uint32_t)p;
    sa[p] = 0;
    sb[p] = (uint32_t)n;
}

// side of the hyperplane for every position of a range that splits at this
// level (0 elsewhere); side[n] = 0 closes the scan; *any = 1 if a range splits.
// Bound by its loads, rows read by single threads: 16 bytes at a time a level
// of 100,000 x 100 takes 19 us, 43 by elements.
template <typename X>
__global__ __launch_bounds__(kBlock) void k_rp_side(const X* __restrict__ Xm, int32_t D,
                                                    const uint32_t* __restrict__ perm,
                                                    const uint32_t* __restrict__ sa,
                                                    const uint32_t* __restrict__ sb, int64_t n,
                                                    int32_t leaf, uint64_t seed, int tree,
                                                    int level, int64_t* __restrict__ side,
                                                    uint32_t* __restrict__ any) {
#pragma clang fp contract(off)
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p > n) return;
    if (p == n) {
        side[n] = 0;
        return;
    }
    const int64_t a = sa[p], m = (int64_t)sb[p] - a;
    int64_t s = 0;
    if (m > leaf) {
        if (p == a) atomicOr(any, 1u);
        if (level < kRpMaxLevel) {
            const int64_t ia = (int64_t)(rp_draw(seed, tree, level, a, 0) % (uint64_t)m);
            int64_t ib = (int64_t)(rp_draw(seed, tree, level, a, 1) % (uint64_t)(m - 1));
            if (ib >= ia) ib++;
            const X* xa = Xm + (int64_t)perm[a + ia] * D;
            const X* xb = Xm + (int64_t)perm[a + ib] * D;
            const X* xi = Xm + (int64_t)perm[p] * D;
            constexpr int V = 16 / sizeof(X);
            double acc = 0.0;
            auto term = [&](X i, X u, X w) {
                const double va = as_f64(u), vb = as_f64(w);
                const double mid = (va + vb) * 0.5;
                const double v = va - vb;
                acc = acc + (as_f64(i) - mid) * v;
            };
            int d = 0;
            for (; d + V <= D; d += V) {
                X i[V], u[V], w[V];
                __builtin_memcpy(i, xi + d, 16);
                __builtin_memcpy(u, xa + d, 16);
                __builtin_memcpy(w, xb + d, 16);
#pragma unroll
                for (int e = 0; e < V; e++) term(i[e], u[e], w[e]);
            }
            for (; d < D; d++) term(xi[d], xa[d], xb[d]);
            s = acc > 0.0 ? 1 : 0;
        }
    }
    side[p] = s;
}

// new place of every position: the left side keeps its order at the front
// of the range, the right side after it; a range that cannot split well
// (a side under k + 1 points, or level >= 48) is cut in the middle in place
__global__ __launch_bounds__(kBlock) void k_rp_scatter(
    const uint32_t* __restrict__ perm, const uint32_t* __restrict__ sa,
    const uint32_t* __restrict__ sb, const int64_t* __restrict__ side,
    const int64_t* __restrict__ ones, int64_t n, int32_t leaf, int32_t k, int level,
    uint32_t* __restrict__ perm2, uint32_t* __restrict__ sa2, uint32_t* __restrict__ sb2) {
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p >= n) return;
    const int64_t a = sa[p], b = sb[p], m = b - a;
    if (m <= leaf) {
        perm2[p] = perm[p];
        sa2[p] = (uint32_t)a;
        sb2[p] = (uint32_t)b;
        return;
    }
    const int64_t right = ones[b] - ones[a];
    const int64_t nl = m - right;
    if (level >= kRpMaxLevel || nl < k + 1 || right < k + 1) {
        const int64_t h = a + m / 2;
        perm2[p] = perm[p];
        sa2[p] = (uint32_t)(p < h ? a : h);
        sb2[p] = (uint32_t)(p < h ? h : b);
        return;
    }
    const int64_t before = ones[p] - ones[a];         // right-side points before p in the range
    int64_t q;
    if (side[p]) {
        q = a + nl + before;
        sa2[q] = (uint32_t)(a + nl);
        sb2[q] = (uint32_t)b;
    } else {
        q = a + (p - a - before);
        sa2[q] = (uint32_t)a;
        sb2[q] = (uint32_t)(a + nl);
    }
    perm2[q] = perm[p];
}

// ---------------------------------------------------------------------------
// List updates, one block of four wavefronts per point.  The point's candidates
// stream through a set in LDS (it holds the point and its current list to begin
// with), which drops repeats.  The new ones gather until there is one for every
// thread; an approximate distance rules out most of those beyond the list's
// k-th entry, and the rest are merged into the list by groups of 64 with their
// distance in FP64, terms in order of d.  The resulting list, the best k of the
// old list and the candidates by (d^2, index), does not depend on the order of
// insertion.  Distances are compared as keys (dist_key): of a row that holds NaN
// they come after all others, by index, and enter a list only while it is short.
//
// A round of exploring at 100,000 x 100 (FP32, k = 90: 8,100 candidates per
// point, 2,700 distinct) is bound by the latency of its row gathers, so what
// counts is wavefronts in flight (32 KB of LDS per block lets five share a CU)
// and bytes in order: 13.6 ms, where one wavefront per point with rows staged
// through LDS took 107, and 26.3 without the first look.  All leaves of a tree
// take 1.4 ms, where they took 5.0.
// ---------------------------------------------------------------------------
constexpr int kMaxSetBits = 12;
constexpr int kProbes = 8;                   // buckets
constexpr int kMaxK = kBlock;                // a thread per list entry in the merge
constexpr int kFlush = 64;                   // merged from this many on
constexpr int kPer = 2;                      // candidates per thread and round

// the precision of the first look at a distance
template <typename X> struct Near { using type = X; };
template <> struct Near<uint8_t> { using type = double; };

struct ListLds {
    uint64_t ld[kMaxK];
    int32_t lj[kMaxK];
    uint64_t ld2[kMaxK];                     // the merged list before it is copied back
    int32_t lj2[kMaxK];
    int32_t gj[kBlock + kFlush];             // candidates that may enter
    uint64_t gd[kBlock + kFlush];
    uint64_t sd[kWave];                      // a group of them, sorted
    int32_t sj[kWave];
    int32_t oj[kMaxK], om[kMaxK];            // exploring: the old list and its entries' lengths
    int32_t pend[kBlock + kPer * kBlock];
    int32_t m, npend, ng, ns;
};

// number of entries of a sorted list (ascending (d, j)) below (d, j)
__device__ __forceinline__ int rank_in(const uint64_t* ld, const int32_t* lj, int m, uint64_t d,
                                       int32_t j) {
    int lo = 0, hi = m;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (knn_less(ld[mid], lj[mid], d, j)) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// True if v was not in the set (and is now).  Four entries share a bucket, so
// that one 16-byte read finds a repeat; entries of a bucket fill in order.  A
// set too full to place v reports it as new, which at worst computes a repeat
// (rejected on insertion).
__device__ __forceinline__ bool set_add(int32_t* set, int bits, int32_t v) {
    if (bits == 0) {
        const uint32_t one = 1u << (v & 31);
        return !(atomicOr(reinterpret_cast<uint32_t*>(set) + (v >> 5), one) & one);
    }
    const uint32_t buckets = 1u << (bits - 2);
    uint32_t h = ((uint32_t)v * 0x9E3779B1u) >> (34 - bits);
#pragma unroll 1
    for (int q = 0; q < kProbes;) {
        int32_t* at = set + 4 * h;
        const int4 c = *reinterpret_cast<const int4*>(at);
        if (c.x == v || c.y == v || c.z == v || c.w == v) return false;
        if (c.w >= 0) {                      // full
            h = (h + 1) & (buckets - 1);
            q++;
            continue;
        }
        const int e = c.x < 0 ? 0 : c.y < 0 ? 1 : c.z < 0 ? 2 : 3;
        const int32_t old = atomicCAS(at + e, -1, v);
        if (old == -1) return true;
        if (old == v) return false;
    }
    return true;
}

// Squared distance of two rows, FP64, terms in order of d, no contraction; 16
// bytes per load, at the rows' own alignment.  Sums of squares of bytes are
// whole numbers, exact in any order.
template <typename X>
__device__ __forceinline__ double row_sqdist(const X* __restrict__ a, const X* __restrict__ b,
                                             int32_t D) {
#pragma clang fp contract(off)
    constexpr int V = 16 / sizeof(X);
    double acc = 0.0;
    int d = 0;
#pragma unroll 4
    for (; d + V <= D; d += V) {
        X u[V], v[V];
        __builtin_memcpy(u, a + d, 16);
        __builtin_memcpy(v, b + d, 16);
        if constexpr (sizeof(X) == 1) {
            uint32_t part = 0;
#pragma unroll
            for (int e = 0; e < V; e++) {
                const int32_t x = (int32_t)u[e] - (int32_t)v[e];
                part += (uint32_t)(x * x);
            }
            acc = acc + (double)part;
        } else {
#pragma unroll
            for (int e = 0; e < V; e++) {
                const double x = (double)u[e] - (double)v[e];
                acc = acc + x * x;
            }
        }
    }
    for (; d < D; d++) {
        const double x = as_f64(a[d]) - as_f64(b[d]);
        acc = acc + x * x;
    }
    return acc;
}

// Approximate squared distances of the wavefront's candidates (lane l's row is
// cand) to row i, in the rows' own precision: four lanes share a row, 64 bytes
// per load, and add up its terms in their own order.
template <typename X>
__device__ __forceinline__ typename Near<X>::type near_sqdist(const X* __restrict__ Xm, int32_t D,
                                                              int64_t i, int32_t cand) {
    using A = typename Near<X>::type;
    constexpr int V = 16 / sizeof(X);
    const int lane = lane_id(), part = lane & 3;
    const X* a = Xm + i * D;
    const X* row[4];
    A acc[4];
#pragma unroll
    for (int p = 0; p < 4; p++) {
        const int32_t c = __shfl(cand, 16 * p + (lane >> 2), kWave);
        row[p] = Xm + (c < 0 ? i : (int64_t)c) * D;
        acc[p] = A(0);
    }
    int d0 = 0;
    for (; d0 + V <= D; d0 += 4 * V) {
        const int d = d0 + part * V;
        if (d + V <= D) {
            X u[V], v[4][V];
            __builtin_memcpy(u, a + d, 16);
#pragma unroll
            for (int p = 0; p < 4; p++) __builtin_memcpy(v[p], row[p] + d, 16);
#pragma unroll
            for (int p = 0; p < 4; p++) {
                if constexpr (sizeof(X) == 1) {
                    uint32_t sum = 0;
#pragma unroll
                    for (int e = 0; e < V; e++) {
                        const int32_t x = (int32_t)u[e] - (int32_t)v[p][e];
                        sum += (uint32_t)(x * x);
                    }
                    acc[p] += (A)sum;
                } else {
#pragma unroll
                    for (int e = 0; e < V; e++) {
                        const A x = u[e] - v[p][e];
                        acc[p] += x * x;
                    }
                }
            }
        }
    }
    for (int d = D / V * V + part; d < D; d += 4)
#pragma unroll
        for (int p = 0; p < 4; p++) {
            const A x = (A)a[d] - (A)row[p][d];
            acc[p] += x * x;
        }
    A out = A(0);
#pragma unroll
    for (int p = 0; p < 4; p++) {
        acc[p] += __shfl_xor(acc[p], 1, kWave);
        acc[p] += __shfl_xor(acc[p], 2, kWave);
        const A v = __shfl(acc[p], 4 * (lane & 15), kWave);
        if (lane >> 4 == p) out = v;
    }
    return out;
}

// True if a sum s of D squares in that precision says that the squared distance
// in FP64 exceeds bound: every term is off by at most 3 roundings and every
// addition by one, all terms are >= 0, and D terms below the smallest normal
// number lose no more than tiny.  An overflow or NaN says nothing.
template <typename A>
__device__ __forceinline__ bool beyond(A s, int32_t D, double bound) {
    const double unit = sizeof(A) == 4 ? 0x1p-24 : 0x1p-53;
    const double tiny = sizeof(A) == 4 ? 0x1p-126 : 0x1p-1022;
    const double low = (double)s * (1.0 - ((double)D + 8.0) * 2.0 * unit) - (double)D * tiny;
    return s <= (sizeof(A) == 4 ? (A)3.4028234663852886e38 : (A)1.7976931348623157e308) &&
           low > bound;
}

// The first ng of the candidates that may enter: their distances, and the merge
// into the list, a group of 64 at a time.
template <typename X>
__device__ __forceinline__ void merge(const X* __restrict__ Xm, int32_t D, int64_t i, int32_t k,
                                      ListLds& s, int ng) {
    const int t = threadIdx.x, lane = lane_id();
    for (int q = t; q < ng; q += kBlock)
        s.gd[q] = dist_key(row_sqdist(Xm + i * D, Xm + (int64_t)s.gj[q] * D, D));
    __syncthreads();
    for (int g0 = 0; g0 < ng; g0 += kWave) {
        const int m0 = s.m;
        if (t < kWave) {
            uint64_t d = g0 + lane < ng ? s.gd[g0 + lane] : ~0ull;
            int32_t j = g0 + lane < ng ? s.gj[g0 + lane] : 0x7FFFFFFF;
            // sort the group, drop repeats (equal pairs: the same index has the
            // same distance), and place every entry of list and group by its
            // rank in the other; the first k form the new list
            wave_sort(d, j);
            const uint64_t pd = __shfl_up(d, 1, kWave);
            const int32_t pj = __shfl_up(j, 1, kWave);
            bool valid = j != 0x7FFFFFFF && !(lane > 0 && pd == d && pj == j);
            const int r_list = valid ? rank_in(s.ld, s.lj, m0, d, j) : 0;
            if (valid && r_list < m0 && s.ld[r_list] == d && s.lj[r_list] == j) valid = false;
            const uint64_t vb = ballot64(valid);
            const int g_rank = __popcll(vb & lanemask_lt());
            if (valid) {
                s.sd[g_rank] = d;
                s.sj[g_rank] = j;
            }
            if (valid && g_rank + r_list < k) {
                s.ld2[g_rank + r_list] = d;
                s.lj2[g_rank + r_list] = j;
            }
            if (lane == 0) s.ns = __popcll(vb);
        }
        __syncthreads();
        const int ns = s.ns, mn = m0 + ns < k ? m0 + ns : k;
        if (t < m0) {
            const int pos = t + rank_in(s.sd, s.sj, ns, s.ld[t], s.lj[t]);
            if (pos < k) {
                s.ld2[pos] = s.ld[t];
                s.lj2[pos] = s.lj[t];
            }
        }
        __syncthreads();
        if (t < mn) {
            s.ld[t] = s.ld2[t];
            s.lj[t] = s.lj2[t];
        }
        if (t == 0) s.m = mn;
        __syncthreads();
    }
}

// this thread's candidate (cand < 0: none): those that may enter the list are
// kept, and merged when there are enough or at the end
template <typename X>
__device__ __forceinline__ void process(const X* __restrict__ Xm, int32_t D, int64_t i, int32_t k,
                                        ListLds& s, int32_t cand, bool end) {
    const int lane = lane_id();
    bool may = cand >= 0;
    if (s.m == k) {
        const auto near = near_sqdist(Xm, D, i, cand);
        may = may && !beyond(near, D, key_dist(s.ld[k - 1]));
    }
    const uint64_t mb = ballot64(may);
    int base = 0;
    if (lane == 0 && mb) base = atomicAdd(&s.ng, __popcll(mb));
    base = __shfl(base, 0, kWave) + __popcll(mb & lanemask_lt());
    if (may) s.gj[base] = cand;
    __syncthreads();
    const int ng = s.ng;
    __syncthreads();
    if (ng >= kFlush || end) {
        merge<X>(Xm, D, i, k, s, ng);
        if (threadIdx.x == 0) s.ng = 0;
        __syncthreads();
    }
}

// MODE 0: the leaf mates of the point at a position of one tree, the list
// updated in place.  MODE 1: one round of exploring for that point: the old
// lists (ld, lj, lm) of it and its neighbours in, the new list (nd, nj, nm)
// out.  The positions are dealt to the XCDs in runs of 64, so that points of one
// leaf, which share neighbours, meet in one L2.  (An eighth of all positions per
// XCD leaves most of them waiting for the largest cluster's: 22.5 ms for the
// round above.)
template <typename X, int MODE>
__global__ __launch_bounds__(kBlock, 5) void k_lists(
    const X* __restrict__ Xm, int32_t D, int64_t b0, int64_t b1, int32_t k, int bits,
    int words, const uint32_t* __restrict__ perm, const uint32_t* __restrict__ sa,
    const uint32_t* __restrict__ sb, const uint64_t* __restrict__ ld,
    const int32_t* __restrict__ lj, const int32_t* __restrict__ lm, uint64_t* __restrict__ nd,
    int32_t* __restrict__ nj, int32_t* __restrict__ nm) {
    __shared__ ListLds s;
    extern __shared__ __attribute__((aligned(16))) int32_t set[];
    const int t = threadIdx.x, lane = lane_id();
    const int64_t x = blockIdx.x / kXcds;
    const int64_t b = b0 + (x / kDeal * kXcds + blockIdx.x % kXcds) * kDeal + x % kDeal;
    if (b >= b1) return;
    const int64_t i = perm[b];
    for (int q = t; q < words; q += kBlock) set[q] = bits ? -1 : 0;
    const int32_t m = lm[i];
    if (t < m) {
        const int32_t j = lj[i * k + t];
        s.ld[t] = ld[i * k + t];
        s.lj[t] = j;
        if (MODE == 1) {
            s.oj[t] = j;
            s.om[t] = lm[j];
        }
    }
    if (t == 0) {
        s.m = m;
        s.npend = 0;
        s.ng = 0;
    }
    __syncthreads();
    // the point itself and its listed neighbours are not candidates
    if (t < m) set_add(set, bits, s.lj[t]);
    if (t == 0) set_add(set, bits, (int32_t)i);
    __syncthreads();
    // the candidate stream: the leaf, or entry c of the list of neighbour a for
    // x = a k + c; a round's are fetched while those before it are worked on
    const int64_t first = MODE == 0 ? sa[b] : 0;
    const int64_t total = MODE == 0 ? (int64_t)sb[b] - first : (int64_t)m * k;
    const uint32_t inv = 0xFFFFFFFFu / (uint32_t)k + 1;      // x / k = x inv >> 32: x k < 2^32
    int32_t next[kPer];
    auto fetch = [&](int64_t x0) {
#pragma unroll
        for (int q = 0; q < kPer; q++) {
            const int64_t x = x0 + q * kBlock + t;
            int32_t v = -1;
            if (x < total) {
                if (MODE == 0) {
                    v = (int32_t)perm[first + x];
                } else {
                    const int32_t a = k == 1 ? (int32_t)x : (int32_t)__umulhi((uint32_t)x, inv);
                    const int32_t c = (int32_t)x - a * k;
                    if (c < s.om[a]) v = lj[(int64_t)s.oj[a] * k + c];
                }
            }
            next[q] = v;
        }
    };
    fetch(0);
    for (int64_t x0 = 0;; x0 += kPer * kBlock) {
        int32_t v[kPer];
#pragma unroll
        for (int q = 0; q < kPer; q++) v[q] = next[q];
        fetch(x0 + kPer * kBlock);
#pragma unroll
        for (int q = 0; q < kPer; q++) {
            const bool fresh = v[q] >= 0 && set_add(set, bits, v[q]);
            const uint64_t fb = ballot64(fresh);
            int base = 0;
            if (lane == 0 && fb) base = atomicAdd(&s.npend, __popcll(fb));
            base = __shfl(base, 0, kWave) + __popcll(fb & lanemask_lt());
            if (fresh) s.pend[base] = v[q];
        }
        __syncthreads();
        // whole blocks of them from the back; the rest after the last round
        const bool last = x0 + kPer * kBlock >= total;
        int np = s.npend;
        while (np >= kBlock || last) {
            const int rest = np > kBlock ? np - kBlock : 0;
            process<X>(Xm, D, i, k, s, rest + t < np ? s.pend[rest + t] : -1, last && rest == 0);
            np = rest;
            if (np == 0) break;
        }
        if (last) break;
        if (t == 0) s.npend = np;
        __syncthreads();
    }
    uint64_t* od = MODE == 0 ? const_cast<uint64_t*>(ld) : nd;
    int32_t* oj = MODE == 0 ? const_cast<int32_t*>(lj) : nj;
    int32_t* om = MODE == 0 ? const_cast<int32_t*>(lm) : nm;
    if (t < s.m) {
        od[i * k + t] = s.ld[t];
        oj[i * k + t] = s.lj[t];
    }
    if (t == 0) om[i] = s.m;
}

// The hash set has room for twice a point's candidates, up to 4,096 entries.  A
// bit per point takes its place where that is no larger: one LDS operation per
// candidate instead of a walk over buckets.  Exploring as above (3,125 words of
// bits, 4,096 of hash set) takes 13.6 ms with bits and 17.3 with the set; a
// tree's leaves (3,125 and 1,024 words, to clear for each point) 1.49 and 1.39.
inline int set_bits(int64_t candidates) {
    int bits = 8;
    while (bits < kMaxSetBits && (1LL << bits) < 2 * candidates) bits++;
    return bits;
}

// All positions, in launches of at most kRun: a grid holds fewer
// than 2^32 threads.
constexpr int64_t kRun = (int64_t)1 << 22;

template <typename X, int MODE>
hipError_t lists(const X* Xm, int32_t D, int64_t n, int32_t k, int64_t candidates,
                 const uint32_t* perm, const uint32_t* sa, const uint32_t* sb, const uint64_t* ld,
                 const int32_t* lj, const int32_t* lm, uint64_t* nd, int32_t* nj, int32_t* nm,
                 hipStream_t s) {
    int bits = set_bits(candidates);
    int words = 1 << bits;
    if (ceil_div(n, 32) <= words) {
        bits = 0;
        words = (int)ceil_div(n, 32);
    }
    for (int64_t b0 = 0; b0 < n; b0 += kRun) {
        const int64_t b1 = n - b0 < kRun ? n : b0 + kRun;
        k_lists<X, MODE><<<dim3((unsigned)(kXcds * kDeal * ceil_div(b1 - b0, kXcds * kDeal))), kBlock,
                           4 * (size_t)words, s>>>(Xm, D, b0, b1, k, bits, words, perm, sa, sb,
                                                        ld, lj, lm, nd, nj, nm);
    }
    return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_lists_out(const uint64_t* __restrict__ ld,
                                                      const int32_t* __restrict__ lj,
                                                      const int32_t* __restrict__ lm, int64_t n,
                                                      int32_t k, int32_t* __restrict__ idx,
                                                      double* __restrict__ d2,
                                                      uint32_t* __restrict__ short_rows) {
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= n * (int64_t)k) return;
    const int64_t i = e / k;
    if (e % k == 0 && lm[i] < k) atomicAdd(short_rows, 1u);
    idx[e] = lj[e];
    d2[e] = key_dist(ld[e]);
}

template <typename X>
hipError_t knn_approx_typed(const X* Xm, int64_t n, int32_t D, int32_t k, int32_t trees,
                            int32_t leaf, int32_t explore, uint64_t seed, int32_t* idx,
                            double* d2, hipStream_t s, std::string* err) {
    uint32_t *perm[2] = {nullptr, nullptr}, *sa[2] = {nullptr, nullptr},
             *sb[2] = {nullptr, nullptr}, *flag = nullptr;
    int64_t *side = nullptr, *ones = nullptr, *tmp = nullptr;
    uint64_t* ld[2] = {nullptr, nullptr};
    int32_t* lj[2] = {nullptr, nullptr};
    int32_t* lm[2] = {nullptr, nullptr};
    hipError_t e = hipSuccess;
    auto cleanup = [&]() {
        for (int h = 0; h < 2; h++) {
            (void)hipFree(perm[h]); (void)hipFree(sa[h]); (void)hipFree(sb[h]);
            (void)hipFree(ld[h]); (void)hipFree(lj[h]); (void)hipFree(lm[h]);
        }
        (void)hipFree(flag); (void)hipFree(side); (void)hipFree(ones); (void)hipFree(tmp);
    };
    const size_t nk = (size_t)n * k;
    for (int h = 0; h < 2 && e == hipSuccess; h++) {
        e = hipMalloc(&perm[h], 4 * (size_t)n);
        if (e == hipSuccess) e = hipMalloc(&sa[h], 4 * (size_t)n);
        if (e == hipSuccess) e = hipMalloc(&sb[h], 4 * (size_t)n);
        if (e == hipSuccess) e = hipMalloc(&ld[h], 8 * nk);
        if (e == hipSuccess) e = hipMalloc(&lj[h], 4 * nk);
        if (e == hipSuccess) e = hipMalloc(&lm[h], 4 * (size_t)n);
    }
    if (e == hipSuccess) e = hipMalloc(&flag, 8);
    if (e == hipSuccess) e = hipMalloc(&side, 8 * (size_t)(n + 1));
    if (e == hipSuccess) e = hipMalloc(&ones, 8 * (size_t)(n + 1));
    if (e == hipSuccess) e = hipMalloc(&tmp, 8 * (size_t)scan_i64_tmp_len(n + 1));
    if (e == hipSuccess) e = hipMemsetAsync(lm[0], 0, 4 * (size_t)n, s);
    // each level at most doubles the number of ranges, so the first levels split
    // one for certain: only those after them ask
    int sure = 0;
    while (sure < kRpMaxLevel && ceil_div(n, (int64_t)1 << sure) > leaf) sure++;
    int cur = 0;
    for (int32_t tr = 0; tr < trees && e == hipSuccess; tr++) {
        cur = 0;
        k_rp_init<<<grid_for(n), kBlock, 0, s>>>(perm[0], sa[0], sb[0], n);
        for (int level = 0; e == hipSuccess; level++) {
            if (level >= sure) e = hipMemsetAsync(flag, 0, 4, s);
            if (e != hipSuccess) break;
            k_rp_side<X><<<grid_for(n + 1), kBlock, 0, s>>>(Xm, D, perm[cur], sa[cur], sb[cur], n,
                                                            leaf, seed, tr, level, side, flag);
            if (level >= sure) {
                uint32_t any = 0;
                e = hipMemcpyAsync(&any, flag, 4, hipMemcpyDeviceToHost, s);
                if (e == hipSuccess) e = hipStreamSynchronize(s);
                if (e != hipSuccess || !any) break;
            }
            e = scan_i64(side, n + 1, ones, tmp, s);
            if (e != hipSuccess) break;
            k_rp_scatter<<<grid_for(n), kBlock, 0, s>>>(perm[cur], sa[cur], sb[cur], side, ones, n,
                                                        leaf, k, level, perm[cur ^ 1], sa[cur ^ 1],
                                                        sb[cur ^ 1]);
            cur ^= 1;
            e = hipGetLastError();
        }
        if (e == hipSuccess) {
            e = lists<X, 0>(Xm, D, n, k, (int64_t)leaf + k, perm[cur], sa[cur], sb[cur], ld[0],
                            lj[0], lm[0], nullptr, nullptr, nullptr, s);
        }
    }
    int L = 0;
    for (int32_t r = 0; r < explore && e == hipSuccess; r++) {
        e = lists<X, 1>(Xm, D, n, k, (int64_t)k * (k + 1), perm[cur], nullptr, nullptr, ld[L],
                        lj[L], lm[L], ld[L ^ 1], lj[L ^ 1], lm[L ^ 1], s);
        L ^= 1;
    }
    uint32_t short_rows = 0;
    if (e == hipSuccess) e = hipMemsetAsync(flag, 0, 4, s);
    if (e == hipSuccess) {
        k_lists_out<<<grid_for((int64_t)nk), kBlock, 0, s>>>(ld[L], lj[L], lm[L], n, k, idx, d2,
                                                             flag);
        e = hipMemcpyAsync(&short_rows, flag, 4, hipMemcpyDeviceToHost, s);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    cleanup();
    if (e == hipSuccess && short_rows) {
        // every leaf holds at least k + 1 points, so this does not happen
        if (err) *err = "approximate kNN left rows with fewer than k neighbours";
        return hipErrorUnknown;
    }
    return e;
}

}  // namespace

hipError_t knn_approx(const void* X, int64_t n, int32_t D, int32_t x_dtype, int32_t k,
                      int32_t trees, int32_t leaf, int32_t explore, uint64_t seed, int32_t* idx,
                      double* d2, hipStream_t s, std::string* err) {
    switch (x_dtype) {
        case PSNE_X_F32:
            return knn_approx_typed<float>((const float*)X, n, D, k, trees, leaf, explore, seed,
                                           idx, d2, s, err);
        case PSNE_X_F64:
            return knn_approx_typed<double>((const double*)X, n, D, k, trees, leaf, explore, seed,
                                            idx, d2, s, err);
        default:
            return knn_approx_typed<uint8_t>((const uint8_t*)X, n, D, k, trees, leaf, explore,
                                             seed, idx, d2, s, err);
    }
}

}  // namespace psne
