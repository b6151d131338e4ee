// One-time setup on gfx950: the sparse affinity matrix P (paper Section 3.2-3.3).
//
//   knn          brute-force k nearest neighbours.  Distance tiles
//                d = |x|^2 + |y|^2 - 2 x.y come from the matrix units: FP16
//                MFMA on rows split into two halves of 11 bits each (three
//                products), or, for uint8 rows, exactly from INT8 MFMA on
//                x - 128; each row keeps a candidate list (global memory,
//                threshold in LDS) that a wavefront cuts to the K' = k + 32
//                best whenever it fills up.  Rows that fall into clusters are
//                put in an order by which whole tiles can be left out.
//                The K' survivors are re-ranked with exact FP64 distances
//                and ties go to the smaller index.
//   perplexity   per-row bisection on the Gaussian precision (FP64)
//   symmetrize   p_ij = (p_{j|i} + p_{i|j}) / 2n on the union pattern -> CSR
#include <math.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <type_traits>
#include <vector>

#include "ctx.h"

namespace psne {

namespace {


constexpr int kQB = 128;       // query rows per block
constexpr int kCB = 256;       // candidate columns per tile
constexpr int kCap = 1024;     // candidate list capacity per row
constexpr int kMargin = 32;    // extra candidates kept for the exact re-rank
constexpr int kCutAt = 512;    // a list longer than this is cut before the next tile, and
constexpr int kCutLow = 320;   // with it every list longer than this
constexpr int kHits = 256;     // passing elements a wavefront gathers per tile
constexpr int kCutSlack = 32;  // entries beyond the kp best that a cut may leave
// Rows from which on an order is looked for: at 17,000 x 50 in 30 clusters the
// search takes 1.5 ms without and 1.8 with it, at 33,000 3.3 and 2.1.
constexpr int64_t kOrderFrom = 1 << 15;
constexpr int kBatch = 1 << 19;   // query rows whose candidates exist at a time
static_assert(kBatch % kQB == 0, "batches are whole blocks");
static_assert(kCutLow >= 256 + kMargin + kCutSlack && kCutAt + kCB <= kCap,
              "a cut list is shorter than kCutLow, and a tile's columns fit");

template <typename X> __device__ __forceinline__ float to_f32(X v) { return (float)v; }

template <typename X>
__device__ __forceinline__ double to_f64(X v) { return (double)v; }

// What the host needs of X: the largest row norm and entry (as float bits,
// ordered like the floats), and whether a norm is not finite.
struct RowStats { uint32_t norm, entry, bad; };

template <typename X>
__global__ __launch_bounds__(256) void k_row_norms(const X* __restrict__ Xm, int64_t n, int D,
                                                   float* __restrict__ nrm,
                                                   RowStats* __restrict__ st) {
    __shared__ float red[4][3];
    const int lane = lane_id(), w = threadIdx.x >> 6;
    float big = 0.f, top = 0.f, bad = 0.f;
    for (int64_t i = (int64_t)blockIdx.x * 4 + w; i < n; i += (int64_t)gridDim.x * 4) {
        double a = 0.0;
        for (int d = lane; d < D; d += 64) {
            const float v = to_f32(Xm[i * D + d]);
            a += (double)v * (double)v;
            top = fmaxf(top, fabsf(v));
        }
        a = wave_sum(a);
        const float f = (float)a;
        if (lane == 0) nrm[i] = f;
        if (isfinite(f)) big = fmaxf(big, f);
        else bad = 1.f;
    }
    top = wave_max(top);
    if (lane == 0) { red[w][0] = big; red[w][1] = top; red[w][2] = bad; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < 4; q++)
            for (int c = 0; c < 3; c++) red[0][c] = fmaxf(red[0][c], red[q][c]);
        atomicMax(&st->norm, __float_as_uint(red[0][0]));
        atomicMax(&st->entry, __float_as_uint(red[0][1]));
        if (red[0][2] > 0.f) atomicOr(&st->bad, 1u);
    }
}

// block-wide bitonic sort of 512 uint64 keys in LDS (256 threads)
__device__ void bitonic512(uint64_t* s) {
    const int t = threadIdx.x;
    for (int k = 2; k <= 512; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            // thread t handles the pair whose lower index has bit j clear
            const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
            const int l = i | j;
            const uint64_t a = s[i], b = s[l];
            const bool up = (i & k) == 0;
            if ((a > b) == up) {
                s[i] = b;
                s[l] = a;
            }
            __syncthreads();
        }
    }
}

// A candidate key is (distance bits << 32 | column): the bits of a
// non-negative float, or an exact integer distance, both ordered as unsigned
// integers.  A row's threshold is the distance bits of its kp-th best key
// (kNoThr while the list is not full).
constexpr uint32_t kNoThr = 0xFFFFFFFFu;

// One wavefront cuts a list of m keys, kp <= m <= kCap, to its smallest, kp of
// them or up to `slack` more (in no order, to `to`, which may be the list), and
// returns their number;
// thr: distance bits that none of the kp best exceeds.  The bits of the
// kp-th distance are found by bisection from the list's smallest to its largest,
// by counts over the wave, until a count within the slack ends the search
// (some five steps; bit by bit from the top took ten, 10.8 ms for 100,000
// Gaussian rows of 8 where this takes 10.1).  Among equal distances at the
// kp-th place the smallest columns are kept.
__device__ __forceinline__ int cut_list(const uint64_t* lst, int m, int kp, int slack,
                                        uint64_t* to, uint32_t& thr) {
    constexpr int kPer = kCap / kWave;
    const int lane = lane_id();
    uint32_t d[kPer], j[kPer];
#pragma unroll
    for (int q = 0; q < kPer; q++) {
        const int e = lane + q * kWave;
        const uint64_t c = e < m ? lst[e] : ~0ull;
        d[q] = (uint32_t)(c >> 32);
        j[q] = (uint32_t)c;
    }
    auto count = [&](auto&& in) {
        int c = 0;
#pragma unroll
        for (int q = 0; q < kPer; q++) c += __popcll(ballot64(in(q)));
        return c;
    };
    // the kept are d < end, or d == end and j <= last
    uint32_t end = ~0u, top = 0, last = 0xFFFFFFFEu;
#pragma unroll
    for (int q = 0; q < kPer; q++) {
        end = d[q] < end ? d[q] : end;
        top = lane + q * kWave < m && d[q] > top ? d[q] : top;
    }
    end = wave_min(end);
    top = wave_max(top);
    bool found = false;
    while (end < top) {             // fewer than kp below end, at least kp up to top
        const uint32_t u = end + (top - end + 1) / 2;
        const int c = count([&](int q) { return d[q] < u; });
        if (c < kp) {
            end = u;
        } else if (c <= kp + slack) {
            end = u - 1;
            found = true;
            break;
        } else {
            top = u - 1;
        }
    }
    if (!found) {
        const int below = count([&](int q) { return d[q] < end; });
        const int equal = count([&](int q) { return d[q] == end && j[q] != 0xFFFFFFFFu; });
        if (equal > kp - below + slack) {
            last = 0;
            for (int b = 30; b >= 0; b--) {
                const uint32_t u = last | (1u << b);
                if (count([&](int q) { return d[q] == end && j[q] < u; }) < kp - below) last = u;
            }
        }
    }
    int at = 0;
#pragma unroll
    for (int q = 0; q < kPer; q++) {
        const bool keep = d[q] < end || (d[q] == end && j[q] <= last);
        const uint64_t b = ballot64(keep);
        if (keep)
            to[at + __popcll(b & lanemask_lt())] = ((uint64_t)d[q] << 32) | (uint64_t)j[q];
        at += __popcll(b);
    }
    thr = end;
    return at;
}

// The matrix operands of a run of rows, as the MFMA units take them: a
// fragment is 32 rows times one instruction's depth, 16 bytes per lane (lane l:
// row l % 32, half l / 32 of the depth), 1 KB in lane order.  Fragments lie by
// [32 rows][depth step][part], so a fragment moves to LDS and to registers in
// whole cache lines and without bank conflicts.  Rows and depth are padded
// with zeros.
//
// FP16: a row times the power of two `scale` is split into two halves of 11
// bits each, x = hi + lo, and x.y = hi.hi + hi.lo + lo.hi up to 2^-22 per
// product.  The sums have fewer roundings than FP32 MFMA's, one depth of 2 after
// another, so the distances are nearer to 64 bits than those: of all pairs of 2,048
// rows of the mixture of 16 / 128 / 784 dimensions the errors' root mean squares are
// 3.8e-5 / 4.3e-4 / 6.3e-3, of the FP32 unit 4.5e-5 / 6.9e-4 / 1.0e-2 (a fourth
// product, lo.lo: 3.6e-5 / 4.3e-4 / 6.3e-3).
struct PartsF16 {
    using Vec = _Float16 __attribute__((ext_vector_type(8)));
    using Acc = float __attribute__((ext_vector_type(16)));
    using Num = float;
    static constexpr int kDepth = 16, kParts = 2, kSteps = 2;
    static __device__ __forceinline__ void product(const Vec* a, const Vec* b, Acc& c) {
        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], b[1], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[1], b[0], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], b[0], c, 0, 0, 0);
    }
    static __device__ __forceinline__ void center_product(const Vec* a, const Vec& y, Acc& c) {
        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[1], y, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], y, c, 0, 0, 0);
    }
    // |y|^2 - 2 x.y, with f = -2 / scale^2
    static __device__ __forceinline__ float part_dist(float dot, float f, float ny) {
        return fmaf(dot, f, ny);
    }
    // the bound on it that keeps a candidate, from a threshold and |x|^2
    static __device__ __forceinline__ float bound(uint32_t thr, float nx) {
        return thr == kNoThr ? INFINITY : __uint_as_float(thr) - nx;
    }
    static __device__ __forceinline__ uint32_t bits(float part, float nx) {
        const float d = nx + part;
        return __float_as_uint(d > 0.0f ? d : 0.0f);
    }
    // no distance of FP32 bits thr or less reaches low2 - err
    static __device__ __forceinline__ bool beyond(float low2, float err, uint32_t thr) {
        return low2 - err > __uint_as_float(thr);
    }
    static __device__ __forceinline__ float none() { return -INFINITY; }
    static __device__ __forceinline__ float far() { return INFINITY; }
};

// INT8: x - 128 for uint8 rows, every distance an exact int32 (D <= 32768).
struct PartsI8 {
    using Vec = int __attribute__((ext_vector_type(4)));
    using Acc = int __attribute__((ext_vector_type(16)));
    using Num = int32_t;
    static constexpr int kDepth = 32, kParts = 1, kSteps = 4;
    static __device__ __forceinline__ void product(const Vec* a, const Vec* b, Acc& c) {
        c = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[0], b[0], c, 0, 0, 0);
    }
    static __device__ __forceinline__ void center_product(const Vec* a, const Vec& y, Acc& c) {
        c = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[0], y, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int32_t part_dist(int32_t dot, float, int32_t ny) {
        return ny - 2 * dot;
    }
    static __device__ __forceinline__ int32_t bound(uint32_t thr, int32_t nx) {
        return thr == kNoThr ? 0x7FFFFFFF : (int32_t)thr - nx;
    }
    static __device__ __forceinline__ uint32_t bits(int32_t part, int32_t nx) {
        return (uint32_t)(nx + part);
    }
    static __device__ __forceinline__ bool beyond(float low2, float, uint32_t thr) {
        return low2 > (float)thr * (1.f + 0x1p-20f);
    }
    static __device__ __forceinline__ int32_t none() { return -0x7FFFFFFF - 1; }
    // a padding row's dot is 0
    static __device__ __forceinline__ int32_t far() { return 0x7FFFFFFF; }
};

inline int64_t pad_rows(int64_t n) { return ceil_div(n, kCB) * kCB; }
template <typename F> inline int pad_steps(int D) {
    return (int)(ceil_div(D, F::kDepth * F::kSteps) * F::kSteps);
}
template <typename F> inline size_t packed_bytes(int64_t n, int D) {
    return (size_t)(pad_rows(n) / 32) * pad_steps<F>(D) * F::kParts * 1024;
}

// One thread per 16-byte piece of the hi (and lo) fragments, from piece `first` on.
template <typename X>
__global__ __launch_bounds__(256) void k_pack_f16(const X* __restrict__ Xm, int64_t n, int64_t np,
                                                  int D, int steps, float scale,
                                                  const uint32_t* __restrict__ perm, int64_t first,
                                                  _Float16* __restrict__ out) {
    const int64_t e = first + (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= np * steps * 2) return;
    const int lane = (int)(e & 63);
    const int64_t f = e >> 6;                               // [32 rows][step]
    const int64_t row = (f / steps) * 32 + (lane & 31);
    const int d0 = (int)(f % steps) * 16 + 8 * (lane >> 5);
    const int64_t src = row < n && perm ? perm[row] : row;
    PartsF16::Vec hi, lo;
#pragma unroll
    for (int q = 0; q < 8; q++) {
        const float v = row < n && d0 + q < D ? to_f32(Xm[src * D + d0 + q]) * scale : 0.f;
        hi[q] = (_Float16)v;
        lo[q] = (_Float16)(v - (float)hi[q]);
    }
    PartsF16::Vec* o = reinterpret_cast<PartsF16::Vec*>(out) + f * 128 + lane;
    o[0] = hi;
    o[64] = lo;
}

__global__ __launch_bounds__(256) void k_pack_i8(const uint8_t* __restrict__ Xm, int64_t n,
                                                 int64_t np, int D, int steps,
                                                 const uint32_t* __restrict__ perm, int64_t first,
                                                 uint4* __restrict__ out) {
    const int64_t e = first + (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= np * steps * 2) return;
    const int lane = (int)(e & 63);
    const int64_t f = e >> 6;
    const int64_t row = (f / steps) * 32 + (lane & 31);
    const int d0 = (int)(f % steps) * 32 + 16 * (lane >> 5);
    union {
        uint4 q;
        uint8_t b[16];
    } v;
    const uint8_t* src = Xm + (row < n && perm ? (int64_t)perm[row] : row) * D + d0;
    if (row < n && d0 + 16 <= D && (reinterpret_cast<uintptr_t>(src) & 15u) == 0) {
        v.q = *reinterpret_cast<const uint4*>(src);
    } else {
#pragma unroll
        for (int q = 0; q < 16; q++) v.b[q] = row < n && d0 + q < D ? src[q] : (uint8_t)128;
    }
    // x - 128 as int8 is the byte with its top bit flipped; padding becomes 0
    v.q.x ^= 0x80808080u;
    v.q.y ^= 0x80808080u;
    v.q.z ^= 0x80808080u;
    v.q.w ^= 0x80808080u;
    out[e] = v.q;
}

__global__ __launch_bounds__(256) void k_row_norms_i8(const uint8_t* __restrict__ Xm, int64_t n,
                                                      int D, int32_t* __restrict__ nrm) {
    const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = lane_id();
    if (i >= n) return;
    int a = 0;
    for (int d = lane; d < D; d += 64) {
        const int v = (int)Xm[i * D + d] - 128;
        a += v * v;
    }
    for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
    if (lane == 0) nrm[i] = a;
}

// ---------------------------------------------------------------------------
// An order of the rows that lets the exact search leave tiles out
//
// Rows are sorted by their nearest of kPivots sample rows.  The sample is taken
// in kRounds rounds, the first evenly, the others with probability proportional
// to the squared distance from the nearest pivot so far (as in the seeding of
// Bahmani et al., 2012), so that small clusters get pivots too; a cluster
// without one would be spread over all others'.  The pivots are numbered along a
// chain from each to its nearest not yet taken.  The rows are then cut into groups of G
// consecutive rows, G a multiple of a tile's columns and large enough that at
// most kMaxGroups remain.  Every group has a centre c, its mean rounded to what
// the matrix units take (any point would do).  For x in group q and y in group
// t, with D = |c_q - c_t|,
//
//   |x - y| >= (x - y).(c_q - c_t) / D = (m_t(x) + m_q(y)) / 2D,
//   m_t(x) = |x - c_t|^2 - |x - c_q|^2 and m_q(y) = |y - c_q|^2 - |y - c_t|^2,
//
// so the smallest m of every group against every centre, one product of all
// rows with all centres (n^2 / G against n^2 of the search), bounds the distance
// of any two rows of two groups from below.  Each group sweeps the groups in the
// order of that bound and stops where it exceeds the block's largest threshold.
// Every row that is left out is further than the threshold, which is what the
// selection asserts of it; rows without structure meet every tile as before.
// ---------------------------------------------------------------------------
constexpr int kPivots = 256, kRounds = 4, kRoundPivots = kPivots / kRounds;
constexpr int kMaxGroups = 4096;
constexpr double kNearShare = 0.35;     // of the pivots' mean squared distance: the rows' at most
constexpr double kApartShare = 0.05;    // of the pairs of groups: apart at least

// centres in fragments of the matrix units, one part
struct CenterF16 {
    static __device__ __forceinline__ float put(void* out, int64_t e, float v, float scale) {
        const _Float16 h = (_Float16)(v * scale);
        reinterpret_cast<_Float16*>(out)[e] = h;
        return (float)h / scale;
    }
};
struct CenterI8 {
    static __device__ __forceinline__ float put(void* out, int64_t e, float v, float) {
        const float c = fminf(fmaxf(rintf(v - 128.f), -128.f), 127.f);
        reinterpret_cast<int8_t*>(out)[e] = (int8_t)c;
        return c;
    }
};

// Centre t (block): the mean of rows first[t] .. first[t] + count - 1 of the
// order; its fragment entries, its coordinates by dimension (ct [D][T]) and |c|^2.
template <typename X, typename F, typename P>
__global__ __launch_bounds__(256) void k_centers(const X* __restrict__ Xm, int64_t n, int D,
                                                 const uint32_t* __restrict__ perm, int64_t stride,
                                                 int64_t count, int steps, float scale,
                                                 void* __restrict__ frag, float* __restrict__ ct,
                                                 typename F::Num* __restrict__ cn) {
    __shared__ double red[4];
    const int t = blockIdx.x, T = gridDim.x, lane = lane_id();
    const int64_t r0 = t * stride < n ? t * stride : n - 1;
    const int64_t r1 = r0 + count < n ? r0 + count : n;
    constexpr int kD = F::kDepth, kHalf = kD / 2;
    double a = 0.0;
    for (int d = threadIdx.x; d < steps * kD; d += 256) {
        float v = 0.f;
        if (d < D) {
            for (int64_t r = r0; r < r1; r++) v += to_f32(Xm[(perm ? (int64_t)perm[r] : r) * D + d]);
            v /= (float)(r1 - r0);
        }
        // entry d of row t: [32 rows][step], lane 32 half + row, kHalf entries each
        const int64_t e = (((int64_t)(t / 32) * steps + d / kD) * 64 + 32 * (d % kD / kHalf) + t % 32) *
                              kHalf + d % kHalf;
        if (d < D) {
            const float c = P::put(frag, e, v, scale);
            ct[(int64_t)d * T + t] = c;
            a += (double)c * c;
        }
    }
    a = wave_sum(a);
    if (lane == 0) red[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) cn[t] = (typename F::Num)(((red[0] + red[1]) + red[2]) + red[3]);
}

// squared distances of all centres, row q (block) of [T][T]
__global__ __launch_bounds__(256) void k_center_d2(const float* __restrict__ ct, int D, int T,
                                                   float* __restrict__ d2) {
    const int q = blockIdx.x;
    for (int t = threadIdx.x; t < T; t += 256) {
        double a = 0.0;
#pragma unroll 8
        for (int d = 0; d < D; d++) {
            const double v = (double)ct[(int64_t)d * T + q] - (double)ct[(int64_t)d * T + t];
            a += v * v;
        }
        d2[(int64_t)q * T + t] = (float)a;
    }
}

// The chain of the pivots, by one wavefront: rank[t] is t's place in it.
__global__ __launch_bounds__(64) void k_chain(const float* __restrict__ d2,
                                              uint32_t* __restrict__ rank) {
    const int lane = lane_id();
    constexpr int kPer = kPivots / kWave;
    bool taken[kPer] = {};
    int at = 0;
    for (int r = 0; r < kPivots; r++) {
        float best = INFINITY;
        int who = kPivots;
#pragma unroll
        for (int q = 0; q < kPer; q++) {
            const int t = q * kWave + lane;
            if (t == at) {
                taken[q] = true;
                rank[t] = (uint32_t)r;
            }
            const float v = d2[(int64_t)at * kPivots + t];
            if (!taken[q] && (v < best || who == kPivots)) {
                best = v;
                who = t;
            }
        }
        for (int o = 32; o > 0; o >>= 1) {
            const float b = __shfl_xor(best, o, kWave);
            const int j = __shfl_xor(who, o, kWave);
            if (j < kPivots && (who == kPivots || b < best || (b == best && j < who))) {
                best = b;
                who = j;
            }
        }
        at = __builtin_amdgcn_readfirstlane(who < kPivots ? who : 0);
    }
}

// All rows against all T centres: a wavefront takes 32 rows, a block one run of
// 256, and four tiles of 32 centres at a time.  ASSIGN: key[row] = rank of the
// nearest centre, or weight[row] its squared distance in units of 1 / unit.
// Else m[group][t] (infinity to begin with) gets the smallest
// |x - c_t|^2 - |x - c_group|^2 of the group's rows, and radius2[group] (bits,
// zero to begin with) the largest |x - c_group|^2.
__device__ __forceinline__ void atomic_min_float(float* at, float v) {
    if (v >= 0.f) atomicMin(reinterpret_cast<int*>(at), __float_as_int(v));
    else atomicMax(reinterpret_cast<unsigned int*>(at), __float_as_uint(v));
}

template <typename F> using Num_t = typename F::Num;

template <typename F, bool ASSIGN>
__global__ __launch_bounds__(512) void k_center_dots(const char* __restrict__ packed, int64_t n,
                                                     int steps, const char* __restrict__ centers,
                                                     const typename F::Num* __restrict__ cn, int T,
                                                     float f, int64_t G,
                                                     const uint32_t* __restrict__ rank,
                                                     uint32_t* __restrict__ key,
                                                     const Num_t<F>* __restrict__ nrm, float unit,
                                                     int64_t* __restrict__ weight,
                                                     float* __restrict__ m,
                                                     uint32_t* __restrict__ radius2) {
    using Vec = typename F::Vec;
    using Num = typename F::Num;
    constexpr int kTiles = 4;
    __shared__ float low[8][32 * kTiles];
    const int t = threadIdx.x, lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t r0 = ((int64_t)blockIdx.x * 8 + w) * 32, group = r0 / G;
    const char* rows = packed + (r0 / 32) * ((int64_t)steps * F::kParts * 1024) + lane * 16;
    const int ctiles = (T + 31) / 32;
    typename F::Acc acc[kTiles];
    auto dots = [&](int c0) {
#pragma unroll
        for (int b = 0; b < kTiles; b++)
#pragma unroll
            for (int v = 0; v < 16; v++) acc[b][v] = 0;
        for (int x = 0; x < steps; x++) {
            Vec a[F::kParts];
#pragma unroll
            for (int p = 0; p < F::kParts; p++)
                a[p] = *reinterpret_cast<const Vec*>(rows + ((int64_t)x * F::kParts + p) * 1024);
#pragma unroll
            for (int b = 0; b < kTiles; b++) {
                const int c = c0 + b < ctiles ? c0 + b : ctiles - 1;
                const Vec y = *reinterpret_cast<const Vec*>(
                    centers + ((int64_t)c * steps + x) * 1024 + lane * 16);
                F::center_product(a, y, acc[b]);
            }
        }
    };
    // element v: row r0 + 8 (v / 4) + 4 (lane / 32) + v % 4, centre lane % 32
    auto row_of = [&](int v) { return r0 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); };
    if constexpr (ASSIGN) {
        Num best[16];
        int id[16];
#pragma unroll
        for (int v = 0; v < 16; v++) {
            best[v] = F::far();
            id[v] = 0;
        }
        for (int c0 = 0; c0 < ctiles; c0 += kTiles) {
            dots(c0);
#pragma unroll
            for (int b = 0; b < kTiles; b++) {
                const int col = 32 * (c0 + b) + (lane & 31);
                if (col >= T) continue;
                const Num c2 = cn[col];
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    const Num d = F::part_dist(acc[b][v], f, c2);
                    if (d < best[v]) {
                        best[v] = d;
                        id[v] = col;
                    }
                }
            }
        }
#pragma unroll
        for (int v = 0; v < 16; v++) {
            for (int o = 16; o > 0; o >>= 1) {
                const Num d = __shfl_xor(best[v], o, kWave);
                const int j = __shfl_xor(id[v], o, kWave);
                if (d < best[v] || (d == best[v] && j < id[v])) {
                    best[v] = d;
                    id[v] = j;
                }
            }
            const int64_t row = row_of(v);
            if ((lane & 31) == 0 && row < n) {
                if (weight) {
                    const float d = fmaxf((float)nrm[row] + (float)best[v], 0.f) * unit;
                    weight[row] = 1 + (int64_t)fminf(d, 0x1p30f);
                } else {
                    key[row] = rank[id[v]];
                }
            }
        }
    } else {
        float own[16], far2 = 0.f;
        {
            const int c = (int)(group / 32) / kTiles * kTiles, b = (int)(group / 32) - c;
            dots(c);
            const Num c2 = cn[group];
#pragma unroll
            for (int v = 0; v < 16; v++) {
                Num d = acc[0][v];
#pragma unroll
                for (int q = 1; q < kTiles; q++) d = b == q ? acc[q][v] : d;
                own[v] = (float)F::part_dist(__shfl(d, (int)(group & 31) | (lane & 32), kWave), f, c2);
                if (row_of(v) < n) far2 = fmaxf(far2, (float)nrm[row_of(v)] + own[v]);
                else own[v] = -INFINITY;
            }
            far2 = wave_max(far2);
            if (lane == 0) atomicMax(&radius2[group], __float_as_uint(far2));
        }
        for (int c0 = 0; c0 < ctiles; c0 += kTiles) {
            dots(c0);
#pragma unroll
            for (int b = 0; b < kTiles; b++) {
                const int col = 32 * (c0 + b) + (lane & 31);
                const Num c2 = col < T ? cn[col] : Num(0);
                float s = INFINITY;
#pragma unroll
                for (int v = 0; v < 16; v++)
                    s = fminf(s, (float)F::part_dist(acc[b][v], f, c2) - own[v]);
                s = fminf(s, __shfl_xor(s, 32, kWave));
                if (lane < 32) low[w][32 * b + lane] = s;
            }
            __syncthreads();
            const int col = 32 * c0 + t;
            if (t < 32 * kTiles && col < T) {
                float s = low[0][t];
#pragma unroll
                for (int q = 1; q < 8; q++) s = fminf(s, low[q][t]);
                atomic_min_float(&m[group * T + col], s);
            }
            __syncthreads();
        }
    }
}

// Group q's (block) list of the groups by their bound on the squared distance,
// rounded down; err: what a value of m may be off by.  apart counts the pairs of
// groups further apart than the rows of the first typically are (for rows at r
// from their mean 2 r^2, squared), far_of those of each first group.
struct GroupAt { float low2; uint32_t group; };

__global__ __launch_bounds__(256) void k_group_order(const float* __restrict__ m,
                                                     const float* __restrict__ d2, int T,
                                                     float err,
                                                     const uint32_t* __restrict__ radius2,
                                                     GroupAt* __restrict__ order,
                                                     uint32_t* __restrict__ far_of,
                                                     unsigned long long* __restrict__ apart) {
    __shared__ uint64_t key[kMaxGroups];
    const int q = blockIdx.x, t = threadIdx.x;
    const float reach2 = 2.f * __uint_as_float(radius2[q]);
    unsigned int far = 0;
    int P = 1;
    while (P < T) P <<= 1;
    for (int g = t; g < P; g += 256) {
        uint64_t k = ~0ull;
        if (g < T) {
            float low2 = 0.f;
            const float D = sqrtf(d2[(int64_t)q * T + g]) * (1.f + 0x1p-20f);
            const float a = m[(int64_t)q * T + g], b = m[(int64_t)g * T + q];
            const float num = (a + b) - 2.f * err - (fabsf(a) + fabsf(b)) * 0x1p-20f;
            if (g != q && num > 0.f && D > 0.f && isfinite(num)) {
                const float low = num / (2.f * D);
                low2 = low * low * (1.f - 0x1p-18f);
            }
            far += low2 > reach2 ? 1u : 0u;
            k = (uint64_t)__float_as_uint(low2) << 32 | (uint32_t)(g == q ? 0 : g + 1);
        }
        key[g] = k;
    }
    for (int o = 32; o > 0; o >>= 1) far += __shfl_xor(far, o, kWave);
    if (lane_id() == 0 && far) {
        atomicAdd(apart, (unsigned long long)far);
        atomicAdd(&far_of[q], far);
    }
    __syncthreads();
    for (int k = 2; k <= P; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int x = t; x < P / 2; x += 256) {
                const int a = ((x & ~(j - 1)) << 1) | (x & (j - 1)), b = a | j;
                const uint64_t u = key[a], v = key[b];
                if ((u > v) == ((a & k) == 0)) {
                    key[a] = v;
                    key[b] = u;
                }
            }
            __syncthreads();
        }
    for (int x = t; x < T; x += 256) {
        const uint32_t g = (uint32_t)key[x];
        order[(int64_t)q * T + x] =
            GroupAt{__uint_as_float((uint32_t)(key[x] >> 32)), g == 0 ? (uint32_t)q : g - 1};
    }
}

// The rows at even steps of the weights' running sum: the next pivots.
__global__ __launch_bounds__(kRoundPivots) void k_pick(const int64_t* __restrict__ sum, int64_t n,
                                                       uint32_t* __restrict__ row) {
    const double at = (double)sum[n] * ((threadIdx.x + 0.5) / kRoundPivots);
    int64_t lo = 0, hi = n;                     // sum[lo] <= at < sum[hi]
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if ((double)sum[mid] <= at) lo = mid;
        else hi = mid;
    }
    row[threadIdx.x] = (uint32_t)lo;
}

__global__ __launch_bounds__(kRoundPivots) void k_even_rows(int64_t n, uint32_t* __restrict__ row) {
    row[threadIdx.x] = (uint32_t)(n / kRoundPivots * threadIdx.x);
}

// The groups by the number of others that are far, fewest first: those that
// will meet the most tiles.
__global__ __launch_bounds__(1024) void k_group_turns(const uint32_t* __restrict__ far_of, int T,
                                                      uint32_t* __restrict__ turn) {
    __shared__ uint64_t key[kMaxGroups];
    const int t = threadIdx.x;
    int P = 1;
    while (P < T) P <<= 1;
    for (int g = t; g < P; g += 1024)
        key[g] = g < T ? (uint64_t)far_of[g] << 32 | (uint32_t)g : ~0ull;
    __syncthreads();
    for (int k = 2; k <= P; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int x = t; x < P / 2; x += 1024) {
                const int a = ((x & ~(j - 1)) << 1) | (x & (j - 1)), b = a | j;
                const uint64_t u = key[a], v = key[b];
                if ((u > v) == ((a & k) == 0)) {
                    key[a] = v;
                    key[b] = u;
                }
            }
            __syncthreads();
        }
    for (int x = t; x < T; x += 1024) turn[x] = (uint32_t)key[x];
}

template <typename V>
__global__ __launch_bounds__(256) void k_permuted(const V* __restrict__ a,
                                                  const uint32_t* __restrict__ perm, int64_t n,
                                                  V* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = a[perm[i]];
}

__global__ __launch_bounds__(256) void k_fill_inf(float* __restrict__ a, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) a[i] = INFINITY;
}

// The order of the rows, or null pointers: the row at a place, the groups' lists,
// the groups' turns, rows per group, number of groups, and what an approximate
// distance may be off by.  Blocks begin in the groups' turns, the longest first:
// 547 blocks of unequal length on 256 CUs (70,000 x 784 bytes) take 3.2 ms, in
// the order of the rows 4.2; 3,125 (400,000 x 128) 22.4 and 23.6.
struct RowOrder {
    const uint32_t* perm;
    const GroupAt* order;
    const uint32_t* turn;
    int64_t G;
    int T;
    float err;
};

// Candidate generation.  Blocks of eight wavefronts, one per CU, take turns of
// kQB query rows; their working lists are a block's (268 MB in all) and each
// row's kp best go to its own place: with working lists for every row, 3.3 GB at
// 400,000, the allocation alone took up to 70 ms once that much memory had been
// released before.  A block sweeps all candidates in tiles of kCB; each
// wavefront computes a 64 x 64 part as 2 x 2 MFMA tiles.  The depth runs in
// stages of F::kSteps
// instructions, staged by loads straight into LDS, the next stage (of this
// tile or of the next) in flight while one is multiplied; with HOLD the
// queries' fragments stay in LDS (depth up to 128 for FP16), else they are
// staged too.  The distances are filtered from the accumulators: per element
// one multiply-add and one comparison with the row's bound, and only elements
// that pass take the way to the lists.
//
// All tiles of 400,000 x 128, three FP16 products, are 123 TFLOP, 50 ms of the
// matrix units; the kernel takes 144: 100 with the loads and the lists taken
// away (barriers of the stages, LDS latency, the filter), the rest for loads
// that come late and for the lists (3,000 entries a row on the way to the last
// 182).  By the groups' lists (100 clusters of unequal size, k = 150) 130 of
// the 1,563 tiles remain for a block on average: 22 ms, a third each for the
// stages, for the lists as they fill and for cutting them, which a block does
// all at once.  Tried: stages half as deep, three in flight, 165; lists cut
// only at 768 entries, 153; the next list read while one is cut, no gain.  The
// FP32 MFMA kernel of 128 x 128 tiles, filtered through LDS, that this replaces
// took 605.  70,000 x 784 bytes: 3.4 ms by the lists, 10.7 with all tiles, 46.6
// by the INT8 kernel of 128 x 128 tiles.
typedef __attribute__((address_space(1))) const void GlobalPtr;
typedef __attribute__((address_space(3))) void LdsPtr;

//
// queries: the packed rows q_first .. of the batch; packed: the candidates, rows
// c_first .. c_first + cols (all of them, or as many as there is room for).
template <typename F, bool HOLD>
__global__ __launch_bounds__(512) void k_knn_candidates(const char* __restrict__ queries,
                                                        const char* __restrict__ packed,
                                                        int64_t n, int64_t c_first, int64_t cols,
                                                        int steps,
                                                        const typename F::Num* __restrict__ nrm,
                                                        float f, int64_t q_first, int kp,
                                                        RowOrder ord, uint32_t blocks,
                                                        uint32_t* __restrict__ ticket,
                                                        unsigned long long* __restrict__ met,
                                                        uint64_t* __restrict__ work,
                                                        uint64_t* __restrict__ cand,
                                                        uint32_t* __restrict__ cand_cnt,
                                                        uint32_t* __restrict__ cand_thr) {
    using Vec = typename F::Vec;
    using Num = typename F::Num;
    constexpr int kFrag = 1024;
    constexpr int kQF = kQB / 32, kCF = kCB / 32;          // fragments of 32 rows
    constexpr int kStageC = kCF * F::kSteps * F::kParts;   // fragments of a stage
    constexpr int kStageQ = kQF * F::kSteps * F::kParts;
    constexpr int kHoldQ = kQF * 8 * F::kParts;            // up to 8 steps held
    __shared__ __attribute__((aligned(16))) char C[2][kStageC * kFrag];
    __shared__ __attribute__((aligned(16))) char Q[(HOLD ? kHoldQ : 2 * kStageQ) * kFrag];
    __shared__ uint32_t cnt[kQB];
    __shared__ __attribute__((aligned(16))) Num bnd[kQB];
    __shared__ Num nq[kQB];
    __shared__ uint32_t thr[kQB];          // every column left out so far is further
    struct Hit { Num part; uint32_t at; };                  // row << 8 | column, in the tile
    __shared__ Hit hits[8][kHits];

    const int t = threadIdx.x, lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wr = w >> 2, wc = w & 3;                      // 64 query rows, 64 columns
    uint64_t* const lists = work + (int64_t)blockIdx.x * (kQB * kCap);
    __shared__ uint32_t s_block;
    for (;;) {
        __syncthreads();
        if (t == 0) s_block = atomicAdd(ticket, 1u);
        __syncthreads();
        int64_t block = __builtin_amdgcn_readfirstlane(s_block);
        if (block >= blocks) return;
        if (ord.turn) {
            const int64_t per = ord.G / kQB;
            block = ord.turn[block / per] * per + block % per;
        }
        const int64_t q0 = q_first + block * kQB;
        if (q0 >= n) continue;
        const int nst = steps / F::kSteps;
        const int64_t tiles = (cols + kCB - 1) / kCB;
        const int64_t q32 = (q0 - q_first) / 32;           // the queries' first fragment
        if (t < kQB) {
            cnt[t] = 0;
            thr[t] = q0 + t < n ? kNoThr : 0u;
            nq[t] = q0 + t < n ? nrm[q0 + t] : Num(0);
            bnd[t] = q0 + t < n ? F::bound(kNoThr, Num(0)) : F::none();
        }
        // A stage takes kPer = 4 fragments of each 32 rows.  Wavefront w loads the
        // fragments w, w + 8, ... of a stage: fragment w % 4 of the rows w / 4,
        // w / 4 + 2, ...
        constexpr int kPer = F::kSteps * F::kParts;
        static_assert(kPer == 4 && kStageC % 8 == 0 && kStageQ % 8 == 0, "whole rounds of loads");
        const int64_t frag_row = (int64_t)steps * F::kParts * kFrag;   // bytes of 32 rows
        const int64_t piece = (w >> 2) * frag_row + (w & 3) * kFrag + lane * 16;
        const char* const mine = packed + piece;
        auto to_lds = [&](const char* src, char* dst) {
            __builtin_amdgcn_global_load_lds((GlobalPtr*)src, (LdsPtr*)dst, 16, 0, 0);
        };
        auto fetch = [&](int64_t tile, int s, int buf) {
            const char* c = mine + tile * (kCF * frag_row) + s * (kPer * kFrag);
#pragma unroll
            for (int y = 0; y < kStageC / 8; y++)
                to_lds(c + y * (2 * frag_row), C[buf] + (w + 8 * y) * kFrag);
            if constexpr (!HOLD) {
                const char* q = queries + piece + q32 * frag_row + s * (kPer * kFrag);
#pragma unroll
                for (int y = 0; y < kStageQ / 8; y++)
                    to_lds(q + y * (2 * frag_row), Q + (buf * kStageQ + w + 8 * y) * kFrag);
            }
        };
        // every load and store of the block is done, in LDS and in the lists
        auto settle = [&]() {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
        };
        auto cut = [&]() {
            // Lists that could overflow during the next tile are cut, 16 rows per
            // wavefront.  The block waits for a wavefront that cuts, so once any
            // list is that long every long one is cut.
            const uint64_t full =
                ballot64(cnt[lane] > (uint32_t)kCutAt || cnt[lane + kWave] > (uint32_t)kCutAt);
            if (full == 0) return;
            uint64_t todo = ballot64(lane < 16 && cnt[w * 16 + (lane & 15)] > (uint32_t)kCutLow);
            while (todo) {
                const int q = w * 16 + __ffsll((long long)todo) - 1;
                todo &= todo - 1;
                uint32_t end;
                uint64_t* const lst = lists + q * kCap;
                const int m = cut_list(lst, (int)cnt[q], kp, kCutSlack, lst, end);
                if (lane == 0) {
                    end = end < thr[q] ? end : thr[q];
                    cnt[q] = (uint32_t)m;
                    thr[q] = end;
                    bnd[q] = F::bound(end, nq[q]);
                }
            }
        };

        if constexpr (HOLD) {
            // all steps of the queries, by [32 rows][8 steps][part]
            for (int x = w; x < kQF * steps * F::kParts; x += 8) {
                const int rb = x / (steps * F::kParts), rest = x % (steps * F::kParts);
                to_lds(queries + (q32 + rb) * frag_row + rest * kFrag + lane * 16,
                       Q + (rb * 8 * F::kParts + rest) * kFrag);
            }
        }
        // the tiles in turn, or by the list of the queries' group
        const GroupAt* const list = ord.order ? ord.order + (q0 / ord.G) * ord.T : nullptr;
        const int64_t sub = ord.order ? ord.G / kCB : 1;
        const int64_t places = ord.order ? ord.T * sub : tiles;
        uint32_t worst = kNoThr;               // the largest threshold of the block's rows
        int64_t place = -1;
        auto next_tile = [&]() -> int64_t {
            while (++place < places) {
                if (!list) return place;
                const GroupAt g = list[place / sub];
                if (worst != kNoThr && F::beyond(g.low2, ord.err, worst)) return -1;
                const int64_t at = (int64_t)g.group * sub + place % sub;
                if (at < tiles) return at;
            }
            return -1;
        };
        int64_t tile = next_tile(), next = -1;
        fetch(tile, 0, 0);
        settle();
        int buf = 0;
        uint32_t swept = 0;
        for (bool begun = false; tile >= 0; tile = next, begun = true) {
            next = next_tile();
            swept++;
            typename F::Acc acc[2][2];
#pragma unroll
            for (int a = 0; a < 2; a++)
#pragma unroll
                for (int b = 0; b < 2; b++)
#pragma unroll
                    for (int v = 0; v < 16; v++) acc[a][b][v] = 0;
            const int64_t c0 = tile * kCB + 64 * wc + (lane & 31);
            const Num nc0 = c0 < cols ? nrm[c_first + c0] : F::far();
            const Num nc1 = c0 + 32 < cols ? nrm[c_first + c0 + 32] : F::far();
            auto stage = [&](int s) {
                if (s + 1 < nst) fetch(tile, s + 1, buf ^ 1);
                else if (next >= 0) fetch(next, 0, buf ^ 1);
                const char* cs = C[buf] + 2 * wc * kPer * kFrag + lane * 16;
                const char* qs = HOLD ? Q + (2 * wr * 8 * F::kParts + s * kPer) * kFrag + lane * 16
                                      : Q + (buf * kStageQ + 2 * wr * kPer) * kFrag + lane * 16;
                constexpr int kQRow = HOLD ? 8 * F::kParts : kPer;     // fragments of 32 queries
#pragma unroll
                for (int k = 0; k < F::kSteps; k++) {
                    Vec av[2][F::kParts], bv[2][F::kParts];
#pragma unroll
                    for (int p = 0; p < F::kParts; p++)
#pragma unroll
                        for (int h = 0; h < 2; h++) {
                            const int x = k * F::kParts + p;
                            av[h][p] = *reinterpret_cast<const Vec*>(qs + (h * kQRow + x) * kFrag);
                            bv[h][p] = *reinterpret_cast<const Vec*>(cs + (h * kPer + x) * kFrag);
                        }
#pragma unroll
                    for (int a = 0; a < 2; a++)
#pragma unroll
                        for (int b = 0; b < 2; b++) F::product(av[a], bv[b], acc[a][b]);
                }
                settle();
                buf ^= 1;
            };
            stage(0);
            // the previous tile's candidates are all in the lists now; the next
            // stage's barrier, or one more, shows the new bounds to everybody
            if (begun) {
                cut();
                if (nst == 1 || list) __syncthreads();
                if (list) {
                    const uint32_t a = thr[lane], b = thr[lane + kWave];
                    worst = wave_max(a > b ? a : b);
                }
            }
            for (int s = 1; s < nst; s++) stage(s);
            // filter: element v of tile (a, b) is row 8 (v / 4) + 4 (lane / 32) + v % 4,
            // column lane % 32.  Each lane collects a bit per element that passes;
            // those few are picked out lane by lane, gather in LDS and go to the
            // lists together.
            int qn = 0;
            auto drain = [&]() {
                __builtin_amdgcn_wave_barrier();
                for (int x = lane; x < qn; x += kWave) {
                    const Hit h = hits[w][x];
                    const uint32_t rl = h.at >> 8;
                    const int64_t lc = tile * kCB + (h.at & 255u), gc = c_first + lc;
                    if (lc < cols && gc != q0 + rl) {
                        const uint32_t pos = atomicAdd(&cnt[rl], 1u);
                        lists[rl * kCap + pos] =
                            ((uint64_t)F::bits(h.part, nq[rl]) << 32) |
                            (uint64_t)(ord.perm ? ord.perm[gc] : (uint32_t)gc);
                    }
                }
                __builtin_amdgcn_wave_barrier();
                qn = 0;
            };
#pragma unroll
            for (int a = 0; a < 2; a++) {
                Num g[16];
#pragma unroll
                for (int v = 0; v < 16; v++)
                    g[v] = bnd[64 * wr + 32 * a + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)];
#pragma unroll
                for (int b = 0; b < 2; b++) {
                    const Num ncv = b ? nc1 : nc0;
                    uint32_t pass = 0;
#pragma unroll
                    for (int v = 15; v >= 0; v--)
                        pass = pass + pass + (F::part_dist(acc[a][b][v], f, ncv) <= g[v] ? 1u : 0u);
                    uint64_t m;
                    while ((m = ballot64(pass != 0u)) != 0) {
                        const int c = __popcll(m);
                        if (qn + c > kHits) drain();
                        const uint32_t v = (uint32_t)__ffs((int)pass) - 1u;
                        // acc[a][b][v], by a tree of selects between values
                        auto pick = [](bool c, Num hi, Num lo) { return c ? hi : lo; };
                        const bool v0 = (v & 1u) != 0, v1 = (v & 2u) != 0, v2 = (v & 4u) != 0,
                                   v3 = (v & 8u) != 0;
                        auto of4 = [&](int q) {
                            return pick(v1, pick(v0, acc[a][b][q + 3], acc[a][b][q + 2]),
                                        pick(v0, acc[a][b][q + 1], acc[a][b][q]));
                        };
                        const Num x = pick(v3, pick(v2, of4(12), of4(8)), pick(v2, of4(4), of4(0)));
                        if (pass != 0u) {
                            const uint32_t rl = (uint32_t)(64 * wr + 32 * a + 4 * (lane >> 5)) +
                                                8u * (v >> 2) + (v & 3u);
                            const uint32_t cl = (uint32_t)(64 * wc + 32 * b + (lane & 31));
                            hits[w][qn + __builtin_amdgcn_mbcnt_hi(
                                             (uint32_t)(m >> 32),
                                             __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0))] =
                                Hit{F::part_dist(x, f, ncv), rl << 8 | cl};
                            pass &= pass - 1u;
                        }
                        qn += c;
                    }
                }
            }
            if (qn > 0) drain();
        }
        settle();
        if (list && t == 0) atomicAdd(met, (unsigned long long)swept);
        // the kp best of each row
        for (int q = 16 * w; q < 16 * w + 16; q++) {
            if (q0 + q >= n) break;
            const int64_t r = q0 - q_first + q;
            const uint64_t* const lst = lists + q * kCap;
            int m = __builtin_amdgcn_readfirstlane((int)cnt[q]);
            uint32_t end = thr[q];
            if (m < kp) {
                for (int e = lane; e < m; e += kWave) cand[r * kp + e] = lst[e];
            } else {
                uint32_t last;
                m = cut_list(lst, m, kp, 0, cand + r * kp, last);
                // kNoThr: all are in the list
                end = kp == n - 1 ? kNoThr : last < end ? last : end;
            }
            if (lane == 0) {
                cand_cnt[r] = (uint32_t)m;
                cand_thr[r] = end;
            }
        }
    }
}

// Exact re-rank: FP64 distances of the candidates, sorted by (d, j); emits
// the first k.  flag[i] = 1 when the error bound of the pre-selection does not
// prove that the k best are among the candidates.
//
// A lane sums its candidate's terms in order of the dimension, its row read 16
// bytes at a time at the rows' own alignment.  400,000 rows of 182 candidates of 128:
// 4.7 ms, 10.7 with the candidates' rows staged through LDS.
template <typename X>
__device__ __forceinline__ double rerank_dist(const X* __restrict__ a, const X* __restrict__ b,
                                              int D) {
    constexpr int V = 16 / sizeof(X);
    double acc = 0.0;
    int d = 0;
#pragma unroll 4
    for (; d + V <= D; d += V) {
        X u[V], v[V];
        __builtin_memcpy(u, a + d, 16);
        __builtin_memcpy(v, b + d, 16);
#pragma unroll
        for (int q = 0; q < V; q++) {
            const double e = to_f64(u[q]) - to_f64(v[q]);
            acc = fma(e, e, acc);
        }
    }
    for (; d < D; d++) {
        const double e = to_f64(a[d]) - to_f64(b[d]);
        acc = fma(e, e, acc);
    }
    return acc;
}

template <typename X>
__global__ __launch_bounds__(256) void k_knn_rerank(const X* __restrict__ Xm, int64_t q_first,
                                                    int D, int k,
                                                    const uint32_t* __restrict__ perm,
                                                    const uint64_t* __restrict__ cand, int kp,
                                                    const uint32_t* __restrict__ cand_cnt,
                                                    const uint32_t* __restrict__ cand_thr,
                                                    const float* __restrict__ nrm, float nrm_max,
                                                    float scale, int32_t* __restrict__ idx,
                                                    double* __restrict__ d2,
                                                    uint32_t* __restrict__ flag) {
    __shared__ double dv[512];
    __shared__ uint32_t jv[512];
    const int64_t l = blockIdx.x, i = perm ? (int64_t)perm[q_first + l] : q_first + l;
    const int t = threadIdx.x;
    const int m = (int)cand_cnt[l];                 // at most 256 + kMargin
    const uint64_t* lst = cand + l * kp;
    for (int e = t; e < 512; e += 256) {
        dv[e] = INFINITY;
        jv[e] = e < m ? (uint32_t)lst[e] : 0xFFFFFFFFu;
    }
    __syncthreads();
    for (int e = t; e < m; e += 256) dv[e] = rerank_dist(Xm + i * D, Xm + (int64_t)jv[e] * D, D);
    __syncthreads();
    for (int kk = 2; kk <= 512; kk <<= 1) {
        for (int j = kk >> 1; j > 0; j >>= 1) {
            const int a = ((t & ~(j - 1)) << 1) | (t & (j - 1));
            const int b = a | j;
            const double da = dv[a], db = dv[b];
            const uint32_t ja = jv[a], jb = jv[b];
            const bool gt = da > db || (da == db && ja > jb);
            const bool up = (a & kk) == 0;
            if (gt == up) {
                dv[a] = db; dv[b] = da;
                jv[a] = jb; jv[b] = ja;
            }
            __syncthreads();
        }
    }
    for (int e = t; e < k; e += 256) {
        idx[i * k + e] = (int32_t)jv[e];
        d2[i * k + e] = dv[e];
    }
    if (t == 0) {
        const uint32_t tb = cand_thr[l];
        if (tb == kNoThr) {
            flag[i] = 0u;                        // every candidate was kept
        } else {
            // Error of a pre-selected distance: 3 D products of the two
            // halves rounded on the way into |x.y| (2 * 3 D 2^-24 |x||y|, and
            // |x||y| <= (|x| + |y|)^2 / 4), the parts left out and the norms
            // (16 2^-24 (|x| + |y|)^2), and half-precision numbers below the
            // normal range, 2^-14 / scale per entry.  A row closer than the
            // k-th has |y| <= |x| + its distance.
            const double tau = (double)__uint_as_float(tb);
            const double sx = sqrt((double)nrm[i]);
            const double sy = fmin(sqrt((double)nrm_max), sx + sqrt(dv[k - 1])), s = sx + sy;
            const double err = 1.01 * ((1.5 * D + 16.0) * 0x1.0p-24 * s * s +
                                       2.0 * sqrt((double)D) * s * (0x1.0p-14 / (double)scale));
            flag[i] = dv[k - 1] < tau - err ? 0u : 1u;
        }
    }
}

// uint8 rows: the kept keys are exact integer distances and a candidate equal
// to the threshold is always kept, so the first k of the sorted list are the
// answer.
__global__ __launch_bounds__(256) void k_knn_emit(const uint64_t* __restrict__ cand, int kp,
                                                  const uint32_t* __restrict__ cand_cnt,
                                                  int64_t q_first, int k,
                                                  const uint32_t* __restrict__ perm,
                                                  int32_t* __restrict__ idx,
                                                  double* __restrict__ d2) {
    __shared__ uint64_t key[512];
    const int64_t l = blockIdx.x, i = perm ? (int64_t)perm[q_first + l] : q_first + l;
    const int t = threadIdx.x, m = (int)cand_cnt[l];
    for (int e = t; e < 512; e += 256) key[e] = e < m ? cand[l * kp + e] : ~0ull;
    __syncthreads();
    bitonic512(key);
    for (int e = t; e < k; e += 256) {
        idx[i * k + e] = (int32_t)(uint32_t)key[e];
        d2[i * k + e] = (double)(uint32_t)(key[e] >> 32);
    }
}

// Rows the bound could not certify.  The k-th distance that the re-ranking
// found bounds the true one from above, so one FP64 pass over all rows collects
// what is not further (k and a few), and a block sorts it.  A single such row at
// 41,273 x 474 took 1.8 s by k passes, 1 ms by this.
constexpr int kMissCap = 2048;     // collected per row
constexpr int kMissRows = 1024;    // rows at a time

template <typename X>
__global__ __launch_bounds__(256) void k_miss_scan(const X* __restrict__ Xm, int64_t n, int D, int k,
                                                   const uint32_t* __restrict__ rows,
                                                   const double* __restrict__ d2,
                                                   uint32_t* __restrict__ cnt,
                                                   double* __restrict__ md,
                                                   uint32_t* __restrict__ mj) {
    const int64_t r = blockIdx.y, i = rows[r];
    const double bound = d2[i * k + k - 1];
    for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n; j += (int64_t)gridDim.x * 256) {
        if (j == i) continue;
        const double d = rerank_dist(Xm + i * D, Xm + j * D, D);
        if (d <= bound) {
            const uint32_t at = atomicAdd(&cnt[r], 1u);
            if (at < (uint32_t)kMissCap) {
                md[r * kMissCap + at] = d;
                mj[r * kMissCap + at] = (uint32_t)j;
            }
        }
    }
}

// (a row with more than kMissCap is left as it is)
__global__ __launch_bounds__(256) void k_miss_sort(const uint32_t* __restrict__ rows, int k,
                                                   const uint32_t* __restrict__ cnt,
                                                   const double* __restrict__ md,
                                                   const uint32_t* __restrict__ mj,
                                                   int32_t* __restrict__ idx,
                                                   double* __restrict__ d2) {
    __shared__ double dv[kMissCap];
    __shared__ uint32_t jv[kMissCap];
    const int64_t r = blockIdx.x, i = rows[r];
    const int t = threadIdx.x, m = cnt[r] <= (uint32_t)kMissCap ? (int)cnt[r] : 0;
    if (m < k) return;
    for (int e = t; e < kMissCap; e += 256) {
        dv[e] = e < m ? md[r * kMissCap + e] : INFINITY;
        jv[e] = e < m ? mj[r * kMissCap + e] : 0xFFFFFFFFu;
    }
    __syncthreads();
    for (int kk = 2; kk <= kMissCap; kk <<= 1)
        for (int j = kk >> 1; j > 0; j >>= 1) {
            for (int x = t; x < kMissCap / 2; x += 256) {
                const int a = ((x & ~(j - 1)) << 1) | (x & (j - 1)), b = a | j;
                const double da = dv[a], db = dv[b];
                const uint32_t ja = jv[a], jb = jv[b];
                if ((da > db || (da == db && ja > jb)) == ((a & kk) == 0)) {
                    dv[a] = db; dv[b] = da;
                    jv[a] = jb; jv[b] = ja;
                }
            }
            __syncthreads();
        }
    for (int e = t; e < k; e += 256) {
        idx[i * k + e] = (int32_t)jv[e];
        d2[i * k + e] = dv[e];
    }
}

// Rows with more than kMissCap others at the bound (ties): block per row,
// FP64 over all n, keeps a sorted top-k in LDS by repeated block passes.
template <typename X>
__global__ __launch_bounds__(256) void k_knn_exact_row(const X* __restrict__ Xm, int64_t n, int D,
                                                       int k, const uint32_t* __restrict__ rows,
                                                       int32_t* __restrict__ idx,
                                                       double* __restrict__ d2) {
    __shared__ double bd[256];
    __shared__ uint32_t bj[256];
    const int64_t i = rows[blockIdx.x];
    const int t = threadIdx.x;
    double last_d = -1.0;
    uint32_t last_j = 0;
    for (int r = 0; r < k; r++) {
        // smallest (d, j) strictly greater than (last_d, last_j)
        double bdv = INFINITY;
        uint32_t bjv = 0xFFFFFFFFu;
        for (int64_t j = t; j < n; j += 256) {
            if (j == i) continue;
            double a = 0.0;
            for (int d = 0; d < D; d++) {
                const double v = to_f64(Xm[i * D + d]) - to_f64(Xm[j * D + d]);
                a += v * v;
            }
            const bool after = a > last_d || (a == last_d && (uint32_t)j > last_j);
            const bool better = a < bdv || (a == bdv && (uint32_t)j < bjv);
            if (after && better) { bdv = a; bjv = (uint32_t)j; }
        }
        bd[t] = bdv; bj[t] = bjv;
        __syncthreads();
        for (int o = 128; o > 0; o >>= 1) {
            if (t < o) {
                const bool better = bd[t + o] < bd[t] || (bd[t + o] == bd[t] && bj[t + o] < bj[t]);
                if (better) { bd[t] = bd[t + o]; bj[t] = bj[t + o]; }
            }
            __syncthreads();
        }
        last_d = bd[0];
        last_j = bj[0];
        if (t == 0) {
            idx[i * k + r] = (int32_t)last_j;
            d2[i * k + r] = last_d;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// perplexity calibration (FP64)
// ---------------------------------------------------------------------------
// W lanes (a power of two) share a row, lane l of them holds its entries l, l + W,
// ...: up to HELD in registers, and for longer rows all are read again for every
// evaluation (HELD = 0).  Bound by the FP64 exponentials, about 20 evaluations of
// k of them per row, so with four entries a lane W is the smallest that holds the
// row.  100,000 rows of 3, 15, 30, 60, 90 and 150: 29, 84, 140, 260, 430 and
// 810 us; with a wavefront per row whatever its length 156, 545, 556, 570, 686 and
// 817; with a thread per row, which read and wrote its row, 8 k bytes from its
// neighbour's, at every evaluation, 34, 273, 664, 1,259, 2,464 and 3,718.
template <int W, int HELD>
__global__ __launch_bounds__(256) void k_perplexity(const double* __restrict__ d2, int64_t n,
                                                    int k, double target, double tol,
                                                    int max_iter, double* __restrict__ P,
                                                    double* __restrict__ beta_out) {
    const int lane = threadIdx.x & (W - 1);
    const int64_t i = (int64_t)blockIdx.x * (256 / W) + threadIdx.x / W;
    if (i >= n) return;
    const double* d = d2 + i * k;
    double* p = P + i * k;
    constexpr int kH = HELD > 0 ? HELD : 1;
    // over the lanes of the row, which leave the loop together
    auto row_sum = [](double v) {
#pragma unroll
        for (int o = W / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, W);
        return v;
    };
    double dh[kH], eh[kH];
    double dmin = INFINITY;
    if constexpr (HELD > 0) {
#pragma unroll
        for (int q = 0; q < HELD; q++) {
            const int j = lane + q * W;
            dh[q] = j < k ? d[j] : INFINITY;
            dmin = fmin(dmin, dh[q]);
        }
    } else {
        for (int j = lane; j < k; j += W) dmin = fmin(dmin, d[j]);
    }
#pragma unroll
    for (int o = W / 2; o > 0; o >>= 1) dmin = fmin(dmin, __shfl_xor(dmin, o, W));
    double b = 1.0, lo = 0.0, hi = 0.0, S = 0.0;
    bool have_lo = false, have_hi = false;
    for (int it = 0; it < max_iter; it++) {
        S = 0.0;
        double SD = 0.0;
        if constexpr (HELD > 0) {
#pragma unroll
            for (int q = 0; q < HELD; q++) {
                eh[q] = 0.0;
                if (lane + q * W < k) {
                    const double dj = dh[q] - dmin;
                    eh[q] = exp(-b * dj);
                    S += eh[q];
                    SD += dj * eh[q];
                }
            }
        } else {
            for (int j = lane; j < k; j += W) {
                const double dj = d[j] - dmin;
                const double e = exp(-b * dj);
                S += e;
                SD += dj * e;
            }
        }
        S = row_sum(S);
        SD = row_sum(SD);
        const double H = log(S) + b * SD / S;
        if (fabs(H - target) < tol || it == max_iter - 1) break;
        if (H > target) {
            lo = b; have_lo = true;
            b = have_hi ? 0.5 * (b + hi) : 2.0 * b;
        } else {
            hi = b; have_hi = true;
            b = have_lo ? 0.5 * (b + lo) : 0.5 * b;
        }
    }
    if constexpr (HELD > 0) {
#pragma unroll
        for (int q = 0; q < HELD; q++)
            if (lane + q * W < k) p[lane + q * W] = eh[q] / S;
    } else {
        for (int j = lane; j < k; j += W) p[j] = exp(-b * (d[j] - dmin)) / S;
    }
    if (beta_out && lane == 0) beta_out[i] = b;
}

// ---------------------------------------------------------------------------
// symmetrisation
// ---------------------------------------------------------------------------
// exclusive scan of int64, three phases (block size 1024 elements)
__global__ __launch_bounds__(256) void k_scan64_reduce(const int64_t* __restrict__ a, int64_t m,
                                                       int64_t* __restrict__ bsum) {
    __shared__ int64_t red[256];
    const int64_t base = (int64_t)blockIdx.x * 1024;
    int64_t s = 0;
    for (int e = threadIdx.x; e < 1024; e += 256)
        if (base + e < m) s += a[base + e];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) bsum[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(1024) void k_scan64_top(int64_t* __restrict__ bsum, int64_t nb) {
    __shared__ int64_t part[1024];
    const int t = threadIdx.x;
    const int64_t per = (nb + 1023) / 1024;
    const int64_t b = t * per, e = b + per < nb ? b + per : nb;
    int64_t s = 0;
    for (int64_t i = b; i < e; i++) s += bsum[i];
    part[t] = s;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        int64_t v = t >= o ? part[t - o] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    int64_t run = t ? part[t - 1] : 0;
    for (int64_t i = b; i < e; i++) {
        int64_t v = bsum[i];
        bsum[i] = run;
        run += v;
    }
}

__global__ __launch_bounds__(256) void k_scan64_apply(const int64_t* __restrict__ a, int64_t m,
                                                      const int64_t* __restrict__ bsum,
                                                      int64_t* __restrict__ out) {
    __shared__ int64_t ws[4];
    const int t = threadIdx.x, w = t >> 6, lane = lane_id();
    const int64_t base = (int64_t)blockIdx.x * 1024 + 4 * t;
    int64_t v[4], sum = 0;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        v[q] = base + q < m ? a[base + q] : 0;
        sum += v[q];
    }
    int64_t x = sum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int64_t y = __shfl_up(x, o, kWave);
        if (lane >= o) x += y;
    }
    if (lane == kWave - 1) ws[w] = x;
    __syncthreads();
    int64_t run = bsum[blockIdx.x] + x - sum;
    for (int q = 0; q < w; q++) run += ws[q];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        if (base + q < m) out[base + q] = run;
        run += v[q];
    }
}

// Row i of P joins the k out-edges i -> j with the in-edges i' -> i.  A stable
// sort of the edges by their target leaves each target's in-edges together
// and, as edge e = i k + t comes before the edges of later rows, ordered by
// their source; the out-edges are sorted by their target in LDS, and the two
// ordered lists are merged by rank.  A pair that is in both is one entry.
// (In-edges placed by atomic counters and then ranked against each other cost
// the square of a row's length: 31.9 ms for the one or two hub rows of 70,000
// byte images, where this takes 0.4.)

// first sorted position of each target's in-edges; start[n] = m
__global__ __launch_bounds__(256) void k_in_start(const uint32_t* __restrict__ target, int64_t m,
                                                  int64_t n, int64_t* __restrict__ start) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e > m) return;
    const int64_t a = e > 0 ? (int64_t)target[e - 1] + 1 : 0;      // rows without in-edges too
    const int64_t b = e < m ? (int64_t)target[e] : n;
    for (int64_t j = a; j <= b; j++) start[j] = e;
}

// position of source j among the in-edges [a, b) (edge numbers, ascending):
// the first whose source is not below j
__device__ __forceinline__ int64_t in_lower(const uint32_t* __restrict__ edge, int64_t a, int64_t b,
                                            uint32_t j, uint32_t k) {
    const uint64_t e0 = (uint64_t)j * k;           // the first edge of row j
    while (a < b) {
        const int64_t mid = (a + b) >> 1;
        if ((uint64_t)edge[mid] < e0) a = mid + 1;
        else b = mid;
    }
    return a;
}
__device__ __forceinline__ bool in_has(const uint32_t* __restrict__ edge, int64_t a, int64_t b,
                                       uint32_t j, uint32_t k) {
    return a < b && edge[a] / k == j;
}

// entries of each row: out-edges and in-edges less the pairs in both (one
// wavefront per row; entry n is 0 for the scan)
__global__ __launch_bounds__(256) void k_sym_count(const int32_t* __restrict__ idx,
                                                   const int64_t* __restrict__ start,
                                                   const uint32_t* __restrict__ edge, int64_t n,
                                                   int k, int64_t* __restrict__ ucnt) {
    const int lane = lane_id();
    const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i > n) return;
    if (i == n) {
        if (lane == 0) ucnt[n] = 0;
        return;
    }
    const int64_t a = start[i], b = start[i + 1];
    int both = 0;
    for (int t = lane; t < k; t += kWave) {
        const uint32_t j = (uint32_t)idx[i * k + t];
        both += in_has(edge, in_lower(edge, a, b, j, (uint32_t)k), b, j, (uint32_t)k) ? 1 : 0;
    }
    both = wave_sum(both);
    if (lane == 0) ucnt[i] = (int64_t)k + (b - a) - both;
}

// One row per block, from row `first` on: k <= 256 out-edges, any number of in-edges.
__global__ __launch_bounds__(256) void k_sym_row(int64_t first, const int32_t* __restrict__ idx,
                                                 const double* __restrict__ Pc,
                                                 const int64_t* __restrict__ start,
                                                 const uint32_t* __restrict__ edge, int k,
                                                 const int64_t* __restrict__ rp, double inv2n,
                                                 uint32_t* __restrict__ col,
                                                 double* __restrict__ val) {
    __shared__ uint32_t own[256];           // out-edges' targets, then sorted
    __shared__ uint32_t sorted[256];
    __shared__ uint32_t both[257];          // sorted targets that are in-edges too, before each
    __shared__ uint32_t wsum[4];
    const int64_t i = first + blockIdx.x;
    const int t = threadIdx.x, w = t >> 6, lane = lane_id();
    const int64_t a = start[i], b = start[i + 1], o = rp[i];
    const uint32_t uk = (uint32_t)k;
    uint32_t j = 0xFFFFFFFFu;
    double v = 0.0;
    if (t < k) {
        j = (uint32_t)idx[i * k + t];
        v = Pc[i * k + t];
        own[t] = j;
    }
    __syncthreads();
    int r = 0;                              // rank among the out-edges (targets are distinct)
    if (t < k) {
        for (int q = 0; q < k; q++) r += own[q] < j ? 1 : 0;
        sorted[r] = j;
    }
    // where the target stands among the in-edges, and whether it is one
    const int64_t at = t < k ? in_lower(edge, a, b, j, uk) : b;
    const bool dup = t < k && in_has(edge, at, b, j, uk);
    if (t < 256) both[t] = 0;
    __syncthreads();
    if (t < k) both[r] = dup ? 1u : 0u;
    __syncthreads();
    // exclusive prefix of the flags over the sorted targets
    uint32_t f = both[t], x = f;
#pragma unroll
    for (int s = 1; s < kWave; s <<= 1) {
        const uint32_t y = __shfl_up(x, s, kWave);
        if (lane >= s) x += y;
    }
    if (lane == kWave - 1) wsum[w] = x;
    __syncthreads();
    for (int q = 0; q < w; q++) x += wsum[q];
    both[t] = x - f;
    if (t == 255) both[256] = x;
    __syncthreads();
    if (t < k) {
        const int64_t pos = o + r + (at - a) - both[r];
        col[pos] = j;
        val[pos] = (dup ? v + Pc[edge[at]] : v) * inv2n;
    }
    for (int64_t e = a + t; e < b; e += 256) {
        const uint32_t src = edge[e] / uk;
        int lo = 0, hi = k;                 // out-edges' targets below src
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (sorted[mid] < src) lo = mid + 1;
            else hi = mid;
        }
        if (lo < k && sorted[lo] == src) continue;      // written with the out-edge
        const int64_t pos = o + (e - a) + lo - both[lo];
        col[pos] = src;
        val[pos] = Pc[edge[e]] * inv2n;
    }
}

hipError_t scan_i64_local(const int64_t* a, int64_t m, int64_t* out, int64_t* tmp, hipStream_t s) {
    const int64_t nb = ceil_div(m, 1024);
    k_scan64_reduce<<<dim3((unsigned)nb), 256, 0, s>>>(a, m, tmp);
    k_scan64_top<<<1, 1024, 0, s>>>(tmp, nb);
    k_scan64_apply<<<dim3((unsigned)nb), 256, 0, s>>>(a, m, tmp, out);
    return hipGetLastError();
}

// Working lists of the blocks that run at a time, one per CU (as LDS allows).
inline int64_t resident_blocks(int64_t rows) {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 0;
    const int64_t most = ceil_div(rows, kQB);
    return cus < 1 ? 1 : (cus < most ? cus : most);
}

struct Lists {
    int64_t resident;                   // blocks that run at a time
    uint32_t* ticket;
    unsigned long long* met;            // tiles that blocks with an order met
    uint64_t *work, *cand;              // [resident][kQB][kCap]; [rows][kp]
    uint32_t *cnt, *thr;
};

// rows first .. of the batch against the candidates c_first .. c_first + cols
template <typename F>
hipError_t launch_candidates(const char* queries, const char* packed, int64_t n, int64_t c_first,
                             int64_t cols, int steps, const typename F::Num* nrm, float f,
                             int64_t first, int64_t rows, int kp, const RowOrder& ord,
                             const Lists& l, hipStream_t s) {
    const int64_t blocks = ord.turn ? ord.T * (ord.G / kQB) : ceil_div(rows, kQB);
    const dim3 g((unsigned)std::min(l.resident, blocks));
    const hipError_t e = hipMemsetAsync(l.ticket, 0, sizeof(uint32_t), s);
    if (e != hipSuccess) return e;
    // the queries' fragments stay in LDS while 8 steps of them fit beside two
    // stages (FP16: depth 128)
    if (steps <= 8)
        k_knn_candidates<F, true><<<g, 512, 0, s>>>(queries, packed, n, c_first, cols, steps, nrm,
                                                    f, first, kp, ord, (uint32_t)blocks, l.ticket,
                                                    l.met, l.work, l.cand, l.cnt, l.thr);
    else
        k_knn_candidates<F, false><<<g, 512, 0, s>>>(queries, packed, n, c_first, cols, steps, nrm,
                                                     f, first, kp, ord, (uint32_t)blocks, l.ticket,
                                                     l.met, l.work, l.cand, l.cnt, l.thr);
    return hipGetLastError();
}

// The kp best of a row's list and of its list from further candidates, one
// wavefront per row: to `best`, with the number kept and the bits of a distance
// that no row left out is nearer than.
__global__ __launch_bounds__(256) void k_join_lists(int64_t rows, int kp,
                                                    const uint64_t* __restrict__ more,
                                                    const uint32_t* __restrict__ more_cnt,
                                                    const uint32_t* __restrict__ more_thr,
                                                    uint64_t* best, uint32_t* __restrict__ cnt,
                                                    uint32_t* __restrict__ thr) {
    __shared__ uint64_t both[256 / kWave][kCap];
    const int lane = lane_id(), w = threadIdx.x >> 6;
    const int64_t r = (int64_t)blockIdx.x * (256 / kWave) + w;
    if (r >= rows) return;
    const int a = (int)cnt[r], b = (int)more_cnt[r];        // at most kp each
    for (int e = lane; e < a; e += kWave) both[w][e] = best[r * kp + e];
    for (int e = lane; e < b; e += kWave) both[w][a + e] = more[r * kp + e];
    __builtin_amdgcn_wave_barrier();
    uint32_t end = thr[r] < more_thr[r] ? thr[r] : more_thr[r];
    int m = a + b;
    if (m < kp) {
        for (int e = a + lane; e < m; e += kWave) best[r * kp + e] = both[w][e];
    } else {
        uint32_t last;
        m = cut_list(both[w], m, kp, 0, best + r * kp, last);
        end = last < end ? last : end;
    }
    if (lane == 0) {
        cnt[r] = (uint32_t)m;
        thr[r] = end;
    }
}

// The order of the rows (see above): packs the rows in their own order, assigns
// them to pivots, sorts them, packs them again and makes the groups' lists.
// pack(perm) packs the rows; nrm_p: the norms in the order; held: the arrays.  Two checks end it where it would not pay.  If the even pivots are
// not much nearer to the rows than to each other, the rows keep their own order
// (66,000 Gaussian rows of 50: 7.5 ms, 9.0 with all of the order made, 7.3 with
// none).  If hardly any groups are apart, neither: a block whose own cluster
// comes late keeps a loose threshold until then, and blocks that take the tiles
// in turn share them in L2 (100,000 Gaussian rows of 8: 10.2 ms without an
// order, 12.5 by the lists; with clusters 4 sigma apart, 7% of the pairs apart,
// 10.0 and 8.8; 100,000 x 100 in such clusters 15.6 and 7.0).
template <typename X, typename F, typename P, typename Pack>
hipError_t order_rows(const X* Xm, int64_t n, int D, int steps, float f, float scale, float err,
                      const Num_t<F>* nrm, float norm_max, char* packed, Pack&& pack, Arena* held,
                      hipStream_t s, RowOrder* ord, const Num_t<F>** nrm_p) {
    using Num = typename F::Num;
    const int64_t G = kCB * ceil_div(ceil_div(n, kCB), kMaxGroups);
    const int T = (int)ceil_div(n, G), most = T > kPivots ? T : kPivots;
    char* frag = nullptr;
    float *ct = nullptr, *d2 = nullptr, *m = nullptr;
    Num *cn = nullptr, *np = nullptr;
    uint32_t *rank = nullptr, *key[2] = {nullptr, nullptr}, *idx[2] = {nullptr, nullptr},
             *hist = nullptr, *dtot = nullptr, *rows = nullptr, *radius2 = nullptr, *far_of = nullptr,
             *turn = nullptr;
    GroupAt* order = nullptr;
    int64_t *weight = nullptr, *sum = nullptr, *tmp = nullptr;
    unsigned long long* apart = nullptr;
    const size_t frags = (size_t)ceil_div(most, 32) * steps * 1024;
    hipError_t e = hipSuccess;
    *nrm_p = nrm;
    held->add(&frag, (int64_t)frags);
    held->add(&ct, (int64_t)D * most);
    held->add(&cn, most);
    held->add(&d2, (int64_t)most * most);
    held->add(&m, (int64_t)T * T);
    held->add(&order, (int64_t)T * T);
    held->add(&radius2, T);
    held->add(&far_of, T);
    held->add(&turn, T);
    held->add(&apart, 1);
    held->add(&rank, kPivots);
    held->add(&rows, kPivots);
    for (int h = 0; h < 2; h++) {
        held->add(&key[h], n);
        held->add(&idx[h], n);
    }
    held->add(&np, n);
    held->add(&weight, n + 1);
    held->add(&sum, n + 1);
    held->add(&tmp, scan_i64_tmp_len(n + 1));
    held->add(&hist, sort_hist_words(n, 8));
    held->add(&dtot, sort_digit_words());
    if ((e = held->make()) != hipSuccess) {
        // no room: the rows keep their order
        (void)hipGetLastError();
        if (e != hipErrorOutOfMemory) return e;
        pack(nullptr);
        return hipGetLastError();
    }
    const dim3 blocks((unsigned)(pad_rows(n) / 256));
    pack(nullptr);
    if ((e = hipMemsetAsync(frag, 0, frags, s)) != hipSuccess) return e;
    if ((e = hipMemsetAsync(weight + n, 0, sizeof(int64_t), s)) != hipSuccess) return e;
    const float unit = 0x1p28f / (norm_max > 0.f ? norm_max : 1.f);
    k_even_rows<<<1, kRoundPivots, 0, s>>>(n, rows);
    for (int r = 1; r <= kRounds; r++) {
        const int count = r * kRoundPivots;
        k_centers<X, F, P><<<count, 256, 0, s>>>(Xm, count, D, rows, 1, 1, steps, scale, frag, ct,
                                                 cn);
        if (r == kRounds) break;
        k_center_dots<F, true><<<blocks, 512, 0, s>>>(packed, n, steps, frag, cn, count, f, G,
                                                      nullptr, nullptr, nrm, unit, weight, nullptr,
                                                      nullptr);
        if ((e = scan_i64_local(weight, n + 1, sum, tmp, s)) != hipSuccess) return e;
        if (r == 1) {
            std::vector<float> between((size_t)count * count);
            int64_t total = 0;
            k_center_d2<<<count, 256, 0, s>>>(ct, D, count, d2);
            e = hipMemcpyAsync(between.data(), d2, 4 * between.size(), hipMemcpyDeviceToHost, s);
            if (e == hipSuccess)
                e = hipMemcpyAsync(&total, sum + n, 8, hipMemcpyDeviceToHost, s);
            if (e == hipSuccess) e = hipStreamSynchronize(s);
            if (e != hipSuccess) return e;
            double all = 0.0;
            for (float v : between) all += v;
            all /= (double)count * (count - 1);
            if (!((double)total / (double)n < kNearShare * all * unit)) return hipSuccess;
        }
        k_pick<<<1, kRoundPivots, 0, s>>>(sum, n, rows + count);
    }
    k_center_d2<<<kPivots, 256, 0, s>>>(ct, D, kPivots, d2);
    k_chain<<<1, kWave, 0, s>>>(d2, rank);
    k_center_dots<F, true><<<blocks, 512, 0, s>>>(packed, n, steps, frag, cn, kPivots, f, G, rank,
                                                  key[0], nrm, 0.f, nullptr, nullptr, nullptr);
    int at = 0;
    if ((e = sort_pairs32(key, idx, n, 8, hist, dtot, s, &at)) != hipSuccess) return e;
    const uint32_t* perm = idx[at];
    pack(perm);
    k_permuted<<<dim3((unsigned)ceil_div(n, 256)), 256, 0, s>>>(nrm, perm, n, np);
    if ((e = hipMemsetAsync(frag, 0, frags, s)) != hipSuccess) return e;
    if ((e = hipMemsetAsync(radius2, 0, sizeof(uint32_t) * T, s)) != hipSuccess) return e;
    if ((e = hipMemsetAsync(far_of, 0, sizeof(uint32_t) * T, s)) != hipSuccess) return e;
    if ((e = hipMemsetAsync(apart, 0, sizeof(*apart), s)) != hipSuccess) return e;
    k_centers<X, F, P><<<dim3((unsigned)T), 256, 0, s>>>(Xm, n, D, perm, G, G, steps, scale, frag, ct,
                                                         cn);
    k_center_d2<<<dim3((unsigned)T), 256, 0, s>>>(ct, D, T, d2);
    k_fill_inf<<<dim3((unsigned)ceil_div((int64_t)T * T, 256)), 256, 0, s>>>(m, (int64_t)T * T);
    k_center_dots<F, false><<<blocks, 512, 0, s>>>(packed, n, steps, frag, cn, T, f, G, nullptr,
                                                   nullptr, np, 0.f, nullptr, m, radius2);
    k_group_order<<<dim3((unsigned)T), 256, 0, s>>>(m, d2, T, 2.f * err, radius2, order, far_of,
                                                    apart);
    k_group_turns<<<1, 1024, 0, s>>>(far_of, T, turn);
    unsigned long long far = 0;
    e = hipMemcpyAsync(&far, apart, sizeof(far), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    if ((double)far >= kApartShare * (double)T * (double)T) {
        // (a batch of rows takes its own in order)
        *ord = RowOrder{perm, order, n <= kBatch ? turn : nullptr, G, T, err};
        *nrm_p = np;
    } else {
        pack(nullptr);
    }
    return hipGetLastError();
}

// What the thread's last exact search did: groups of the rows' order (0: none was
// taken), tiles of kQB x kCB met by it, and tiles of all pairs.
struct SearchTrace { int64_t groups, met, all; };
thread_local SearchTrace g_trace;

// What a search holds at a time: the lists of `rows` queries, `cols` candidates
// packed, working lists of `resident` blocks.
struct Room {
    int64_t rows, cols, resident;
    // half of everything; false once there is nothing to halve
    bool shrink() {
        if (rows <= kQB && cols <= kCB && resident <= 1) return false;
        rows = ceil_div(ceil_div(rows, 2), kQB) * kQB;
        cols = ceil_div(ceil_div(cols, 2), kCB) * kCB;
        resident = ceil_div(resident, 2);
        return true;
    }
};

template <typename X>
hipError_t knn_typed(const X* Xm, int64_t n, int32_t D, int32_t k, int32_t* idx, double* d2,
                     hipStream_t s, std::string* err) {
    const int kp = (int)((int64_t)(k + kMargin) < n - 1 ? (k + kMargin) : (n - 1));
    // exact while 256^2 D fits an int32
    const bool exact = std::is_same<X, uint8_t>::value && D <= 32768;
    const int steps = exact ? pad_steps<PartsI8>(D) : pad_steps<PartsF16>(D);
    auto bytes = [&](int64_t rows) {
        return (int64_t)(exact ? packed_bytes<PartsI8>(rows, D) : packed_bytes<PartsF16>(rows, D));
    };
    float* nrm = nullptr;
    int32_t* nrm_i = nullptr;
    char *packed = nullptr, *queries = nullptr;
    Lists lists{}, more{};
    uint32_t* flag = nullptr;
    RowStats* st = nullptr;
    hipError_t e = hipSuccess;
    RowOrder ord{};
    Arena own, held;
    auto fail = [&](hipError_t x) {
        own.release();
        held.release();
        return x;
    };
    // All rows are packed at once, 4 bytes an element (1 for bytes) of padded depth.
    // Where there is no room for that, runs of candidates are packed in turn for
    // each batch of queries and their lists joined; the rows keep their order then.
    Room room{n < kBatch ? n : kBatch, n, 0};
    room.resident = resident_blocks(room.rows);
    for (;;) {
        const bool whole = room.cols >= n;
        own.add(&lists.ticket, 1);
        own.add(&lists.met, 1);
        own.add(&lists.work, room.resident * (kQB * kCap));
        for (Lists* l : {&lists, &more}) {
            if (l == &more && whole) break;
            own.add(&l->cand, room.rows * kp);
            own.add(&l->cnt, room.rows);
            own.add(&l->thr, room.rows);
        }
        own.add(&packed, bytes(room.cols));
        if (!whole) own.add(&queries, bytes(room.rows));
        if (exact) {
            own.add(&nrm_i, n);
        } else {
            own.add(&nrm, n);
            own.add(&flag, n);
            own.add(&st, 1);
        }
        if ((e = own.make()) == hipSuccess) break;
        if (e != hipErrorOutOfMemory || !room.shrink()) return fail(e);
        (void)hipGetLastError();
        own.reset();
    }
    lists.resident = more.resident = room.resident;
    more.ticket = lists.ticket;
    more.met = lists.met;
    more.work = lists.work;
    const bool whole = room.cols >= n;
    g_trace = SearchTrace{0, 0, ceil_div(n, kQB) * ceil_div(n, kCB)};
    auto trace = [&]() {         // after the launches, before a synchronisation
        g_trace.groups = ord.order ? ord.T : 0;
        return ord.order ? hipMemcpyAsync(&g_trace.met, lists.met, sizeof(*lists.met),
                                          hipMemcpyDeviceToHost, s)
                         : hipSuccess;
    };
    // launch(first, blocks) over the pieces of np packed rows; a grid holds fewer than
    // 2^32 threads, which a packed copy of 64 GB would pass
    auto by_pieces = [&](int64_t np, auto&& launch) {
        constexpr int64_t kRun = (int64_t)1 << 26;
        const int64_t all = np * steps * 2;
        for (int64_t e0 = 0; e0 < all; e0 += kRun)
            launch(e0, dim3((unsigned)ceil_div(std::min(kRun, all - e0), 256)));
    };
    // the candidates of queries first .. first + m, by pack(rows, count, perm, to)
    auto search = [&](auto parts, const auto* nrm_p, float f, int64_t first, int64_t m,
                      auto&& pack) {
        using F = decltype(parts);
        if (whole)
            return launch_candidates<F>(packed + bytes(kCB) / kCB * first, packed, n, 0, n, steps,
                                        nrm_p, f, first, m, kp, ord, lists, s);
        pack(first, m, nullptr, queries);
        for (int64_t c = 0; c < n; c += room.cols) {
            const int64_t cols = std::min(room.cols, n - c);
            pack(c, cols, nullptr, packed);
            const hipError_t x = launch_candidates<F>(queries, packed, n, c, cols, steps, nrm_p, f,
                                                      first, m, kp, ord, c ? more : lists, s);
            if (x != hipSuccess) return x;
            if (c)
                k_join_lists<<<dim3((unsigned)ceil_div(m, 256 / kWave)), 256, 0, s>>>(
                    m, kp, more.cand, more.cnt, more.thr, lists.cand, lists.cnt, lists.thr);
        }
        return hipGetLastError();
    };
    if (exact) {
        // uint8 rows: exact integer distances from INT8 MFMA
        k_row_norms_i8<<<dim3((unsigned)ceil_div(n, 4)), 256, 0, s>>>((const uint8_t*)Xm, n, D,
                                                                     nrm_i);
        auto pack = [&](int64_t first, int64_t count, const uint32_t* perm, char* to) {
            const int64_t np = pad_rows(count);
            by_pieces(np, [&](int64_t e0, dim3 g) {
                k_pack_i8<<<g, 256, 0, s>>>((const uint8_t*)Xm + first * D, count, np, D, steps,
                                            perm, e0, (uint4*)to);
            });
        };
        auto pack_all = [&](const uint32_t* perm) { pack(0, n, perm, packed); };
        // the distances' halves reach 2^30: as floats they are off by 2^7
        const int32_t* nrm_p = nrm_i;
        if (whole && n >= kOrderFrom)
            e = order_rows<X, PartsI8, CenterI8>(Xm, n, D, steps, 0.f, 1.f, 128.f, nrm_i,
                                                 16384.f * D, packed, pack_all, &held, s, &ord,
                                                 &nrm_p);
        else if (whole)
            pack_all(nullptr);
        if (e == hipSuccess && ord.order) e = hipMemsetAsync(lists.met, 0, sizeof(*lists.met), s);
        if (e != hipSuccess) return fail(e);
        for (int64_t first = 0; first < n; first += room.rows) {
            const int64_t m = std::min(room.rows, n - first);
            if ((e = search(PartsI8{}, nrm_p, 0.f, first, m, pack)) != hipSuccess) return fail(e);
            k_knn_emit<<<dim3((unsigned)m), 256, 0, s>>>(lists.cand, kp, lists.cnt, first, k,
                                                         ord.perm, idx, d2);
        }
        if ((e = hipGetLastError()) != hipSuccess) return fail(e);
        if ((e = trace()) != hipSuccess) return fail(e);
        return fail(hipStreamSynchronize(s));
    }
    if ((e = hipMemsetAsync(st, 0, sizeof(RowStats), s)) != hipSuccess) return fail(e);
    const int64_t nblk = ceil_div(n, 4) < 2048 ? ceil_div(n, 4) : 2048;
    k_row_norms<X><<<dim3((unsigned)nblk), 256, 0, s>>>(Xm, n, D, nrm, st);
    RowStats h;
    if ((e = hipMemcpyAsync(&h, st, sizeof(h), hipMemcpyDeviceToHost, s)) != hipSuccess)
        return fail(e);
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return fail(e);
    if (h.bad) {
        if (err) *err = "X contains non-finite values";
        return fail(hipErrorInvalidValue);
    }
    float norm_max, entry_max;
    memcpy(&norm_max, &h.norm, 4);
    memcpy(&entry_max, &h.entry, 4);
    // the largest entry just below FP16's range, 2^14 <= |x| < 2^15 (and 1 /
    // scale^2 in range)
    int ex = 0;
    if (entry_max > 0.f) (void)frexpf(entry_max, &ex);
    const int sh = 15 - ex < -60 ? -60 : (15 - ex > 60 ? 60 : 15 - ex);
    const float scale = ldexpf(1.f, sh), f = ldexpf(-2.f, -2 * sh);
    auto pack = [&](int64_t first, int64_t count, const uint32_t* perm, char* to) {
        const int64_t np = pad_rows(count);
        by_pieces(np, [&](int64_t e0, dim3 g) {
            k_pack_f16<X><<<g, 256, 0, s>>>(Xm + first * D, count, np, D, steps, scale, perm, e0,
                                            (_Float16*)to);
        });
    };
    auto pack_all = [&](const uint32_t* perm) { pack(0, n, perm, packed); };
    const float* nrm_p = nrm;
    if (whole && n >= kOrderFrom) {
        // the error bound of k_knn_rerank for any two rows; a centre's norm is no
        // larger than the largest row's, but for its rounding to 11 bits
        const double sum = 2.0 * sqrt((double)norm_max) * (1.0 + 0x1.0p-10);
        const double err = 1.01 * ((1.5 * D + 16.0) * 0x1.0p-24 * sum * sum +
                                   2.0 * sqrt((double)D) * sum * (0x1.0p-14 / (double)scale));
        e = order_rows<X, PartsF16, CenterF16>(Xm, n, D, steps, f, scale, (float)(1.001 * err), nrm,
                                               norm_max, packed, pack_all, &held, s, &ord, &nrm_p);
    } else if (whole) {
        pack_all(nullptr);
    }
    if (e == hipSuccess && ord.order) e = hipMemsetAsync(lists.met, 0, sizeof(*lists.met), s);
    if (e != hipSuccess) return fail(e);
    for (int64_t first = 0; first < n; first += room.rows) {
        const int64_t m = std::min(room.rows, n - first);
        if ((e = search(PartsF16{}, nrm_p, f, first, m, pack)) != hipSuccess) return fail(e);
        k_knn_rerank<X><<<dim3((unsigned)m), 256, 0, s>>>(Xm, first, D, k, ord.perm, lists.cand, kp,
                                                          lists.cnt, lists.thr, nrm, norm_max,
                                                          scale, idx, d2, flag);
    }
    if ((e = hipGetLastError()) != hipSuccess) return fail(e);
    if ((e = trace()) != hipSuccess) return fail(e);
    std::vector<uint32_t> hf(n);
    if ((e = hipMemcpyAsync(hf.data(), flag, sizeof(uint32_t) * n, hipMemcpyDeviceToHost, s)) != hipSuccess)
        return fail(e);
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return fail(e);
    std::vector<uint32_t> miss;
    for (int64_t i = 0; i < n; i++)
        if (hf[i]) miss.push_back((uint32_t)i);
    if (!miss.empty()) {
        if ((e = hipMemcpyAsync(flag, miss.data(), sizeof(uint32_t) * miss.size(),
                                hipMemcpyHostToDevice, s)) != hipSuccess)
            return fail(e);
        uint32_t *cnt = nullptr, *mj = nullptr;
        double* md = nullptr;
        // the order's scratch is done with; short of memory fewer rows go at a time, and
        // where not one has room all take the passes below
        held.release();
        int64_t at_once = std::min((int64_t)miss.size(), (int64_t)kMissRows);
        Arena found;
        auto stop = [&](hipError_t x) {
            found.release();
            return fail(x);
        };
        for (; at_once > 0; at_once /= 2) {
            found.add(&cnt, (int64_t)miss.size());
            found.add(&md, at_once * kMissCap);
            found.add(&mj, at_once * kMissCap);
            if ((e = found.make()) == hipSuccess) break;
            if (e != hipErrorOutOfMemory) return stop(e);
            (void)hipGetLastError();
            found.reset();
        }
        size_t left = miss.size();
        if (at_once > 0) {
            if ((e = hipMemsetAsync(cnt, 0, sizeof(uint32_t) * miss.size(), s)) != hipSuccess)
                return stop(e);
            const int64_t chunks = std::min(ceil_div(n, 256), (int64_t)1024);
            for (int64_t r = 0; r < (int64_t)miss.size(); r += at_once) {
                const int64_t m = std::min((int64_t)miss.size() - r, at_once);
                k_miss_scan<X><<<dim3((unsigned)chunks, (unsigned)m), 256, 0, s>>>(
                    Xm, n, D, k, flag + r, d2, cnt + r, md, mj);
                k_miss_sort<<<dim3((unsigned)m), 256, 0, s>>>(flag + r, k, cnt + r, md, mj, idx, d2);
            }
            std::vector<uint32_t> hc(miss.size());
            if ((e = hipMemcpyAsync(hc.data(), cnt, sizeof(uint32_t) * hc.size(), hipMemcpyDeviceToHost,
                                    s)) != hipSuccess)
                return stop(e);
            if ((e = hipStreamSynchronize(s)) != hipSuccess) return stop(e);
            left = 0;
            for (size_t r = 0; r < miss.size(); r++)
                if (hc[r] > (uint32_t)kMissCap) miss[left++] = miss[r];
        }
        if (left > 0) {
            if ((e = hipMemcpyAsync(flag, miss.data(), sizeof(uint32_t) * left,
                                    hipMemcpyHostToDevice, s)) != hipSuccess)
                return stop(e);
            k_knn_exact_row<X><<<dim3((unsigned)left), 256, 0, s>>>(Xm, n, D, k, flag, idx, d2);
            if ((e = hipGetLastError()) != hipSuccess) return stop(e);
            if ((e = hipStreamSynchronize(s)) != hipSuccess) return stop(e);
        }
        found.release();
    }
    return fail(hipSuccess);
}

// ---------------------------------------------------------------------------
// initial numbering: three random +-1 projections of each row, quantised and
// interleaved into a Morton code (points close in X get close codes)
// ---------------------------------------------------------------------------
__device__ __forceinline__ float rademacher(int axis, int d) {
    uint32_t h = (uint32_t)d * 0x9E3779B1u ^ (uint32_t)(axis + 1) * 0x85EBCA77u;
    h ^= h >> 15;
    h *= 0x2C1B3C6Du;
    h ^= h >> 12;
    return (h & 1u) ? 1.0f : -1.0f;
}

// one wavefront per row; proj [n][3]; per-block min/max of each axis
template <typename X>
__global__ __launch_bounds__(256) void k_project(const X* __restrict__ Xm, int64_t n, int D,
                                                 float* __restrict__ proj,
                                                 float* __restrict__ part) {
    __shared__ float red[4][6];
    const int w = threadIdx.x >> 6, lane = lane_id();
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int64_t i = (int64_t)blockIdx.x * 4 + w; i < n; i += (int64_t)gridDim.x * 4) {
        float a[3] = {0.f, 0.f, 0.f};
        for (int d = lane; d < D; d += 64) {
            const float v = to_f32(Xm[i * D + d]);
#pragma unroll
            for (int q = 0; q < 3; q++) a[q] += rademacher(q, d) * v;
        }
#pragma unroll
        for (int q = 0; q < 3; q++) {
            a[q] = wave_sum(a[q]);
            mn[q] = fminf(mn[q], a[q]);
            mx[q] = fmaxf(mx[q], a[q]);
        }
        if (lane == 0) {
            proj[3 * i + 0] = a[0];
            proj[3 * i + 1] = a[1];
            proj[3 * i + 2] = a[2];
        }
    }
    if (lane == 0)
        for (int q = 0; q < 3; q++) {
            red[w][q] = mn[q];
            red[w][3 + q] = mx[q];
        }
    __syncthreads();
    if (threadIdx.x < 6) {
        const int q = threadIdx.x;
        float v = red[0][q];
        for (int k = 1; k < 4; k++) v = q < 3 ? fminf(v, red[k][q]) : fmaxf(v, red[k][q]);
        part[6 * blockIdx.x + q] = v;
    }
}

__device__ __forceinline__ uint32_t spread3(uint32_t v) {     // 10 bits -> every third bit
    v &= 0x3FFu;
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

__global__ __launch_bounds__(256) void k_project_keys(const float* __restrict__ proj, int64_t n,
                                                      const float* __restrict__ part, int nb,
                                                      uint32_t* __restrict__ keys) {
    __shared__ float lo[3], hi[3];
    if (threadIdx.x < 3) {
        float a = INFINITY, b = -INFINITY;
        for (int k = 0; k < nb; k++) {
            a = fminf(a, part[6 * k + threadIdx.x]);
            b = fmaxf(b, part[6 * k + 3 + threadIdx.x]);
        }
        lo[threadIdx.x] = a;
        hi[threadIdx.x] = b;
    }
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    uint32_t code = 0;
#pragma unroll
    for (int q = 0; q < 3; q++) {
        const float span = hi[q] - lo[q];
        float f = span > 0.f ? (proj[3 * i + q] - lo[q]) / span * 1024.f : 0.f;
        f = f < 0.f ? 0.f : (f > 1023.f ? 1023.f : f);
        code |= spread3((uint32_t)f) << q;
    }
    keys[i] = code;
}

}  // namespace

hipError_t projection_keys(const void* X, int64_t n, int32_t D, int32_t x_dtype, uint32_t* keys,
                           hipStream_t s) {
    const int nb = (int)(ceil_div(n, 4) < 1024 ? ceil_div(n, 4) : 1024);
    float *proj = nullptr, *part = nullptr;
    hipError_t e = hipMalloc(&proj, sizeof(float) * 3 * (size_t)n);
    if (e == hipSuccess) e = hipMalloc(&part, sizeof(float) * 6 * (size_t)nb);
    if (e == hipSuccess) {
        switch (x_dtype) {
            case PSNE_X_F32:
                k_project<float><<<nb, 256, 0, s>>>((const float*)X, n, D, proj, part);
                break;
            case PSNE_X_F64:
                k_project<double><<<nb, 256, 0, s>>>((const double*)X, n, D, proj, part);
                break;
            default:
                k_project<uint8_t><<<nb, 256, 0, s>>>((const uint8_t*)X, n, D, proj, part);
                break;
        }
        k_project_keys<<<dim3((unsigned)ceil_div(n, 256)), 256, 0, s>>>(proj, n, part, nb, keys);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipFree(proj);
    (void)hipFree(part);
    return e;
}

hipError_t scan_i64(const int64_t* a, int64_t m, int64_t* out, int64_t* tmp, hipStream_t s) {
    return scan_i64_local(a, m, out, tmp, s);
}

int64_t scan_i64_tmp_len(int64_t m) { return ceil_div(m, 1024) + 1; }

hipError_t knn(const void* X, int64_t n, int32_t D, int32_t x_dtype, int32_t k, int32_t* idx,
               double* d2, hipStream_t s, std::string* err) {
    switch (x_dtype) {
        case PSNE_X_F32: return knn_typed<float>((const float*)X, n, D, k, idx, d2, s, err);
        case PSNE_X_F64: return knn_typed<double>((const double*)X, n, D, k, idx, d2, s, err);
        case PSNE_X_U8: return knn_typed<uint8_t>((const uint8_t*)X, n, D, k, idx, d2, s, err);
        default: return hipErrorInvalidValue;
    }
}

hipError_t perplexity(const double* d2, int64_t n, int32_t k, double u, double* P, double* beta,
                      hipStream_t s) {
    const double target = log(u);
    // a grid holds fewer than 2^32 threads, up to 64 of them to a row
    constexpr int64_t kRun = (int64_t)1 << 22;
    for (int64_t r0 = 0; r0 < n; r0 += kRun) {
        const int64_t m = n - r0 < kRun ? n - r0 : kRun;
        const double* d = d2 + r0 * k;
        double *p = P + r0 * k, *b = beta ? beta + r0 : nullptr;
        auto run = [&](auto w, auto held) {
            constexpr int W = decltype(w)::value, HELD = decltype(held)::value;
            k_perplexity<W, HELD><<<dim3((unsigned)ceil_div(m, 256 / W)), 256, 0, s>>>(
                d, m, k, target, 1e-5, 200, p, b);
        };
        auto by4 = [&](auto w) { run(w, std::integral_constant<int, 4>()); };
        if (k <= 4) by4(std::integral_constant<int, 1>());
        else if (k <= 8) by4(std::integral_constant<int, 2>());
        else if (k <= 16) by4(std::integral_constant<int, 4>());
        else if (k <= 32) by4(std::integral_constant<int, 8>());
        else if (k <= 64) by4(std::integral_constant<int, 16>());
        else if (k <= 128) by4(std::integral_constant<int, 32>());
        else if (k <= 256) by4(std::integral_constant<int, 64>());
        else run(std::integral_constant<int, 64>(), std::integral_constant<int, 0>());
    }
    return hipGetLastError();
}

hipError_t symmetrize(const int32_t* idx, const double* Pc, int64_t n, int32_t k,
                      int64_t** row_ptr_out, uint32_t** col_out, double** val_out, int64_t* nnz_out,
                      hipStream_t s) {
    const int64_t m = n * (int64_t)k;
    // edge numbers are 32 bits: 2^32 edges need 155 GB here and 86 GB for the
    // lists they come from
    if (m >= ((int64_t)1 << 32)) return hipErrorOutOfMemory;
    uint32_t *key[2] = {nullptr, nullptr}, *edge[2] = {nullptr, nullptr};
    uint32_t *hist = nullptr, *dtot = nullptr, *col = nullptr;
    int64_t *start = nullptr, *tmp = nullptr, *ucnt = nullptr, *rp = nullptr;
    double* val = nullptr;
    hipError_t e = hipSuccess;
    Arena own;
    auto fail = [&](hipError_t x) {
        own.release();
        (void)hipFree(rp); (void)hipFree(col); (void)hipFree(val);
        return x;
    };
    int bits = 1, at = 0;
    while (((int64_t)1 << bits) < n) bits++;
    for (int h = 0; h < 2; h++) {
        own.add(&key[h], m);
        own.add(&edge[h], m);
    }
    own.add(&hist, sort_hist_words(m, bits));
    own.add(&dtot, sort_digit_words());
    own.add(&start, n + 1);
    own.add(&tmp, scan_i64_tmp_len(n + 1));
    own.add(&ucnt, n + 1);
    if ((e = own.make()) != hipSuccess) return fail(e);
    if ((e = hipMalloc(&rp, 8 * (n + 1))) != hipSuccess) return fail(e);
    if ((e = hipMemcpyAsync(key[0], idx, 4 * m, hipMemcpyDeviceToDevice, s)) != hipSuccess)
        return fail(e);
    if ((e = sort_pairs32(key, edge, m, bits, hist, dtot, s, &at)) != hipSuccess) return fail(e);
    k_in_start<<<dim3((unsigned)ceil_div(m + 1, 256)), 256, 0, s>>>(key[at], m, n, start);
    k_sym_count<<<dim3((unsigned)ceil_div(n + 1, 4)), 256, 0, s>>>(idx, start, edge[at], n, k, ucnt);
    if ((e = scan_i64_local(ucnt, n + 1, rp, tmp, s)) != hipSuccess) return fail(e);
    int64_t nnz = 0;
    if ((e = hipMemcpyAsync(&nnz, rp + n, 8, hipMemcpyDeviceToHost, s)) != hipSuccess) return fail(e);
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return fail(e);
    if ((e = hipMalloc(&col, 4 * (nnz > 0 ? nnz : 1))) != hipSuccess) return fail(e);
    if ((e = hipMalloc(&val, 8 * (nnz > 0 ? nnz : 1))) != hipSuccess) return fail(e);
    // a grid holds fewer than 2^32 threads
    constexpr int64_t kRun = (int64_t)1 << 22;
    for (int64_t i = 0; i < n; i += kRun)
        k_sym_row<<<dim3((unsigned)std::min(kRun, n - i)), 256, 0, s>>>(
            i, idx, Pc, start, edge[at], k, rp, 1.0 / (2.0 * (double)n), col, val);
    if ((e = hipGetLastError()) != hipSuccess) return fail(e);
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return fail(e);
    own.release();
    *row_ptr_out = rp;
    *col_out = col;
    *val_out = val;
    *nnz_out = nnz;
    return hipSuccess;
}

}  // namespace psne

// For the tests, which cannot see from the lists whether tiles were left out.
extern "C" void psne_knn_trace(int64_t* groups, int64_t* met, int64_t* all) {
    *groups = psne::g_trace.groups;
    *met = psne::g_trace.met;
    *all = psne::g_trace.all;
}
