// Embedding quality: the k nearest neighbours of every point in the 2-D
// embedding and the neighbourhood precision of Eq. (14),
//   (1 / kN) sum_i |N_D^(k)(i) intersect N_d^(k)(i)|,
// with N_D the high-dimensional neighbours (an input) and N_d the 2-D ones.
#include <string>
#include <vector>

#include "ctx.h"
#include "nearest.h"

namespace psne {

namespace {

constexpr int kB = 256;
constexpr int kK2 = 32;      // 2-D neighbours kept per point

// Brute-force 2-D kNN in the embedding metric d^2 = b1 dx^2 + b2 dy^2 (FP64,
// pixel frame), ties to the smaller caller index, without meeting most pairs:
// the points are sorted along a Morton curve, 64 consecutive ones form a tile
// with a bounding box, 64 tiles a group with its own, and a point meets the
// tiles whose box is no further than its 32nd best so far.  The box distance
// takes the same rounded steps as a point's and each step is monotone, so it
// never exceeds the distance of a point inside and the lists are those of all
// pairs.
constexpr int kTile = kWave;
constexpr int32_t kNoIndex = 0x7FFFFFFF;

__device__ __forceinline__ double metric(double b1, double b2, double dx, double dy) {
#pragma clang fp contract(off)
    return __builtin_fma(b1 * dx, dx, (b2 * dy) * dy);
}

// keys on a 2^16 x 2^16 grid over the screen
template <typename T>
__global__ __launch_bounds__(kB) void k_near_keys(const T* __restrict__ zh,
                                                  const DevScalars* __restrict__ sc, int64_t n,
                                                  int r, T per_pixel, uint32_t* __restrict__ key) {
    const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (i >= n) return;
    const v2_t<T> p = norm_pos<T>(zh, sc, i, r);
    key[i] = spread_bits16((uint32_t)(p.x * per_pixel)) |
             (spread_bits16((uint32_t)(p.y * per_pixel)) << 1);
}

// positions and caller indices in sorted order, the tiles' boxes
// [lo x, lo y, hi x, hi y] (a coordinate that is no number is in no box, and in
// nobody's list)
template <typename T>
__global__ __launch_bounds__(kB) void k_near_tiles(const uint32_t* __restrict__ perm,
                                                   const T* __restrict__ zh,
                                                   const DevScalars* __restrict__ sc,
                                                   const uint32_t* __restrict__ orig, int64_t n,
                                                   int r, T* __restrict__ zs,
                                                   uint32_t* __restrict__ us,
                                                   T* __restrict__ box) {
    using V = v2_t<T>;
    const int64_t s = (int64_t)blockIdx.x * kB + threadIdx.x;
    V lo = V{(T)INFINITY, (T)INFINITY}, hi = V{-(T)INFINITY, -(T)INFINITY};
    if (s < n) {
        const uint32_t i = perm[s];
        const V p = norm_pos<T>(zh, sc, i, r);
        reinterpret_cast<V*>(zs)[s] = p;
        us[s] = orig[i];
        if (p.x == p.x && p.y == p.y) lo = hi = p;
    }
    lo.x = wave_min(lo.x);
    lo.y = wave_min(lo.y);
    hi.x = wave_max(hi.x);
    hi.y = wave_max(hi.y);
    if (lane_id() == 0 && s < n) {
        V* b = reinterpret_cast<V*>(box) + 2 * (s / kTile);
        b[0] = lo;
        b[1] = hi;
    }
}

// one wavefront per 64 boxes
template <typename T>
__global__ __launch_bounds__(kWave) void k_near_groups(const T* __restrict__ box, int64_t m,
                                                       T* __restrict__ group) {
    using V = v2_t<T>;
    const int64_t t = (int64_t)blockIdx.x * kWave + threadIdx.x;
    const V* b = reinterpret_cast<const V*>(box);
    V lo = t < m ? b[2 * t] : V{(T)INFINITY, (T)INFINITY};
    V hi = t < m ? b[2 * t + 1] : V{-(T)INFINITY, -(T)INFINITY};
    lo.x = wave_min(lo.x);
    lo.y = wave_min(lo.y);
    hi.x = wave_max(hi.x);
    hi.y = wave_max(hi.y);
    if (threadIdx.x == 0) {
        V* g = reinterpret_cast<V*>(group) + 2 * (int64_t)blockIdx.x;
        g[0] = lo;
        g[1] = hi;
    }
}

// distance of a point to a box (infinite for an empty one)
template <typename T>
__device__ __forceinline__ double box_metric(const T* __restrict__ box, int64_t t, double b1,
                                             double b2, double x, double y) {
    const v2_t<T> lo = reinterpret_cast<const v2_t<T>*>(box)[2 * t];
    const v2_t<T> hi = reinterpret_cast<const v2_t<T>*>(box)[2 * t + 1];
    const double dx = fmax(fmax((double)lo.x - x, x - (double)hi.x), 0.0);
    const double dy = fmax(fmax((double)lo.y - y, y - (double)hi.y), 0.0);
    return metric(b1, b2, dx, dy);
}

__device__ __forceinline__ double lane_double(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// One wavefront per point, one candidate per lane.  Lanes 0..31 hold the best
// 32 in order.  Candidates that would enter gather in LDS and are sorted in by
// the 64 (bitonic), which a point pays a few times, where a list per lane was
// shifted in registers at every entry of any of 64 points, by 940 wavefronts
// at 60,000 points.  The caller's rows are written whole.  60,000 points,
// late layout: 0.3 ms where all pairs took 40.9.
template <typename T>
__global__ __launch_bounds__(kB) void k_knn2d(const T* __restrict__ zs,
                                              const uint32_t* __restrict__ us,
                                              const T* __restrict__ box,
                                              const T* __restrict__ group,
                                              const DevScalars* __restrict__ sc, int64_t first,
                                              int64_t n, int32_t* __restrict__ out) {
    __shared__ double pend_d[kB / kWave][kWave];
    __shared__ int32_t pend_j[kB / kWave][kWave];
    const int lane = lane_id(), w = threadIdx.x >> 6;
    const int64_t s =
        first + (int64_t)blockIdx.x * (kB / kWave) + __builtin_amdgcn_readfirstlane(w);
    if (s >= n) return;                         // no barrier below
    const double s0 = sc->s[0], s1 = sc->s[1];
    const double b1 = s0 * s0, b2 = s1 * s1;
    const v2_t<T> p = reinterpret_cast<const v2_t<T>*>(zs)[s];
    const double x = (double)p.x, y = (double)p.y;
    double bd = INFINITY;                       // the list: lanes 0..31
    int32_t bj = kNoIndex;
    double worst = INFINITY;                    // its last entry
    int32_t worst_j = kNoIndex;
    int np = 0;                                 // candidates gathered

    auto merge = [&]() {
        __builtin_amdgcn_wave_barrier();
        double d = lane < np ? pend_d[w][lane] : INFINITY;
        int32_t j = lane < np ? pend_j[w][lane] : kNoIndex;
        __builtin_amdgcn_wave_barrier();
        wave_sort(d, j);
        // the list ascending below, the 32 best candidates descending above:
        // a bitonic sequence, whose lower half after one exchange holds the
        // 32 best of both
        const double rd = __shfl(d, 63 - lane, kWave);
        const int32_t rj = __shfl(j, 63 - lane, kWave);
        if (lane >= kK2) {
            bd = rd;
            bj = rj;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double od = __shfl_xor(bd, o, kWave);
            const int32_t oj = __shfl_xor(bj, o, kWave);
            const bool low = (lane & o) == 0;
            if (low ? knn_less(od, oj, bd, bj) : knn_less(bd, bj, od, oj)) {
                bd = od;
                bj = oj;
            }
        }
        worst = lane_double(bd, kK2 - 1);
        worst_j = __builtin_amdgcn_readlane(bj, kK2 - 1);
        np = 0;
    };
    auto meet = [&](int64_t t) {
        const int64_t q = t * kTile + lane;
        double d = INFINITY;
        int32_t j = kNoIndex;
        if (q < n && q != s) {
            const v2_t<T> c = reinterpret_cast<const v2_t<T>*>(zs)[q];
            d = metric(b1, b2, x - (double)c.x, y - (double)c.y);
            j = (int32_t)us[q];
        }
        bool in = j != kNoIndex && knn_less(d, j, worst, worst_j);
        uint64_t b = ballot64(in);
        if (b == 0) return;
        if (np + __popcll(b) > kWave) {
            merge();
            in = in && knn_less(d, j, worst, worst_j);
            b = ballot64(in);
        }
        if (in) {
            const int at = np + __popcll(b & lanemask_lt());
            pend_d[w][at] = d;
            pend_j[w][at] = j;
        }
        np += __popcll(b);
    };

    const int64_t tiles = (n + kTile - 1) / kTile, groups = (tiles + kWave - 1) / kWave;
    const int64_t own = s / kTile;
    meet(own);
    if (own > 0) meet(own - 1);
    if (own + 1 < tiles) meet(own + 1);
    merge();
    for (int64_t g0 = 0; g0 < groups; g0 += kWave) {
        const double gl = g0 + lane < groups ? box_metric(group, g0 + lane, b1, b2, x, y) : INFINITY;
        uint64_t gm = ballot64(!(gl > worst) && g0 + lane < groups);
        while (gm) {
            const int a = __ffsll((long long)gm) - 1;
            gm &= gm - 1;
            if (lane_double(gl, a) > worst) continue;
            const int64_t t = (g0 + a) * kWave + lane;
            const double tl = t < tiles ? box_metric(box, t, b1, b2, x, y) : INFINITY;
            uint64_t tm = ballot64(t < tiles && !(tl > worst) && (t > own + 1 || t + 1 < own));
            while (tm) {
                const int c = __ffsll((long long)tm) - 1;
                tm &= tm - 1;
                if (!(lane_double(tl, c) > worst)) meet((g0 + a) * kWave + c);
            }
        }
    }
    if (np > 0) merge();
    if (lane < kK2) out[(int64_t)us[s] * kK2 + lane] = bj == kNoIndex ? -1 : bj;
}

// per-point overlap counts for each requested k, summed per block
__global__ __launch_bounds__(kB) void k_overlap(const int32_t* __restrict__ hi, int k_hi,
                                                const int32_t* __restrict__ lo, int64_t n,
                                                const int32_t* __restrict__ ks, int nk,
                                                unsigned long long* __restrict__ part) {
    __shared__ unsigned long long red[kB];
    const int64_t u = (int64_t)blockIdx.x * kB + threadIdx.x;
    for (int q = 0; q < nk; q++) {
        const int k = ks[q];
        unsigned long long c = 0;
        if (u < n) {
            for (int a = 0; a < k; a++) {
                const int32_t h = hi[u * k_hi + a];
                for (int b = 0; b < k; b++) c += (lo[u * kK2 + b] == h) ? 1ull : 0ull;
            }
        }
        red[threadIdx.x] = c;
        __syncthreads();
        for (int o = kB / 2; o > 0; o >>= 1) {
            if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
            __syncthreads();
        }
        if (threadIdx.x == 0) part[(int64_t)blockIdx.x * nk + q] = red[0];
        __syncthreads();
    }
}

// The sorted points, their tiles' and groups' boxes live in the context's
// buffers for the renumbering, which hold nothing between calls.
template <typename T>
hipError_t knn2d_typed(const pixelsne_ctx* c, int32_t* out) {
    const int64_t n = c->n, tiles = ceil_div(n, kTile), groups = ceil_div(tiles, kWave);
    const dim3 g((unsigned)ceil_div(n, kB));
    uint32_t* const key[2] = {(uint32_t*)c->len_tmp, (uint32_t*)c->len_tmp + n};
    uint32_t* const idx[2] = {(uint32_t*)c->ch_tmp, (uint32_t*)c->ch_tmp + n};
    T *zs = (T*)c->zh2, *box = (T*)c->u2, *group = (T*)c->g2;
    uint32_t* us = c->orig2;
    k_near_keys<T><<<g, kB, 0, c->stream>>>((const T*)c->zh, c->sc, n, c->r,
                                            (T)(65536.0 / c->r), key[0]);
    int sorted = 0;
    hipError_t e = sort_pairs32(key, idx, n, 32, c->tb.hist, c->tb.dtot, c->stream, &sorted);
    if (e != hipSuccess) return e;
    k_near_tiles<T><<<g, kB, 0, c->stream>>>(idx[sorted], (const T*)c->zh, c->sc, c->orig, n, c->r,
                                             zs, us, box);
    k_near_groups<T><<<dim3((unsigned)groups), kWave, 0, c->stream>>>(box, tiles, group);
    // a grid holds fewer than 2^32 threads, 64 of them to a point
    constexpr int64_t kRun = (int64_t)1 << 20;
    for (int64_t s0 = 0; s0 < n; s0 += kRun)
        k_knn2d<T><<<dim3((unsigned)ceil_div(n - s0 < kRun ? n - s0 : kRun, kB / kWave)), kB, 0,
                     c->stream>>>(zs, us, box, group, c->sc, s0, n, out);
    return hipGetLastError();
}

hipError_t knn2d(const pixelsne_ctx* c, int32_t* out) {
    return c->prm.precision == PSNE_FP64 ? knn2d_typed<double>(c, out)
                                         : knn2d_typed<float>(c, out);
}

}  // namespace
}  // namespace psne

using namespace psne;

extern "C" {

psne_status pixelsne_knn2d(const pixelsne_ctx* c, int32_t* idx) {
    if (!c || !is_device_ptr(idx)) { set_error("knn2d: null context or non-device output"); return PSNE_E_INVAL; }
    if (c->n - 1 < kK2) { set_error("knn2d needs n > 32"); return PSNE_E_UNSUPPORTED; }
    hipError_t e = knn2d(c, idx);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return device_error(const_cast<pixelsne_ctx*>(c), e, "knn2d");
    return PSNE_OK;
}

psne_status pixelsne_neighborhood_precision(const pixelsne_ctx* c, const int32_t* hi_knn,
                                            int32_t k_hi, const int32_t* ks, int32_t nk,
                                            double* out) {
    if (!c || !is_device_ptr(hi_knn) || !ks || !out || nk < 1 || nk > 64 || k_hi < 1) {
        set_error("neighborhood_precision: bad arguments");
        return PSNE_E_INVAL;
    }
    for (int q = 0; q < nk; q++)
        if (ks[q] < 1 || ks[q] > k_hi || ks[q] > kK2) {
            set_error("neighborhood_precision: every k must be in [1, min(k_hi, 32)]");
            return PSNE_E_INVAL;
        }
    if (c->n - 1 < kK2) { set_error("neighborhood_precision needs n > 32"); return PSNE_E_UNSUPPORTED; }
    const int64_t nb = ceil_div(c->n, kB);
    int32_t *lo = nullptr, *kd = nullptr;
    unsigned long long* part = nullptr;
    hipError_t e = hipMalloc(&lo, sizeof(int32_t) * (size_t)c->n * kK2);
    if (e == hipSuccess) e = hipMalloc(&kd, sizeof(int32_t) * nk);
    if (e == hipSuccess) e = hipMalloc(&part, sizeof(unsigned long long) * (size_t)nb * nk);
    if (e == hipSuccess) e = hipMemcpyAsync(kd, ks, sizeof(int32_t) * nk, hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = knn2d(c, lo);
    if (e == hipSuccess) {
        k_overlap<<<dim3((unsigned)nb), kB, 0, c->stream>>>(hi_knn, k_hi, lo, c->n, kd, nk, part);
        e = hipGetLastError();
    }
    std::vector<unsigned long long> h((size_t)nb * nk);
    if (e == hipSuccess)
        e = hipMemcpyAsync(h.data(), part, h.size() * sizeof(unsigned long long),
                           hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    (void)hipFree(lo); (void)hipFree(kd); (void)hipFree(part);
    if (e != hipSuccess) return device_error(const_cast<pixelsne_ctx*>(c), e, "neighborhood_precision");
    for (int q = 0; q < nk; q++) {
        unsigned long long s = 0;
        for (int64_t b = 0; b < nb; b++) s += h[(size_t)b * nk + q];
        out[q] = (double)s / ((double)ks[q] * (double)c->n);
    }
    return PSNE_OK;
}

}  // extern "C"
