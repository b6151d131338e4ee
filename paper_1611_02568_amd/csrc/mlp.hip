// Learned placement network on gfx950: Linear-GELU-Linear-GELU-Linear(2),
// trained with the mean squared error against screen positions z / r of a
// converged embedding.  Matrix products use bfloat16 operands on the MFMA
// units (v_mfma_f32_16x16x32_bf16) with FP32 accumulation; master weights and
// Adam moments are FP32.  The 2-wide output layer runs on the vector units.
//
// Cast points (operands rounded to bfloat16, round to nearest even):
//   forward   X^, W1 | H1, W2 | H2, W3
//   backward  dA2, H1, W2 (dW2, dH1) and dA1, X^ (dW1); the head uses H2, W3.
//
// Every operand of a matrix product lies in memory as the MFMA units take it,
// in fragments of 16 rows by 32 of the reduction (512 elements, 16 bytes per
// lane, in lane order): an operand's fragments move to LDS by loads straight
// into it and are read without bank conflicts.  The kernel that computes a
// matrix writes it in the order of each product that reads it: X^, H1, dA2
// by rows (reduction along the columns) and by columns (reduction along the
// batch), dA1 by columns, the weights after each step.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <random>
#include <string>
#include <vector>

#include "ctx.h"

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

struct pixelsne_mlp {
    int32_t d = 0, h1 = 0, h2 = 0;
    int64_t n_params = 0;
    hipStream_t stream = nullptr;
    uint64_t seed = 0;
    int64_t step = 0;                   // Adam step count
    int64_t cap_batch = 0;              // rows the work buffers hold
    float* theta = nullptr;             // FP32 master parameters (flat)
    float* m1 = nullptr;                // Adam first moment
    float* m2 = nullptr;                // Adam second moment
    uint16_t* w1p = nullptr;            // W1: fragments of rows h1, reduction d
    uint16_t* w2p = nullptr;            // W2: rows h2, reduction h1 (forward)
    uint16_t* w2q = nullptr;            // W2: rows h1, reduction h2 (backward)
    uint16_t* w3b = nullptr;            // W3 [h2][2]
    float* mean = nullptr;              // input standardisation
    float* inv_std = nullptr;
    // work buffers of a forward pass (rows padded to whole tiles)
    uint16_t* xp = nullptr;             // X^: rows batch, reduction d
    uint16_t* h1p = nullptr;            // H1: rows batch, reduction h1
    uint16_t* h2b = nullptr;            // H2 [B][h2]
    int64_t cap_train = 0;              // rows the training buffers hold
    int64_t train_steps = 0;            // depth steps of the batch they are laid out for
    uint16_t* xq = nullptr;             // X^: rows d, reduction batch
    uint16_t* h1q = nullptr;            // H1: rows h1, reduction batch
    uint16_t* da2p = nullptr;           // dA2: rows batch, reduction h2
    uint16_t* da2q = nullptr;           // dA2: rows h2, reduction batch
    uint16_t* da1q = nullptr;           // dA1: rows h1, reduction batch
    float* yb = nullptr;                // targets [B][2]
    float* a1 = nullptr;                // pre-activations [B][h1], [B][h2]
    float* a2 = nullptr;
    float* dout = nullptr;              // [B][2]
    float* da2 = nullptr;               // [B][h2]
    float* da1 = nullptr;               // [B][h1]
    float* splitk = nullptr;            // split-K partials
    int64_t splitk_len = 0;
    float* part = nullptr;              // row-slice partial sums of the batch reductions
    double* lossbuf = nullptr;          // loss partials, one per four rows
    int64_t lossbuf_len = 0;
    uint32_t* order = nullptr;          // batch row order (device)
    int64_t order_len = 0;
    std::vector<void*> allocs;
};

namespace psne {
namespace {

constexpr int kT = 256;
constexpr int64_t kForwardRows = 32768;

__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ float gelu_f(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float x) {
    return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) +
           x * expf(-0.5f * x * x) * 0.39894228040143268f;
}

constexpr int kXcds = 8;
constexpr int kFrag = 512;                     // elements of a fragment
constexpr int kTileRows = 128;                 // rows of an operand are padded to this

// depth steps (of 32) of a reduction, padded to whole stages of two
__host__ __device__ inline int depth_steps(int64_t k) { return 2 * (int)((k + 63) / 64); }
inline int64_t pad_tile(int64_t r) { return ceil_div(r, kTileRows) * kTileRows; }
inline int64_t frag_elems(int64_t rows, int64_t k) { return pad_tile(rows) * depth_steps(k) * 32; }

// element (r, k) of an operand with `steps` depth steps
__device__ __forceinline__ int64_t frag_at(int64_t r, int k, int steps) {
    return ((r >> 4) * steps + (k >> 5)) * kFrag + (((r & 15) + 16 * ((k & 31) >> 3)) << 3) +
           (k & 7);
}

// rows of an operand that exist in memory
__device__ __forceinline__ int pad_cols(int r) { return (r + kTileRows - 1) / kTileRows * kTileRows; }

// C[n][m] = sum_k B[n][k] A[m][k] over the depth steps step0 .. step0 + n_steps of
// the operands' sa and sb, for a TM x TN tile at row fragments ma and nb, by
// WM x WN wavefronts.  Stages of KS steps, the next one in flight while one is
// multiplied.  Lane l ends with the elements m = l % 16, n = 4 (l / 16) + 0..3
// of each 16 x 16 tile, so four consecutive columns of one row.  The depth runs
// in instructions of 32 in ascending order, whatever the tile.
template <int TM, int TN, int WM, int WN, int KS>
struct Tile {
    static constexpr int kWaves = WM * WN;
    static constexpr int kA = TM / 16, kB = TN / 16;        // fragments per step
    static constexpr int kLds = 2 * KS * (kA + kB) * kFrag; // elements, two stages
    static constexpr int kMi = TM / WM / 16, kNj = TN / WN / 16;   // a wavefront's
    static_assert(KS * (kA + kB) % kWaves == 0, "every wavefront loads as many fragments");
    v4f acc[kNj][kMi];

    __device__ __forceinline__ void run(const uint16_t* __restrict__ A, int sa, int64_t ma,
                                        const uint16_t* __restrict__ B, int sb, int64_t nb,
                                        int step0, int n_steps, uint16_t* lds) {
        const int t = threadIdx.x, lane = t & 63;
        const int w = __builtin_amdgcn_readfirstlane(t >> 6);
        const int wm = w / WN, wn = w % WN;
#pragma unroll
        for (int j = 0; j < kNj; j++)
#pragma unroll
            for (int i = 0; i < kMi; i++) acc[j][i] = v4f{0.f, 0.f, 0.f, 0.f};
        const int stages = (n_steps + KS - 1) / KS, end = step0 + n_steps;
        // a stage holds [A fragments][KS steps], then B's; wavefront w loads
        // fragments w, w + kWaves, ...
        auto fetch = [&](int st, int buf) {
            uint16_t* to = lds + buf * (kLds / 2);
            const int s = step0 + KS * st;
#pragma unroll
            for (int y = 0; y < KS * (kA + kB) / kWaves; y++) {
                const int x = w + kWaves * y, f = x / KS;
                const int q = s + x % KS < end ? s + x % KS : end - 1;     // an odd last stage
                const uint16_t* src = f < kA ? A + ((ma + f) * sa + q) * kFrag
                                             : B + ((nb + (f - kA)) * sb + q) * kFrag;
                __builtin_amdgcn_global_load_lds(
                    (__attribute__((address_space(1))) const void*)(src + 8 * lane),
                    (__attribute__((address_space(3))) void*)(to + x * kFrag), 16, 0, 0);
            }
        };
        auto settle = [&]() {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
        };
        auto step = [&](const uint16_t* from, int h) {
            v8bf a[kMi], b[kNj];
#pragma unroll
            for (int i = 0; i < kMi; i++)
                a[i] = *reinterpret_cast<const v8bf*>(from + ((wm * kMi + i) * KS + h) * kFrag +
                                                      8 * lane);
#pragma unroll
            for (int j = 0; j < kNj; j++)
                b[j] = *reinterpret_cast<const v8bf*>(from + ((kA + wn * kNj + j) * KS + h) * kFrag +
                                                      8 * lane);
#pragma unroll
            for (int j = 0; j < kNj; j++)
#pragma unroll
                for (int i = 0; i < kMi; i++)
                    acc[j][i] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[j][i], 0, 0, 0);
        };
        fetch(0, 0);
        settle();
        for (int st = 0; st < stages; st++) {
            const int buf = st & 1;
            if (st + 1 < stages) fetch(st + 1, buf ^ 1);
            const uint16_t* from = lds + buf * (kLds / 2);
            step(from, 0);
            if (KS == 2 && 2 * st + 1 < n_steps) step(from, 1);
            settle();
        }
    }

    // fn(mf, nf, values) for every 16 x 16 tile, mf and nf its (uniform) place in
    // units of 16; the lane's four elements are row 16 mf + lane_m(), columns
    // 16 nf + lane_n() + 0..3
    template <typename Fn>
    __device__ __forceinline__ void each(int64_t m0, int n0, Fn&& fn) const {
        const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        const int wm = w / WN, wn = w % WN;
#pragma unroll
        for (int j = 0; j < kNj; j++)
#pragma unroll
            for (int i = 0; i < kMi; i++)
                fn(m0 / 16 + wm * kMi + i, n0 / 16 + wn * kNj + j, acc[j][i]);
    }
};
__device__ __forceinline__ int lane_m() { return threadIdx.x & 15; }
__device__ __forceinline__ int lane_n() { return 4 * ((threadIdx.x & 63) >> 4); }

// A lane's four elements of tile (mf, nf): to fragments by rows (one 8-byte
// store), and by columns (a 2-byte store each; 16 lanes fill two 16-byte
// pieces).
__device__ __forceinline__ void put_rows(uint16_t* __restrict__ P, int steps, int64_t mf, int nf,
                                         const uint16_t* h) {
    const int n = 16 * (nf & 1) + lane_n();
    uint16_t* base = P + (mf * steps + (nf >> 1)) * kFrag;
    *reinterpret_cast<uint2*>(base + ((lane_m() + 16 * (n >> 3)) << 3) + (n & 7)) =
        uint2{(uint32_t)h[0] | (uint32_t)h[1] << 16, (uint32_t)h[2] | (uint32_t)h[3] << 16};
}
__device__ __forceinline__ void put_cols(uint16_t* __restrict__ Q, int steps, int64_t mf, int nf,
                                         const uint16_t* h) {
    const int k = 16 * (int)(mf & 1) + lane_m();
    uint16_t* base = Q + ((int64_t)nf * steps + (mf >> 1)) * kFrag + ((16 * (k >> 3)) << 3) + (k & 7);
#pragma unroll
    for (int e = 0; e < 4; e++) base[(lane_n() + e) << 3] = h[e];
}

// and to a row-major matrix of N columns
template <typename V, typename E>
__device__ __forceinline__ void put_flat(E* __restrict__ C, int64_t m, int n, int M, int N,
                                         const E* v) {
    E* p = C + m * N + n;
    if (N % 4 == 0) {
        if (m < M && n < N) *reinterpret_cast<V*>(p) = *reinterpret_cast<const V*>(v);
    } else {
#pragma unroll
        for (int e = 0; e < 4; e++)
            if (m < M && n + e < N) p[e] = v[e];
    }
}

// Blocks b, b + 8, ... share an L2 (blocks go round the XCDs): those of one XCD
// take all column tiles of one row tile before the next row tile, so that a row
// tile of A is read once per chip and B stays in each L2.

// A layer: H = gelu(A B^T + bias) for M rows and N columns.  pre (training):
// the pre-activations [M][N]; rowsP / colsQ / flat: where H goes.  Rows past M
// and columns past N become zeros in the fragments.  What bounds it is GELU
// (erff is 40 vector instructions per element, on both sides of a branch) and
// the latency of the short depth loop, so wavefronts per CU count for more than
// LDS traffic.  A million rows of two 1,024-wide layers, all kernels: tiles of
// 128 x 128 with four wavefronts and stages of two steps 9.4 ms, with eight 7.2,
// with stages of one step (half the LDS) 6.4, in the order above 5.8.  One layer
// of 32,768 rows takes 77 us; all layers together 4.8 ms, where products of
// row-major operands took 17.3.
template <int TM, int TN, int WM, int WN, int KS>
__global__ __launch_bounds__(64 * WM * WN) void k_layer(const uint16_t* __restrict__ A,
                                                        const uint16_t* __restrict__ B, int steps,
                                                        int M, int N,
                                                        const float* __restrict__ bias,
                                                        float* __restrict__ pre,
                                                        uint16_t* __restrict__ rowsP,
                                                        uint16_t* __restrict__ colsQ, int sq,
                                                        uint16_t* __restrict__ flat) {
    using T = Tile<TM, TN, WM, WN, KS>;
    __shared__ __attribute__((aligned(16))) uint16_t lds[T::kLds];
    const int nt = (N + TN - 1) / TN, q = (int)blockIdx.x / kXcds;
    const int64_t m0 = ((int64_t)(q / nt) * kXcds + blockIdx.x % kXcds) * TM;
    const int n0 = q % nt * TN, sp = depth_steps(N);
    if (m0 >= 32 * (int64_t)depth_steps(M)) return;
    T c;
    c.run(A, steps, m0 / 16, B, steps, n0 / 16, 0, steps, lds);
    c.each(m0, n0, [&](int64_t mf, int nf, const v4f& v) {
        const int64_t m = 16 * mf + lane_m();
        const int n = 16 * nf + lane_n();
        __attribute__((aligned(16))) float a[4];
        __attribute__((aligned(8))) uint16_t h[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const bool in = m < M && n + e < N;
            a[e] = v[e] + (in ? bias[n + e] : 0.f);
            h[e] = in ? f2bf(gelu_f(a[e])) : (uint16_t)0;
        }
        if (pre) put_flat<float4>(pre, m, n, M, N, a);
        if (flat) put_flat<uint2>(flat, m, n, M, N, h);
        if (nf < 2 * sp) {
            if (rowsP) put_rows(rowsP, sp, mf, nf, h);
            if (colsQ && mf < 2 * sq) put_cols(colsQ, sq, mf, nf, h);
        }
    });
}

// dA = (A B^T) * gelu'(pre): M rows, N columns; FP32 [M][N] and by columns
template <int TM, int TN, int WM, int WN, int KS>
__global__ __launch_bounds__(64 * WM * WN) void k_layer_back(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ B, int steps, int M, int N,
    const float* __restrict__ pre, float* __restrict__ da, uint16_t* __restrict__ colsQ, int sq) {
    using T = Tile<TM, TN, WM, WN, KS>;
    __shared__ __attribute__((aligned(16))) uint16_t lds[T::kLds];
    const int nt = (N + TN - 1) / TN, q = (int)blockIdx.x / kXcds;
    const int64_t m0 = ((int64_t)(q / nt) * kXcds + blockIdx.x % kXcds) * TM;
    const int n0 = q % nt * TN;
    if (m0 >= 32 * (int64_t)sq) return;
    T c;
    c.run(A, steps, m0 / 16, B, steps, n0 / 16, 0, steps, lds);
    c.each(m0, n0, [&](int64_t mf, int nf, const v4f& v) {
        const int64_t m = 16 * mf + lane_m();
        const int n = 16 * nf + lane_n();
        __attribute__((aligned(16))) float d[4];
        uint16_t h[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const bool in = m < M && n + e < N;
            d[e] = in ? v[e] * gelu_grad_f(pre[m * N + n + e]) : 0.f;
            h[e] = f2bf(d[e]);
        }
        put_flat<float4>(da, m, n, M, N, d);
        if (mf < 2 * sq && 16 * nf < pad_cols(N)) put_cols(colsQ, sq, mf, nf, h);
    });
}

// X^ rows of a batch: standardise, round to bfloat16.  A wavefront writes one
// fragment, a lane eight consecutive features of one row (16 bytes), so that
// reads are 128-byte runs of 16 rows and writes 1 KiB in a row.  wide: the
// rows of X begin on 16 bytes.  32,768 rows of 100 take 7 us; with a row's
// pieces in consecutive lanes, whose writes lie 256 bytes apart, 20.
__global__ __launch_bounds__(kT) void k_stage_x(const float* __restrict__ X, int d, int steps,
                                                int64_t b0, int Bn, int64_t rows, bool wide,
                                                const float* __restrict__ mean,
                                                const float* __restrict__ inv_std,
                                                uint16_t* __restrict__ xp) {
    const int64_t f = (int64_t)blockIdx.x * (kT / 64) + (threadIdx.x >> 6);
    if (f >= rows / 16 * steps) return;
    const int lane = threadIdx.x & 63;
    const int64_t r = 16 * (f / steps) + (lane & 15);
    const int c0 = 32 * (int)(f % steps) + 8 * (lane >> 4);
    union {
        uint4 q;
        uint16_t h[8];
    } v;
    __attribute__((aligned(16))) float x[8];
    const float* row = X + (b0 + r) * d + c0;
    if (wide && r < Bn && c0 + 8 <= d) {
        *reinterpret_cast<float4*>(x) = *reinterpret_cast<const float4*>(row);
        *reinterpret_cast<float4*>(x + 4) = *reinterpret_cast<const float4*>(row + 4);
    } else {
#pragma unroll
        for (int e = 0; e < 8; e++) x[e] = r < Bn && c0 + e < d ? row[e] : 0.f;
    }
#pragma unroll
    for (int e = 0; e < 8; e++) {
        const int c = c0 + e;
        v.h[e] = r < Bn && c < d ? f2bf((x[e] - mean[c]) * inv_std[c]) : (uint16_t)0;
    }
    *reinterpret_cast<uint4*>(xp + f * kFrag + 8 * lane) = v.q;
}

// The same for training, in both orders, and the targets: a thread takes one
// feature of eight rows (a 16-byte piece of the order by columns).
__global__ __launch_bounds__(kT) void k_stage_train(const float* __restrict__ X, int d, int steps,
                                                    const uint32_t* __restrict__ order, int64_t b0,
                                                    int Bn, int sq, const float* __restrict__ mean,
                                                    const float* __restrict__ inv_std,
                                                    uint16_t* __restrict__ xp,
                                                    uint16_t* __restrict__ xq,
                                                    const float* __restrict__ Y,
                                                    float* __restrict__ yb) {
    const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
    const int cols = 32 * steps;
    if (i >= (int64_t)4 * sq * cols) return;
    const int64_t r0 = 8 * (i / cols);
    const int c = (int)(i % cols);
    const float mu = c < d ? mean[c] : 0.f, is = c < d ? inv_std[c] : 0.f;
    union {
        uint4 q;
        uint16_t h[8];
    } v;
#pragma unroll
    for (int e = 0; e < 8; e++) {
        const int64_t r = r0 + e;
        uint16_t h = 0;
        if (r < Bn) {
            const int64_t src = order ? order[b0 + r] : b0 + r;
            if (c < d) h = f2bf((X[src * d + c] - mu) * is);
            if (c == 0) {
                yb[r * 2] = Y[src * 2];
                yb[r * 2 + 1] = Y[src * 2 + 1];
            }
        }
        v.h[e] = h;
        xp[frag_at(r, c, steps)] = h;
    }
    if (c < pad_cols(d)) *reinterpret_cast<uint4*>(xq + frag_at(c, (int)r0, sq)) = v.q;
}

// R rows of the head, out = H2 W3 + b3, by one wavefront: lane l adds columns
// l, l + 64, ... of each.  Rows from Bn on repeat the last.
template <int R>
__device__ __forceinline__ void head_rows(const uint16_t* __restrict__ h2b, int64_t r0, int Bn,
                                          int h2, const uint16_t* __restrict__ w3b,
                                          const float* __restrict__ b3, float2* out) {
    float s0[R], s1[R];
    const uint16_t* row[R];
#pragma unroll
    for (int q = 0; q < R; q++) {
        s0[q] = s1[q] = 0.f;
        row[q] = h2b + (r0 + q < Bn ? r0 + q : Bn - 1) * h2;
    }
#pragma unroll 4
    for (int j = threadIdx.x & 63; j < h2; j += 64) {
        const float w0 = bf2f(w3b[2 * j]), w1 = bf2f(w3b[2 * j + 1]);
#pragma unroll
        for (int q = 0; q < R; q++) {
            const float h = bf2f(row[q][j]);
            s0[q] += h * w0;
            s1[q] += h * w1;
        }
    }
#pragma unroll
    for (int q = 0; q < R; q++)
        out[q] = float2{psne::wave_sum(s0[q]) + b3[0], psne::wave_sum(s1[q]) + b3[1]};
}

// Bound by the rate of its 2-byte loads, so four rows per wavefront share those
// of W3: 32,768 rows of 1,024 in 12 us, 26 with a row per wavefront.
constexpr int kPlaceRows = 4;
__global__ __launch_bounds__(kT) void k_head(const uint16_t* __restrict__ h2b, int h2,
                                             const uint16_t* __restrict__ w3b,
                                             const float* __restrict__ b3, int Bn,
                                             float* __restrict__ out) {
    const int64_t r = ((int64_t)blockIdx.x * (kT / 64) + (threadIdx.x >> 6)) * kPlaceRows;
    if (r >= Bn) return;
    float2 o[kPlaceRows];
    head_rows<kPlaceRows>(h2b, r, Bn, h2, w3b, b3, o);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int q = 0; q < kPlaceRows; q++)
            if (r + q < Bn) reinterpret_cast<float2*>(out)[r + q] = o[q];
}

// The head in training, 16 rows per block: out and the loss partials of every
// four rows, dout, then dA2 = (dout W3^T) * GELU'(A2) in FP32 and in both
// orders of the products that read it (zeros past the batch).  A wavefront per
// row, then a thread per eight elements of a column: 4,096 rows of 512 leave
// one block per CU, so its sixteen wavefronts are all there is to hide the
// latency (29 us with four wavefronts, 11 with sixteen).
constexpr int kHeadRows = 16, kHeadT = 64 * kHeadRows;

__global__ __launch_bounds__(kHeadT) void k_head_train(const uint16_t* __restrict__ h2b, int h2,
                                                   const uint16_t* __restrict__ w3b,
                                                   const float* __restrict__ b3, int Bn,
                                                   const float* __restrict__ yb,
                                                   const float* __restrict__ a2,
                                                   float* __restrict__ dout,
                                                   double* __restrict__ lossp,
                                                   float* __restrict__ da2, int sp,
                                                   uint16_t* __restrict__ da2p, int sq,
                                                   uint16_t* __restrict__ da2q) {
    __shared__ double red[kHeadRows];
    __shared__ float dl[kHeadRows][2];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t r0 = (int64_t)blockIdx.x * kHeadRows;
    const int64_t r = r0 + w;
    double l = 0.0;
    float d0 = 0.f, d1 = 0.f;
    if (r < Bn) {
        float2 o;
        head_rows<1>(h2b, r, Bn, h2, w3b, b3, &o);
        const float e0 = o.x - yb[2 * r], e1 = o.y - yb[2 * r + 1];
        d0 = 2.f * e0 / (float)Bn;
        d1 = 2.f * e1 / (float)Bn;
        l = (double)e0 * e0 + (double)e1 * e1;
    }
    if (lane == 0) {
        red[w] = l;
        dl[w][0] = d0;
        dl[w][1] = d1;
        if (r < Bn) {
            dout[2 * r] = d0;
            dout[2 * r + 1] = d1;
        }
    }
    __syncthreads();
    if (t < kHeadRows / 4 && r0 + 4 * t < Bn)
        lossp[r0 / 4 + t] = ((red[4 * t] + red[4 * t + 1]) + red[4 * t + 2]) + red[4 * t + 3];
    const int cols = pad_cols(h2);
    for (int x = t; x < 2 * cols; x += kHeadT) {
        const int j = x % cols, m0 = 8 * (x / cols);        // eight rows of one column
        const float w0 = j < h2 ? bf2f(w3b[2 * j]) : 0.f, w1 = j < h2 ? bf2f(w3b[2 * j + 1]) : 0.f;
        union {
            uint4 q;
            uint16_t h[8];
        } v;
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const int64_t r = r0 + m0 + e;
            float d = 0.f;
            if (r < Bn && j < h2) {
                const float g = dl[m0 + e][0] * w0 + dl[m0 + e][1] * w1;
                d = g * gelu_grad_f(a2[r * h2 + j]);
                da2[r * h2 + j] = d;
            }
            v.h[e] = f2bf(d);
            if (j < 32 * sp) da2p[frag_at(r, j, sp)] = v.h[e];
        }
        *reinterpret_cast<uint4*>(da2q + frag_at(j, (int)(r0 + m0), sq)) = v.q;
    }
}

// dW3[j][d] = sum_b H2[b][j] dout[b][d];  db3[d] = sum_b dout[b][d]
// Batch reductions are split into kSlices row slices: block (x, z) sums its
// slice for 64 columns (4 row phases x 64 columns, then the phases in order)
// into part[z][...]; k_sum_slices adds the slices in slice order.
constexpr int kSlices = 32;

// dW3[j][c] = sum_b H2[b][j] dout[b][c]; columns j < h2 give 2 outputs each,
// and block x == 0 also sums dout itself (db3) into part[z][2 h2 + c]
__device__ __forceinline__ void head_wgrad(const uint16_t* __restrict__ h2b, int h2,
                                           const float* __restrict__ dout, int Bn, int bx, int bz,
                                           float* __restrict__ part, float (*red)[64][3]) {
    const int t = threadIdx.x, cj = t & 63, ph = (t >> 6) & 3;
    const int j = bx * 64 + cj;
    const int per = (Bn + kSlices - 1) / kSlices;
    const int b0 = bz * per, b1 = b0 + per < Bn ? b0 + per : Bn;
    float s0 = 0.f, s1 = 0.f, d0 = 0.f, d1 = 0.f;
    for (int b = b0 + ph; b < b1; b += 4) {
        const float o0 = dout[2 * b], o1 = dout[2 * b + 1];
        if (j < h2) {
            const float h = bf2f(h2b[(int64_t)b * h2 + j]);
            s0 += h * o0;
            s1 += h * o1;
        }
        d0 += o0;
        d1 += o1;
    }
    red[ph][cj][0] = s0;
    red[ph][cj][1] = s1;
    red[ph][cj][2] = cj == 0 ? d0 : (cj == 1 ? d1 : 0.f);
    __syncthreads();
    if (ph == 0) {
        const float a0 = ((red[0][cj][0] + red[1][cj][0]) + red[2][cj][0]) + red[3][cj][0];
        const float a1 = ((red[0][cj][1] + red[1][cj][1]) + red[2][cj][1]) + red[3][cj][1];
        float* p = part + (int64_t)bz * (2 * h2 + 2);
        if (j < h2) {
            p[2 * j] = a0;
            p[2 * j + 1] = a1;
        }
        if (bx == 0 && cj < 2)
            p[2 * h2 + cj] = ((red[0][cj][2] + red[1][cj][2]) + red[2][cj][2]) + red[3][cj][2];
    }
}

// column sums over the batch (bias gradients), per row slice
__device__ __forceinline__ void column_sums(const float* __restrict__ a, int rows, int cols,
                                            int bx, int bz, float* __restrict__ part,
                                            float (*red)[64][3]) {
    const int t = threadIdx.x, cj = t & 63, ph = (t >> 6) & 3;
    const int j = bx * 64 + cj;
    const int per = (rows + kSlices - 1) / kSlices;
    const int b0 = bz * per, b1 = b0 + per < rows ? b0 + per : rows;
    float s = 0.f;
    if (j < cols)
        for (int b = b0 + ph; b < b1; b += 4) s += a[(int64_t)b * cols + j];
    red[ph][cj][0] = s;
    __syncthreads();
    if (ph == 0 && j < cols)
        part[(int64_t)bz * cols + j] =
            ((red[0][cj][0] + red[1][cj][0]) + red[2][cj][0]) + red[3][cj][0];
}

// All gradients of a batch that need nothing but dA1 and dA2, in one launch:
// the split-K partials of dW2 = H1^T dA2 and dW1 = X^T dA1, the column sums of
// dA1 and dA2 and the head's.  No part fills the chip alone, side by side they
// do: 22 us for 4,096 rows of 128-512-512.  Blocks of one batch slice share an
// L2 (every eighth block with 8 slices; its operands are 1.7 MB), and the tiles
// take sixteen wavefronts, as in the small layers.
constexpr int kGradT = 1024, kGradSlices = kGradT / 256;   // row slices of a block of sums
constexpr int kSliceBlocks = kSlices / kGradSlices;
// blocks of a launch: a grid holds fewer than 2^32 threads, which networks of a
// billion weights would pass
constexpr int64_t kGradBlocks = 1 << 15;
struct GradArgs {
    const uint16_t *h1q, *da2q, *xq, *da1q, *h2b;
    const float *da1, *da2, *dout;
    float *pw2, *pw1;                       // [slices][h1][h2], [slices][d][h1]
    float *pb1, *pb2, *ph;                  // [kSlices][...]
    int d, h1, h2, Bn, sq;                  // sq: depth steps of the batch
    int slice_steps, slices;                // split-K
    int g2, g1;                             // blocks of dW2 and dW1
    int c1, c2;                             // groups of 64 columns of the sums (the head's last)
    int first;                              // the launch's first block
};

__global__ __launch_bounds__(kGradT) void k_grads(GradArgs g) {
    using T = Tile<64, 64, 4, 4, 2>;
    union Room {
        uint16_t lds[T::kLds];
        float red[kGradSlices][4][64][3];
        __device__ Room() {}
    };
    __shared__ __attribute__((aligned(16))) Room room;
    int b = g.first + (int)blockIdx.x;
    if (b < g.g2 + g.g1) {
        const bool two = b < g.g2;
        if (!two) b -= g.g2;
        const int M = two ? g.h1 : g.d, N = two ? g.h2 : g.h1;
        const int nt = (N + 63) / 64;
        const int z = b % g.slices, x = b / g.slices;
        const int n0 = 64 * (x % nt), m0 = 64 * (x / nt);
        const int s0 = z * g.slice_steps, total = (g.Bn + 31) / 32;
        const int ns = s0 + g.slice_steps < total ? g.slice_steps : total - s0;
        T c;
        c.run(two ? g.h1q : g.xq, g.sq, m0 / 16, two ? g.da2q : g.da1q, g.sq, n0 / 16, s0, ns,
              room.lds);
        float* p = (two ? g.pw2 : g.pw1) + (int64_t)z * M * N;
        c.each(m0, n0, [&](int64_t mf, int nf, const v4f& v) {
            const int64_t m = 16 * mf + lane_m();
            const int n = 16 * nf + lane_n();
            __attribute__((aligned(16))) const float a[4] = {v[0], v[1], v[2], v[3]};
            put_flat<float4>(p, m, n, M, N, a);
        });
        return;
    }
    b -= g.g2 + g.g1;
    const int ws = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);
    const int bx = b / kSliceBlocks, bz = (b % kSliceBlocks) * kGradSlices + ws;
    if (bx < g.c1) column_sums(g.da1, g.Bn, g.h1, bx, bz, g.pb1, room.red[ws]);
    else if (bx < g.c1 + g.c2)
        column_sums(g.da2, g.Bn, g.h2, bx - g.c1, bz, g.pb2, room.red[ws]);
    else head_wgrad(g.h2b, g.h2, g.dout, g.Bn, bx - g.c1 - g.c2, bz, g.ph, room.red[ws]);
}

// One parameter per thread: its gradient (the partials summed in their order,
// or a caller's), one Adam step on it, and the bfloat16 copies of a weight in
// the orders of the products that read it.
struct FinishArgs {
    float *th, *m1, *m2, *grad_out;         // grad_out may be null
    const float* grad_in;                   // a caller's gradient, or null: the partials
    const float *pw2, *pw1, *pb1, *pb2, *ph;
    uint16_t *w1p, *w2p, *w2q, *w3b;
    int64_t np, o_b1, o_w2, o_b2, o_w3;
    int d, h1, h2, slices;
    int adam;
    float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ float sum_parts(const float* __restrict__ p, int64_t stride, int n) {
    float s = 0.f;
    for (int z = 0; z < n; z++) s += p[z * stride];
    return s;
}

// the bfloat16 copies of parameter i (biases have none)
__device__ __forceinline__ void put_weight(const FinishArgs& a, int64_t i, float v) {
    const uint16_t h = f2bf(v);
    if (i < a.o_b1) {
        a.w1p[frag_at(i % a.h1, (int)(i / a.h1), depth_steps(a.d))] = h;
    } else if (i >= a.o_w2 && i < a.o_b2) {
        const int64_t q = i - a.o_w2;
        const int k = (int)(q / a.h2), n = (int)(q % a.h2);
        a.w2p[frag_at(n, k, depth_steps(a.h1))] = h;
        a.w2q[frag_at(k, n, depth_steps(a.h2))] = h;
    } else if (i >= a.o_w3 && i < a.o_w3 + 2 * (int64_t)a.h2) {
        a.w3b[i - a.o_w3] = h;
    }
}

__global__ __launch_bounds__(kT) void k_finish(FinishArgs a) {
    const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (i >= a.np) return;
    float gi;
    if (a.grad_in) gi = a.grad_in[i];
    else if (i < a.o_b1) gi = sum_parts(a.pw1 + i, (int64_t)a.d * a.h1, a.slices);
    else if (i < a.o_w2) gi = sum_parts(a.pb1 + (i - a.o_b1), a.h1, kSlices);
    else if (i < a.o_b2) gi = sum_parts(a.pw2 + (i - a.o_w2), (int64_t)a.h1 * a.h2, a.slices);
    else if (i < a.o_w3) gi = sum_parts(a.pb2 + (i - a.o_b2), a.h2, kSlices);
    else gi = sum_parts(a.ph + (i - a.o_w3), 2 * a.h2 + 2, kSlices);
    if (a.grad_out) a.grad_out[i] = gi;
    if (!a.adam) return;
    const float m = a.b1 * a.m1[i] + (1.f - a.b1) * gi;
    const float v = a.b2 * a.m2[i] + (1.f - a.b2) * gi * gi;
    a.m1[i] = m;
    a.m2[i] = v;
    const float th = a.th[i] - a.lr * (m / a.c1) / (sqrtf(v / a.c2) + a.eps);
    a.th[i] = th;
    put_weight(a, i, th);
}

__global__ __launch_bounds__(kT) void k_weights(FinishArgs a) {
    const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (i < a.np) put_weight(a, i, a.th[i]);
}

// per-feature mean and 1/std over n rows, FP64 accumulation (one block per feature)
__global__ __launch_bounds__(kT) void k_feature_stats(const float* __restrict__ X, int64_t n, int d,
                                                      float* __restrict__ mean,
                                                      float* __restrict__ inv_std) {
    __shared__ double r1[kT], r2[kT];
    const int c = blockIdx.x;
    double s = 0.0, q = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += kT) {
        const double v = X[i * d + c];
        s += v;
        q += v * v;
    }
    r1[threadIdx.x] = s;
    r2[threadIdx.x] = q;
    __syncthreads();
    for (int o = kT / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            r1[threadIdx.x] += r1[threadIdx.x + o];
            r2[threadIdx.x] += r2[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double mu = r1[0] / (double)n;
        double var = r2[0] / (double)n - mu * mu;
        if (!(var > 0.0)) var = 1.0;
        mean[c] = (float)mu;
        inv_std[c] = (float)(1.0 / sqrt(var));
    }
}

// placed embedding: y = clamp(out, 0, 1 - 2^-24) * r * s  (double [n][2])
__global__ __launch_bounds__(kT) void k_place(const float* __restrict__ out, int64_t n, double r,
                                              double sx, double sy, double* __restrict__ Y) {
    const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (i >= n) return;
    const double top = 1.0 - 0x1.0p-24;
    double a = (double)out[2 * i], b = (double)out[2 * i + 1];
    a = a < 0.0 ? 0.0 : (a > top ? top : a);
    b = b < 0.0 ? 0.0 : (b > top ? top : b);
    Y[2 * i] = a * r * sx;
    Y[2 * i + 1] = b * r * sy;
}

inline dim3 g1(int64_t n) { return dim3((unsigned)ceil_div(n > 0 ? n : 1, kT)); }

template <typename P>
hipError_t mal(pixelsne_mlp* m, P** p, size_t bytes) {
    void* q = nullptr;
    hipError_t e = hipMalloc(&q, bytes ? bytes : 1);
    if (e != hipSuccess) return e;
    m->allocs.push_back(q);
    *p = (P*)q;
    return hipSuccess;
}

int64_t off_W1(const pixelsne_mlp*) { return 0; }
int64_t off_b1(const pixelsne_mlp* m) { return (int64_t)m->d * m->h1; }
int64_t off_W2(const pixelsne_mlp* m) { return off_b1(m) + m->h1; }
int64_t off_b2(const pixelsne_mlp* m) { return off_W2(m) + (int64_t)m->h1 * m->h2; }
int64_t off_W3(const pixelsne_mlp* m) { return off_b2(m) + m->h2; }
int64_t off_b3(const pixelsne_mlp* m) { return off_W3(m) + (int64_t)m->h2 * 2; }

// a zeroed buffer of fragments (the padding of rows and depth stays zero)
hipError_t mal_frags(pixelsne_mlp* m, uint16_t** p, int64_t rows, int64_t k) {
    const size_t bytes = 2 * (size_t)frag_elems(rows, k);
    hipError_t e = mal(m, p, bytes);
    return e == hipSuccess ? hipMemsetAsync(*p, 0, bytes, m->stream) : e;
}

// buffers of a forward pass over B rows: all of them, or those that were there
hipError_t ensure_forward(pixelsne_mlp* m, int64_t B) {
    if (B <= m->cap_batch) return hipSuccess;
    const size_t had = m->allocs.size();
    uint16_t *xp = nullptr, *h1p = nullptr, *h2b = nullptr;
    hipError_t e = mal_frags(m, &xp, B, m->d);
    if (e == hipSuccess) e = mal_frags(m, &h1p, B, m->h1);
    if (e == hipSuccess) e = mal(m, &h2b, 2 * (size_t)B * m->h2);
    if (e != hipSuccess) {
        for (; m->allocs.size() > had; m->allocs.pop_back()) (void)hipFree(m->allocs.back());
        return e;
    }
    m->xp = xp;
    m->h1p = h1p;
    m->h2b = h2b;
    m->cap_batch = B;
    return hipSuccess;
}

int splits_for(int64_t K) {
    int s = (int)(K / 512);
    return s < 1 ? 1 : (s > 16 ? 16 : s);
}

// weight-gradient elements of one batch slice
int64_t slice_len(const pixelsne_mlp* m) {
    return (int64_t)m->h1 * m->h2 + (int64_t)m->d * m->h1;
}

// and of a training batch of B rows; the orders by columns are laid out for
// their batch, so another size starts from zeroed ones
hipError_t ensure_train(pixelsne_mlp* m, int64_t B) {
    hipError_t e = ensure_forward(m, B);
    if (e != hipSuccess) return e;
    if (B > m->cap_train) {
        if ((e = mal_frags(m, &m->xq, m->d, B)) != hipSuccess) return e;
        if ((e = mal_frags(m, &m->h1q, m->h1, B)) != hipSuccess) return e;
        if ((e = mal_frags(m, &m->da2p, B, m->h2)) != hipSuccess) return e;
        if ((e = mal_frags(m, &m->da2q, m->h2, B)) != hipSuccess) return e;
        if ((e = mal_frags(m, &m->da1q, m->h1, B)) != hipSuccess) return e;
        if ((e = mal(m, &m->yb, 8 * (size_t)B)) != hipSuccess) return e;
        if ((e = mal(m, &m->a1, 4 * (size_t)B * m->h1)) != hipSuccess) return e;
        if ((e = mal(m, &m->a2, 4 * (size_t)B * m->h2)) != hipSuccess) return e;
        if ((e = mal(m, &m->dout, 8 * (size_t)B)) != hipSuccess) return e;
        if ((e = mal(m, &m->da2, 4 * (size_t)B * m->h2)) != hipSuccess) return e;
        if ((e = mal(m, &m->da1, 4 * (size_t)B * m->h1)) != hipSuccess) return e;
        m->cap_train = B;
        m->train_steps = depth_steps(B);
    }
    if (m->train_steps != depth_steps(B)) {
        const int64_t rows[4] = {m->d, m->h1, m->h2, m->h1};
        uint16_t* q[4] = {m->xq, m->h1q, m->da2q, m->da1q};
        for (int x = 0; x < 4; x++)
            if ((e = hipMemsetAsync(q[x], 0, 2 * (size_t)frag_elems(rows[x], B), m->stream)) !=
                hipSuccess)
                return e;
        m->train_steps = depth_steps(B);
    }
    // partials for as many batch slices as there is room for, at least one
    const int64_t slice = slice_len(m);
    for (int64_t splits = splits_for(B); splits * slice > m->splitk_len; splits /= 2) {
        e = mal(m, &m->splitk, 4 * (size_t)(splits * slice));
        if (e == hipSuccess) {
            m->splitk_len = splits * slice;
            break;
        }
        if (e != hipErrorOutOfMemory || splits == 1) return e;
        (void)hipGetLastError();
    }
    if (!m->part &&
        (e = mal(m, &m->part, 4 * (size_t)kSlices * (m->h1 + 3 * (int64_t)m->h2 + 2))) != hipSuccess)
        return e;
    return hipSuccess;
}

hipError_t ensure_loss(pixelsne_mlp* m, int64_t partials) {
    if (partials <= m->lossbuf_len) return hipSuccess;
    hipError_t e = mal(m, &m->lossbuf, 8 * (size_t)partials);
    if (e == hipSuccess) m->lossbuf_len = partials;
    return e;
}

// 128 x 128 tiles of eight wavefronts when they give every CU two blocks (LDS
// and L2 traffic per product halves), else 64 x 64 tiles of sixteen.  A
// million rows through 1,024-wide layers take 4.98 ms with the large tiles and
// 7.88 with the small, an epoch of 100,000 rows at 512 wide in batches of 4,096
// (256 large tiles per layer) 3.07 with the large and 2.34 with the small.
bool large_tiles(int64_t M, int64_t N) { return ceil_div(M, 128) * ceil_div(N, 128) >= 512; }

dim3 layer_grid(int64_t M, int TM, int64_t N, int TN) {
    return dim3((unsigned)(ceil_div(ceil_div(M, TM), kXcds) * kXcds * ceil_div(N, TN)));
}

hipError_t layer(pixelsne_mlp* m, const uint16_t* A, const uint16_t* B, int64_t K, int M, int N,
                 const float* bias, float* pre, uint16_t* rowsP, uint16_t* colsQ, int sq,
                 uint16_t* flat) {
    const int steps = depth_steps(K);
    if (large_tiles(M, N))
        k_layer<128, 128, 2, 4, 1><<<layer_grid(M, 128, N, 128), 512, 0, m->stream>>>(
            A, B, steps, M, N, bias, pre, rowsP, colsQ, sq, flat);
    else
        k_layer<64, 64, 4, 4, 2><<<layer_grid(M, 64, N, 64), 1024, 0, m->stream>>>(
            A, B, steps, M, N, bias, pre, rowsP, colsQ, sq, flat);
    return hipGetLastError();
}

// staged rows xp[0..Bn) through both layers; training keeps the
// pre-activations and H1 by columns
hipError_t forward_layers(pixelsne_mlp* m, int Bn, bool train) {
    const int sq = depth_steps(Bn);
    hipError_t e = layer(m, m->xp, m->w1p, m->d, Bn, m->h1, m->theta + off_b1(m),
                         train ? m->a1 : nullptr, m->h1p, train ? m->h1q : nullptr, sq, nullptr);
    if (e != hipSuccess) return e;
    return layer(m, m->h1p, m->w2p, m->h1, Bn, m->h2, m->theta + off_b2(m),
                 train ? m->a2 : nullptr, nullptr, nullptr, 0, m->h2b);
}

FinishArgs finish_args(pixelsne_mlp* m) {
    FinishArgs a{};
    a.th = m->theta;
    a.m1 = m->m1;
    a.m2 = m->m2;
    a.w1p = m->w1p;
    a.w2p = m->w2p;
    a.w2q = m->w2q;
    a.w3b = m->w3b;
    a.np = m->n_params;
    a.o_b1 = off_b1(m);
    a.o_w2 = off_W2(m);
    a.o_b2 = off_b2(m);
    a.o_w3 = off_W3(m);
    a.d = m->d;
    a.h1 = m->h1;
    a.h2 = m->h2;
    return a;
}

// Gradient partials of a staged batch: seven launches with the staging and
// k_finish.  lossp: the batch's loss partials, one per four rows.
hipError_t grad_batch(pixelsne_mlp* m, int Bn, double* lossp, FinishArgs& fin) {
    hipError_t e = forward_layers(m, Bn, true);
    if (e != hipSuccess) return e;
    const int sq = depth_steps(Bn);
    k_head_train<<<dim3((unsigned)(32 * sq / kHeadRows)), kHeadT, 0, m->stream>>>(
        m->h2b, m->h2, m->w3b, m->theta + off_b3(m), Bn, m->yb, m->a2, m->dout, lossp, m->da2,
        depth_steps(m->h2), m->da2p, sq, m->da2q);
    // dA1 = (dA2 W2^T) * GELU'(A1)
    const int steps = depth_steps(m->h2);
    if (large_tiles(Bn, m->h1))
        k_layer_back<128, 128, 2, 4, 1><<<layer_grid(Bn, 128, m->h1, 128), 512, 0, m->stream>>>(
            m->da2p, m->w2q, steps, Bn, m->h1, m->a1, m->da1, m->da1q, sq);
    else
        k_layer_back<64, 64, 4, 4, 2><<<layer_grid(Bn, 64, m->h1, 64), 1024, 0, m->stream>>>(
            m->da2p, m->w2q, steps, Bn, m->h1, m->a1, m->da1, m->da1q, sq);
    GradArgs g{};
    g.h1q = m->h1q;
    g.da2q = m->da2q;
    g.xq = m->xq;
    g.da1q = m->da1q;
    g.h2b = m->h2b;
    g.da1 = m->da1;
    g.da2 = m->da2;
    g.dout = m->dout;
    g.d = m->d;
    g.h1 = m->h1;
    g.h2 = m->h2;
    g.Bn = Bn;
    g.sq = sq;
    const int64_t splits = std::min((int64_t)splits_for(Bn), m->splitk_len / slice_len(m));
    g.slice_steps = (int)ceil_div(ceil_div(Bn, splits), 32);
    g.slices = (int)ceil_div(Bn, 32 * (int64_t)g.slice_steps);
    g.pw2 = m->splitk;
    g.pw1 = m->splitk + (int64_t)g.slices * m->h1 * m->h2;
    g.pb1 = m->part;
    g.pb2 = g.pb1 + (int64_t)kSlices * m->h1;
    g.ph = g.pb2 + (int64_t)kSlices * m->h2;
    const int64_t t1 = ceil_div(m->h1, 64), t2 = ceil_div(m->h2, 64);
    const int64_t g2 = t1 * t2 * g.slices, g1 = ceil_div(m->d, 64) * t1 * g.slices;
    const int64_t total = g2 + g1 + (t1 + 2 * t2) * kSliceBlocks;
    if (total >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    g.g2 = (int)g2;
    g.g1 = (int)g1;
    g.c1 = (int)t1;
    g.c2 = (int)t2;
    for (int64_t b = 0; b < total; b += kGradBlocks) {
        g.first = (int)b;
        k_grads<<<dim3((unsigned)(total - b < kGradBlocks ? total - b : kGradBlocks)), kGradT, 0,
                  m->stream>>>(g);
    }
    fin = finish_args(m);
    fin.pw2 = g.pw2;
    fin.pw1 = g.pw1;
    fin.pb1 = g.pb1;
    fin.pb2 = g.pb2;
    fin.ph = g.ph;
    fin.slices = g.slices;
    return hipGetLastError();
}

hipError_t stage_train(pixelsne_mlp* m, const float* X, const float* Y, const uint32_t* order,
                       int64_t b0, int Bn) {
    const int steps = depth_steps(m->d), sq = depth_steps(Bn);
    k_stage_train<<<g1((int64_t)4 * sq * 32 * steps), kT, 0, m->stream>>>(
        X, m->d, steps, order, b0, Bn, sq, m->mean, m->inv_std, m->xp, m->xq, Y, m->yb);
    return hipGetLastError();
}

hipError_t refresh_bf16(pixelsne_mlp* m) {
    k_weights<<<g1(m->n_params), kT, 0, m->stream>>>(finish_args(m));
    return hipGetLastError();
}

// One Adam step (Kingma & Ba, 2015; beta 0.9 / 0.999, eps 1e-8, bias-corrected)
// on the master weights, with the bfloat16 weight copies.
hipError_t adam_update(pixelsne_mlp* m, FinishArgs a, float lr) {
    a.adam = 1;
    a.b1 = 0.9f;
    a.b2 = 0.999f;
    a.eps = 1e-8f;
    a.lr = lr;
    m->step++;
    a.c1 = 1.f - powf(a.b1, (float)m->step);
    a.c2 = 1.f - powf(a.b2, (float)m->step);
    k_finish<<<g1(m->n_params), kT, 0, m->stream>>>(a);
    return hipGetLastError();
}

psne_status mlp_error(hipError_t e, const char* where) {
    (void)hipGetLastError();     // the status reports it: nobody else's next call should
    set_error(std::string(where) + ": " + hipGetErrorString(e));
    return e == hipErrorOutOfMemory ? PSNE_E_NOMEM : PSNE_E_DEVICE;
}

// The generator of the initial weights.  Its steps are inlined, and as a type of this
// file's own it has the distribution's code inlined beside them: 1.15 million weights
// take 12 ms.  As shared functions of the C++ library they took 45 ms or 78, which of
// the two hung on where the linker put them.
struct WeightRng {
    using result_type = std::mt19937_64::result_type;
    std::mt19937_64 rng;
    static constexpr result_type min() { return std::mt19937_64::min(); }
    static constexpr result_type max() { return std::mt19937_64::max(); }
    __attribute__((always_inline)) result_type operator()() {
        [[clang::always_inline]] return rng();
    }
};

// He-normal weights of the three layers
__attribute__((noinline)) void initial_weights(float* th, uint64_t seed, const int64_t* off,
                                               const int64_t* rows, const int64_t* cols) {
    WeightRng rng{std::mt19937_64(seed)};
    std::normal_distribution<float> nd(0.f, 1.f);
#pragma clang loop unroll(disable)
    for (int l = 0; l < 3; l++) {
        const float sc = sqrtf(2.f / (float)rows[l]);
        float* w = th + off[l];
        for (int64_t i = 0; i < rows[l] * cols[l]; i++) w[i] = nd(rng) * sc;
    }
}

bool dev_ptr(const void* p) {
    if (!p) return false;
    hipPointerAttribute_t a;
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return a.type == hipMemoryTypeDevice || a.type == hipMemoryTypeManaged;
}

}  // namespace
}  // namespace psne

using namespace psne;

extern "C" {

psne_status pixelsne_mlp_forward(pixelsne_mlp* m, const float* X, int64_t n, float* Y01_out);

pixelsne_mlp* pixelsne_mlp_create(int32_t d_in, int32_t h1, int32_t h2, uint64_t seed,
                                  void* stream) {
    if (d_in < 1 || h1 < 1 || h2 < 1 || d_in > 65536 || h1 > 65536 || h2 > 65536) {
        set_error("MLP sizes must be in [1, 65536]");
        return nullptr;
    }
    pixelsne_mlp* m = new pixelsne_mlp();
    m->d = d_in;
    m->h1 = h1;
    m->h2 = h2;
    m->seed = seed;
    m->stream = (hipStream_t)stream;
    m->n_params = (int64_t)d_in * h1 + h1 + (int64_t)h1 * h2 + h2 + (int64_t)h2 * 2 + 2;
    hipError_t e = mal(m, &m->theta, 4 * m->n_params);
    if (e == hipSuccess) e = mal(m, &m->m1, 4 * m->n_params);
    if (e == hipSuccess) e = mal(m, &m->m2, 4 * m->n_params);
    if (e == hipSuccess) e = mal_frags(m, &m->w1p, h1, d_in);
    if (e == hipSuccess) e = mal_frags(m, &m->w2p, h2, h1);
    if (e == hipSuccess) e = mal_frags(m, &m->w2q, h1, h2);
    if (e == hipSuccess) e = mal(m, &m->w3b, 2 * (size_t)h2 * 2);
    if (e == hipSuccess) e = mal(m, &m->mean, 4 * (size_t)d_in);
    if (e == hipSuccess) e = mal(m, &m->inv_std, 4 * (size_t)d_in);
    if (e != hipSuccess) {
        mlp_error(e, "mlp_create");
        pixelsne_mlp_destroy(m);
        return nullptr;
    }
    // He-style initialisation from a seeded host generator, zero biases
    std::vector<float> th(m->n_params, 0.f);
    const int64_t off[3] = {off_W1(m), off_W2(m), off_W3(m)}, rows[3] = {d_in, h1, h2},
                  cols[3] = {h1, h2, 2};
    initial_weights(th.data(), seed, off, rows, cols);
    std::vector<float> ones(d_in, 1.f), zeros(d_in, 0.f);
    e = hipMemcpyAsync(m->theta, th.data(), 4 * m->n_params, hipMemcpyHostToDevice, m->stream);
    if (e == hipSuccess) e = hipMemsetAsync(m->m1, 0, 4 * m->n_params, m->stream);
    if (e == hipSuccess) e = hipMemsetAsync(m->m2, 0, 4 * m->n_params, m->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(m->mean, zeros.data(), 4 * d_in, hipMemcpyHostToDevice, m->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(m->inv_std, ones.data(), 4 * d_in, hipMemcpyHostToDevice, m->stream);
    if (e == hipSuccess) e = refresh_bf16(m);
    if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
    if (e != hipSuccess) {
        mlp_error(e, "mlp_create");
        pixelsne_mlp_destroy(m);
        return nullptr;
    }
    return m;
}

void pixelsne_mlp_destroy(pixelsne_mlp* m) {
    if (!m) return;
    (void)hipStreamSynchronize(m->stream);
    for (void* p : m->allocs) (void)hipFree(p);
    delete m;
}

int64_t pixelsne_mlp_num_params(const pixelsne_mlp* m) { return m ? m->n_params : -1; }

psne_status pixelsne_mlp_set_params(pixelsne_mlp* m, const float* theta) {
    if (!m || !dev_ptr(theta)) { set_error("mlp_set_params: null mlp or non-device theta"); return PSNE_E_INVAL; }
    hipError_t e = hipMemcpyAsync(m->theta, theta, 4 * m->n_params, hipMemcpyDeviceToDevice, m->stream);
    if (e == hipSuccess) e = refresh_bf16(m);
    if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
    return e == hipSuccess ? PSNE_OK : mlp_error(e, "mlp_set_params");
}

psne_status pixelsne_mlp_get_params(const pixelsne_mlp* m, float* theta) {
    if (!m || !dev_ptr(theta)) { set_error("mlp_get_params: null mlp or non-device theta"); return PSNE_E_INVAL; }
    hipError_t e = hipMemcpyAsync(theta, m->theta, 4 * m->n_params, hipMemcpyDeviceToDevice, m->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
    return e == hipSuccess ? PSNE_OK : mlp_error(e, "mlp_get_params");
}

psne_status pixelsne_mlp_set_norm(pixelsne_mlp* m, const float* mean, const float* inv_std) {
    if (!m || !dev_ptr(mean) || !dev_ptr(inv_std)) { set_error("mlp_set_norm: bad arguments"); return PSNE_E_INVAL; }
    hipError_t e = hipMemcpyAsync(m->mean, mean, 4 * (size_t)m->d, hipMemcpyDeviceToDevice, m->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(m->inv_std, inv_std, 4 * (size_t)m->d, hipMemcpyDeviceToDevice, m->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
    return e == hipSuccess ? PSNE_OK : mlp_error(e, "mlp_set_norm");
}

psne_status pixelsne_mlp_fit_norm(pixelsne_mlp* m, const float* X, int64_t n) {
    if (!m || !dev_ptr(X) || n < 1) { set_error("mlp_fit_norm: bad arguments"); return PSNE_E_INVAL; }
    k_feature_stats<<<dim3((unsigned)m->d), kT, 0, m->stream>>>(X, n, m->d, m->mean, m->inv_std);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
    return e == hipSuccess ? PSNE_OK : mlp_error(e, "mlp_fit_norm");
}

psne_status pixelsne_mlp_grad(pixelsne_mlp* m, const float* X, const float* Y01, int64_t n,
                              float* grads_out, double* loss) {
    if (!m || !dev_ptr(X) || !dev_ptr(Y01) || n < 1 || n > (1 << 20)) {
        set_error("mlp_grad: bad arguments (n must be in [1, 2^20])");
        return PSNE_E_INVAL;
    }
    if (grads_out && !dev_ptr(grads_out)) { set_error("mlp_grad: grads_out must be a device pointer"); return PSNE_E_INVAL; }
    hipError_t e = ensure_train(m, n);
    if (e == hipSuccess) e = ensure_loss(m, ceil_div(n, 4));
    if (e != hipSuccess) return mlp_error(e, "mlp_grad");
    FinishArgs fin;
    e = stage_train(m, X, Y01, nullptr, 0, (int)n);
    if (e == hipSuccess) e = grad_batch(m, (int)n, m->lossbuf, fin);
    if (e == hipSuccess && grads_out) {
        fin.grad_out = grads_out;
        k_finish<<<g1(m->n_params), kT, 0, m->stream>>>(fin);
        e = hipGetLastError();
    }
    std::vector<double> lp(m->lossbuf_len);
    const int64_t nb = ceil_div(n, 4);
    if (e == hipSuccess)
        e = hipMemcpyAsync(lp.data(), m->lossbuf, 8 * nb, hipMemcpyDeviceToHost, m->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
    if (e != hipSuccess) return mlp_error(e, "mlp_grad");
    if (loss) {
        double s = 0.0;
        for (int64_t i = 0; i < nb; i++) s += lp[i];
        *loss = s / (double)n;
    }
    return PSNE_OK;
}

psne_status pixelsne_mlp_train(pixelsne_mlp* m, const float* X, const float* Y01, int64_t n,
                               int32_t epochs, int32_t batch, float lr, double* last_epoch_loss) {
    if (!m || !dev_ptr(X) || !dev_ptr(Y01) || n < 1 || epochs < 0 || batch < 1 ||
        batch > (1 << 20) || !(lr > 0.f)) {
        set_error("mlp_train: bad arguments");
        return PSNE_E_INVAL;
    }
    const int64_t B = batch < n ? batch : n;
    const int64_t nbatch = n / B;                // full batches only
    const int64_t nl = ceil_div(B, 4);           // loss partials per batch
    hipError_t e = ensure_train(m, B);
    if (e == hipSuccess) e = ensure_loss(m, nbatch * nl);
    if (e == hipSuccess && m->order_len < n) {
        e = mal(m, &m->order, 4 * (size_t)n);
        if (e == hipSuccess) m->order_len = n;
    }
    if (e != hipSuccess) return mlp_error(e, "mlp_train");
    std::vector<uint32_t> ord(n);
    for (int64_t i = 0; i < n; i++) ord[i] = (uint32_t)i;
    std::mt19937_64 rng(m->seed ^ 0x5DEECE66DULL);
    double epoch_loss = 0.0;
    for (int32_t ep = 0; ep < epochs && e == hipSuccess; ep++) {
        std::shuffle(ord.begin(), ord.end(), rng);
        e = hipMemcpyAsync(m->order, ord.data(), 4 * (size_t)n, hipMemcpyHostToDevice, m->stream);
        if (e != hipSuccess) return mlp_error(e, "mlp_train");
        for (int64_t bi = 0; bi < nbatch && e == hipSuccess; bi++) {
            FinishArgs fin;
            e = stage_train(m, X, Y01, m->order, bi * B, (int)B);
            if (e == hipSuccess) e = grad_batch(m, (int)B, m->lossbuf + bi * nl, fin);
            if (e == hipSuccess) e = adam_update(m, fin, lr);
        }
    }
    if (e == hipSuccess && epochs > 0 && nbatch > 0) {
        // the last epoch's partials, added in their order
        std::vector<double> lp((size_t)(nbatch * nl));
        e = hipMemcpyAsync(lp.data(), m->lossbuf, 8 * lp.size(), hipMemcpyDeviceToHost, m->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
        double acc = 0.0;
        for (double v : lp) acc += v;
        epoch_loss = acc / (double)(nbatch * B);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
    if (e != hipSuccess) return mlp_error(e, "mlp_train");
    if (last_epoch_loss) *last_epoch_loss = epoch_loss;
    return PSNE_OK;
}

psne_status pixelsne_mlp_adam_step(pixelsne_mlp* m, const float* grad, float lr) {
    if (!m || !dev_ptr(grad) || !(lr > 0.f)) {
        set_error("mlp_adam_step: bad arguments");
        return PSNE_E_INVAL;
    }
    FinishArgs fin = finish_args(m);
    fin.grad_in = grad;
    hipError_t e = adam_update(m, fin, lr);
    if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
    return e == hipSuccess ? PSNE_OK : mlp_error(e, "mlp_adam_step");
}

psne_status pixelsne_mlp_place(pixelsne_mlp* m, const float* X, int64_t n, int32_t screen,
                               const double* s, double* Y_out) {
    if (!m || !dev_ptr(X) || !dev_ptr(Y_out) || n < 1 || screen < 2 || !s || !(s[0] > 0.0) ||
        !(s[1] > 0.0)) {
        set_error("mlp_place: bad arguments");
        return PSNE_E_INVAL;
    }
    float* tmp = nullptr;
    hipError_t e = hipMalloc(&tmp, 8 * (size_t)n);
    if (e != hipSuccess) return mlp_error(e, "mlp_place");
    psne_status st = pixelsne_mlp_forward(m, X, n, tmp);
    if (st == PSNE_OK) {
        k_place<<<g1(n), kT, 0, m->stream>>>(tmp, n, (double)screen, s[0], s[1], Y_out);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
        if (e != hipSuccess) st = mlp_error(e, "mlp_place");
    }
    (void)hipFree(tmp);
    return st;
}

psne_status pixelsne_mlp_forward(pixelsne_mlp* m, const float* X, int64_t n, float* Y01_out) {
    if (!m || !dev_ptr(X) || !dev_ptr(Y01_out) || n < 1) {
        set_error("mlp_forward: bad arguments");
        return PSNE_E_INVAL;
    }
    // rows per pass: whole rounds of 128 x 128 tiles, 140 MB of activations at
    // 1,024 wide; fewer where there is no room for as many
    int64_t B = n < kForwardRows ? n : kForwardRows;
    hipError_t e = ensure_forward(m, B);
    while (e == hipErrorOutOfMemory && B > kTileRows) {
        (void)hipGetLastError();
        B = ceil_div(B, 2);
        e = ensure_forward(m, B);
    }
    const int steps = depth_steps(m->d);
    for (int64_t b0 = 0; b0 < n && e == hipSuccess; b0 += B) {
        const int Bn = (int)(n - b0 < B ? n - b0 : B);
        const int64_t rows = pad_tile(Bn);
        k_stage_x<<<g1(rows * 4 * steps), kT, 0, m->stream>>>(
            X, m->d, steps, b0, Bn, rows, m->d % 4 == 0 && (uintptr_t)X % 16 == 0, m->mean,
            m->inv_std, m->xp);
        e = forward_layers(m, Bn, false);
        if (e == hipSuccess) {
            k_head<<<dim3((unsigned)ceil_div(Bn, kPlaceRows * (kT / 64))), kT, 0, m->stream>>>(
                m->h2b, m->h2, m->w3b, m->theta + off_b3(m), Bn, Y01_out + 2 * b0);
            e = hipGetLastError();
        }
    }
    if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
    return e == hipSuccess ? PSNE_OK : mlp_error(e, "mlp_forward");
}

}  // extern "C"
