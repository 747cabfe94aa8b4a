// Angle-predictor MLP: 131 -> 256 -> GELU -> 256 -> GELU -> 2, bfloat16
// operands on the matrix cores (v_mfma_f32_16x16x32_bf16), float32 accumulation.
//
// The paper proposes deriving G-QAOA angles from statistics of the density of
// states (Sec. V) and observes that optimized single-angle pairs cluster
// (Sec. III.B); the network maps the normalized level histogram and (n, d, p)
// to one (beta, gamma) pair.
//
// Storage points in bfloat16 (round to nearest even): inputs, weights,
// post-GELU activations, and the pre-activation gradients that enter the
// backward products. Pre-activations z1, z2, outputs and all gradients of
// parameters are float32; the float32 master weights are updated by Adam.
//
// A training step's products are small (a batch of 512 against 256 units), so
// its launches and the latency of each are what it costs. The forward pass is
// one launch and the backward pass two: a block takes ROWS rows of the batch
// through all layers with a whole weight matrix in LDS at a time; the weight
// gradients, sums over the batch, take 32x32 tiles of all matrices (and the
// bias sums) in one launch.
#include "internal.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace gqaoa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
// The same in global memory. Parameters and the activation cache are the caller's
// and may lie at any float's address (the rows of a stack of networks are 8 bytes
// off a multiple of 16), where one 16-byte access still serves.
typedef f32x4 f32x4_g __attribute__((aligned(4)));
typedef u16x8 u16x8_g __attribute__((aligned(4)));
typedef unsigned int u32x2_g __attribute__((ext_vector_type(2), aligned(4)));

constexpr int kDIn = 131, kDInPad = 160, kDH = 256, kDOut = 2;
constexpr size_t kOffW1 = 0;
constexpr size_t kOffB1 = kOffW1 + (size_t)kDInPad * kDH;
constexpr size_t kOffW2 = kOffB1 + kDH;
constexpr size_t kOffB2 = kOffW2 + (size_t)kDH * kDH;
constexpr size_t kOffW3 = kOffB2 + kDH;
constexpr size_t kOffB3 = kOffW3 + (size_t)kDH * kDOut;
constexpr size_t kNParams = kOffB3 + kDOut;
static_assert(kNParams == GQAOA_MLP_NPARAMS, "parameter packing");

// Round a float to bfloat16, nearest with ties to even (one v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
// Two of them, the first in the low half.
__device__ __forceinline__ uint32_t f2bf2(float lo, float hi) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad(float z) {
    const float cdf = 0.5f * (1.0f + erff(z * 0.70710678118654752f));
    const float pdf = 0.39894228040143268f * expf(-0.5f * z * z);
    return cdf + z * pdf;
}

// ---- activation cache layout ---------------------------------------------------
struct ActLayout {
    size_t xb, z1, h1, z2, h2, dz, dz1, wb, total;
};
static size_t al256(size_t x) { return (x + 255) & ~size_t(255); }
static ActLayout act_layout(int batch) {
    ActLayout L{};
    const size_t B = (size_t)batch;
    size_t o = 0;
    L.xb = o;  o += al256(B * kDInPad * 2);   // bf16 inputs, padded to 160
    L.z1 = o;  o += al256(B * kDH * 4);       // float z1
    L.h1 = o;  o += al256(B * kDH * 2);       // bf16 h1
    L.z2 = o;  o += al256(B * kDH * 4);       // float z2
    L.h2 = o;  o += al256(B * kDH * 2);       // bf16 h2
    L.dz = o;  o += al256(B * kDH * 2);       // bf16 dz2
    L.dz1 = o; o += al256(B * kDH * 2);       // bf16 dz1
    L.wb = o;  o += al256(kNParams * 2);      // bf16 copies of W1, W2, W3 (same packing)
    L.total = o;
    return L;
}
size_t mlp_act_bytes(int batch) { return act_layout(batch).total; }

// ---- training forward and backward --------------------------------------------
// MFMA operands (16x16x32): lane l holds row (column) l % 16 and the 8
// consecutive k values from 8 (l / 16); C's lane holds rows 4 (l / 16) .. + 3
// of column l % 16. Every product accumulates its k steps in one ascending
// chain, so a product's bits do not depend on the tiling.
constexpr int kPad = 8;                                    // row padding of the LDS images
constexpr int kW1Ld = kDInPad + kPad, kW2Ld = kDH + kPad, kXLd = kDInPad + kPad;
constexpr int kTrThreads = 1024;                           // 16 waves, 16 units each

__device__ __forceinline__ f32x4 mfma_bf16(const uint16_t *a, const uint16_t *b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(
        __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8 *>(a)),
        __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8 *>(b)), c, 0, 0, 0);
}

// A [64 Q or fewer rows][256] float matrix in registers: wave w's lane l holds,
// for q < Q, the 4x4 block at rows 64 q + 4 w, columns 4 l. Whole rows per load
// instruction: with lanes over rows 4 KiB apart the same loads took three
// times as long (16,000 against 5,500 clocks per 256 KiB).
template <int ROWS, int Q = (ROWS + 63) / 64>
__device__ __forceinline__ void load_blocks(const float *__restrict__ w, f32x4 (&v)[Q][4]) {
    const int k = 4 * (threadIdx.x >> 6), n = 4 * (threadIdx.x & 63);
#pragma unroll
    for (int q = 0; q < Q; ++q)
        if (64 * q + k < ROWS)  // whole waves
#pragma unroll
            for (int r = 0; r < 4; ++r) v[q][r] = *reinterpret_cast<const f32x4_g *>(w + (size_t)(64 * q + k + r) * kDH + n);
}
// LDS image of a transposed weight matrix: column n's bfloat16 k values in a
// row of 512 bytes, its 16-byte chunk c (k = 8 c ..) at chunk c ^ (n's bits 3,
// 2, 5, 4). So the transposing writes (lanes 4 columns apart, one k) and the
// operand reads (16 consecutive columns, 4 chunks) both spread over all banks.
constexpr int kWLd = kDH;
__device__ __forceinline__ int w_at(int n, int chunk) {
    return n * kWLd + ((chunk ^ ((n & 12) | (n >> 4 & 3))) << 3);
}
template <int ROWS, int Q = (ROWS + 63) / 64>
__device__ __forceinline__ void put_transposed(const f32x4 (&v)[Q][4], uint16_t *dst) {
    const int k = 4 * (threadIdx.x >> 6), n = 4 * (threadIdx.x & 63);
#pragma unroll
    for (int q = 0; q < Q; ++q)
        if (64 * q + k < ROWS) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<uint2 *>(dst + w_at(n + i, (64 * q + k) >> 3) + (k & 4)) =
                    make_uint2(f2bf2(v[q][0][i], v[q][1][i]), f2bf2(v[q][2][i], v[q][3][i]));
        }
}

// The bfloat16 copy of W2 for the backward pass, from the blocks in registers:
// row i by block i mod P, P the largest power of two up to the grid and 32.
__device__ __forceinline__ void keep_w2(const f32x4 (&v)[kDH / 64][4], uint16_t *__restrict__ wb) {
    const uint32_t P = 1u << (31 - __clz((int)min(gridDim.x, 32u)));
    if (blockIdx.x >= P) return;
    const int k = 4 * (threadIdx.x >> 6), n = 4 * (threadIdx.x & 63);
#pragma unroll
    for (int q = 0; q < kDH / 64; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (((uint32_t)(k + r) & (P - 1)) == blockIdx.x)  // 64 q is a multiple of P
                *reinterpret_cast<u32x2_g *>(wb + (size_t)(64 * q + k + r) * kDH + n) =
                    u32x2_g{f2bf2(v[q][r][0], v[q][r][1]), f2bf2(v[q][r][2], v[q][r][3])};
}

// acc = A B over KS k steps: A rows [ROWS] and B columns (this wave's 16) in
// LDS; B in the w_at layout or, with SWZ false, in rows of kW2Ld.
template <int ROWS, int KS, bool SWZ>
__device__ __forceinline__ void wave_product(const uint16_t *a, int lda, const uint16_t *b,
                                             f32x4 (&acc)[ROWS / 16]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r16 = lane & 15, kg = (lane >> 4) * 8;
#pragma unroll
    for (int i = 0; i < ROWS / 16; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int i = 0; i < ROWS / 16; ++i)
            acc[i] = mfma_bf16(a + (i * 16 + r16) * lda + ks * 32 + kg,
                               b + (SWZ ? w_at(wave * 16 + r16, ks * 4 + (lane >> 4))
                                        : (wave * 16 + r16) * kW2Ld + ks * 32 + kg),
                               acc[i]);
}

struct ActPtrs {
    uint16_t *xb, *h1, *h2, *dz2, *dz1, *wb;
    float *z1, *z2;
};

// z = acc + bias and h = bf16(gelu(z)) of this block's rows, to the cache and to LDS.
template <int ROWS>
__device__ __forceinline__ void hidden_epilogue(const f32x4 (&acc)[ROWS / 16], float bn, int row0, int batch, float *__restrict__ z, uint16_t *__restrict__ h,
                                                uint16_t *s) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = wave * 16 + (lane & 15);
#pragma unroll
    for (int i = 0; i < ROWS / 16; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = i * 16 + 4 * (lane >> 4) + r;
            const float v = acc[i][r] + bn;
            const uint16_t b = f2bf(gelu(v));
            s[m * kW2Ld + n] = b;
            if (row0 + m < batch) {
                z[(size_t)(row0 + m) * kDH + n] = v;
                h[(size_t)(row0 + m) * kDH + n] = b;
            }
        }
}

// Forward pass of ROWS batch rows: x -> z1, h1 -> z2, h2 -> out, keeping what
// the backward pass reads (and bfloat16 copies of W2 and W3 as they are now).
// Bound by latency and by what one CU can load (0.43 MB of float weights per
// block): two weight matrices through LDS, the second one loaded while the
// first product runs. A batch of 512: 12 us in one launch, where packing
// launches, two 64x64-tile products with 2-byte loads and the output layer took
// 45 us in five.
template <int ROWS>
__global__ void __launch_bounds__(kTrThreads) mlp_forward_kernel(const float *__restrict__ prm,
                                                                 const float *__restrict__ x, int batch,
                                                                 float *__restrict__ out, ActPtrs a) {
    __shared__ __attribute__((aligned(16))) uint16_t w[kDH * kWLd];
    __shared__ __attribute__((aligned(16))) uint16_t s[ROWS * kW2Ld];  // the rows' x, then h1, then h2
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row0 = blockIdx.x * ROWS, rows = min(ROWS, batch - row0);
    // what the later stages need, asked for before the first wait
    const float bn1 = prm[kOffB1 + wave * 16 + (lane & 15)], bn2 = prm[kOffB2 + wave * 16 + (lane & 15)];
    const float b30 = prm[kOffB3], b31 = prm[kOffB3 + 1];
    const uint16_t w3v = f2bf(prm[kOffW3 + tid % (kDH * kDOut)]);
    float w30[kDH / 64], w31[kDH / 64];
#pragma unroll
    for (int q = 0; q < kDH / 64; ++q) {
        w30[q] = bf2f(f2bf(prm[kOffW3 + 2 * (lane + 64 * q)]));
        w31[q] = bf2f(f2bf(prm[kOffW3 + 2 * (lane + 64 * q) + 1]));
    }
    {
        f32x4 v[(kDInPad + 63) / 64][4];
        load_blocks<kDInPad>(prm + kOffW1, v);
        constexpr int kX = (ROWS * kXLd + kTrThreads - 1) / kTrThreads;
        float xv[kX];
#pragma unroll
        for (int q = 0; q < kX; ++q) {
            // clamped, not skipped: all loads go out together
            const int i = tid + kTrThreads * q, r = i / kXLd, k = i % kXLd;
            const float e = x[(size_t)(row0 + min(r, rows - 1)) * kDIn + min(k, kDIn - 1)];
            xv[q] = r < rows && k < kDIn ? e : 0.f;
        }
#pragma unroll
        for (int q = 0; q < kX; ++q)
            if (tid + kTrThreads * q < ROWS * kXLd) s[tid + kTrThreads * q] = f2bf(xv[q]);
        put_transposed<kDInPad>(v, w);
    }
    __syncthreads();
    f32x4 v2[kDH / 64][4];
    load_blocks<kDH>(prm + kOffW2, v2);
    for (int i = tid; i < rows * (kDInPad / 8); i += kTrThreads) {
        const int r = i / (kDInPad / 8), c = i % (kDInPad / 8) * 8;
        *reinterpret_cast<u16x8_g *>(a.xb + (size_t)(row0 + r) * kDInPad + c) =
            *reinterpret_cast<const u16x8 *>(s + r * kXLd + c);
    }
    f32x4 acc[ROWS / 16];
    wave_product<ROWS, kDInPad / 32, true>(s, kXLd, w, acc);
    __syncthreads();  // x and W1 are read
    put_transposed<kDH>(v2, w);
    keep_w2(v2, a.wb + kOffW2);
    if (blockIdx.x == 0 && tid < kDH * kDOut) a.wb[kOffW3 + tid] = w3v;
    hidden_epilogue<ROWS>(acc, bn1, row0, batch, a.z1, a.h1, s);
    __syncthreads();
    wave_product<ROWS, kDH / 32, true>(s, kW2Ld, w, acc);
    __syncthreads();  // h1 is read
    hidden_epilogue<ROWS>(acc, bn2, row0, batch, a.z2, a.h2, s);
    __syncthreads();
    // o[b][c] = sum_j h2[b][j] W3[j][c] + b3[c]; one wave per row
    for (int r = wave; r < rows; r += kTrThreads / 64) {
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int q = 0; q < kDH / 64; ++q) {
            const float h = bf2f(s[r * kW2Ld + lane + 64 * q]);
            s0 += h * w30[q];
            s1 += h * w31[q];
        }
        s0 = wave_sum(s0);
        s1 = wave_sum(s1);
        if (lane == 0) {
            out[(size_t)(row0 + r) * 2] = s0 + b30;
            out[(size_t)(row0 + r) * 2 + 1] = s1 + b31;
        }
    }
}

// Backward pass of ROWS batch rows: dz2 = bf16((dout W3^T) gelu'(z2)) and
// dz1 = bf16((dz2 W2^T) gelu'(z1)); W2's rows are k-contiguous as they are. A
// batch of 512: 7 us (25 us in two launches before).
template <int ROWS>
__global__ void __launch_bounds__(kTrThreads) mlp_back_rows_kernel(const float *__restrict__ dout, int batch,
                                                                   ActPtrs a) {
    __shared__ __attribute__((aligned(16))) uint16_t w[kDH * kW2Ld];
    __shared__ __attribute__((aligned(16))) uint16_t s[ROWS * kW2Ld];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row0 = blockIdx.x * ROWS;
    constexpr int kCopies = kDH * kDH / 8 / kTrThreads;
    u16x8 c[kCopies];
#pragma unroll
    for (int q = 0; q < kCopies; ++q)
        c[q] = *reinterpret_cast<const u16x8_g *>(a.wb + kOffW2 + (size_t)(tid + kTrThreads * q) * 8);
    // every load of the block before its first use: this thread's z2 (unit j of
    // rows tid / 256 + 4 q) and the z1 of its rows of the product
    const int j = tid % kDH, n = wave * 16 + (lane & 15);
    const float w30 = bf2f(a.wb[kOffW3 + 2 * j]), w31 = bf2f(a.wb[kOffW3 + 2 * j + 1]);
    float z2[ROWS / 4], d0[ROWS / 4], d1[ROWS / 4], z1[ROWS / 16][4];
#pragma unroll
    for (int q = 0; q < ROWS / 4; ++q) {
        const int b = min(row0 + tid / kDH + 4 * q, batch - 1);
        z2[q] = a.z2[(size_t)b * kDH + j];
        d0[q] = dout[(size_t)b * 2];
        d1[q] = dout[(size_t)b * 2 + 1];
    }
#pragma unroll
    for (int i = 0; i < ROWS / 16; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            z1[i][r] = a.z1[(size_t)min(row0 + i * 16 + 4 * (lane >> 4) + r, batch - 1) * kDH + n];
#pragma unroll
    for (int q = 0; q < ROWS / 4; ++q) {
        const int r = tid / kDH + 4 * q, b = row0 + r;
        const float dh = d0[q] * w30 + d1[q] * w31;
        const uint16_t d = b < batch ? f2bf(dh * gelu_grad(z2[q])) : (uint16_t)0;
        if (b < batch) a.dz2[(size_t)b * kDH + j] = d;
        s[r * kW2Ld + j] = d;
    }
#pragma unroll
    for (int q = 0; q < kCopies; ++q) {
        const int i = (tid + kTrThreads * q) * 8;
        *reinterpret_cast<u16x8 *>(w + (i / kDH) * kW2Ld + i % kDH) = c[q];
    }
    __syncthreads();
    f32x4 acc[ROWS / 16];
    wave_product<ROWS, kDH / 32, false>(s, kW2Ld, w, acc);
#pragma unroll
    for (int i = 0; i < ROWS / 16; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int b = row0 + i * 16 + 4 * (lane >> 4) + r;
            if (b < batch) a.dz1[(size_t)b * kDH + n] = f2bf(acc[i][r] * gelu_grad(z1[i][r]));
        }
}

// Sums over the batch, one launch. Blocks [0, 64): 32x32 tiles of gW2 = h1^T
// dz2; [64, 104): of gW1 = xb^T dz1; [104, 112): gb2, [112, 120): gb1, 32
// columns each; [120, 128): 32 rows of gW3 = h2^T dout (the first also gb3). A
// batch of 512: 6.5 us (64 us in four launches before, on 28 blocks of 64x64).
constexpr int kGwTile = 32, kGwK = 256, kGwLd = kGwK + kPad;
constexpr int kGwBlocks2 = (kDH / kGwTile) * (kDH / kGwTile), kGwBlocks1 = (kDInPad / kGwTile) * (kDH / kGwTile);
constexpr int kSumBlocks = kDH / 32;

// The part of one operand [k][cols] for a tile: thread t (of 128) takes 8 of
// the tile's 32 columns and, per step, 4 consecutive k.
struct GwOperand {
    const uint16_t *p;
    int ld;
    __device__ __forceinline__ void load(int k0, int batch, u16x8 (&v)[kGwK / 128][4]) const {
        const int t = threadIdx.x & 127, c = (t & 3) * 8, kr = (t >> 2) * 4;
#pragma unroll
        for (int q = 0; q < kGwK / 128; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int k = k0 + 128 * q + kr + r;
                v[q][r] = u16x8{0, 0, 0, 0, 0, 0, 0, 0};
                if (k < batch) v[q][r] = *reinterpret_cast<const u16x8_g *>(p + (size_t)k * ld + c);
            }
    }
    __device__ __forceinline__ void put(const u16x8 (&v)[kGwK / 128][4], uint16_t *dst) const {
        const int t = threadIdx.x & 127, c = (t & 3) * 8, kr = (t >> 2) * 4;
#pragma unroll
        for (int q = 0; q < kGwK / 128; ++q)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                *reinterpret_cast<uint2 *>(dst + (c + e) * kGwLd + 128 * q + kr) =
                    make_uint2(v[q][0][e] | (uint32_t)v[q][1][e] << 16, v[q][2][e] | (uint32_t)v[q][3][e] << 16);
    }
};

// g[c] (and, with dout, both outputs) of 32 columns: 64 row groups of 4
// threads, 8 columns each; double sums in a fixed order.
template <bool OUT>
__device__ __forceinline__ void column_sums(const uint16_t *__restrict__ src, const float *__restrict__ dout,
                                            int batch, int c0, float *__restrict__ g, double *red) {
    const int tid = threadIdx.x, c = c0 + (tid & 3) * 8, rg = tid >> 2;
    constexpr int NO = OUT ? 2 : 1;
    double s[8][NO];
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int o = 0; o < NO; ++o) s[e][o] = 0.0;
    for (int b = rg; b < batch; b += 64) {
        const u16x8 v = *reinterpret_cast<const u16x8_g *>(src + (size_t)b * kDH + c);
        double d[NO];
#pragma unroll
        for (int o = 0; o < NO; ++o) d[o] = OUT ? (double)dout[(size_t)b * 2 + o] : 1.0;
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int o = 0; o < NO; ++o) s[e][o] += (double)bf2f(v[e]) * d[o];
    }
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 8; ++e) red[rg * 33 + (tid & 3) * 8 + e] = s[e][o];
        __syncthreads();
        if (tid < 32) {
            double t = 0.0;
            for (int r = 0; r < 64; ++r) t += red[r * 33 + tid];
            g[(c0 + tid) * NO + o] = (float)t;
        }
    }
}

__global__ void __launch_bounds__(256) mlp_back_weights_kernel(const float *__restrict__ dout, int batch, ActPtrs a,
                                                               float *__restrict__ grads) {
    __shared__ __attribute__((aligned(16))) uint16_t As[kGwTile * kGwLd];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[kGwTile * kGwLd];
    __shared__ double red[64 * 33];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int blk = blockIdx.x;
    if (blk >= kGwBlocks2 + kGwBlocks1) {
        blk -= kGwBlocks2 + kGwBlocks1;
        const int c0 = blk % kSumBlocks * 32;
        if (blk < kSumBlocks) {
            column_sums<false>(a.dz2, nullptr, batch, c0, grads + kOffB2, red);
        } else if (blk < 2 * kSumBlocks) {
            column_sums<false>(a.dz1, nullptr, batch, c0, grads + kOffB1, red);
        } else {
            column_sums<true>(a.h2, dout, batch, c0, grads + kOffW3, red);
            if (c0 == 0) {
                double v[2] = {0.0, 0.0};
                for (int b = tid; b < batch; b += 256) {
                    v[0] += dout[(size_t)b * 2];
                    v[1] += dout[(size_t)b * 2 + 1];
                }
                __syncthreads();
                block_sum<2, 256>(v, red);
                if (tid == 0) {
                    grads[kOffB3] = (float)v[0];
                    grads[kOffB3 + 1] = (float)v[1];
                }
            }
        }
        return;
    }
    const bool second = blk < kGwBlocks2;
    if (!second) blk -= kGwBlocks2;
    const int m0 = blk / (kDH / kGwTile) * kGwTile, n0 = blk % (kDH / kGwTile) * kGwTile;
    // threads 0..127 stage A, 128..255 B
    const bool isA = tid < 128;
    const GwOperand op = isA ? (second ? GwOperand{a.h1 + m0, kDH} : GwOperand{a.xb + m0, kDInPad})
                             : GwOperand{(second ? a.dz2 : a.dz1) + n0, kDH};
    uint16_t *dst = isA ? As : Bs;
    u16x8 v[kGwK / 128][4];
    op.load(0, batch, v);
    f32x4 acc{0.f, 0.f, 0.f, 0.f};
    const int r16 = lane & 15, kg = (lane >> 4) * 8;
    const int wm = (wave >> 1) * 16, wn = (wave & 1) * 16;
    for (int k0 = 0; k0 < batch; k0 += kGwK) {
        op.put(v, dst);
        __syncthreads();
        if (k0 + kGwK < batch) op.load(k0 + kGwK, batch, v);
        const int steps = min(kGwK / 32, (batch - k0 + 31) / 32);
        for (int ks = 0; ks < steps; ++ks)
            acc = mfma_bf16(As + (wm + r16) * kGwLd + ks * 32 + kg, Bs + (wn + r16) * kGwLd + ks * 32 + kg, acc);
        __syncthreads();
    }
    float *out = grads + (second ? kOffW2 : kOffW1);
#pragma unroll
    for (int r = 0; r < 4; ++r) out[(size_t)(m0 + wm + 4 * (lane >> 4) + r) * kDH + n0 + wn + r16] = acc[r];
}

// Loss of the angle regression and its gradient with respect to the raw outputs:
// beta = 2 pi sigmoid(o0), gamma = pi sigmoid(o1),
// L = mean_b ((beta-beta*)/(2 pi))^2 + ((gamma-gamma*)/pi)^2.
__global__ void __launch_bounds__(256) loss_kernel(const float *__restrict__ out, const float *__restrict__ tgt,
                                                   int batch, float *__restrict__ dout, float *__restrict__ loss) {
    __shared__ double red[4];
    double s = 0.0;
    const float invB = 1.0f / (float)batch;
    for (int b = threadIdx.x; b < batch; b += 256) {
        const float s0 = 1.f / (1.f + expf(-out[(size_t)b * 2]));
        const float s1 = 1.f / (1.f + expf(-out[(size_t)b * 2 + 1]));
        const float rb = s0 - tgt[(size_t)b * 2] * (0.5f / (float)M_PI);
        const float rg = s1 - tgt[(size_t)b * 2 + 1] * (1.0f / (float)M_PI);
        s += (double)(rb * rb + rg * rg);
        dout[(size_t)b * 2] = 2.f * rb * s0 * (1.f - s0) * invB;
        dout[(size_t)b * 2 + 1] = 2.f * rg * s1 * (1.f - s1) * invB;
    }
    double v[1] = {s};
    block_sum<1, 256>(v, red);
    if (threadIdx.x == 0) *loss = (float)(v[0] / batch);
}

__global__ void adam_kernel(float *__restrict__ prm, const float *__restrict__ grd, float *__restrict__ m,
                            float *__restrict__ v, float lr, float b1, float b2, float eps, float c1,
                            float c2) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kNParams) return;
    // rows 131..159 of W1 stay zero
    if (i < kOffB1 && (i / kDH) >= (size_t)kDIn) return;
    const float g = grd[i];
    const float mi = b1 * m[i] + (1.f - b1) * g;
    const float vi = b2 * v[i] + (1.f - b2) * g * g;
    m[i] = mi;
    v[i] = vi;
    prm[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// Features: w_k = N_k / 2^n for k < 128 (zero beyond m), n/24, d/8, log2(p)/6.
__global__ void features_kernel(const unsigned long long *__restrict__ hists, int hist_stride,
                                const int32_t *__restrict__ n, const int32_t *__restrict__ m,
                                const int32_t *__restrict__ p, int batch, float *__restrict__ x) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)batch * kDIn) return;
    const int b = (int)(i / kDIn), c = (int)(i % kDIn);
    float v;
    if (c < 128) v = c <= m[b] && c < hist_stride ? (float)((double)hists[(size_t)b * hist_stride + c] * ldexp(1.0, -n[b])) : 0.f;
    else if (c == 128) v = (float)n[b] / 24.f;
    else if (c == 129) v = (float)((double)m[b] / (double)n[b] / 8.0);
    else v = (float)(log2((double)p[b]) / 6.0);
    x[i] = v;
}

// ---- host entry points ---------------------------------------------------------------
static ActPtrs act_ptrs(void *act, int batch) {
    const ActLayout L = act_layout(batch);
    char *a = reinterpret_cast<char *>(act);
    auto u16 = [&](size_t o) { return reinterpret_cast<uint16_t *>(a + o); };
    return ActPtrs{u16(L.xb),  u16(L.h1), u16(L.h2), u16(L.dz), u16(L.dz1), u16(L.wb),
                   reinterpret_cast<float *>(a + L.z1), reinterpret_cast<float *>(a + L.z2)};
}

// Rows per block: 16 until that gives every CU a block, then 32, which halves
// the reads of the weights (L2) per row.
template <typename F>
static void by_rows(int batch, const DeviceInfo &dev, F f) {
    if (batch <= 16 * dev.num_cus) f(std::integral_constant<int, 16>{}, (batch + 15) / 16);
    else f(std::integral_constant<int, 32>{}, (batch + 31) / 32);
}

int run_mlp_forward(const float *prm, int batch, const float *x, float *out, void *act, hipStream_t st) {
    DeviceInfo dev;
    int s = device_info(&dev);
    if (s) return s;
    const ActPtrs a = act_ptrs(act, batch);
    by_rows(batch, dev, [&](auto rows, int blocks) {
        hipLaunchKernelGGL(mlp_forward_kernel<decltype(rows)::value>, dim3(blocks), dim3(kTrThreads), 0, st, prm, x,
                           batch, out, a);
    });
    GQ_LAUNCH_CHECK();
    return GQAOA_OK;
}

int run_mlp_backward(const float *prm, int batch, const void *act, const float *dout, float *grads,
                     hipStream_t st) {
    (void)prm;  // the weights of the forward pass, kept in act
    DeviceInfo dev;
    int s = device_info(&dev);
    if (s) return s;
    const ActPtrs a = act_ptrs(const_cast<void *>(act), batch);
    by_rows(batch, dev, [&](auto rows, int blocks) {
        hipLaunchKernelGGL(mlp_back_rows_kernel<decltype(rows)::value>, dim3(blocks), dim3(kTrThreads), 0, st, dout,
                           batch, a);
    });
    GQ_LAUNCH_CHECK();
    hipLaunchKernelGGL(mlp_back_weights_kernel, dim3(kGwBlocks2 + kGwBlocks1 + 3 * kSumBlocks), dim3(256), 0, st, dout,
                       batch, a, grads);
    GQ_LAUNCH_CHECK();
    return GQAOA_OK;
}

int run_mlp_adam(float *prm, const float *grads, float *state, int step, float lr, float b1, float b2,
                 float eps, hipStream_t st) {
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((kNParams + 255) / 256)), dim3(256), 0, st, prm, grads,
                       state, state + kNParams, lr, b1, b2, eps, c1, c2);
    GQ_LAUNCH_CHECK();
    return GQAOA_OK;
}

int run_mlp_loss(int batch, const float *out, const float *tgt, float *dout, float *loss, hipStream_t st) {
    hipLaunchKernelGGL(loss_kernel, dim3(1), dim3(256), 0, st, out, tgt, batch, dout, loss);
    GQ_LAUNCH_CHECK();
    return GQAOA_OK;
}

int run_mlp_features(int batch, const uint64_t *hists, int hist_stride, const int32_t *n, const int32_t *m,
                     const int32_t *p, float *x, hipStream_t st) {
    const size_t nx = (size_t)batch * kDIn;
    hipLaunchKernelGGL(features_kernel, dim3((unsigned)((nx + 255) / 256)), dim3(256), 0, st,
                       reinterpret_cast<const unsigned long long *>(hists), hist_stride, n, m, p, batch, x);
    GQ_LAUNCH_CHECK();
    return GQAOA_OK;
}

// ---- inference: weights stationary in LDS ----------------------------------------------
// A small kernel packs the LDS images of W1^T and W2^T (bfloat16) into the
// workspace; then two persistent kernels of 512 threads (8 waves) run over
// tiles of 128 rows, each block copying its weight image with 16-byte loads; a
// wave owns 16 rows and all 256 hidden units (16 MFMA tiles, 64 accumulator
// registers). Kernel 1 keeps W1^T (bfloat16) in LDS, stages the tile's x rows
// (contiguous in memory) through LDS and writes h1 = bf16(gelu(x W1 + b1)).
// Kernel 2 keeps W2^T in LDS, loads h1 fragments straight into the MFMA
// operand layout and folds the output layer into its epilogue, so h2 never
// leaves registers. The MFMA k-order equals the training GEMM's, so h1 and
// h2 are bit-identical to the training forward; only the output layer's
// 256-term sum is taken in another order.
constexpr int kInfThreads = 512, kInfRows = 128;

constexpr size_t kW1Image = (size_t)kDH * kW1Ld * 2, kW2Image = (size_t)kDH * kW2Ld * 2;  // bytes

// workspace: [W1^T LDS image | W2^T LDS image | h1 (bfloat16 [batch][256])]
size_t mlp_infer_bytes(int batch) { return al256(kW1Image) + al256(kW2Image) + al256((size_t)batch * kDH * 2); }

// The LDS images of both weight matrices, bfloat16, transposed ([n][k]) and
// padded, so every block of the inference kernels loads them with 16-byte
// copies.
__global__ void mlp_pack_images_kernel(const float *__restrict__ prm, uint16_t *__restrict__ w1t,
                                       uint16_t *__restrict__ w2t) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kDH * kW1Ld) {
        const int n = i / kW1Ld, k = i % kW1Ld;
        w1t[i] = k < kDIn ? f2bf(prm[kOffW1 + (size_t)k * kDH + n]) : (uint16_t)0;
    }
    if (i < kDH * kW2Ld) {
        const int n = i / kW2Ld, k = i % kW2Ld;
        w2t[i] = k < kDH ? f2bf(prm[kOffW2 + (size_t)k * kDH + n]) : (uint16_t)0;
    }
}

// 16-byte copy of an LDS image (bytes a multiple of 16) by a whole block.
__device__ __forceinline__ void load_image(uint16_t *dst, const uint16_t *__restrict__ src, size_t bytes) {
    const uint4 *s = reinterpret_cast<const uint4 *>(src);
    uint4 *d = reinterpret_cast<uint4 *>(dst);
    for (size_t i = threadIdx.x; i < bytes / 16; i += blockDim.x) d[i] = s[i];
}

__global__ void __launch_bounds__(kInfThreads) mlp_infer_l1_kernel(const float *__restrict__ prm,
                                                                    const uint16_t *__restrict__ w1t,
                                                                    const float *__restrict__ x, int batch,
                                                                    int x_aligned, uint16_t *__restrict__ h1) {
    __shared__ __attribute__((aligned(16))) uint16_t w[kDH * kW1Ld];        // W1^T: [n][k]
    __shared__ __attribute__((aligned(16))) uint16_t xs[kInfRows * kXLd];   // the tile's inputs: [row][k]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    load_image(w, w1t, kW1Image);
    const int r16 = lane & 15, kg = (lane >> 4) * 8;
    float b1[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) b1[t] = prm[kOffB1 + t * 16 + r16];
    const int ntiles = (batch + kInfRows - 1) / kInfRows;
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int row0 = tile * kInfRows;
        const int rows = min(kInfRows, batch - row0);
        __syncthreads();  // the previous tile's reads of xs (and, first time, the W1 staging) are done
        // the tile's rows are contiguous and, when x is 16-byte aligned, start
        // 16-byte aligned (row0 is a multiple of 4): float4 loads over the
        // valid part, zeros past the batch
        const float *src = x + (size_t)row0 * kDIn;
        const int nvalid = rows * kDIn;
        for (int j = tid; j < (kInfRows * kDIn) / 4; j += kInfThreads) {
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (x_aligned && 4 * j + 3 < nvalid) {
                v = reinterpret_cast<const float4 *>(src)[j];
            } else {
                if (4 * j < nvalid) v.x = src[4 * j];
                if (4 * j + 1 < nvalid) v.y = src[4 * j + 1];
                if (4 * j + 2 < nvalid) v.z = src[4 * j + 2];
                if (4 * j + 3 < nvalid) v.w = src[4 * j + 3];
            }
            const float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = 4 * j + q, r = i / kDIn, k = i % kDIn;
                xs[r * kXLd + k] = f2bf(e[q]);
            }
        }
        for (int i = tid; i < kInfRows * (kDInPad - kDIn); i += kInfThreads) {
            const int r = i / (kDInPad - kDIn), k = kDIn + i % (kDInPad - kDIn);
            xs[r * kXLd + k] = 0;
        }
        __syncthreads();
        f32x4 acc[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < kDInPad / 32; ++ks) {
            const u16x8 av = *reinterpret_cast<const u16x8 *>(&xs[(wave * 16 + r16) * kXLd + ks * 32 + kg]);
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const u16x8 bv = *reinterpret_cast<const u16x8 *>(&w[(t * 16 + r16) * kW1Ld + ks * 32 + kg]);
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av),
                                                                 __builtin_bit_cast(bf16x8, bv), acc[t], 0, 0, 0);
            }
        }
        // lane holds C[4*(lane/16) + r][lane % 16] of each 16x16 tile
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = row0 + wave * 16 + 4 * (lane >> 4) + r;
            if (row >= batch) continue;
            uint16_t *dst = h1 + (size_t)row * kDH + r16;
#pragma unroll
            for (int t = 0; t < 16; ++t) dst[t * 16] = f2bf(gelu(acc[t][r] + b1[t]));
        }
    }
}

__global__ void __launch_bounds__(kInfThreads) mlp_infer_l23_kernel(const float *__restrict__ prm,
                                                                     const uint16_t *__restrict__ w2t,
                                                                     const uint16_t *__restrict__ h1, int batch,
                                                                     float *__restrict__ out) {
    __shared__ __attribute__((aligned(16))) uint16_t w[kDH * kW2Ld];        // W2^T: [n][k]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    load_image(w, w2t, kW2Image);
    const int r16 = lane & 15, kg = (lane >> 4) * 8;
    float b2[16], w30[16], w31[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        const int n = t * 16 + r16;
        b2[t] = prm[kOffB2 + n];
        w30[t] = bf2f(f2bf(prm[kOffW3 + (size_t)n * kDOut]));
        w31[t] = bf2f(f2bf(prm[kOffW3 + (size_t)n * kDOut + 1]));
    }
    const float b30 = prm[kOffB3], b31 = prm[kOffB3 + 1];
    __syncthreads();
    const int ntiles = (batch + kInfRows - 1) / kInfRows;
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int row0 = tile * kInfRows;
        const int arow = row0 + wave * 16 + r16;  // the A-operand row of this lane
        const bool live = arow < batch;
        const uint16_t *src = h1 + (size_t)(live ? arow : 0) * kDH + kg;
        f32x4 acc[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
        for (int ks = 0; ks < kDH / 32; ++ks) {
            u16x8 av = *reinterpret_cast<const u16x8 *>(src + ks * 32);
            if (!live) av = u16x8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const u16x8 bv = *reinterpret_cast<const u16x8 *>(&w[(t * 16 + r16) * kW2Ld + ks * 32 + kg]);
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av),
                                                                 __builtin_bit_cast(bf16x8, bv), acc[t], 0, 0, 0);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float s0 = 0.f, s1 = 0.f;
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const float h = bf2f(f2bf(gelu(acc[t][r] + b2[t])));
                s0 += h * w30[t];
                s1 += h * w31[t];
            }
            // the 16 lanes of a group hold the same rows, different columns
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) {
                s0 += __shfl_xor(s0, off, kWave);
                s1 += __shfl_xor(s1, off, kWave);
            }
            const int row = row0 + wave * 16 + 4 * (lane >> 4) + r;
            if (r16 == 0 && row < batch) {
                out[(size_t)row * kDOut] = s0 + b30;
                out[(size_t)row * kDOut + 1] = s1 + b31;
            }
        }
    }
}

int run_mlp_infer(const float *prm, int batch, const float *x, float *out, void *ws, hipStream_t st) {
    DeviceInfo dev;
    int s = device_info(&dev);
    if (s) return s;
    char *base = reinterpret_cast<char *>(ws);
    uint16_t *w1t = reinterpret_cast<uint16_t *>(base);
    uint16_t *w2t = reinterpret_cast<uint16_t *>(base + al256(kW1Image));
    uint16_t *h1 = reinterpret_cast<uint16_t *>(base + al256(kW1Image) + al256(kW2Image));
    const int img = std::max(kDH * kW1Ld, kDH * kW2Ld);
    hipLaunchKernelGGL(mlp_pack_images_kernel, dim3((img + 255) / 256), dim3(256), 0, st, prm, w1t, w2t);
    GQ_LAUNCH_CHECK();
    const int ntiles = (batch + kInfRows - 1) / kInfRows;
    const int blocks = std::min(ntiles, dev.num_cus);
    const int x_aligned = (reinterpret_cast<uintptr_t>(x) & 15) == 0;
    hipLaunchKernelGGL(mlp_infer_l1_kernel, dim3(blocks), dim3(kInfThreads), 0, st, prm, w1t, x, batch, x_aligned,
                       h1);
    GQ_LAUNCH_CHECK();
    hipLaunchKernelGGL(mlp_infer_l23_kernel, dim3(blocks), dim3(kInfThreads), 0, st, prm, w2t, h1, batch, out);
    GQ_LAUNCH_CHECK();
    return GQAOA_OK;
}

}  // namespace gqaoa
