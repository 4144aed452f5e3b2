// Inference of the surrogate network at hidden width 256 in one launch: rows in,
// outputs out, no activation in memory.  The arithmetic is that of the
// layer-by-layer kernels in mlp.hip, bit for bit: every product rounds both
// operands to FP16 and accumulates in FP32 over 32 terms per matrix
// instruction in the same order, biases and GELU are FP32, and the head's sum
// keeps the shape of its tree.
#include "internal.hpp"

namespace pwa {
namespace {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned u2 __attribute__((ext_vector_type(2)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));

constexpr int kPH = 256;            // hidden width
constexpr int kPT = 1024;           // threads per block: 16 waves, four per SIMD
constexpr int kPTiles = kPH / 16;   // feature tiles of a layer

// GELU in FP32, then rounded to FP16: two roundings, as where the FP32 value goes
// through memory.  The empty statement keeps the compiler from rounding the last
// product once, straight to FP16 (one activation in some 35,000 came out different).
__device__ __forceinline__ _Float16 gelu16(float x) {
    float h = 0.5f * x * (1.f + erff(x * 0.70710678118654752f));
    __asm__ volatile("" : "+v"(h));
    return (_Float16)h;
}

// Operand order of a layer's output.  With features as rows and samples as
// columns, lane (q, r16) holds features 4 q + e of tiles 2 s (a) and 2 s + 1 (b)
// of sample r16 after a layer, and feeds features 32 s + 8 q + 0..7 of the same
// sample to the next: lane row q needs the halves of two lane rows, which the
// 32- and 16-lane row swaps deliver (a: rows a0 a1 a2 a3 -> a0 a2 b0 b2; b: ->
// a1 a3 b1 b3).
__device__ __forceinline__ h8 as_operand(h4 a, h4 b) {
    u2 x = __builtin_bit_cast(u2, a), y = __builtin_bit_cast(u2, b);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const auto p = __builtin_amdgcn_permlane32_swap(x[i], y[i], false, false);
        const auto r = __builtin_amdgcn_permlane16_swap(p[0], p[1], false, false);
        x[i] = r[0];
        y[i] = r[1];
    }
    return __builtin_bit_cast(h8, u4{x[0], x[1], y[0], y[1]});
}

// 16-byte piece of fp16 weights: W[r][c .. c + 7] of a row-major FP32 matrix,
// zero past the row's `in` columns.
__device__ __forceinline__ h8 weights8(const float *W, int in, int r, int c) {
    h8 v;
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = (_Float16)(c + i < in ? W[(int64_t)r * in + c + i] : 0.f);
    return v;
}

// A wave takes 16 rows through the whole network.  The block's FP16 weights sit
// in LDS in operand order (16 bytes per lane, 1 KB per 16 x 32 piece), 144 KB at
// up to 32 inputs and 160 KB, all of it, at up to 64; each layer's output goes
// to the next layer's operand registers with lane-row swaps.  Waves take row
// tiles in turn, the blocks fastest, so that the last round spreads over all
// SIMDs.
//
// Bound: vector arithmetic, 512 GELU per row (an erf of about 40 instructions
// each).  10^5 rows, 32 inputs: 54 us; layer by layer through memory in chunks of
// 8192 rows (26 products of 16 us, 13 heads of 6.5 us) 0.52 ms.
template <int INP>
__global__ __launch_bounds__(kPT) void mlp_predict_kernel(const float *P, int in, const float *X, int64_t n,
                                                          float *y) {
    constexpr int KS1 = INP / 32;                       // k-steps of layer 1
    constexpr int KS2 = kPH / 32;                       // k-steps of layer 2
    __shared__ __attribute__((aligned(16))) h8 w1[kPTiles * KS1 * 64];
    __shared__ __attribute__((aligned(16))) h8 w2[kPTiles * KS2 * 64];
    const float *W1 = P, *b1 = W1 + (int64_t)kPH * in, *W2 = b1 + kPH, *b2 = W2 + kPH * kPH, *w3 = b2 + kPH,
                *b3 = w3 + kPH;
    const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, r16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // piece (t, s) of W2: lane (q, r16) holds W2[16 t + r16][32 s + 8 q .. + 7]
    for (int i = tid; i < kPTiles * KS1 * 64; i += kPT)
        w1[i] = weights8(W1, in, 16 * (i / (KS1 * 64)) + (i & 15), 32 * (i / 64 % KS1) + 8 * (i / 16 % 4));
    for (int i = tid; i < kPTiles * KS2 * 64; i += kPT) {
        const float *src = W2 + (16 * (i / (KS2 * 64)) + (i & 15)) * kPH + 32 * (i / 64 % KS2) + 8 * (i / 16 % 4);
        const f4 lo = *reinterpret_cast<const f4 *>(src), hi = *reinterpret_cast<const f4 *>(src + 4);
        w2[i] = h8{(_Float16)lo[0], (_Float16)lo[1], (_Float16)lo[2], (_Float16)lo[3],
                   (_Float16)hi[0], (_Float16)hi[1], (_Float16)hi[2], (_Float16)hi[3]};
    }
    __syncthreads();

    const bool vec = in % 4 == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0;
    const float head_b = b3[0];
    const int64_t ntiles = (n + 15) / 16;
    for (int64_t tile = (int64_t)wave * gridDim.x + blockIdx.x; tile < ntiles; tile += 16 * (int64_t)gridDim.x) {
        // this lane's sample (the last tile's missing rows repeat the last row)
        const int64_t row = 16 * tile + r16 < n ? 16 * tile + r16 : n - 1;
        const float *xr = X + row * in;
        h8 xs[KS1];
#pragma unroll
        for (int s = 0; s < KS1; ++s) {
            const int c = 32 * s + 8 * q;
            if (vec && c + 8 <= in) {
                const f4 lo = *reinterpret_cast<const f4 *>(xr + c), hi = *reinterpret_cast<const f4 *>(xr + c + 4);
                xs[s] = h8{(_Float16)lo[0], (_Float16)lo[1], (_Float16)lo[2], (_Float16)lo[3],
                           (_Float16)hi[0], (_Float16)hi[1], (_Float16)hi[2], (_Float16)hi[3]};
            } else {
                xs[s] = weights8(xr, in, 0, c);
            }
        }
        // layer 1, two feature tiles (one k-step of layer 2) at a time
        h8 h1[KS2];
#pragma unroll 1
        for (int s = 0; s < KS2; ++s) {
            h4 half[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int t = 2 * s + h;
                f4 acc = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KS1; ++ks)
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(w1[(t * KS1 + ks) * 64 + lane], xs[ks], acc, 0, 0, 0);
                const f4 bias = *reinterpret_cast<const f4 *>(b1 + 16 * t + 4 * q);
#pragma unroll
                for (int e = 0; e < 4; ++e) half[h][e] = gelu16(acc[e] + bias[e]);
            }
            const h8 op = as_operand(half[0], half[1]);
#pragma unroll
            for (int i = 0; i < KS2; ++i)
                if (i == s) h1[i] = op;
        }
        // layer 2 and the head's products, tiles u, u + 8, u + 4, u + 12 together:
        // the head adds products 128 apart, then 64, 32, 16 (tiles 8, 4, 2, 1 apart),
        // then 8, 4, 2, 1 within a tile
        f4 part[4];
#pragma unroll 1
        for (int g = 0; g < 4; ++g) {
            const int u = g;
            f4 acc[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KS2; ++s)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int t = u + 4 * i;
                    acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w2[(t * KS2 + s) * 64 + lane], h1[s], acc[i], 0, 0,
                                                                    0);
                }
            f4 prod[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int f = 16 * (u + 4 * i) + 4 * q;
                const f4 bias = *reinterpret_cast<const f4 *>(b2 + f), w = *reinterpret_cast<const f4 *>(w3 + f);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    prod[i][e] = (float)gelu16(acc[i][e] + bias[e]) * (float)(_Float16)w[e];
            }
            // tiles 8 apart, then 4 apart
            const f4 sum = (prod[0] + prod[2]) + (prod[1] + prod[3]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (i == g) part[i] = sum;
        }
        f4 v = (part[0] + part[2]) + (part[1] + part[3]);       // tiles 2 apart, then 1 apart
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] += __shfl_xor(v[e], 32);                       // features 8 apart
            v[e] += __shfl_xor(v[e], 16);                       // 4 apart
        }
        const float out = ((v[0] + v[2]) + (v[1] + v[3])) + head_b;
        if (q == 0 && 16 * tile + r16 < n) y[row] = out;
    }
}

}  // namespace

// Inputs beyond 64 would need more LDS than a CU has next to W2; other hidden
// widths take the general products.
bool mlp_predict_ok(const MlpBuffers &m) { return m.hidden == kPH && m.in <= 64; }

hipError_t mlp_predict(const MlpBuffers &m, int cu_count, const float *X, int64_t n, float *y, hipStream_t s) {
    if (!mlp_predict_ok(m) || n < 0 || cu_count < 1) return hipErrorInvalidValue;
    if (n == 0) return hipSuccess;
    // one block per CU (its LDS holds one); fewer when there are fewer tiles
    const int blocks = (int)std::min<int64_t>(cu_count, (n + 15) / 16);
    if (m.in <= 32)
        hipLaunchKernelGGL(mlp_predict_kernel<32>, dim3(blocks), dim3(kPT), 0, s, m.P, m.in, X, n, y);
    else
        hipLaunchKernelGGL(mlp_predict_kernel<64>, dim3(blocks), dim3(kPT), 0, s, m.P, m.in, X, n, y);
    return hipGetLastError();
}

}  // namespace pwa
