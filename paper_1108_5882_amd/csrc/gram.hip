// MC integral matrix of the expanded likelihood (Berger, Section 2, Eq. 3):
//   M_ab = (1/N_gen) sum_j w_j conj(A_ja) A_jb
// While only the production amplitudes V vary, M is fixed; each evaluation
// then needs S = V^H M V and M V (O(k^2)) instead of a pass over the MC rows.
//
// Built once per MC sample.  With the stored row X_j = (Re A_j0, Im A_j0,
// Re A_j1, ...) of 2k reals, G = sum_j w_j X_j X_j^T holds everything:
//   Re M_ab = G[2a][2b] + G[2a+1][2b+1],   Im M_ab = G[2a][2b+1] - G[2a+1][2b],
// a symmetric rank-N update, so it runs on the FP64 matrix cores
// (v_mfma_f64_16x16x4f64 on the 16 x 16 tiles of G's upper triangle).  Products
// of FP32 amplitudes are exact in FP64; every sum is FP64.
#include <utility>

#include "internal.hpp"

namespace pwa {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kGramThreads = 256;
constexpr int kGramWaves = kGramThreads / 64;
// k-steps (of four rows) in flight per stage: fewer where the tiles fill the
// registers, so that two waves fit a SIMD
constexpr int gram_steps(int nt) { return nt == 1 ? 8 : nt <= 3 ? 4 : nt == 4 ? 2 : 1; }
constexpr int kGramMaxTiles = 21;                  // accumulator tiles per wave (168 registers)
constexpr int kGramSlices = 16;                    // threads that share one entry's block sum

// Upper-triangle tiles of the NT x NT grid, numbered row by row.
constexpr int gram_tiles(int nt) { return nt * (nt + 1) / 2; }
constexpr int gram_tile_p(int t, int nt) {
    int p = 0;
    while (t >= nt - p) {
        t -= nt - p;
        ++p;
    }
    return p;
}
constexpr int gram_tile_q(int t, int nt) {
    int p = 0;
    while (t >= nt - p) {
        t -= nt - p;
        ++p;
    }
    return p + t;
}
int gram_nt(int k) { return (2 * k + 15) / 16; }

template <int NT, int T0, int... I>
__device__ __forceinline__ void gram_mfma(d4 *acc, const double *wx, const double *x,
                                          std::integer_sequence<int, I...>) {
    ((acc[I] = __builtin_amdgcn_mfma_f64_16x16x4f64(
          wx[std::integral_constant<int, gram_tile_p(T0 + I, NT)>::value],
          x[std::integral_constant<int, gram_tile_q(T0 + I, NT)>::value], acc[I], 0, 0, 0)),
     ...);
}

// Tiles T0 .. T0 + NTL - 1 of G over the block's rows.  Both operands of a
// tile come straight from the stored row: lane (er, ec) of a k-step feeds row
// 4 s + er, real column 16 c + ec of every column block c, which is the
// instruction's A operand (row index ec) and its B operand (column ec) alike,
// so nothing passes through LDS and each element is loaded once per wave.
// Weights multiply the A operand (W: there are weights).
//
// Bound: the FP64 matrix cores from 2 tiles on (K = 24 takes 6 instructions of
// 64 cycles per four rows), HBM below.  While an FP64 MFMA runs, its SIMD issues
// no vector instruction of any wave (measured: eight integer additions per MFMA
// take it from 66 to 88 cycles, eight FP64 FMAs to 104), so the loop holds little
// else: stages that exist whole take a wave-uniform base and fixed lane offsets,
// without clamps or masks, and the columns past the row are read as column 0
// (they reach only entries of G past 2k, which nobody reads).  10^6 rows: 31 us
// at K = 16, 56 us at K = 24 (55 TFLOP/s executed, 70% of the FP64 peak; 71 us
// with clamped and masked loads), 178 us at K = 48; rows staged in LDS with one
// thread per entry of M and five LDS reads per two products took 519 us at K = 24.
template <typename T, int NT, int T0, int NTL, bool W>
__global__ __launch_bounds__(kGramThreads) void gram_partial_kernel(const T *__restrict__ A,
                                                                    const T *__restrict__ w, int64_t n, int64_t ld,
                                                                    int ntu, double *__restrict__ partials) {
    constexpr int STEPS = gram_steps(NT), STAGE = 4 * STEPS;    // STAGE: rows of one wave's stage
    __shared__ double red[NTL * 256];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int er = lane >> 4, ec = lane & 15;
    const int width = (int)(2 * ld);                            // reals per row
    unsigned off[NT];                                           // bytes from the k-step's first row
#pragma unroll
    for (int c = 0; c < NT; ++c)
        off[c] = (unsigned)((er * width + (16 * c + ec < width ? 16 * c + ec : 0)) * (int)sizeof(T));
    d4 acc[NTL];
#pragma unroll
    for (int i = 0; i < NTL; ++i) acc[i] = d4{0.0, 0.0, 0.0, 0.0};

    T x[STEPS][NT], wt[STEPS];
    auto fetch = [&](int64_t st) {                              // stage st exists whole
        const char *base = reinterpret_cast<const char *>(A + st * STAGE * width);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
#pragma unroll
            for (int c = 0; c < NT; ++c)
                x[s][c] = *reinterpret_cast<const T *>(base + (int64_t)(4 * s) * width * (int)sizeof(T) + off[c]);
            if constexpr (W) wt[s] = (w + (st * STAGE + 4 * s))[(unsigned)er];
        }
    };
    auto multiply = [&](const double (&xd)[NT], double wd) {
        if constexpr (W) {
            double wx[NT];
#pragma unroll
            for (int c = 0; c < NT; ++c) wx[c] = wd * xd[c];
            gram_mfma<NT, T0>(acc, wx, xd, std::make_integer_sequence<int, NTL>{});
        } else {
            gram_mfma<NT, T0>(acc, xd, xd, std::make_integer_sequence<int, NTL>{});
        }
    };
    // whole stages dealt to the waves of the grid in turn, the next one's loads
    // ahead of the MFMAs
    const int64_t nfull = n / STAGE, nwaves = (int64_t)gridDim.x * kGramWaves;
    int64_t st = (int64_t)blockIdx.x * kGramWaves + wave;
    if (st < nfull) fetch(st);
    for (; st < nfull; st += nwaves) {
        double xd[STEPS][NT], wd[STEPS];
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
#pragma unroll
            for (int c = 0; c < NT; ++c) xd[s][c] = (double)x[s][c];
            if constexpr (W) wd[s] = (double)wt[s];
        }
        if (st + nwaves < nfull) fetch(st + nwaves);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) multiply(xd[s], W ? wd[s] : 1.0);
    }
    // the rows after the last whole stage: one wave, rows past the sample count as zero
    if (st == nfull) {
        for (int64_t r0 = nfull * STAGE; r0 < n; r0 += 4) {
            const bool in = r0 + er < n;
            const char *row = reinterpret_cast<const char *>(A + (r0 - (in ? 0 : er)) * width);
            double xd[NT];
#pragma unroll
            for (int c = 0; c < NT; ++c) {
                const T v = *reinterpret_cast<const T *>(row + off[c]);
                xd[c] = in ? (double)v : 0.0;
            }
            multiply(xd, W && in ? (double)w[r0 + er] : 0.0);
        }
    }
    // the waves' tiles added in wave order; item j of a lane is row er + 4 j, column ec
#pragma unroll
    for (int v = 0; v < kGramWaves; ++v) {
        if (v > 0) __syncthreads();
        if (wave == v) {
#pragma unroll
            for (int i = 0; i < NTL; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    double &g = red[i * 256 + (er + 4 * j) * 16 + ec];
                    g = v == 0 ? acc[i][j] : g + acc[i][j];
                }
        }
    }
    __syncthreads();
    double *out = partials + ((int64_t)blockIdx.x * ntu + T0) * 256;
    for (int i = tid; i < NTL * 256; i += kGramThreads) out[i] = red[i];
}

// M from the block partials.  A workgroup forms four entries M_ab (a <= b) and
// their conjugates: each needs the 2 x 2 block of G at (2a, 2b), which lies in
// one tile, so 16 entries of G are summed by 16 threads each (thread r adds
// blocks r, r + 16, ... in block order with 32 loads in flight, then the 16
// sums in r order).  One thread per entry adding every block in turn took
// 123 us for 512 blocks at K = 24.
__global__ __launch_bounds__(256) void gram_finish_kernel(const double *__restrict__ partials, int nblocks, int k,
                                                          int nt, double inv_ngen, double *__restrict__ M) {
    __shared__ double part[kGramSlices][16];
    const int tid = threadIdx.x, el = tid & 15, r = tid >> 4;
    const int o = blockIdx.x * 4 + (el >> 2), a = o / k, b = o % k;
    const bool mine = a < k && a <= b;
    const int gr = 2 * a + ((el >> 1) & 1), gc = 2 * b + (el & 1);
    double s = 0.0;
    if (mine) {
        const int p = gr >> 4, q = gc >> 4;
        const int64_t stride = (int64_t)gram_tiles(nt) * 256;
        const double *src = partials + (p * nt - p * (p - 1) / 2 + (q - p)) * 256 + (gr & 15) * 16 + (gc & 15);
        for (int b0 = r; b0 < nblocks; b0 += 32 * kGramSlices) {
            double v[32];
#pragma unroll
            for (int u = 0; u < 32; ++u) {
                const int i = b0 + u * kGramSlices;
                v[u] = i < nblocks ? src[i * stride] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 32; ++u) s += v[u];
        }
    }
    part[r][el] = s;
    __syncthreads();
    if (r == 0) {
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < kGramSlices; ++q) t += part[q][el];
        part[0][el] = t;
    }
    __syncthreads();
    if (r == 0 && (el & 3) == 0 && mine) {
        const double *g = &part[0][el];             // rr, ri, ir, ii
        const double re = (g[0] + g[3]) * inv_ngen;
        const double im = a == b ? 0.0 * re : (g[1] - g[2]) * inv_ngen;
        M[2 * (a * k + b)] = re;
        M[2 * (a * k + b) + 1] = im;
        M[2 * (b * k + a)] = re;
        M[2 * (b * k + a) + 1] = -im;
    }
}

template <typename T, int NT, int T0>
hipError_t launch_tiles(const T *A, const T *w, int64_t n, int64_t ld, double *partials, int blocks, hipStream_t s) {
    constexpr int NTU = gram_tiles(NT), NG = (NTU + kGramMaxTiles - 1) / kGramMaxTiles, NTLM = (NTU + NG - 1) / NG;
    constexpr int NTL = NTU - T0 < NTLM ? NTU - T0 : NTLM;
    if (w)
        hipLaunchKernelGGL((gram_partial_kernel<T, NT, T0, NTL, true>), dim3(blocks), dim3(kGramThreads), 0, s, A, w, n,
                           ld, NTU, partials);
    else
        hipLaunchKernelGGL((gram_partial_kernel<T, NT, T0, NTL, false>), dim3(blocks), dim3(kGramThreads), 0, s, A, w,
                           n, ld, NTU, partials);
    const hipError_t e = hipGetLastError();
    if constexpr (T0 + NTLM < NTU) {
        if (e == hipSuccess) return launch_tiles<T, NT, T0 + NTLM>(A, w, n, ld, partials, blocks, s);
    }
    return e;
}

template <typename T>
hipError_t launch_partial(const T *A, const T *w, int64_t n, int64_t ld, int k, double *partials, int blocks,
                          hipStream_t s) {
    switch (gram_nt(k)) {
        case 1: return launch_tiles<T, 1, 0>(A, w, n, ld, partials, blocks, s);
        case 2: return launch_tiles<T, 2, 0>(A, w, n, ld, partials, blocks, s);
        case 3: return launch_tiles<T, 3, 0>(A, w, n, ld, partials, blocks, s);
        case 4: return launch_tiles<T, 4, 0>(A, w, n, ld, partials, blocks, s);
        case 5: return launch_tiles<T, 5, 0>(A, w, n, ld, partials, blocks, s);
        case 6: return launch_tiles<T, 6, 0>(A, w, n, ld, partials, blocks, s);
        case 7: return launch_tiles<T, 7, 0>(A, w, n, ld, partials, blocks, s);
        case 8: return launch_tiles<T, 8, 0>(A, w, n, ld, partials, blocks, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

// Two blocks per CU keep the matrix cores fed; up to 16 waves, bound by HBM
// instead, four keep more loads in flight.  Fewer where a wave would get less
// than 16 rows.
int gram_blocks(int cu_count, int k, int64_t n) {
    const int64_t need = (n + 16 * kGramWaves - 1) / (16 * kGramWaves);
    return (int)std::max<int64_t>(1, std::min<int64_t>((gram_nt(k) <= 2 ? 4 : 2) * (int64_t)cu_count, need));
}

size_t gram_partial_doubles(int k, int blocks) { return (size_t)blocks * gram_tiles(gram_nt(k)) * 256; }

hipError_t launch_gram(pwa_prec prec, const void *A, const void *w, int64_t n, int64_t ld, int k,
                       double n_gen, double *partials, int blocks, double *M, hipStream_t stream) {
    if (k < 1 || k > PWA_MAX_K || ld < k || n < 1 || blocks < 1) return hipErrorInvalidValue;
    const hipError_t e = prec == PWA_F32
                             ? launch_partial(static_cast<const float *>(A), static_cast<const float *>(w), n, ld, k,
                                              partials, blocks, stream)
                             : launch_partial(static_cast<const double *>(A), static_cast<const double *>(w), n, ld, k,
                                              partials, blocks, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(gram_finish_kernel, dim3((k * k + 3) / 4), dim3(256), 0, stream, partials, blocks, k,
                       gram_nt(k), 1.0 / n_gen, M);
    return hipGetLastError();
}

}  // namespace pwa
