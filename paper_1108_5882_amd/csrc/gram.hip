// MC integral matrix of the expanded likelihood (Berger, Section 2, Eq. 3):
//   M_ab = (1/N_gen) sum_j w_j conj(A_ja) A_jb
// While only the production amplitudes V vary, M is fixed; each evaluation
// then needs S = V^H M V and M V (O(k^2)) instead of a pass over the MC rows.
//
// Built once per MC sample: every block takes one contiguous chunk of rows and
// adds each entry's terms in row order in FP64 (products of FP32 amplitudes are
// exact in FP64); a second kernel adds the block partials in block order and
// divides by N_gen.
//
// The order of these sums is kept: a fit in Gram form carries the last bits of
// M through its iterations (24 L-BFGS iterations from 200 starts turned a
// difference of 1e-16 into 2e-5 of the result), so a sum in another order, as
// the FP64 matrix cores make it, gives another trajectory.  (They would take
// 63 us instead of 185 us for 10^6 weighted rows at K = 24.)
#include "internal.hpp"

namespace pwa {
namespace {

constexpr int kGramRows = 32;       // rows per stage (two stages in LDS)

// Shapes by the number of waves: tiles of TA x TB entries, the row length KP of a
// stage in LDS (fixed, so that its reads take immediate offsets), threads of a
// chunk (at most) and chunks side by side in a block, rows whose operands are read
// ahead of the arithmetic, and values a thread stages (at most).
struct GramShape {
    int ta, tb, kp, threads, chunks, ahead, per;
};
constexpr GramShape kGramShapes[4] = {
    {1, 1, 8, 64, 2, 8, 4}, {1, 2, 20, 128, 2, 4, 8}, {2, 2, 32, 192, 2, 4, 8}, {2, 2, 64, 576, 1, 2, 8}};

typedef double d2 __attribute__((ext_vector_type(2)));

// N consecutive complex values of a row in LDS: two FP32 ones in one 16-byte read
// (N = 2 starts at an even column of an even row length).
template <typename V, int N>
__device__ __forceinline__ void read_tile(V (&v)[N], const V *p) {
    if constexpr (N == 2 && sizeof(V) == 8) {
        typedef float f4 __attribute__((ext_vector_type(4)));
        const f4 q = *reinterpret_cast<const f4 *>(p);
        v[0] = V{q.x, q.y};
        v[1] = V{q.z, q.w};
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = p[i];
    }
}

// Tiles of TA x TB entries that hold an entry of the upper triangle: row tile
// ti has the column tiles from (ti TA) / TB on.
constexpr int gram_tiles(int k, int ta, int tb) {
    int n = 0;
    for (int ti = 0; ti * ta < k; ++ti) n += (k + tb - 1) / tb - ti * ta / tb;
    return n;
}

// One thread per tile of TA x TB entries of M's upper triangle (a <= b), all
// rows of the block's chunk in order.  The rows pass through LDS as stored, two
// stages of 32 rows, the next one loaded while the current one is used; the
// lower triangle is the conjugate (for FP64 amplitudes its imaginary part is
// summed on its own: there the products round).
//
// Bound: FP64 vector arithmetic of few waves (6 TA TB operations and the
// conversions of TA + TB values per row and tile, some 4.4 cycles each): the
// number of chunks is fixed by the order of the sums, and larger tiles, which
// need fewer LDS reads, leave SIMDs without a wave.  Up to K = 32 two chunks
// share a block, so that their waves spread over all four SIMDs of a CU.
// 10^6 weighted rows at K = 24: 185 us; 519 us when each thread summed single
// entries of the full matrix, five LDS reads per entry and row.  Unweighted:
// 71 us at K = 8, 118 us at 16, 166 us at 24, 283 us at 32, 515 us at 48.
template <typename T, int SH, bool W>
__global__ __launch_bounds__(kGramShapes[SH].threads * kGramShapes[SH].chunks) void
gram_partial_kernel(const T *__restrict__ A, const T *__restrict__ w, int64_t n, int64_t ld, int k, int nchunks,
                    int per_block, double *__restrict__ partials) {
    typedef T t2 __attribute__((ext_vector_type(2)));
    extern __shared__ d2 lds_raw[];                // rows [2][kGramRows][KP] as stored, then the weights [2][kGramRows]
    constexpr bool LOWER = sizeof(T) == 8;
    constexpr int TA = kGramShapes[SH].ta, TB = kGramShapes[SH].tb, KP = kGramShapes[SH].kp;
    constexpr int U = kGramShapes[SH].ahead, PER = kGramShapes[SH].per;
    constexpr int UNITS = 2 * kGramRows * KP + 2 * kGramRows * 8 / (int)(2 * sizeof(T));     // of LDS per chunk
    // one or two chunks per block: the threads of a chunk are whole waves
    const int nt = blockDim.x / per_block, side = threadIdx.x / nt, tid = threadIdx.x - side * nt;
    const int kp = (k + 1) & ~1;                   // columns staged (an even number)
    t2 *lds = reinterpret_cast<t2 *>(lds_raw) + side * UNITS;
    const int chunk_id = blockIdx.x * per_block + side;
    double *lw = reinterpret_cast<double *>(lds + 2 * kGramRows * KP);
    const int64_t chunk = (n + nchunks - 1) / nchunks;
    const int64_t r0 = (int64_t)chunk_id * chunk;
    const int64_t r1 = chunk_id >= nchunks ? r0 : r0 + chunk < n ? r0 + chunk : n;
    // this thread's tile
    int a0 = 0, left = tid;
    const int ncol = (k + TB - 1) / TB;
    while (a0 < k && left >= ncol - a0 / TB) {
        left -= ncol - a0 / TB;
        a0 += TA;
    }
    const bool live = a0 < k;
    const int b0 = live ? (a0 / TB + left) * TB : 0;
    if (!live) a0 = 0;

    double sr[TA][TB], si[TA][TB], sl[TA][TB];
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) sr[i][j] = si[i][j] = sl[i][j] = 0.0;

    // The values this thread stages: row of the stage, offset in the sample and place
    // in LDS (a padding column reads the row's first value and stores zero; a thread
    // past the stage's values repeats the stage's first).  Rows past the chunk are
    // read as its first row and not used: no load hangs on a branch, at whose join
    // the compiler would wait for it.
    t2 x[PER];
    T wr = T(1);
    int xr[PER], xo[PER], xl[PER];
    bool pad[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int e = tid + i * nt < kGramRows * kp ? tid + i * nt : 0;
        xr[i] = e / kp;
        const int c = e - xr[i] * kp;
        pad[i] = c >= k;
        xo[i] = 2 * (int)(xr[i] * ld + (pad[i] ? 0 : c));
        xl[i] = xr[i] * KP + c;
    }
    const T *wl = W ? w : A;
    auto load = [&](int64_t base) {
        const T *src = A + 2 * base * ld;
        const int rows = r1 - base < kGramRows ? (int)(r1 - base) : kGramRows;
#pragma unroll
        for (int i = 0; i < PER; ++i) x[i] = *reinterpret_cast<const t2 *>(src + (xr[i] < rows ? xo[i] : 0));
        if constexpr (W) wr = wl[base + (tid < rows ? tid : 0)];
    };
    auto stage = [&](int b) {
#pragma unroll
        for (int i = 0; i < PER; ++i) lds[b * kGramRows * KP + xl[i]] = pad[i] ? t2{} : x[i];
        if constexpr (W)
            if (tid < kGramRows) lw[b * kGramRows + tid] = (double)wr;
    };
    if (r0 < r1) {
        load(r0);
        stage(0);
    }
    __syncthreads();
    int b = 0;
    // every thread of the block makes the trips of a whole chunk
    for (int64_t base = r0; base < r0 + chunk; base += kGramRows, b ^= 1) {
        if (base + kGramRows < r1) load(base + kGramRows);
        struct Row {
            t2 a[TA], b[TB];
            double w;
        };
        const t2 *stg = lds + b * kGramRows * KP;
        const double *pw = lw + b * kGramRows;
        auto fetch = [&](Row &v, int r) {
            read_tile(v.a, stg + r * KP + a0);
            read_tile(v.b, stg + r * KP + b0);
            v.w = W ? pw[r] : 1.0;
        };
        auto add = [&](const Row &v) {
#pragma unroll
            for (int i = 0; i < TA; ++i)
#pragma unroll
                for (int j = 0; j < TB; ++j) {
                    // conj(A_a) A_b = (ar br + ai bi) + i (ar bi - ai br)
                    const double ar = v.a[i].x, ai = v.a[i].y, br = v.b[j].x, bi = v.b[j].y;
                    const double pr = fma(ar, br, ai * bi);
                    const double pi = fma(ar, bi, -(ai * br));
                    sr[i][j] = W ? fma(v.w, pr, sr[i][j]) : sr[i][j] + pr;
                    si[i][j] = W ? fma(v.w, pi, si[i][j]) : si[i][j] + pi;
                    if constexpr (LOWER) {
                        const double pl = fma(br, ai, -(bi * ar));
                        sl[i][j] = W ? fma(v.w, pl, sl[i][j]) : sl[i][j] + pl;
                    }
                }
        };
        if (live && base < r1) {
            if (r1 - base >= kGramRows) {
                Row cur[U], nxt[U];
#pragma unroll
                for (int u = 0; u < U; ++u) fetch(cur[u], u);
#pragma unroll
                for (int r = 0; r < kGramRows; r += U) {
                    if (r + U < kGramRows) {
#pragma unroll
                        for (int u = 0; u < U; ++u) fetch(nxt[u], r + U + u);
                    }
                    __builtin_amdgcn_sched_barrier(0);      // the reads stay ahead of the arithmetic
#pragma unroll
                    for (int u = 0; u < U; ++u) add(cur[u]);
#pragma unroll
                    for (int u = 0; u < U; ++u) cur[u] = nxt[u];
                }
            } else {
                for (int r = 0; r < (int)(r1 - base); ++r) {
                    Row v;
                    fetch(v, r);
                    add(v);
                }
            }
        }
        if (base + kGramRows < r1) stage(b ^ 1);
        __syncthreads();
    }
    if (!live || chunk_id >= nchunks) return;
    double *out = partials + (int64_t)chunk_id * 2 * k * k;
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) {
            const int a = a0 + i, c = b0 + j;
            if (a < k && c < k && a <= c) {
                out[2 * (a * k + c)] = sr[i][j];
                out[2 * (a * k + c) + 1] = si[i][j];
                if (LOWER && a < c) out[2 * (c * k + a) + 1] = sl[i][j];
            }
        }
}

// M from the block partials: a workgroup takes 16 consecutive numbers of the
// k x k complex matrix, stages their partials of 256 blocks at a time in LDS (16
// loads in flight per thread) and adds them in block order.  The numbers that the
// first kernel did not store come from their conjugates.  One thread per number
// adding 512 partials in memory took 123 us.
constexpr int kGramFinish = 256;
__global__ __launch_bounds__(kGramFinish) void gram_finish_kernel(const double *__restrict__ partials, int nblocks,
                                                                  int k, int lower, double inv_ngen,
                                                                  double *__restrict__ M) {
    __shared__ double part[kGramFinish][17];
    const int tid = threadIdx.x, el = tid & 15, r = tid >> 4;
    const int kk2 = 2 * k * k, e = blockIdx.x * 16 + el;
    const int a = e / 2 / k, b = e / 2 % k, c = e & 1;
    const bool mine = e < kk2 && (a <= b || (lower && c));
    double s = 0.0;
    for (int b0 = 0; b0 < nblocks; b0 += kGramFinish) {
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int i = b0 + r + 16 * u;
            v[u] = mine && i < nblocks ? partials[(int64_t)i * kk2 + e] : 0.0;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 16; ++u) part[r + 16 * u][el] = v[u];
        __syncthreads();
        if (r == 0) {
            const int cnt = nblocks - b0 < kGramFinish ? nblocks - b0 : kGramFinish;
            int i = 0;
            for (; i + 16 <= cnt; i += 16) {
#pragma unroll
                for (int u = 0; u < 16; ++u) s += part[i + u][el];
            }
            for (; i < cnt; ++i) s += part[i][el];
        }
    }
    if (r != 0 || !mine) return;
    const double m = s * inv_ngen;
    M[e] = m;
    if (a < b) {                                    // the conjugate's real part, and its imaginary part if not stored
        if (c == 0) M[2 * (b * k + a)] = m;
        else if (!lower) M[2 * (b * k + a) + 1] = -m;
    }
}

template <typename T, int SH>
hipError_t launch_partial(const T *A, const T *w, int64_t n, int64_t ld, int k, double *partials, int blocks,
                          hipStream_t s) {
    constexpr GramShape S = kGramShapes[SH];
    const int threads = (gram_tiles(k, S.ta, S.tb) + 63) / 64 * 64, kp = (k + 1) & ~1;
    if (threads > S.threads || kp > S.kp || kGramRows * kp > S.per * threads) return hipErrorInvalidValue;
    const int per = blocks > 1 ? S.chunks : 1;
    const dim3 grid((blocks + per - 1) / per), block(per * threads);
    const size_t lds = per * (2 * sizeof(T) * 2 * kGramRows * S.kp + sizeof(double) * 2 * kGramRows);
    if (w)
        hipLaunchKernelGGL((gram_partial_kernel<T, SH, true>), grid, block, lds, s, A, w, n, ld, k, blocks, per,
                           partials);
    else
        hipLaunchKernelGGL((gram_partial_kernel<T, SH, false>), grid, block, lds, s, A, w, n, ld, k, blocks, per,
                           partials);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_pass(const T *A, const T *w, int64_t n, int64_t ld, int k, double *partials, int blocks,
                       hipStream_t s) {
    // small matrices take smaller tiles, so that a chunk's entries reach two waves
    if (k <= 8) return launch_partial<T, 0>(A, w, n, ld, k, partials, blocks, s);
    if (k <= 20) return launch_partial<T, 1>(A, w, n, ld, k, partials, blocks, s);
    if (k <= 32) return launch_partial<T, 2>(A, w, n, ld, k, partials, blocks, s);
    return launch_partial<T, 3>(A, w, n, ld, k, partials, blocks, s);
}

}  // namespace

size_t gram_partial_doubles(int k, int blocks) { return (size_t)blocks * 2 * k * k; }

hipError_t launch_gram(pwa_prec prec, const void *A, const void *w, int64_t n, int64_t ld, int k,
                       double n_gen, double *partials, int blocks, double *M, hipStream_t stream) {
    if (k < 1 || k > PWA_MAX_K || blocks < 1) return hipErrorInvalidValue;
    const hipError_t e = prec == PWA_F32 ? launch_pass(static_cast<const float *>(A), static_cast<const float *>(w), n,
                                                       ld, k, partials, blocks, stream)
                                         : launch_pass(static_cast<const double *>(A), static_cast<const double *>(w),
                                                       n, ld, k, partials, blocks, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(gram_finish_kernel, dim3((2 * k * k + 15) / 16), dim3(kGramFinish), 0, stream, partials, blocks, k,
                       prec == PWA_F64 ? 1 : 0, 1.0 / n_gen, M);
    return hipGetLastError();
}

}  // namespace pwa
