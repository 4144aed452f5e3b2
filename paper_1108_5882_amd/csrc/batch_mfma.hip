// Many production vectors at once on the matrix cores (Berger, Section 2:
// repeated fits from many starting points; Eq. 1-3 for each vector).
//
// For nv vectors the per-event coherent sums of all vectors form a dense
// contraction: with A_r the N x 2K real view of the amplitude rows
// (re, im interleaved) and W the 2K x 2nv real matrix whose columns for V_b
// are (Re V_b, -Im V_b) and (Im V_b, Re V_b) interleaved per wave,
//     Z = A_r W            (Re z_ib, Im z_ib in columns 2b, 2b + 1).
// The adjoint sums are a second contraction over events,
//     P = U^T A_r,  U_ib = z_ib / I_ib (data) or w_i z_ib (MC),
//     Re G_ba = P[ur_b, 2a] + P[ui_b, 2a+1],  Im G_ba = P[ui_b, 2a] - P[ur_b, 2a+1].
// Both run on v_mfma_f32_16x16x32_* in one kernel per event tile; U never
// leaves registers: the forward's output layout is the adjoint's A operand
// once the adjoint's event order is permuted the same way in both operands.
//
// Operand planes: the split amplitudes do not depend on V, so they are formed
// once per sample (batch_planes_kernel) in the order and layout the tile's LDS
// buffers take them, 32-event tiles one after another; per tile a block
// copies them to LDS with 16-byte loads and stores and no conversion.
//
// Arithmetic (split): the forward uses two-term FP16 splits (hi + lo) of the
// amplitudes, scaled by a power of two per wave, and of W, scaled by a power
// of two per column: products hi*hi + hi*lo + lo*hi, 22-bit operands.  The
// adjoint uses two-term BF16 splits of U and of the amplitudes (BF16 keeps
// FP32's range, so the unbounded z/I needs no scale): 3 products.  MFMA
// accumulation is FP32 within a block; each block covers at most
// kTilesPerBlock tiles of one sample (spread evenly over whole rounds of
// compute units) and writes FP64 partials per vector,
// which a second kernel adds in block order (FP64) before forming NLL and
// gradient per vector.
#include "internal.hpp"
#include "lane_ops.hpp"
#include "lbfgs_device.hpp"
#include "row_norm.hpp"

#include <algorithm>
#include <cmath>

// v_writelane_b32 (the LLVM intrinsic): writes a wave-uniform value into one lane
// of a register, leaving the other lanes as they are
__device__ unsigned writelane_u32(unsigned v, int lane, unsigned old) __asm("llvm.amdgcn.writelane.i32");

namespace pwa {
namespace {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));

constexpr int kTile = 32;          // events per tile (two 16-row MFMA tiles)
constexpr int kWaves = 8;          // waves per block
constexpr int kThreads = 64 * kWaves;

__device__ __forceinline__ int dpp_xor1(int x) {
    return __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
}
__device__ __forceinline__ float xor1_f(float x) { return __int_as_float(dpp_xor1(__float_as_int(x))); }

// Block b covers tiles [b tpb, (b + 1) tpb) of one segment (SEG: 0 data,
// 1 MC) for the vectors of blockIdx.y; each wave takes VPW = 8 CT vectors
// (2 CT real columns in CT column tiles: re and im of 16 vectors per tile
// pair).  Lanes of vectors past nv compute on zero weights and are never
// written out; only the last, partial tile of the data segment masks events
// (an absent data row would give z = 0 and a non-finite z / I, while an absent
// MC row has weight 0).
template <int KS, int CT>
struct BatchSmem {
    static constexpr int K2 = 32 * KS;          // padded real width
    // row stride (halfs) of the row-major FP16 planes: 16 halfs of padding (measured:
    // fewer LDS bank conflicts than 8 or 24, none is worse by 3.5x)
    static constexpr int RS16 = K2 + 16;
    static constexpr int RST = kTile + 8;       // row stride (bf16) of the transposed planes (16-byte rows)
    _Float16 ah[kTile * RS16];
    _Float16 al[kTile * RS16];
    __bf16 bh[K2 * RST];
    __bf16 bl[K2 * RST];
    float wts[kTile];
};

// Two LDS buffers (one barrier per tile: the next tile is staged into the
// other buffer after the current one is computed) when they fit in 64 KB.
template <int KS, int CT>
constexpr int batch_buffers() { return 2 * sizeof(BatchSmem<KS, CT>) <= 64 * 1024 ? 2 : 1; }

// REF (data segment only): events whose coherent sum is small against the
// bound |z| <= |V| |A_i| (|Z'|^2 < c^2 t_v^2 |V|^2 |A_i|^2, c^2 = p.cthr2) are
// left out of the sums and marked in p.flags, one 64-bit lane mask per
// (vector group, tile, group g, rt, e), in that order of significance, so the
// words of one vector group over consecutive tiles are contiguous;
// batch_refine_kernel adds them exactly.
template <int KS, int CT, int SEG, bool REF>
__device__ __forceinline__ void batch_block(const BatchArgs &p, BatchSmem<KS, CT> *bufs, int bseg) {
    constexpr int NB = batch_buffers<KS, CT>();
    constexpr int kVPerWave = 8 * CT;
    constexpr int K2 = BatchSmem<KS, CT>::K2;
    constexpr int RS16 = BatchSmem<KS, CT>::RS16;
    constexpr int RST = BatchSmem<KS, CT>::RST;
    constexpr int kChunks = 16 * K2;            // 16-byte chunks of a tile's four planes
    constexpr int kPer = (kChunks + kThreads - 1) / kThreads;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int q = lane >> 4, r16 = lane & 15;
    const int64_t n = p.n[SEG];
    const float *A = p.A[SEG];
    const float *w = SEG ? p.w : nullptr;
    const int64_t tile0 = (int64_t)bseg * p.tpb;
    const int64_t ntiles = (n + kTile - 1) / kTile;
    const int64_t tile1 = tile0 + p.tpb < ntiles ? tile0 + p.tpb : ntiles;
    const int vg = (int)blockIdx.y * kWaves + wave;          // this wave's vector group
    const int v0 = vg * kVPerWave;
    const bool active = v0 < p.nv;                           // wave-uniform
    constexpr bool kRef = REF && SEG == 0;
    // flag thresholds of this lane's vectors: c^2 t_v^2 |V|^2 (-1 for vectors past nv),
    // and 1 / t_v^2 (a power of two): the log is taken of the unscaled I = I' / t_v^2,
    // whose magnitude keeps the FP32 log and the FP32 tile sums accurate
    float thr[CT / 2], inv_t2[CT / 2];
#pragma unroll
    for (int g = 0; g < CT / 2; ++g) {
        thr[g] = -1.f;
        inv_t2[g] = 1.f;
        const int v = v0 + 16 * g + r16;
        if (SEG == 0 && v < p.nv) {
            const double tv = p.vscale[2 * v], n2 = p.vscale[2 * v + 1];
            inv_t2[g] = (float)(1.0 / (tv * tv));
            if (kRef) thr[g] = (float)((double)p.cthr2 * tv * tv * n2);
        }
    }

    // forward weights of this wave's vectors, fragment order [hi/lo][ct][ks][lane]
    h8 wh[CT][KS], wl[CT][KS];
    {
        const h8 *src = reinterpret_cast<const h8 *>(p.wfrag) + (int64_t)vg * 2 * CT * KS * 64;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                wh[ct][ks] = src[((0 * CT + ct) * KS + ks) * 64 + lane];
                wl[ct][ks] = src[((1 * CT + ct) * KS + ks) * 64 + lane];
            }
    }

    // adjoint accumulators D[ct][rtile]: lane holds rows 4q+e (columns of U) x col r16 (real)
    f4 D[CT][2 * KS];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int rt = 0; rt < 2 * KS; ++rt) D[ct][rt] = f4{0.f, 0.f, 0.f, 0.f};
    double tsum[CT / 2];            // per lane: sum over its events for vectors 16g + r16
#pragma unroll
    for (int g = 0; g < CT / 2; ++g) tsum[g] = 0.0;

    const int nreal = 2 * p.k;                      // real columns present in a row
    // The next tile's operand planes are loaded into registers while the current
    // tile is computed; each thread holds kPer 16-byte chunks and one MC weight.
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    const u4 *planes = static_cast<const u4 *>(p.planes[SEG]);
    u4 xr[kPer];
    float wr = 0.f;
    auto load_tile = [&](int64_t t) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int c = tid + i * kThreads;
            if (c < kChunks) {
                typedef const u4 __attribute__((address_space(1))) *gptr;
                xr[i] = __builtin_nontemporal_load((gptr)(planes + t * kChunks + c));
            }
        }
        if ((SEG || kRef) && tid < kTile) {
            const int64_t row = t * kTile + tid;
            wr = row < n ? (SEG ? (w ? w[row] : 1.f) : p.rnorm[row]) : 0.f;
        }
    };

    // epilogue of one tile: per (event, vector) I, log2 I (data) or w I (MC),
    // and U = z / I (data) or w z (MC), split into BF16 hi/lo in the adjoint's
    // operand order (slot 4 rt + e holds event 16 rt + 4 q + e)
    // (column group g: column tiles 2g and 2g + 1, vectors 16 g + r16)
    auto epilogue = [&](const float (&wv)[8], const f4 (&Z)[2][CT], b8 (&uh)[CT], b8 (&ul)[CT], int nvalid,
                        int64_t t, const int g) {
        {
            float ts = 0.f;
            // the flag masks of (g, slot): with one k-step (KS = 1) lane `slot` gathers
            // them for one store per group; with more, registers are short (the
            // gather costs spills) and every lane stores each (wave-uniform) mask to
            // its word, one store instruction with no branch around it (a store by
            // lane 0 alone put an exec-mask branch per slot into the epilogue, whose
            // blocks the scheduler cannot interleave matrix products across)
            unsigned fw_lo = 0u, fw_hi = 0u;
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int slot = 4 * rt + e;
                    const float zr = Z[rt][2 * g][e], zi = Z[rt][2 * g + 1][e];
                    const float I = fmaf(zr, zr, zi * zi);
                    float ur, ui;
                    if (SEG == 0) {
                        const bool absent = nvalid < kTile && 16 * rt + 4 * q + e >= nvalid;
                        const bool flag = kRef && !absent && I < thr[g] * wv[slot];
                        if (kRef) {
                            const unsigned long long mask = __ballot(flag);
                            if constexpr (KS == 1) {
                                fw_lo = writelane_u32((unsigned)mask, slot, fw_lo);
                                fw_hi = writelane_u32((unsigned)(mask >> 32), slot, fw_hi);
                            } else {
                                p.flags[((int64_t)vg * ntiles + t) * (8 * (CT / 2)) + 8 * g + slot] = mask;
                            }
                        }
                        if (absent || flag) {
                            ur = ui = 0.f;
                        } else {
                            ts += __log2f(I * inv_t2[g]);
                            const float rI = __builtin_amdgcn_rcpf(I);
                            ur = zr * rI;
                            ui = zi * rI;
                        }
                    } else {
                        ts = fmaf(wv[slot], I, ts);
                        ur = wv[slot] * zr;
                        ui = wv[slot] * zi;
                    }
                    const __bf16 hr = (__bf16)ur, hi_ = (__bf16)ui;
                    uh[2 * g][slot] = hr;
                    uh[2 * g + 1][slot] = hi_;
                    ul[2 * g][slot] = (__bf16)(ur - (float)hr);
                    ul[2 * g + 1][slot] = (__bf16)(ui - (float)hi_);
                }
            tsum[g] += (double)ts;
            if (kRef && KS == 1 && lane < 8)
                p.flags[((int64_t)vg * ntiles + t) * (8 * (CT / 2)) + 8 * g + lane] =
                    ((unsigned long long)fw_hi << 32) | fw_lo;
        }
    };

    // stage a tile from the registers into buffer b: plane 0 / 1 are the FP16 hi /
    // lo row-major planes (K2 halfs per event), plane 2 / 3 the BF16 hi / lo
    // transposed planes (32 events per real column, in the adjoint's operand
    // order); each 16-byte chunk goes to its place in the padded LDS rows
    auto stage = [&](BatchSmem<KS, CT> &b) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int c = tid + i * kThreads;
            if (c < kChunks) {
                const int plane = c / (4 * K2), u = 8 * (c % (4 * K2));
                u4 *dst;
                if (plane < 2) {
                    const int e = u / K2, r = u % K2;
                    dst = reinterpret_cast<u4 *>((plane == 0 ? b.ah : b.al) + e * RS16 + r);
                } else {
                    const int rr = u / kTile, pos = u % kTile;
                    dst = reinterpret_cast<u4 *>((plane == 2 ? b.bh : b.bl) + rr * RST + pos);
                }
                *dst = xr[i];
            }
        }
        if ((SEG || kRef) && tid < kTile) b.wts[tid] = wr;
    };

    // forward, epilogue and adjoint of the tile in buffer sm
    // forward products of column group g only (used when the groups are interleaved)
    auto forward_g = [&](const BatchSmem<KS, CT> &sm, f4 (&Z)[2][CT], const int g) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                const int off = (16 * rt + r16) * RS16 + 32 * ks + 8 * q;
                const h8 a_h = *reinterpret_cast<const h8 *>(&sm.ah[off]);
                const h8 a_l = *reinterpret_cast<const h8 *>(&sm.al[off]);
#pragma unroll
                for (int ct = 2 * g; ct < 2 * g + 2; ++ct) {
                    Z[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a_h, wh[ct][ks], Z[rt][ct], 0, 0, 0);
                    Z[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a_h, wl[ct][ks], Z[rt][ct], 0, 0, 0);
                    Z[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a_l, wh[ct][ks], Z[rt][ct], 0, 0, 0);
                }
            }
    };
    // adjoint D[ct][rt] += U^T (16 columns x 32 events) . A (32 events x 16 reals) for the
    // column tiles [c0, c1)
    auto adjoint = [&](const BatchSmem<KS, CT> &sm, const b8 (&uh)[CT], const b8 (&ul)[CT], const int c0,
                       const int c1) {
#pragma unroll
        for (int rt = 0; rt < 2 * KS; ++rt) {
            const int rr = 16 * rt + r16;
            const b8 b_h = *reinterpret_cast<const b8 *>(&sm.bh[rr * RST + 8 * q]);
            const b8 b_l = *reinterpret_cast<const b8 *>(&sm.bl[rr * RST + 8 * q]);
#pragma unroll
            for (int ct = c0; ct < c1; ++ct) {
                D[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(uh[ct], b_h, D[ct][rt], 0, 0, 0);
                D[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(uh[ct], b_l, D[ct][rt], 0, 0, 0);
                D[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ul[ct], b_h, D[ct][rt], 0, 0, 0);
            }
        }
    };

    // one tile; nvalid < kTile only for the data segment's last tile
    auto tile_body = [&](const BatchSmem<KS, CT> &sm, int64_t t, const int nvalid) __attribute__((always_inline)) {
        f4 Z[2][CT];
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) Z[rt][ct] = f4{0.f, 0.f, 0.f, 0.f};
        b8 uh[CT], ul[CT];
        float wv[8];                // MC weights, or the rows' |A|^2 when flagging
        auto load_wv = [&]() __attribute__((always_inline)) {
            if (SEG || kRef) {
                const f4 w0 = *reinterpret_cast<const f4 *>(&sm.wts[4 * q]);
                const f4 w1 = *reinterpret_cast<const f4 *>(&sm.wts[16 + 4 * q]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    wv[e] = w0[e];
                    wv[4 + e] = w1[e];
                }
            }
        };

        if constexpr (KS == 1 || CT < 4) {
            // forward of all column tiles (one A fragment load each), epilogue, adjoint
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int rt = 0; rt < 2; ++rt) {
                    const int off = (16 * rt + r16) * RS16 + 32 * ks + 8 * q;
                    const h8 a_h = *reinterpret_cast<const h8 *>(&sm.ah[off]);
                    const h8 a_l = *reinterpret_cast<const h8 *>(&sm.al[off]);
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        Z[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a_h, wh[ct][ks], Z[rt][ct], 0, 0, 0);
                        Z[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a_h, wl[ct][ks], Z[rt][ct], 0, 0, 0);
                        Z[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a_l, wh[ct][ks], Z[rt][ct], 0, 0, 0);
                    }
                }
            load_wv();
            if (nvalid < kTile) {
#pragma unroll
                for (int g = 0; g < CT / 2; ++g) epilogue(wv, Z, uh, ul, nvalid, t, g);
            } else {
#pragma unroll
                for (int g = 0; g < CT / 2; ++g) epilogue(wv, Z, uh, ul, kTile, t, g);
            }
            adjoint(sm, uh, ul, 0, CT);
        } else {
            // two column groups with two or more k-steps: the matrix products of one
            // group are interleaved with the vector epilogue of the other (F0 | F1 with
            // E0 | A0 with E1 | A1), one product per three vector instructions; the two
            // waves sharing a SIMD otherwise run the same phase of a tile
            constexpr int kM = 12 * KS;                 // products per group and direction
            forward_g(sm, Z, 0);
            forward_g(sm, Z, 1);
            load_wv();
            epilogue(wv, Z, uh, ul, nvalid, t, 0);
            adjoint(sm, uh, ul, 0, 2);
            epilogue(wv, Z, uh, ul, nvalid, t, 1);
            adjoint(sm, uh, ul, 2, 4);
#pragma unroll
            for (int i = 0; i < kM; ++i) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
#pragma unroll
            for (int i = 0; i < 2 * kM; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
            }
#pragma unroll
            for (int i = 0; i < kM; ++i) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
    };
    auto compute = [&](const BatchSmem<KS, CT> &sm, int64_t t) {
        const int64_t left = n - t * kTile;
        tile_body(sm, t, (SEG == 0 && left < kTile) ? (int)left : kTile);
    };

    if (tile0 < tile1) load_tile(tile0);
    if (NB == 2) {
        // stage the first tile, then per tile: compute it, stage the next one
        // into the other buffer, load the one after into registers, one barrier
        if (tile0 < tile1) {
            stage(bufs[0]);
            if (tile0 + 1 < tile1) load_tile(tile0 + 1);
        }
        __syncthreads();
        for (int64_t t = tile0; t < tile1; ++t) {
            const int cur = (int)((t - tile0) & 1);
            if (active) compute(bufs[cur], t);
            if (t + 1 < tile1) {
                stage(bufs[cur ^ 1]);
                if (t + 2 < tile1) load_tile(t + 2);
            }
            __syncthreads();
        }
    } else {
        for (int64_t t = tile0; t < tile1; ++t) {
            __syncthreads();
            stage(bufs[0]);
            __syncthreads();
            if (t + 1 < tile1) load_tile(t + 1);
            if (active) compute(bufs[0], t);
        }
    }
    if (!active) return;

    // ---- per-vector scalar sums: lanes r16, r16 + 16, r16 + 32, r16 + 48 share a vector
#pragma unroll
    for (int g = 0; g < CT / 2; ++g) {
        tsum[g] += __shfl_xor(tsum[g], 16);
        tsum[g] += __shfl_xor(tsum[g], 32);
    }
    // partial layout [v][block][1 + 2 ld]: [0] scalar, [1 + 2a + c] complex sums
    const int pst = p.pstride;
    const int nblk = p.nb[0] + p.nb[1];
    if (q == 0) {
#pragma unroll
        for (int g = 0; g < CT / 2; ++g) {
            const int v = v0 + 16 * g + r16;
            if (v < p.nv) p.partials[((int64_t)v * nblk + blockIdx.x) * pst] = tsum[g];
        }
    }
    // gradient sums: lane pairs (2a, 2a+1) in r16 hold the re and im real rows of wave a
#pragma unroll
    for (int g = 0; g < CT / 2; ++g)
#pragma unroll
        for (int rt = 0; rt < 2 * KS; ++rt)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float pr = D[2 * g][rt][e];       // P[ur_v, real r]
                const float pi = D[2 * g + 1][rt][e];   // P[ui_v, real r]
                const float pr_o = xor1_f(pr), pi_o = xor1_f(pi);   // the odd real row
                const int v = v0 + 16 * g + 4 * q + e;
                const int rr = 16 * rt + r16;
                if ((r16 & 1) == 0 && v < p.nv && rr < nreal) {
                    const int a = rr >> 1;
                    double *dst = p.partials + ((int64_t)v * nblk + blockIdx.x) * pst + 1 + 2 * a;
                    dst[0] = (double)pr + (double)pi_o;      // Re G = P[ur, 2a] + P[ui, 2a+1]
                    dst[1] = (double)pi - (double)pr_o;      // Im G = P[ui, 2a] - P[ur, 2a+1]
                }
            }
}

template <int KS, int CT, bool REF>
__global__ __launch_bounds__(kThreads) void nll_batch_kernel(BatchArgs p) {
    __shared__ __attribute__((aligned(16))) BatchSmem<KS, CT> bufs[batch_buffers<KS, CT>()];
    if ((int)blockIdx.x < p.nb[0])
        batch_block<KS, CT, 0, REF>(p, bufs, (int)blockIdx.x);
    else
        batch_block<KS, CT, 1, REF>(p, bufs, (int)blockIdx.x - p.nb[0]);
}

// Exact terms of the flagged data events, in the units of the block partials
// (log2 I, conj(A) z / (I t_v)), added to the partial of their vector and block:
// block (b, y) takes the flag words of data block b's tiles for the vector groups
// 8 y .. 8 y + 7.  A wave takes one group, or with fewer groups than waves a share
// of its vectors.  It reads 512 words at a time and goes through its vectors: the
// vector's flagged events are listed in tile, word and bit order, SG lanes (lane =
// wave a) form each event's z in FP64 from the FP32 amplitudes, like the single-V
// path, 64 / SG events side by side and four such rounds of rows in flight, and
// the terms are added to the partial in list order.  Every partial is updated by
// one wave, in that fixed order.
//
// Bound: latency (flag words, then rows; few events are flagged).  256 vectors at
// K = 32, 2 10^6 data rows, of the cases in perf/cases.py (115,709 events flagged,
// 33,758 of them by one vector): 132 us, and 207 us when one wave per group took one
// event after the other, each with a row load, twelve lane shuffles through LDS and an
// update of the partial in memory.  On the sample of the same size in synth (80,844
// flagged, at most 5,672 by one vector) there is less to put side by side: 106 us, 103
// one after the other.  32 vectors at K = 8 on 4000 rows (one group): 5.6 us on average
// over a fit, 13.3 one after the other.  Not kept: the next 512 words asked for during
// the present ones (155 and 140 us: they queue ahead of the rows).
constexpr int kRefineLoads = 8;                     // flag words per lane and chunk
constexpr int kRefineRounds = 4;                    // rounds of rows in flight
constexpr unsigned long long kEveryRow16 = 0x0001000100010001ull;

template <int CT, int SG>
__global__ __launch_bounds__(kThreads) void batch_refine_kernel(BatchArgs p) {
    constexpr int kVPerWave = 8 * CT;
    constexpr int kWords = 8 * (CT / 2);
    constexpr int E = 64 / SG;                      // events side by side
    __shared__ unsigned short list[kWaves][64 * kRefineLoads * 4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int a = lane & (SG - 1), es = lane / SG;
    // waves per vector group: a power of two
    const int ng = min(kWaves, (p.nv + kVPerWave - 1) / kVPerWave - (int)blockIdx.y * kWaves);
    int sub = 1;
    while (2 * sub * ng <= kWaves) sub *= 2;
    if (wave >= ng * sub) return;
    const int vg = (int)blockIdx.y * kWaves + wave / sub;
    const int c0 = 16 / sub * (wave % sub), c1 = c0 + 16 / sub;      // vectors 16 g + c0 .. 16 g + c1 - 1
    const unsigned long long mine = (((1ull << (c1 - c0)) - 1) << c0) * kEveryRow16;
    const int64_t ntiles = (p.n[0] + kTile - 1) / kTile;
    const int64_t tile0 = (int64_t)blockIdx.x * p.tpb;
    const int64_t tile1 = tile0 + p.tpb < ntiles ? tile0 + p.tpb : ntiles;
    const int nblk = p.nb[0] + p.nb[1], k = p.k;
    unsigned short *events = list[wave];
    const unsigned long long below = (1ull << lane) - 1;
    // the group's words for tiles [tile0, tile1) are contiguous
    const int64_t nwords = (tile1 - tile0) * kWords;
    const unsigned long long *fw = p.flags + ((int64_t)vg * ntiles + tile0) * kWords;
    for (int64_t base = 0; base < nwords; base += 64 * kRefineLoads) {
        unsigned long long mw[kRefineLoads], any = 0;
#pragma unroll
        for (int j = 0; j < kRefineLoads; ++j) {
            const int64_t i = base + 64 * j + lane;
            mw[j] = i < nwords ? fw[i] : 0ull;
        }
#pragma unroll
        for (int j = 0; j < kRefineLoads; ++j) any |= mw[j] &= mine;
        if (!__ballot(any != 0)) continue;
        for (int c = c0; c < c1; ++c) {
            if (!__ballot((any >> c & kEveryRow16) != 0)) continue;
            for (int g = 0; g < CT / 2; ++g) {
                // this vector's bits (word i of a chunk belongs to column group (i % kWords) / 8)
                const bool my_g = lane % kWords / 8 == g;
                int total = 0;
#pragma unroll
                for (int j = 0; j < kRefineLoads; ++j) {
                    const unsigned long long bits = my_g ? mw[j] >> c & kEveryRow16 : 0ull;
                    if (!__ballot(bits != 0)) continue;
                    int at = total, here = 0;
                    unsigned long long row[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        row[q] = __ballot((bits >> (16 * q) & 1) != 0);
                        at += __popcll(row[q] & below);
                        total += __popcll(row[q]);
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (bits >> (16 * q) & 1) events[at + here++] = (unsigned short)((64 * j + lane) * 4 + q);
                }
                if (total == 0) continue;
                // LDS operations of one wave complete in order; the fences keep the compiler's order
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                const int v = vg * kVPerWave + 16 * g + c;
                const double *V = p.V + (int64_t)v * p.vstride;
                const double vr = a < k ? V[2 * a] : 0.0, vi = a < k ? V[2 * a + 1] : 0.0, tv = p.vscale[2 * v];
                double *dst = p.partials + ((int64_t)v * nblk + blockIdx.x) * p.pstride;
                double acc_t = dst[0], acc_r = a < k ? dst[1 + 2 * a] : 0.0, acc_i = a < k ? dst[2 + 2 * a] : 0.0;
                for (int s = 0; s < total; s += E * kRefineRounds) {
                    float2 x[kRefineRounds];
#pragma unroll
                    for (int u = 0; u < kRefineRounds; ++u) {
                        const int i = s + u * E + es;
                        x[u] = float2{0.f, 0.f};
                        if (i < total && a < k) {
                            const int q = events[i] & 3;
                            const int64_t w = base + (events[i] >> 2);
                            const int wi = (int)(w % kWords) % 8;
                            const int64_t r = (tile0 + w / kWords) * kTile + 16 * (wi / 4) + 4 * q + wi % 4;
                            x[u] = *reinterpret_cast<const float2 *>(p.A[0] + 2 * (r * p.ld + a));
                        }
                    }
#pragma unroll
                    for (int u = 0; u < kRefineRounds; ++u) {
                        if (s + u * E >= total) break;
                        const double ar = (double)x[u].x, ai = (double)x[u].y;
                        const double zr = lane_sum<SG>(fma(vr, ar, -(vi * ai)));
                        const double zi = lane_sum<SG>(fma(vr, ai, vi * ar));
                        const double I = fma(zr, zr, zi * zi);
                        const double ur = zr / (I * tv), ui = zi / (I * tv);
                        const double tt = log2(I);
                        const double tr = fma(ar, ur, ai * ui);          // Re conj(A_a) u
                        const double ti = fma(ar, ui, -(ai * ur));       // Im conj(A_a) u
#pragma unroll
                        for (int e = 0; e < E; ++e) {
                            if (s + u * E + e >= total) break;
                            acc_t += E == 1 ? tt : __shfl(tt, e * SG);
                            acc_r += E == 1 ? tr : __shfl(tr, e * SG + a);
                            acc_i += E == 1 ? ti : __shfl(ti, e * SG + a);
                        }
                    }
                }
                if (lane == 0) dst[0] = acc_t;
                if (es == 0 && a < k) {
                    dst[1 + 2 * a] = acc_r;
                    dst[2 + 2 * a] = acc_i;
                }
            }
        }
    }
}

// Operand planes of one sample, tile after tile (4 planes x 32 x K2 values of 2
// bytes per tile): FP16 hi / lo of the amplitudes scaled by the power of two
// of their wave (event-major rows), then BF16 hi / lo of the unscaled
// amplitudes transposed (real-column-major, event e at position
// 8 ((e mod 16) / 4) + (e mod 4) + 4 (e / 16)).  Rows past n and columns past
// 2k hold zeros.
//
// Bound by memory (4 bytes read and 8 written per real column).  A block takes tiles
// in turn: the rows pass through LDS, the next tile's already on their way, and a
// thread forms 16 bytes of a hi and a lo plane from 8 values, so that a wave writes
// whole lines.  LDS rows of K2 + 4 floats keep the reads of 16 columns at 4 event
// groups on distinct banks.  K = 32, 10^7 rows: 1.8 ms; 6.8 ms when a thread wrote the
// 2-byte values of one event and column pair, 64 bytes apart in the transposed planes.
template <int KS>
__global__ __launch_bounds__(256) void batch_planes_kernel(const float *A, int64_t n, int64_t ld, int nreal,
                                                           int64_t ntiles, const float *ascale, unsigned short *out) {
    constexpr int K2 = 32 * KS, ST = K2 + 4, PER = kTile * K2 / 2 / 256;
    typedef unsigned short us8 __attribute__((ext_vector_type(8)));
    typedef float f2r __attribute__((ext_vector_type(2)));
    typedef float f4r __attribute__((ext_vector_type(4)));
    __shared__ __attribute__((aligned(16))) float rows[kTile * ST];
    __shared__ __attribute__((aligned(16))) float scale[K2];
    const int tid = threadIdx.x;
    for (int i = tid; i < K2; i += 256) scale[i] = ascale[i];
    f2r x[PER];
    auto load = [&](int64_t t) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int c = tid + 256 * i, r = 2 * (c % (K2 / 2));
            const int64_t e = t * kTile + c / (K2 / 2);
            // values outside the sample are read from inside it and replaced when they are staged
            x[i] = *reinterpret_cast<const f2r *>(A + 2 * (e < n ? e : n - 1) * ld + (r < nreal ? r : 0));
        }
    };
    int64_t t = blockIdx.x;
    if (t < ntiles) load(t);
    for (; t < ntiles; t += gridDim.x) {
        __syncthreads();                                // the previous tile's reads are done
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int c = tid + 256 * i, r = 2 * (c % (K2 / 2)), e = c / (K2 / 2);
            *reinterpret_cast<f2r *>(rows + e * ST + r) = t * kTile + e < n && r < nreal ? x[i] : f2r{0.f, 0.f};
        }
        __syncthreads();
        if (t + gridDim.x < ntiles) load(t + gridDim.x);
        unsigned short *base = out + t * (128 * (int64_t)K2);
        for (int u = tid; u < 4 * K2; u += 256) {       // event-major: columns 8 j .. 8 j + 7 of one event
            const int e = u / (K2 / 8), r = 8 * (u % (K2 / 8));
            us8 hi, lo;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f4r v = *reinterpret_cast<const f4r *>(rows + e * ST + r + 4 * h) *
                              *reinterpret_cast<const f4r *>(scale + r + 4 * h);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const _Float16 y = (_Float16)v[i];
                    hi[4 * h + i] = __builtin_bit_cast(unsigned short, y);
                    lo[4 * h + i] = __builtin_bit_cast(unsigned short, (_Float16)(v[i] - (float)y));
                }
            }
            *reinterpret_cast<us8 *>(base + e * K2 + r) = hi;
            *reinterpret_cast<us8 *>(base + kTile * K2 + e * K2 + r) = lo;
        }
        for (int u = tid; u < 4 * K2; u += 256) {       // transposed: events 4 q .. and 16 + 4 q .. of one column
            const int r = u >> 2, q = u & 3;
            us8 hi, lo;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float v = rows[(16 * (i >> 2) + 4 * q + (i & 3)) * ST + r];
                const __bf16 y = (__bf16)v;
                hi[i] = __builtin_bit_cast(unsigned short, y);
                lo[i] = __builtin_bit_cast(unsigned short, (__bf16)(v - (float)y));
            }
            *reinterpret_cast<us8 *>(base + 2 * kTile * K2 + r * kTile + 8 * q) = hi;
            *reinterpret_cast<us8 *>(base + 3 * kTile * K2 + r * kTile + 8 * q) = lo;
        }
    }
}

// |A_i|^2 of each row (FP64 sums of the FP32 values, stored as FP32): 8 lanes per
// row, summed over the 8 lanes.  Only the first k complex values count (a borrowed
// sample's padding is not read as data).
__global__ void rownorm_kernel(const float *A, int64_t n, int64_t ld, int k, float *out) {
    typedef float f2r __attribute__((ext_vector_type(2)));
    typedef float f4r __attribute__((ext_vector_type(4)));
    const int sub = threadIdx.x & 7;
    const int64_t groups = (int64_t)gridDim.x * blockDim.x / 8;
    // the 8 lanes of a row share r, so they leave the loop together
    for (int64_t r = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 8; r < n; r += groups) {
        const float *row = A + 2 * r * ld;
        double s = row_norm_share(
            k, ld % 2 == 0, sub, [=](int c) { return reinterpret_cast<const f4r *>(row)[c]; },
            [=](int a) { return reinterpret_cast<const f2r *>(row)[a]; });
        s += __shfl_xor(s, 1);
        s += __shfl_xor(s, 2);
        s += __shfl_xor(s, 4);
        if (sub == 0) out[r] = (float)s;
    }
}

// The FP16 hi + lo pair the forward weights carry for a weight x (scaled by
// t / s); the combine evaluates the same expression to know the weights the
// matrix cores used.
struct WeightSplit {
    _Float16 hi, lo;
};
__device__ __forceinline__ WeightSplit split_weight(double x) {
    const _Float16 hi = (_Float16)(float)x;
    return WeightSplit{hi, (_Float16)(float)(x - (double)(float)hi)};
}

// Forward weights of one vector by one wave: lane i holds elements i and i + 64 of
// V (those past 2k are not used) and the scales of their columns.  t_v is the power of two with
// max_a |V_a| / s_a * t_v in [2^13, 2^14); W' = W t_v / s_r is split into FP16 hi +
// lo and stored in the B-operand fragment order [group][hi/lo][ct][ks][lane][8] that
// the batched kernel loads; a vector past nv stores zeros.  (t_v, |V|^2) go to
// vscale; |V|^2 is added in index order from the lanes' values in LDS (vs, 128 doubles).
// p.vscale and p.wfrag are outputs here.
template <int KS, int CT>
__device__ __forceinline__ void vector_weights(const BatchArgs &p, int v, const LbVec &V, const float (&sc)[kLbfgsPer],
                                               double *vs) {
    const int lane = threadIdx.x & 63;
    double m = 0.0;
#pragma unroll
    for (int u = 0; u < kLbfgsPer; ++u) {
        const double s = (double)__shfl(sc[u], lane & ~1);
        if (lane + 64 * u < 2 * p.k) m = fmax(m, fabs(V.e[u]) / s);
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) m = fmax(m, __shfl_xor(m, off));
    double t = 1.0;
    if (m > 0.0) {
        int e;
        frexp(m, &e);                 // m in [2^(e-1), 2^e)
        t = ldexp(1.0, 14 - e);
    }
    const int grp = v / (8 * CT), ct = v % (8 * CT) / 16 * 2, col = v % 16;
    const LbVec o = lb_pair(V);
    _Float16 *wf = reinterpret_cast<_Float16 *>(const_cast<void *>(p.wfrag));
#pragma unroll
    for (int u = 0; u < kLbfgsPer; ++u) {
        const int r = lane + 64 * u;
        if (r >= 32 * KS) continue;
        const size_t at = ((size_t)(r / 32) * 64 + 16 * (r % 32 / 8) + col) * 8 + r % 8;
#pragma unroll
        for (int c = 0; c < 2; ++c) {                 // the columns of z's real and imaginary part
            const double w = c == 0 ? (lane & 1 ? -V.e[u] : V.e[u]) : o.e[u];
            const WeightSplit ws = split_weight(r < 2 * p.k ? w * t / (double)sc[u] : 0.0);
            wf[(((size_t)grp * 2 + 0) * CT + ct + c) * KS * 512 + at] = ws.hi;
            wf[(((size_t)grp * 2 + 1) * CT + ct + c) * KS * 512 + at] = ws.lo;
        }
    }
    if (v >= p.nv) return;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
#pragma unroll
    for (int u = 0; u < kLbfgsPer; ++u) vs[lane + 64 * u] = V.e[u];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    double n2 = 0.0;
#pragma unroll 8
    for (int i = 0; i < 2 * p.k; ++i) n2 = fma(vs[i], vs[i], n2);
    if (lane == 0) {
        double *vsc = const_cast<double *>(p.vscale);
        vsc[2 * v] = t;
        vsc[2 * v + 1] = n2;
    }
}

// The scales of the columns that lane i's elements i and i + 64 belong to.
__device__ __forceinline__ void lane_scales(const BatchArgs &p, float (&sc)[kLbfgsPer]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int u = 0; u < kLbfgsPer; ++u) sc[u] = lane + 64 * u < 2 * p.k ? p.ascale[lane + 64 * u] : 1.f;
}

// Per vector v (one block each): add the block partials of each segment in
// block order, undo the per-vector scale t_v of the forward weights, and form
// NLL and gradient (Eq. 2 or Eq. 3 form; streamed MC or the MC matrix).
//
// The matrix cores summed with the weights V~ the FP16 hi + lo pairs hold,
// not V; the difference dV = V - V~ (about 2^-22 |V|) is the same for every
// event, so it does not average out over the sums.  Its first-order effect is
// added here from the adjoint sums the pass produced:
//   sum_i ln I_i(V) = sum_i ln I_i(V~) + 2 Re sum_a dV_a conj(G_a),
//   sum_j w_j I_j(V) = sum_j w_j I_j(V~) + 2 Re sum_a dV_a conj(H_a),
// with G_a = sum_i conj(A_ia) z_i / I_i and H_a = sum_j w_j conj(A_ja) z_j
// (the second-order terms are about 2^-44 of the sums).
// The block partials of a segment are summed by G = kCombineSlots / pstride
// groups (group g takes blocks g, g + G, ...; slots of a group take the pstride
// values of a block, so each block's partial row is read contiguously), then the
// G group sums are added in group order: the order is fixed.  A thread holds four
// slots of both segments, four loads of each in flight: one block per vector
// reads up to a few MB of partials.  t_v is a power of two, so its reciprocal and the
// products with either are exact.
//
// All threads of the block call it; the results are valid in wave 0 (the NLL, the
// domain flag and the gradient's elements of the lane).
constexpr int kCombineThreads = 256;
constexpr int kCombineSlots = 1024;

struct CombineSmem {
    double tot[2][1 + 2 * PWA_MAX_K];
    double grp[2][kCombineSlots];
    double V[2 * PWA_MAX_K], dv[2 * PWA_MAX_K], mv[2 * PWA_MAX_K];
    double pl[64 * kLbfgsPer], ps[64 * kLbfgsPer];
};

__device__ __forceinline__ void combine_vector(const BatchArgs &p, int v, CombineSmem &sm, double &nll, unsigned &flags,
                                               LbVec &grad) {
    constexpr int kSlots = kCombineSlots / kCombineThreads;
    const int tid = threadIdx.x, lane = tid & 63;
    const int pst = p.pstride;
    const int nblk = p.nb[0] + p.nb[1];
    const int k = p.k;
    const double *base = p.partials + (int64_t)v * nblk * pst;
    const int G = kCombineSlots / pst;
    const double tv = p.vscale[2 * v], itv = 1.0 / tv;
    for (int i = tid; i < 2 * k; i += kCombineThreads) {
        const double x = p.V[(int64_t)v * p.vstride + i], sr = (double)p.ascale[i];
        const WeightSplit ws = split_weight(x * tv / sr);
        sm.V[i] = x;
        sm.dv[i] = x - ((double)ws.hi + (double)ws.lo) * sr * itv;
    }
    constexpr int kAhead = 4;
    double s[2][kSlots];
    int off[kSlots], b[kSlots];
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
        const int slot = tid + u * kCombineThreads;
        s[0][u] = s[1][u] = 0.0;
        off[u] = slot % pst;
        b[u] = slot < G * pst ? slot / pst : nblk;              // blocks b, b + G, ... of both segments
    }
    // every slot's terms in block order; a slot past its last block reads that block and keeps its sum
    for (int j = 0; j < max(p.nb[0], p.nb[1]); j += kAhead * G) {
        double x[2][kAhead][kSlots];
#pragma unroll
        for (int sg = 0; sg < 2; ++sg) {
            const double *seg = base + (sg ? (int64_t)p.nb[0] * pst : 0);
            if (j < p.nb[sg]) {
#pragma unroll
                for (int i = 0; i < kAhead; ++i)
#pragma unroll
                    for (int u = 0; u < kSlots; ++u)
                        x[sg][i][u] = seg[(int64_t)min(b[u] + j + i * G, p.nb[sg] - 1) * pst + off[u]];
            }
        }
#pragma unroll
        for (int sg = 0; sg < 2; ++sg)
#pragma unroll
            for (int i = 0; i < kAhead; ++i)
#pragma unroll
                for (int u = 0; u < kSlots; ++u)
                    if (b[u] + j + i * G < p.nb[sg]) s[sg][u] += x[sg][i][u];
    }
#pragma unroll
    for (int sg = 0; sg < 2; ++sg)
#pragma unroll
        for (int u = 0; u < kSlots; ++u) sm.grp[sg][tid + u * kCombineThreads] = s[sg][u];
    __syncthreads();
    for (int i = tid; i < 2 * pst; i += kCombineThreads) {
        const int sg = i >= pst, c = i - sg * pst;
        double s = 0.0;
#pragma unroll 8
        for (int h = 0; h < G; ++h) s += sm.grp[sg][h * pst + c];
        sm.tot[sg][c] = s;
    }
    if (p.gram) {
        for (int a = tid; a < k; a += kCombineThreads) {
            double r = 0.0, i = 0.0;
            for (int b = 0; b < k; ++b) {
                const double mr = p.gram[2 * (a * k + b)], mi = p.gram[2 * (a * k + b) + 1];
                r += mr * sm.V[2 * b] - mi * sm.V[2 * b + 1];
                i += mr * sm.V[2 * b + 1] + mi * sm.V[2 * b];
            }
            sm.mv[2 * a] = r;
            sm.mv[2 * a + 1] = i;
        }
    }
    __syncthreads();
    if (tid >= 64) return;
    // Z' = t_v z: the data sums hold log2 I (unscaled) and conj(A) u / t_v; sum w I = sum w I' / t_v^2
    // first-order terms of the weight rounding (data: G = t_v x data sums;
    // MC: H = MC sums / t_v); the data's log sum is of the unscaled I
    const double nd = p.nd_total;
#pragma unroll
    for (int u = 0; u < kLbfgsPer; ++u) {
        const int i = lane + 64 * u;
        if (i < 2 * k) {
            sm.pl[i] = sm.dv[i] * sm.tot[0][1 + i] * tv;
            sm.ps[i] = sm.dv[i] * sm.tot[1][1 + i] * itv;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    double dlog = 0.0, ds = 0.0;
#pragma unroll 8
    for (int i = 0; i < 2 * k; ++i) {
        dlog += sm.pl[i];
        ds += sm.ps[i];
    }
    const double sum_log = sm.tot[0][0] * 0.69314718055994530942 + 2.0 * dlog;
    double S, c;
    if (p.gram) {
        double s = 0.0;
        for (int a = 0; a < k; ++a) s += sm.V[2 * a] * sm.mv[2 * a] + sm.V[2 * a + 1] * sm.mv[2 * a + 1];
        S = s;
        c = p.extended ? 1.0 : nd / S;
    } else {
        const double s_raw = sm.tot[1][0] / (tv * tv) + 2.0 * ds;
        S = s_raw / p.n_gen;
        c = p.extended ? 1.0 / p.n_gen : nd / s_raw;
    }
    const bool zero = !p.extended && nd == 0.0;
    flags = 0;
    if (zero) {
        nll = 0.0;
        c = 0.0;
    } else {
        nll = p.extended ? -sum_log + S : -sum_log + nd * log(S);
        if (!isfinite(nll) || (!p.extended && !(S > 0.0))) {
            nll = INFINITY;
            flags = 1;
        }
    }
    // data sums carry u = t_v Z'/I' (x t_v); MC sums carry w Z' = t_v w z (/ t_v)
#pragma unroll
    for (int u = 0; u < kLbfgsPer; ++u) {
        const int i = lane + 64 * u;
        grad.e[u] = 0.0;
        if (i < 2 * k && !zero) {
            const double g = sm.tot[0][1 + i] * tv;
            const double h = p.gram ? sm.mv[i] : sm.tot[1][1 + i] * itv;
            grad.e[u] = 2.0 * (-g + c * h);
        }
    }
}

__global__ __launch_bounds__(kCombineThreads) void nll_batch_combine_kernel(BatchArgs p) {
    __shared__ CombineSmem sm;
    const int v = blockIdx.x;
    double nll;
    unsigned flags;
    LbVec grad;
    combine_vector(p, v, sm, nll, flags, grad);
    if (threadIdx.x >= 64) return;
    double *out = p.out + (int64_t)v * p.ostride;
    lb_store(out + 1, grad, 2 * p.k, threadIdx.x);
    if (threadIdx.x == 0) {
        out[0] = nll;
        out[1 + 2 * p.k] = (double)flags;
    }
}

// What lies between two passes of a fit, in one launch: the vector's sums, its
// L-BFGS update and the weights of its next trial point, which the update leaves in
// the state (p.V points into it).  Bound by latency; the state is loaded before the
// partials' sums, and the two parametrisations are kernels of their own: the code runs
// once per launch, so its size counts (86 KB of it with both: 15.0 us, 26 KB: 12.5).
// 32 vectors at K = 8, 20000 rows: 12.5 us; 23 us in four launches (combine 7.3,
// update 6.2, scales 4.5, fragments 4.7), one vector's |V|^2 formed by every block of
// the pass (12.6 us, now 8.5).
template <int KS, int CT, bool POLAR>
__global__ __launch_bounds__(kCombineThreads) void batch_step_kernel(BatchArgs p, LbfgsState *states, double c1,
                                                                     double ftol, double rmin) {
    __shared__ CombineSmem sm;
    const int v = blockIdx.x, n = 2 * p.k;
    const bool first = threadIdx.x < 64;
    LbRegs r;
    float sc[kLbfgsPer];
    if (first) {
        lbfgs_load(r, states + v, n, POLAR);
        lane_scales(p, sc);
    }
    double nll;
    unsigned flags;
    LbVec grad;
    combine_vector(p, v, sm, nll, flags, grad);
    if (!first) return;
    const LbVec next = lbfgs_advance(states + v, r, n, nll, grad, c1, ftol, POLAR, rmin, sm.pl);
    vector_weights<KS, CT>(p, v, next, sc, sm.ps);
}

// Largest |re| or |im| of each wave over a sample's rows (FP32), as float bits
// in an atomicMax (non-negative floats order like their bit patterns).
__global__ void amax_kernel(const float *A, int64_t n, int64_t ld, int k, unsigned *out) {
    __shared__ unsigned sm[PWA_MAX_K];
    for (int a = threadIdx.x; a < k; a += blockDim.x) sm[a] = 0u;
    __syncthreads();
    const int64_t total = n * (int64_t)k;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t row = i / k;
        const int a = (int)(i % k);
        const float *x = A + 2 * (row * ld + a);
        const float m = fmaxf(fabsf(x[0]), fabsf(x[1]));
        atomicMax(&sm[a], __float_as_uint(m));
    }
    __syncthreads();
    for (int a = threadIdx.x; a < k; a += blockDim.x) atomicMax(&out[a], sm[a]);
}

// The weights of all vectors, one wave each, the padding groups included.
template <int KS, int CT>
__global__ __launch_bounds__(256) void batch_weights_kernel(BatchArgs p, int nvectors) {
    __shared__ double vs[4][64 * kLbfgsPer];
    const int wave = threadIdx.x >> 6, v = blockIdx.x * 4 + wave;
    if (v >= nvectors) return;
    LbVec V{};
    float sc[kLbfgsPer];
    if (v < p.nv) V = lb_load(p.V + (int64_t)v * p.vstride, 2 * p.k, threadIdx.x & 63);
    lane_scales(p, sc);
    vector_weights<KS, CT>(p, v, V, sc, vs[wave]);
}

}  // namespace

hipError_t launch_batch_weights(const BatchArgs &args, hipStream_t stream) {
    const int gpad = (batch_vector_groups(args.nv, args.k) + kWaves - 1) / kWaves * kWaves;
    const int nvectors = gpad * batch_vectors_per_wave(args.k);
    const dim3 grid((nvectors + 3) / 4);
    switch (batch_ks(args.k)) {
        case 1: hipLaunchKernelGGL((batch_weights_kernel<1, 4>), grid, dim3(256), 0, stream, args, nvectors); break;
        case 2: hipLaunchKernelGGL((batch_weights_kernel<2, 4>), grid, dim3(256), 0, stream, args, nvectors); break;
        case 3: hipLaunchKernelGGL((batch_weights_kernel<3, 2>), grid, dim3(256), 0, stream, args, nvectors); break;
        case 4: hipLaunchKernelGGL((batch_weights_kernel<4, 2>), grid, dim3(256), 0, stream, args, nvectors); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

size_t batch_partial_doubles(int64_t n0, int64_t n1, int tpb, int nv, int k) {
    const int64_t nb = batch_blocks(n0, tpb) + batch_blocks(n1, tpb);
    return (size_t)nb * (size_t)nv * (size_t)(1 + 2 * k);
}

int batch_tiles_per_block(int64_t n0, int64_t n1, int cu) {
    const int64_t tiles = (n0 + kTile - 1) / kTile + (n1 + kTile - 1) / kTile;
    if (tiles == 0 || cu < 1) return kTilesPerBlock;
    const int64_t rounds = (tiles + (int64_t)cu * kTilesPerBlock - 1) / ((int64_t)cu * kTilesPerBlock);
    const int64_t tpb = (tiles + rounds * cu - 1) / (rounds * cu);
    return (int)(tpb < 1 ? 1 : tpb);
}

int64_t batch_blocks(int64_t n, int tpb) {
    const int64_t tiles = (n + kTile - 1) / kTile;
    return (tiles + tpb - 1) / tpb;
}

int batch_ks(int k) { return (2 * k + 31) / 32; }

int batch_ct(int k) { return batch_ks(k) <= 2 ? 4 : 2; }

int batch_vectors_per_wave(int k) { return 8 * batch_ct(k); }

int batch_vector_groups(int nv, int k) {
    const int vpw = batch_vectors_per_wave(k);
    return (nv + vpw - 1) / vpw;
}

hipError_t launch_amax(const float *A, int64_t n, int64_t ld, int k, unsigned *out,
                       hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const int64_t blocks64 = (n * k + 255) / 256;
    const int blocks = (int)(blocks64 < 4096 ? blocks64 : 4096);
    hipLaunchKernelGGL(amax_kernel, dim3(blocks), dim3(256), 0, stream, A, n, ld, k, out);
    return hipGetLastError();
}

hipError_t launch_batch(const BatchArgs &args, bool refine, hipStream_t stream) {
    const int nblk = args.nb[0] + args.nb[1];
    if (nblk > 0) {
        const int gy = (batch_vector_groups(args.nv, args.k) + kWaves - 1) / kWaves;
        const dim3 grid(nblk, gy);
#define PWA_BATCH_LAUNCH(KS_, CT_)                                                                   \
    do {                                                                                             \
        if (refine)                                                                                  \
            hipLaunchKernelGGL((nll_batch_kernel<KS_, CT_, true>), grid, dim3(kThreads), 0, stream, args);  \
        else                                                                                         \
            hipLaunchKernelGGL((nll_batch_kernel<KS_, CT_, false>), grid, dim3(kThreads), 0, stream, args); \
    } while (0)
        switch (batch_ks(args.k)) {
            case 1: PWA_BATCH_LAUNCH(1, 4); break;
            case 2: PWA_BATCH_LAUNCH(2, 4); break;
            case 3: PWA_BATCH_LAUNCH(3, 2); break;
            case 4: PWA_BATCH_LAUNCH(4, 2); break;
            default: return hipErrorInvalidValue;
        }
#undef PWA_BATCH_LAUNCH
        return hipGetLastError();
    }
    return hipSuccess;
}

hipError_t launch_batch_refine(const BatchArgs &args, hipStream_t stream) {
    if (args.nb[0] == 0) return hipSuccess;
    const int gy = (batch_vector_groups(args.nv, args.k) + kWaves - 1) / kWaves;
    const dim3 grid(args.nb[0], gy);
    // the fewest lanes that hold the event's waves
    if (args.k <= 8)
        hipLaunchKernelGGL((batch_refine_kernel<4, 8>), grid, dim3(kThreads), 0, stream, args);
    else if (args.k <= 16)
        hipLaunchKernelGGL((batch_refine_kernel<4, 16>), grid, dim3(kThreads), 0, stream, args);
    else if (args.k <= 32)
        hipLaunchKernelGGL((batch_refine_kernel<4, 32>), grid, dim3(kThreads), 0, stream, args);
    else
        hipLaunchKernelGGL((batch_refine_kernel<2, 64>), grid, dim3(kThreads), 0, stream, args);
    return hipGetLastError();
}

size_t batch_flag_words(int64_t n0, int nv, int k) {
    const int64_t tiles = (n0 + kTile - 1) / kTile;
    const int gpad = (batch_vector_groups(nv, k) + kWaves - 1) / kWaves * kWaves;
    return (size_t)tiles * gpad * 8 * (batch_ct(k) / 2);
}

size_t batch_plane_bytes(int64_t n, int k) {
    const int64_t ntiles = (n + kTile - 1) / kTile;
    return (size_t)ntiles * 256 * (size_t)(32 * batch_ks(k));
}

hipError_t launch_batch_planes(const float *A, int64_t n, int64_t ld, int k, const float *ascale, void *out,
                               hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const int64_t ntiles = (n + kTile - 1) / kTile;
    const dim3 grid((unsigned)std::min<int64_t>(ntiles, 2048)), block(256);
    unsigned short *o = static_cast<unsigned short *>(out);
    switch (batch_ks(k)) {
        case 1: hipLaunchKernelGGL(batch_planes_kernel<1>, grid, block, 0, stream, A, n, ld, 2 * k, ntiles, ascale, o); break;
        case 2: hipLaunchKernelGGL(batch_planes_kernel<2>, grid, block, 0, stream, A, n, ld, 2 * k, ntiles, ascale, o); break;
        case 3: hipLaunchKernelGGL(batch_planes_kernel<3>, grid, block, 0, stream, A, n, ld, 2 * k, ntiles, ascale, o); break;
        case 4: hipLaunchKernelGGL(batch_planes_kernel<4>, grid, block, 0, stream, A, n, ld, 2 * k, ntiles, ascale, o); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_rownorm(const float *A, int64_t n, int64_t ld, int k, float *out, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const int blocks = (int)std::min<int64_t>((8 * n + 255) / 256, 16384);
    hipLaunchKernelGGL(rownorm_kernel, dim3(blocks), dim3(256), 0, stream, A, n, ld, k, out);
    return hipGetLastError();
}

hipError_t launch_batch_combine(const BatchArgs &args, hipStream_t stream) {
    hipLaunchKernelGGL(nll_batch_combine_kernel, dim3(args.nv), dim3(kCombineThreads), 0, stream, args);
    return hipGetLastError();
}

hipError_t launch_batch_step(const BatchArgs &args, LbfgsState *states, double c1, double ftol, bool polar, double rmin,
                             hipStream_t stream) {
    const dim3 grid(args.nv), block(kCombineThreads);
#define PWA_BATCH_STEP(KS_, CT_)                                                                                      \
    do {                                                                                                              \
        if (polar)                                                                                                    \
            hipLaunchKernelGGL((batch_step_kernel<KS_, CT_, true>), grid, block, 0, stream, args, states, c1, ftol,   \
                               rmin);                                                                                 \
        else                                                                                                          \
            hipLaunchKernelGGL((batch_step_kernel<KS_, CT_, false>), grid, block, 0, stream, args, states, c1, ftol,  \
                               rmin);                                                                                 \
    } while (0)
    switch (batch_ks(args.k)) {
        case 1: PWA_BATCH_STEP(1, 4); break;
        case 2: PWA_BATCH_STEP(2, 4); break;
        case 3: PWA_BATCH_STEP(3, 2); break;
        default: return hipErrorInvalidValue;          // fits have at most kMultiMaxLd waves
    }
#undef PWA_BATCH_STEP
    return hipGetLastError();
}

}  // namespace pwa
