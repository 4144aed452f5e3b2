// Fused training pass of the surrogate network at hidden width 256, in two
// launches.  The row pass takes one workgroup per slice of 16 mini-batch rows:
// forward pass, loss, dZ2 and dZ1 of the slice, written to HBM as FP16 planes
// whose rows are features (X, H1, dZ2 and dZ1 transposed, in the order the
// weight pass's operands take), and the slice's sums for the bias and head
// gradients.  The
// weight pass takes one workgroup per 16 x 16 tile of W2 or W1: dW = dZ^T H
// over every row of the mini-batch on the matrix cores (wave w takes the 32-row
// chunks w, w + 4, ..., the four waves' sums are added in wave order), then
// Adam on the tile (or the summed gradient); thirteen more workgroups add the
// slices' sums of the bias and head gradients and of the loss in a fixed order.
// The arithmetic is that of the layer-by-layer kernels in mlp.hip: every
// matrix product rounds both operands to FP16 and accumulates in FP32
// (v_mfma_f32_16x16x32_f16), biases and activations are FP32, the head and the
// weight-3 gradient use the FP16-rounded activations.  Only the order in which
// the rows of a mini-batch are added differs, and that an activation goes to FP16
// without a stop in FP32 memory.
#include "internal.hpp"

namespace pwa {
namespace {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kFR = 16;                 // rows per slice (one workgroup of the row pass)
constexpr int kFH = 256;                // hidden width of the fused path
constexpr int kFT = 256;                // threads per workgroup of the weight pass
constexpr int kFRT = 1024;              // threads per workgroup of the row pass
constexpr int kSH = kFH + 8;            // row stride (halfs) of [16][256] planes in LDS
constexpr int kFV = 3 * kFH + 8;        // floats per slice of vector sums: db1, db2, dw3, db3, loss

// GELU and its derivative from t = 1 + erf(x / sqrt 2)
__device__ __forceinline__ float erf1(float x) { return 1.f + erff(x * 0.70710678118654752f); }
__device__ __forceinline__ float gelu(float x, float t) { return 0.5f * x * t; }
__device__ __forceinline__ float gelu_d(float x, float t) {
    return fmaf(x * 0.39894228040143268f, expf(-0.5f * x * x), 0.5f * t);
}

struct FusedArgs {
    const float *P;                     // parameters W1 [H][in], b1, W2 [H][H], b2, w3, b3
    const float *X, *t;                 // features [n][in] and targets [n]
    const int *perm;                    // null: rows 0 .. B-1 of X; else rows perm[*batch B + r]
    const int *batch;                   // mini-batch index (with perm)
    const int *step;                    // Adam steps taken
    int *tnext;                         // for the Adam update that follows: its step t = *step + 1,
                                        // then 1 - 0.9^t and 1 - 0.999^t (floats)
    int64_t n;
    int B, in;
    _Float16 *act;                      // planes H1^T, dZ2^T, dZ1^T [256][bp] and X^T [INP][bp], operand order
    int64_t bp;                         // their columns: B rounded up to 32
    float *vsum;                        // [slice][kFV] vector sums of the slice's rows
    const _Float16 *w1h;                // fp16(W1) [256][INP] (zero past in), operand order
    const _Float16 *w2h;                // fp16(W2) [256][256], operand order
    const _Float16 *w2th;               // fp16(W2) transposed, operand order
    int *bad;
};

// Position of W[r][c] (W has 32 ks columns) in its FP16 copy: operand order, 1 KB
// per 16 x 32 piece, so that a wave reads its operand of one product step as 16
// consecutive bytes per lane.  (Row order, 64 bytes from each of 16 rows per load,
// held the row pass up for 6 us.)
__device__ __forceinline__ int operand_at(int r, int c, int ks) {
    return (((r >> 4) * ks + (c >> 5)) * 64 + ((c >> 3) & 3) * 16 + (r & 15)) * 8 + (c & 7);
}

// The planes hold, for features as rows and mini-batch rows as columns, 16 x 32
// pieces in operand order too: the weight pass reads 1 KB per wave and load.
// Piece (t, s) of features 16 t .. and mini-batch rows 32 s .., of bp / 32 pieces per t:
__device__ __forceinline__ int64_t piece_at(int t, int64_t s, int64_t bp) { return (t * (bp >> 5) + s) * 512; }

// Row pass: one workgroup of 16 waves per slice of 16 rows.  Wave w owns the 16
// features 16 w .. 16 w + 15 of every layer: its operands of W1, W2 and W2
// transposed are read once, straight from the FP16 copies into registers, and
// are in flight while the rows are gathered; item e of lane (q, r16) of a product
// is row 4 q + e, feature 16 w + r16, in all three products alike, so Z1 and Z2
// stay in registers and only the FP16 activations pass between waves (LDS).
//
// Bound: one dependent chain per slice (gather, three products, five erf or exp
// evaluations per element, six barriers) on as many CUs as there are slices.
// Batch 1024, 32 inputs: 9.0 us; 20.5 us with four waves that staged every weight chunk
// through LDS between two barriers.
template <int INP>
struct RowSmem {
    static constexpr int SX = INP + 8;
    _Float16 xr[kFR * SX];              // X, rows
    _Float16 h1r[kFR * kSH];            // fp16(H1), rows
    _Float16 h2r[kFR * kSH];            // fp16(H2), rows
    _Float16 d2r[kFR * kSH];            // fp16(dZ2), rows
    float w3[kFH];                      // fp16(w3)
    float tgt[kFR], dy[kFR], lrow[kFR];
    int src[kFR];
};

// Barrier that orders LDS only: global loads stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Sum of x[e] y[e] over the lane rows q = 0 .. 3 and e = 0 .. 3 in row order, one
// fused multiply-add after the other from 0.  Valid in lane row 3.
__device__ __forceinline__ float rows_in_order(const float (&x)[4], const float (&y)[4], int q) {
    float s = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const float up = t ? __shfl_up(s, 16) : 0.f;
        if (q == t) s = fmaf(x[3], y[3], fmaf(x[2], y[2], fmaf(x[1], y[1], fmaf(x[0], y[0], up))));
    }
    return s;
}

template <int INP>
__global__ __launch_bounds__(kFRT) void mlp_rows_kernel(FusedArgs a) {
    __shared__ __attribute__((aligned(16))) RowSmem<INP> sm;
    constexpr int SX = RowSmem<INP>::SX, KS1 = INP / 32, KS2 = kFH / 32;
    const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, r16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slice = blockIdx.x, in = a.in;
    const float *W1 = a.P, *b1 = W1 + (int64_t)kFH * in, *b2 = b1 + kFH + (int64_t)kFH * kFH, *w3 = b2 + kFH,
                *b3 = w3 + kFH;
    const int64_t bp = a.bp, rb = (int64_t)slice * kFR;  // first row of the slice
    _Float16 *H1T = a.act, *D2T = H1T + kFH * bp, *D1T = D2T + kFH * bp, *XT = D1T + kFH * bp;
    float *V = a.vsum + (int64_t)slice * kFV;
    const int rows = a.B - slice * kFR < kFR ? a.B - slice * kFR : kFR;
    const int f = 16 * wave + r16;                       // this lane's feature
    // this lane's rows 4 q .. 4 q + 3 of its feature in a plane
    const int64_t at = piece_at(wave, slice >> 1, bp) + ((2 * (slice & 1) + (q >> 1)) * 16 + r16) * 8 + 4 * (q & 1);

    if (slice * kFR >= a.B) {                            // the last workgroup: Adam's corrections
        if (tid == 0) {
            const int t = *a.step + 1;
            float *corr = reinterpret_cast<float *>(a.tnext + 1);
            *a.tnext = t;
            corr[0] = 1.f - powf(0.9f, (float)t);
            corr[1] = 1.f - powf(0.999f, (float)t);
        }
        return;
    }
    // rows of the slice (a bad permutation entry reads row 0 and raises the flag)
    const int64_t first = a.perm ? (int64_t)(*a.batch) * a.B : 0;
    const float head_b = b3[0];
    int my_src = -1;
    if (tid < rows) {
        const int64_t gr = rb + tid;
        int64_t s = a.perm ? (int64_t)a.perm[first + gr] : gr;
        if (s < 0 || s >= a.n) {
            atomicOr(a.bad, 1);
            s = 0;
        }
        my_src = (int)s;
    }
    if (tid < kFR) sm.src[tid] = my_src;
    const float bias1 = b1[f], bias2 = b2[f];
    h8 w1[KS1], w2[KS2], w2t[KS2];
#pragma unroll
    for (int s = 0; s < KS1; ++s) w1[s] = reinterpret_cast<const h8 *>(a.w1h)[(wave * KS1 + s) * 64 + lane];
    const float w3v = w3[tid % kFH];
    lds_barrier();
    // X rows and targets (row and column clamped into the arrays, zero past the
    // slice's rows and past in)
    constexpr int XN = (kFR * INP + kFRT - 1) / kFRT;
    float xv[XN];
    bool xlive[XN];
#pragma unroll
    for (int i = 0; i < XN; ++i) {
        const int it = tid + i * kFRT, r = it / INP % kFR, c = it % INP;
        const int s = sm.src[r];
        xlive[i] = s >= 0 && c < in;
        xv[i] = a.X[(int64_t)(s >= 0 ? s : 0) * in + (c < in ? c : 0)];
    }
    const float tv = a.t[my_src >= 0 ? my_src : 0];
#pragma unroll
    for (int i = 0; i < XN; ++i) {
        const int it = tid + i * kFRT;
        if (it < kFR * INP) sm.xr[it / INP * SX + it % INP] = (_Float16)(xlive[i] ? xv[i] : 0.f);
    }
    if (tid < kFR) sm.tgt[tid] = my_src >= 0 ? tv : 0.f;
    if (tid < kFH) sm.w3[tid] = (float)(_Float16)w3v;
    lds_barrier();

    // Each product's weights are asked for one product ahead (any earlier and
    // they queue in front of the rows)
#pragma unroll
    for (int s = 0; s < KS2; ++s) w2[s] = reinterpret_cast<const h8 *>(a.w2h)[(wave * KS2 + s) * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
    // layer 1: Z1 = X W1^T + b1, H1 = GELU(Z1)
    float z1[4], t1[4];                                  // Z1 and 1 + erf(Z1 / sqrt 2)
    {
        f4 acc = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS1; ++s)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                *reinterpret_cast<const h8 *>(sm.xr + r16 * SX + 32 * s + 8 * q), w1[s], acc, 0, 0, 0);
        h4 hv;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            z1[e] = acc[e] + bias1;
            t1[e] = erf1(z1[e]);
            hv[e] = (_Float16)gelu(z1[e], t1[e]);
            sm.h1r[(4 * q + e) * kSH + f] = hv[e];
        }
        *reinterpret_cast<h4 *>(H1T + at) = hv;
    }
    lds_barrier();
#pragma unroll
    for (int s = 0; s < KS2; ++s) w2t[s] = reinterpret_cast<const h8 *>(a.w2th)[(wave * KS2 + s) * 64 + lane];
    float g1[4], g2[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) g1[e] = gelu_d(z1[e], t1[e]);
    __builtin_amdgcn_sched_barrier(0);
    // layer 2: Z2 = H1 W2^T + b2, fp16(H2) rows
    float z2[4], t2[4], h2[4];
    {
        f4 acc = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS2; ++s)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                *reinterpret_cast<const h8 *>(sm.h1r + r16 * kSH + 32 * s + 8 * q), w2[s], acc, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            z2[e] = acc[e] + bias2;
            t2[e] = erf1(z2[e]);
            const _Float16 h = (_Float16)gelu(z2[e], t2[e]);
            h2[e] = (float)h;
            sm.h2r[(4 * q + e) * kSH + f] = h;
        }
    }
    lds_barrier();
    // head: y = fp16(H2) . fp16(w3) + b3 (wave = row; 16 lanes, lane-order sums), dy, loss
    {
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < kFH; j += 16) s += (float)sm.h2r[wave * kSH + j + r16] * sm.w3[j + r16];
        s += __shfl_xor(s, 1);
        s += __shfl_xor(s, 2);
        s += __shfl_xor(s, 4);
        s += __shfl_xor(s, 8);
        if (lane == 0) {
            const float yb = s + head_b;
            const bool ok = wave < rows;
            sm.dy[wave] = ok ? 2.f * (yb - sm.tgt[wave]) : 0.f;
            sm.lrow[wave] = ok ? (yb - sm.tgt[wave]) * (yb - sm.tgt[wave]) : 0.f;
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) g2[e] = gelu_d(z2[e], t2[e]);      // while the sums cross the waves
    lds_barrier();
    // dZ2 = dy fp16(w3) GELU'(Z2) (rows into LDS, the feature's rows into dZ2^T)
    float dyw[4], dy[4];
    {
        const float wj = sm.w3[f];
        h4 dv;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            dy[e] = sm.dy[4 * q + e];
            dyw[e] = dy[e] * wj;
            dv[e] = (_Float16)(dyw[e] * g2[e]);
            sm.d2r[(4 * q + e) * kSH + f] = dv[e];
        }
        *reinterpret_cast<h4 *>(D2T + at) = dv;
    }
    lds_barrier();
    // dH1 = dZ2 W2, dZ1 = dH1 GELU'(Z1) (the feature's rows into dZ1^T)
    float d1[4];
    {
        f4 acc = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS2; ++s)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                *reinterpret_cast<const h8 *>(sm.d2r + r16 * kSH + 32 * s + 8 * q), w2t[s], acc, 0, 0, 0);
        h4 dv;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            d1[e] = acc[e] * g1[e];
            __asm__ volatile("" : "+v"(d1[e]));          // FP32 first, then FP16: dZ1 is summed in FP32 too
            dv[e] = (_Float16)d1[e];
        }
        *reinterpret_cast<h4 *>(D1T + at) = dv;
    }
    // per feature the slice's db1, db2 and dw3 (rows in order)
    {
        const float one[4] = {1.f, 1.f, 1.f, 1.f};
        const float s1 = rows_in_order(d1, one, q), s2 = rows_in_order(dyw, g2, q), sw = rows_in_order(dy, h2, q);
        if (q == 3) {
            V[f] = s1;
            V[kFH + f] = s2;
            V[2 * kFH + f] = sw;
        }
    }
    if (tid == 0) {                                      // db3 and the loss
        float sd = 0.f, sl = 0.f;
        for (int r = 0; r < kFR; ++r) {
            sd += sm.dy[r];
            sl += sm.lrow[r];
        }
        V[3 * kFH] = sd;
        V[3 * kFH + 1] = sl;
    }
    // X transposed (the slice's 16 rows of feature c), by the last waves
    const int c = kFRT - 1 - tid;
    if (c < INP) {
        h8 lo, hi;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            lo[r] = sm.xr[r * SX + c];
            hi[r] = sm.xr[(r + 8) * SX + c];
        }
        _Float16 *xt = XT + piece_at(c >> 4, slice >> 1, bp) + (2 * (slice & 1) * 16 + (c & 15)) * 8;
        *reinterpret_cast<h8 *>(xt) = lo;
        *reinterpret_cast<h8 *>(xt + 16 * 8) = hi;
    }
}

struct UpdateArgs {
    const _Float16 *act;                // the row pass's planes
    int64_t bp;                         // their columns
    int S;                              // slices (plane columns 16 S .. bp - 1 were not written)
    const float *vsum;                  // [slice][kFV]
    int in, B, adam;
    float gscale, lr;
    float *P, *M1, *M2, *G, *loss, *hist;
    _Float16 *w1h, *w2h, *w2th;
    const int *tnext;
    int *step, *batch;
};

// Adam on parameter i with gradient sum g (the update of mlp.hip's Adam
// kernel), from the parameter and moments read beforehand; or g into G.
// Returns the new parameter.
struct AdamIn {
    float p, m1, m2;
};
__device__ __forceinline__ AdamIn adam_load(const UpdateArgs &a, int64_t i) {
    return a.adam ? AdamIn{a.P[i], a.M1[i], a.M2[i]} : AdamIn{0.f, 0.f, 0.f};
}
__device__ __forceinline__ float apply(const UpdateArgs &a, int64_t i, const AdamIn &o, float g, const float *corr) {
    if (!a.adam) {
        a.G[i] = g;
        return 0.f;
    }
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f, c1 = corr[0], c2 = corr[1];
    const float gi = g * a.gscale;
    const float mi = b1 * o.m1 + (1.f - b1) * gi;
    const float vi = b2 * o.m2 + (1.f - b2) * gi * gi;
    a.M1[i] = mi;
    a.M2[i] = vi;
    const float p = o.p - a.lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    a.P[i] = p;
    return p;
}

constexpr int kVecBlocks = 3 * (kFH / 64) + 1;   // workgroups of the vector sums

// Weight pass: workgroups 0 .. 255 the tiles of W2, then the tiles of W1
// (16 x INP/16), then the vector sums: 64 entries of b1, b2 or w3 per
// workgroup, and one for b3 and the loss.  A tile's Adam state is read before
// its products.  With Adam the tile workgroups refresh the fp16 weight copies;
// the loss workgroup writes the loss (hist[*batch] too) and advances *step and
// *batch (no other workgroup reads them).
// Bound: latency (a launch, one round of loads, one of stores).  Batch 1024: 4.5 us;
// 7.6 us when each workgroup first computed Adam's two powers from the step and its
// operands were 64 bytes from each of 16 rows per load.
template <int INP>
__global__ __launch_bounds__(kFT) void mlp_update_kernel(UpdateArgs a) {
    constexpr int N2 = (kFH / 16) * (kFH / 16), N1 = (kFH / 16) * (INP / 16);
    __shared__ float red[4][256];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, q = lane >> 4, r16 = lane & 15;
    const float *corr = reinterpret_cast<const float *>(a.tnext + 1);
    const int in = a.in;
    const int64_t o2 = (int64_t)kFH * in + kFH, e2 = o2 + (int64_t)kFH * kFH;
    const int bt = blockIdx.x;
    if (bt < N2 + N1) {
        const int64_t bp = a.bp, rows = (int64_t)kFR * a.S;
        const _Float16 *H1T = a.act, *D2T = H1T + kFH * bp, *D1T = D2T + kFH * bp, *XT = D1T + kFH * bp;
        const bool w2 = bt < N2;
        const int ti = w2 ? bt / (kFH / 16) : (bt - N2) / (INP / 16);
        const int tj = w2 ? bt % (kFH / 16) : (bt - N2) % (INP / 16);
        // this thread's parameter: row tid / 16, column tid % 16 of the tile
        const int row = 16 * ti + (tid >> 4), col = 16 * tj + (tid & 15);
        const bool mine = w2 || col < in;
        const int64_t ip = w2 ? o2 + (int64_t)row * kFH + col : (int64_t)row * in + col;
        const AdamIn st = mine ? adam_load(a, ip) : AdamIn{0.f, 0.f, 0.f};
        const _Float16 *pa = (w2 ? D2T : D1T) + piece_at(ti, 0, bp) + lane * 8;
        const _Float16 *pb = (w2 ? H1T : XT) + piece_at(tj, 0, bp) + lane * 8;
        // D[i][j] = sum_r A[i][r] B[j][r] over the wave's chunks in order (rows
        // 16 S .. bp - 1 count as zero); eight chunks' loads in flight
        f4 acc = f4{0.f, 0.f, 0.f, 0.f};
        for (int64_t k0 = 32 * wave; k0 < rows; k0 += 1024) {
            h8 av[8], bv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t kk = k0 + 128 * u;
                const bool ok = kk + 8 * q < rows;
                av[u] = ok ? *reinterpret_cast<const h8 *>(pa + kk * 16) : h8{};
                bv[u] = ok ? *reinterpret_cast<const h8 *>(pb + kk * 16) : h8{};
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[u], bv[u], acc, 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) red[wave][(4 * q + e) * 16 + r16] = acc[e];
        __syncthreads();
        const float g = ((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid];
        if (!mine) return;
        const float p = apply(a, ip, st, g, corr);
        if (a.adam) {
            if (w2) {
                a.w2h[operand_at(row, col, kFH / 32)] = (_Float16)p;
                a.w2th[operand_at(col, row, kFH / 32)] = (_Float16)p;
            } else {
                a.w1h[operand_at(row, col, INP / 32)] = (_Float16)p;
            }
        }
        return;
    }
    // vector sums: entry c (64 per workgroup) of vector v (db1, db2, dw3; v = 3:
    // db3 and the loss); wave w adds slices w, w + 4, ... in order (sixteen
    // loads in flight), the waves' sums are added in wave order
    const int vb = bt - N2 - N1, v = vb / (kFH / 64), c = 64 * (vb % (kFH / 64)) + lane;
    const bool live = v < 3 || c < 2;
    const int64_t off = (int64_t)v * kFH + (live ? c : 0);
    const int64_t ip = v == 0 ? (int64_t)kFH * in + c : v == 1 ? e2 + c : v == 2 ? e2 + kFH + c : e2 + 2 * kFH;
    const bool param = live && !(v == 3 && c == 1);
    const AdamIn st = param && wave == 0 ? adam_load(a, ip) : AdamIn{0.f, 0.f, 0.f};
    float sum = 0.f;
    for (int s0 = wave; s0 < a.S; s0 += 64) {
        float x[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int sl = s0 + 4 * u;
            x[u] = a.vsum[(int64_t)(sl < a.S ? sl : a.S - 1) * kFV + off];
            if (sl >= a.S) x[u] = 0.f;
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) sum += x[u];
    }
    red[wave][lane] = sum;
    __syncthreads();
    if (wave != 0 || !live) return;
    const float g = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
    if (param) {
        apply(a, ip, st, g, corr);
        return;
    }
    *a.loss = g / (float)a.B;                           // v = 3, c = 1: the loss
    if (a.hist) a.hist[*a.batch] = g / (float)a.B;
    if (a.adam) {
        *a.step = *a.tnext;
        *a.batch += 1;
    }
}

// fp16 copies of W1 (rows padded to inp with zeros) and W2 (and its transpose) in
// operand order.
__global__ void mlp_fused_weights_kernel(const float *P, int in, int inp, _Float16 *w1h, _Float16 *w2h,
                                         _Float16 *w2th) {
    const float *W1 = P, *W2 = P + (int64_t)kFH * in + kFH;
    const int n1 = kFH * inp, n2 = kFH * kFH;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n1 + n2; i += gridDim.x * blockDim.x) {
        if (i < n1) {
            const int f = i / inp, c = i % inp;
            w1h[operand_at(f, c, inp / 32)] = (_Float16)(c < in ? W1[f * in + c] : 0.f);
        } else {
            const int j = i - n1, o = j / kFH, c = j % kFH;
            const _Float16 h = (_Float16)W2[j];
            w2h[operand_at(o, c, kFH / 32)] = h;
            w2th[operand_at(c, o, kFH / 32)] = h;
        }
    }
}

template <int INP>
hipError_t launch_fused(const FusedArgs &a, const UpdateArgs &u, int S, hipStream_t s) {
    hipLaunchKernelGGL(mlp_rows_kernel<INP>, dim3(S + 1), dim3(kFRT), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    constexpr int blocks = (kFH / 16) * (kFH / 16) + (kFH / 16) * (INP / 16) + kVecBlocks;
    hipLaunchKernelGGL(mlp_update_kernel<INP>, dim3(blocks), dim3(kFT), 0, s, u);
    return hipGetLastError();
}

int64_t plane_stride(int B) { return ((int64_t)B + 31) / 32 * 32; }

}  // namespace

bool mlp_fused_ok(const MlpBuffers &m) { return m.hidden == kFH && m.in >= 1 && m.in <= 128 && m.fact; }

int mlp_fused_slices(int B) { return (B + kFR - 1) / kFR; }

size_t mlp_fused_wh_halfs() { return (size_t)kFH * 128 + 2 * (size_t)kFH * kFH; }

size_t mlp_fused_act_halfs(int max_batch) { return (size_t)(3 * kFH + 128) * (size_t)plane_stride(max_batch); }

size_t mlp_fused_vec_floats(int max_batch) { return (size_t)mlp_fused_slices(max_batch) * kFV; }

hipError_t mlp_fused_weights(const MlpBuffers &m, hipStream_t s) {
    if (!mlp_fused_ok(m)) return hipErrorInvalidValue;
    const int inp = (m.in + 31) / 32 * 32;
    hipLaunchKernelGGL(mlp_fused_weights_kernel, dim3(256), dim3(256), 0, s, m.P, m.in, inp, m.fwh,
                       m.fwh + (size_t)kFH * 128, m.fwh + (size_t)kFH * 128 + (size_t)kFH * kFH);
    return hipGetLastError();
}

hipError_t mlp_fused_pass(const MlpBuffers &m, int B, const float *X, const float *t, const int *perm, int64_t n,
                          bool adam, float gscale, float lr, float *hist, hipStream_t s) {
    if (!mlp_fused_ok(m) || B < 1 || B > m.max_batch) return hipErrorInvalidValue;
    const int S = mlp_fused_slices(B);
    const int inp = (m.in + 31) / 32 * 32;
    const int64_t bp = plane_stride(B);
    _Float16 *w1h = m.fwh, *w2h = w1h + (size_t)kFH * 128, *w2th = w2h + (size_t)kFH * kFH;
    const FusedArgs a{m.P, X, t, perm, m.batch, m.step, m.ftnext, n, B, m.in, m.fact, bp, m.fvec, w1h, w2h, w2th,
                      m.bad};
    const UpdateArgs u{m.fact, bp,   S,      m.fvec, m.in, B,       adam ? 1 : 0, gscale,  lr,     m.P,
                       m.M1,   m.M2, m.G,    m.loss, hist, w1h,     w2h,          w2th,    m.ftnext, m.step,
                       m.batch};
    return inp == 32   ? launch_fused<32>(a, u, S, s)
           : inp == 64 ? launch_fused<64>(a, u, S, s)
           : inp == 96 ? launch_fused<96>(a, u, S, s)
                       : launch_fused<128>(a, u, S, s);
}

}  // namespace pwa
