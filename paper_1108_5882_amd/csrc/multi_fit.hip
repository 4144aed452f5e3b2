// Many independent fits in one persistent launch (Berger, Section 2: fits are
// repeated from many starting points and models, each needing the likelihood
// of Eq. 2 and its gradient at every iteration).
//
// Every fit f has its own samples (N_D, N_MC, K_f) and its own trial vector.
// The rows of all fits are cut into work items (one sample of one fit, a
// range of tiles); blocks take items from an atomic counter, stream the rows
// of the item with the fused single-V arithmetic (FP32 storage, FP64 z, I,
// z/I and sums) and write one FP64 partial per item.  Because each item has
// its own slot, results do not depend on which block took which item.  A
// combine kernel adds each fit's item partials in item order, forms NLL and
// gradient and advances the fit's L-BFGS state: two launches per step.
//
// Row widths differ between fits (K from 4 to 48): each item carries its
// width and the block dispatches to the compiled tile shape for it.
#include "lbfgs_device.hpp"
#include "nll_stream_impl.hpp"

namespace pwa {
namespace {

using stream_detail::EventMath;
using stream_detail::Stage;

constexpr int kMT = kStreamThreads;     // threads per block
constexpr int kMW = kMT / 64;

// Streams tiles [t0, t1) of one sample with shape (L, C, U); waves take tiles
// t0 + wave, t0 + wave + kMW, ...; returns the block's partial in red.
constexpr int kRedSlot = 2 * 6 + 1;      // largest 2C + 1 of the shapes below

// Wave index of lane j's local complex c.  Contiguous (CH = false): lane j
// holds waves [jC, jC + C).  Chunked (CH = true, C even): lane j holds the
// 2-wave chunks j, j + L, j + 2L, ..., so each 16-byte load instruction of a
// lane group covers one contiguous span of the row (used for rows of 24 and
// 48 waves, which three contiguous waves per lane would read in 8-byte pieces).
template <int L, int C, bool CH>
__device__ __forceinline__ int wave_of(int j, int c) {
    if constexpr (CH) return 2 * (j + L * (c >> 1)) + (c & 1);
    else return j * C + c;
}

// Row loads of the chunked layout (same registers as Stage::load fills), row
// stride L * C complex.  FULL: every row of the tile exists (wave-uniform tile
// base, constant offsets, no clamping; SEG 1 then needs W); otherwise rows
// are clamped into [0, n).
template <int L, int C, int U, int SEG, bool FULL>
__device__ __forceinline__ void load_chunked(Stage<float, L, C, U, SEG> &st, const float *__restrict__ A,
                                             const float *__restrict__ W, int64_t n, int64_t tile,
                                             int g, int j) {
    typedef float f4c __attribute__((ext_vector_type(4)));
    typedef const f4c __attribute__((address_space(1))) *gp4;
    typedef const float __attribute__((address_space(1))) *gpf;
    constexpr int G = 64 / L;
    constexpr int64_t LD = L * C;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        int64_t row = tile * (G * U) + (int64_t)u * G + g;
        if constexpr (!FULL) row = row < n ? row : n - 1;
        if constexpr (SEG == 1) st.w[u] = FULL || W ? __builtin_nontemporal_load((gpf)(W + row)) : 1.f;
#pragma unroll
        for (int i = 0; i < C / 2; ++i) {
            const f4c v = __builtin_nontemporal_load((gp4)(A + 2 * (row * LD + 2 * (j + L * i))));
            st.a[u][4 * i + 0] = v.x;
            st.a[u][4 * i + 1] = v.y;
            st.a[u][4 * i + 2] = v.z;
            st.a[u][4 * i + 3] = v.w;
        }
    }
}

// grab() asks for the block's next item and is called once the first rows are on
// their way; fetch() follows the barrier that publishes the answer.
template <int L, int C, int U, int SEG, bool CH = false, typename Grab, typename Fetch>
__device__ __forceinline__ void multi_item(const MultiItem &it, double *slot, double *red, Grab grab, Fetch fetch) {
    constexpr int SLOT = 2 * C + 1;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int g = lane / L, j = lane % L;
    const float *A = it.A;
    const float *W = SEG ? it.w : nullptr;
    const int64_t n = it.n;
    // waves past k read wave 0 (a load under a mask would be waited for before the rows are asked for)
    typedef const stream_detail::d2v __attribute__((address_space(1))) *gpv;
    stream_detail::d2v v[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int a = wave_of<L, C, CH>(j, c);
        v[c] = *((gpv)it.V + (a < it.k ? a : 0));
    }
    // row stride L * C (the item's width selected this shape)
    auto ld_stage = [&](Stage<float, L, C, U, SEG> &st, int64_t tt) {
        if constexpr (CH) load_chunked<L, C, U, SEG, false>(st, A, W, n, tt, g, j);
        else st.load(A, W, n, (int64_t)(L * C), tt, g, j);
    };
    auto ld_full = [&](Stage<float, L, C, U, SEG> &st, int64_t tt) {
        if constexpr (CH) load_chunked<L, C, U, SEG, true>(st, A, W, n, tt, g, j);
        else st.load_full(A, W, tt, g, j);
    };
    double acc_t = 0.0, acc_r[C], acc_i[C];
#pragma unroll
    for (int c = 0; c < C; ++c) acc_r[c] = acc_i[c] = 0.0;
    constexpr int ROWS = (64 / L) * U;
    const int64_t nfull = n / ROWS;   // tiles whose rows all exist
    int64_t t = it.t0 + wid;
    Stage<float, L, C, U, SEG> s0, s1;
    // the same two-stage schedule as the single-fit pass: whole tiles
    // without clamping or masks while they last, then the clamped loads
    // (a wave without a tile loads clamped rows it does not use)
    const bool whole = t + kMW < it.t1 && t + 2 * kMW < nfull;
    if (whole) ld_full(s0, t);
    else ld_stage(s0, t);
    grab();
    double vr[C], vi[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const bool there = wave_of<L, C, CH>(j, c) < it.k;
        vr[c] = there ? v[c].x : 0.0;
        vi[c] = there ? v[c].y : 0.0;
    }
    if (t < it.t1) {
        if (whole) {
            do {
                ld_full(s1, t + kMW);
                stream_detail::fence_sched();
                s0.template compute<false>(n, t, g, vr, vi, acc_t, acc_r, acc_i);
                t += kMW;
                ld_full(s0, t + kMW);
                stream_detail::fence_sched();
                s1.template compute<false>(n, t, g, vr, vi, acc_t, acc_r, acc_i);
                t += kMW;
            } while (t + kMW < it.t1 && t + 2 * kMW < nfull);
        }
        // s0 holds tile t
        while (t < it.t1) {
            ld_stage(s1, t + kMW);
            stream_detail::fence_sched();
            s0.template compute<true>(n, t, g, vr, vi, acc_t, acc_r, acc_i);
            t += kMW;
            if (t >= it.t1) break;
            ld_stage(s0, t + kMW);
            stream_detail::fence_sched();
            s1.template compute<true>(n, t, g, vr, vi, acc_t, acc_r, acc_i);
            t += kMW;
        }
    }
#pragma unroll
    for (int off = L; off < 64; off <<= 1) {
        acc_t += __shfl_xor(acc_t, off);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            acc_r[c] += __shfl_xor(acc_r[c], off);
            acc_i[c] += __shfl_xor(acc_i[c], off);
        }
    }
    auto R = [&](int w, int jj, int s_) -> double & { return red[(w * 64 + jj) * SLOT + s_]; };
    if (lane < L) {
        R(wid, j, 0) = acc_t;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            R(wid, j, 1 + 2 * c) = acc_r[c];
            R(wid, j, 2 + 2 * c) = acc_i[c];
        }
    }
    __syncthreads();
    fetch();
    const int ps = 1 + 2 * L * C;
    for (int idx = threadIdx.x; idx < ps; idx += kMT) {
        double s = 0.0;
        if (idx == 0) {
            for (int w = 0; w < kMW; ++w) s += R(w, 0, 0);
        } else {
            const int a = (idx - 1) >> 1, q = (idx - 1) & 1;
            // lane and local complex of wave a (inverse of wave_of)
            int jj, cc;
            if constexpr (CH) {
                jj = (a >> 1) % L;
                cc = 2 * ((a >> 1) / L) + (a & 1);
            } else {
                jj = a / C;
                cc = a % C;
            }
            for (int w = 0; w < kMW; ++w) s += R(w, jj, 1 + 2 * cc + q);
        }
        slot[idx] = s;
    }
    __syncthreads();
}

template <int SEG, typename Grab, typename Fetch>
__device__ __forceinline__ void dispatch_item(const MultiItem &it, double *slot, double *red, Grab grab, Fetch fetch) {
    switch (it.ld) {
        case 4: multi_item<2, 2, 4, SEG>(it, slot, red, grab, fetch); break;
        case 6: multi_item<2, 3, 2, SEG>(it, slot, red, grab, fetch); break;
        case 8: multi_item<4, 2, 4, SEG>(it, slot, red, grab, fetch); break;
        case 12: multi_item<4, 3, 2, SEG>(it, slot, red, grab, fetch); break;
        case 16: multi_item<8, 2, 4, SEG>(it, slot, red, grab, fetch); break;
        case 24: multi_item<4, 6, 2, SEG, true>(it, slot, red, grab, fetch); break;
        case 32: multi_item<16, 2, 4, SEG>(it, slot, red, grab, fetch); break;
        default: multi_item<8, 6, 2, SEG, true>(it, slot, red, grab, fetch); break;      // 48
    }
}

// A block asks for its next item while it streams the current one, and reads that
// item's descriptor during the current one's reduction.  One block per compute unit:
// the widest rows take more than half of its registers, and its four waves keep enough
// rows in flight (with a bound of 256 registers two blocks fit, and a step of 436 MB
// took 116 us with two and 110 with one).  Shares of the rows fixed per block, of equal
// bytes, were slower (the blocks differ in speed).
// 24 fits, 436 MB of rows: 86 us; 101 us when a block asked after it had finished and
// read descriptor, fit and V in turn.
__global__ __launch_bounds__(kMT) void multi_stream_kernel(MultiArgs p) {
    __shared__ int s_next;
    __shared__ double red[kMW * 64 * kRedSlot];
    // descriptors through the scalar cache, apart from the rows in flight
    typedef const MultiItem __attribute__((address_space(4))) *citem;
    const citem items = (citem)p.items;
    auto descriptor = [&](int i) {
        const citem c = items + (i < p.n_items ? i : 0);
        return MultiItem{c->A, c->w, c->V, c->n, c->t0, c->t1, c->ld, c->k, c->seg, 0};
    };
    int item = blockIdx.x;                             // the grid has at most n_items blocks
    if (item >= p.n_items) return;                     // no items at all
    MultiItem it = descriptor(item);
    while (item < p.n_items) {
        double *slot = p.partials + (int64_t)item * kMultiSlot;
        int next = 0;
        MultiItem ahead;
        auto grab = [&]() {
            if (threadIdx.x == 0) s_next = (int)(gridDim.x + atomicAdd(p.item_counter, 1u));
        };
        auto fetch = [&]() {
            next = __builtin_amdgcn_readfirstlane(s_next);
            ahead = descriptor(next);
        };
        // MC rows with weights (segment kind 1) or unit weights (2): a
        // compile-time choice, so the row loop holds no branch on it
        if (it.seg == 0)
            dispatch_item<0>(it, slot, red, grab, fetch);
        else if (it.w)
            dispatch_item<1>(it, slot, red, grab, fetch);
        else
            dispatch_item<2>(it, slot, red, grab, fetch);
        item = next;
        it = ahead;
    }
}

// One block per fit: adds the fit's item partials and forms NLL and gradient
// (Eq. 2 form).  Slice s of a column adds items i0 + s, i0 + s + kSlices, ...; the
// slices are then added in slice order, so the result does not depend on which
// block evaluated which item.  A wave takes two slices, its lanes the columns (two
// each in fits of more than 31 waves), so that a slice's items are counted per wave
// and whole partials are read; the first items of both samples are read together.
//
// With STEP the first wave then advances the fit's L-BFGS state, loaded ahead of the
// partials; otherwise the result goes to out[fit][2k + 2].  Bound by latency with few
// items per fit, by what one CU reads with many.  64 fits, 11.8 GB of rows, sums alone:
// 328 us in items of 64 KB, 94 of 256 KB, 28 of 1 MB, 9.7 of 4 MB; 428, 120, 34 and
// 12.2 us with one sum per thread and a load of its own for each (1024 threads), 487,
// 138, 39 and 12.7 us when a thread read an item for all of its sums in every round,
// whether they had one or not.  With the update 22.7 us (4 MB).
constexpr int kCombineThreads = 512;
constexpr int kSlices = 16;
constexpr int kWaveSlices = kSlices / (kCombineThreads / 64);
constexpr int kAhead = 4;                              // items of a slice in flight

// Sums of a wave's slices of one sample: items first + sl + 16 t of n, t in order.
// NC: columns per lane; lanes past the last column read it again.
template <int NC>
struct SliceSums {
    typedef const double __attribute__((address_space(1))) *gptr;
    gptr src[NC];
    int last;                                          // of the sample's items, from src on
    int count[kWaveSlices];                            // items of each slice
    double s[kWaveSlices][NC], x[kAhead][kWaveSlices][NC];

    __device__ __forceinline__ SliceSums(const double *partials, int first, int n, int sl, int ps) {
        const int lane = threadIdx.x & 63;
        // a sample without items reads the first partial
        gptr base = (gptr)partials + (n > 0 ? (int64_t)(first + (sl < n ? sl : 0)) * kMultiSlot : 0);
        last = max(n - 1 - sl, 0);
#pragma unroll
        for (int c = 0; c < NC; ++c) src[c] = base + min(lane + 64 * c, ps - 1);
#pragma unroll
        for (int j = 0; j < kWaveSlices; ++j) {
            count[j] = n > sl + j ? (n - sl - j + kSlices - 1) / kSlices : 0;
#pragma unroll
            for (int c = 0; c < NC; ++c) s[j][c] = 0.0;
        }
    }
    // items t .. t + kAhead - 1; in the place of those past the slice's last, the
    // sample's last one (no branch around the loads, at whose join they would be waited for)
    __device__ __forceinline__ void load(int t) {
#pragma unroll
        for (int h = 0; h < kAhead; ++h)
#pragma unroll
            for (int j = 0; j < kWaveSlices; ++j) {
                const int64_t i = min((t + h) * kSlices + j, last);
#pragma unroll
                for (int c = 0; c < NC; ++c) x[h][j][c] = src[c][i * kMultiSlot];
            }
    }
    __device__ __forceinline__ void add(int t) {
#pragma unroll
        for (int h = 0; h < kAhead; ++h)
#pragma unroll
            for (int j = 0; j < kWaveSlices; ++j)
#pragma unroll
                for (int c = 0; c < NC; ++c) s[j][c] += t + h < count[j] ? x[h][j][c] : 0.0;     // no sum is -0
    }
};

template <int NC>
__device__ __forceinline__ void slice_sums(const MultiArgs &p, const MultiFit &fit, int ps,
                                           double (*part)[2][1 + 2 * kMultiMaxLd]) {
    const int lane = threadIdx.x & 63, sl = kWaveSlices * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    SliceSums<NC> d(p.partials, fit.item_data0, fit.item_data1 - fit.item_data0, sl, ps);
    SliceSums<NC> m(p.partials, fit.item_mc0, fit.item_mc1 - fit.item_mc0, sl, ps);
    if (d.count[0] + m.count[0] > 0) {
        d.load(0);
        m.load(0);
        d.add(0);
        m.add(0);
    }
    for (int t = kAhead; t < d.count[0]; t += kAhead) {
        d.load(t);
        d.add(t);
    }
    for (int t = kAhead; t < m.count[0]; t += kAhead) {
        m.load(t);
        m.add(t);
    }
#pragma unroll
    for (int j = 0; j < kWaveSlices; ++j)
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (lane + 64 * c < ps) {
                part[sl + j][0][lane + 64 * c] = d.s[j][c];
                part[sl + j][1][lane + 64 * c] = m.s[j][c];
            }
}

template <bool STEP>
__global__ __launch_bounds__(kCombineThreads) void multi_combine_kernel(MultiArgs p, LbfgsState *states, double c1,
                                                                        double ftol) {
    __shared__ double part[kSlices][2][1 + 2 * kMultiMaxLd];
    __shared__ double tot[2][1 + 2 * kMultiMaxLd];
    __shared__ double prod[64 * kLbfgsPer];
    const int f = blockIdx.x, tid = threadIdx.x;
    const MultiFit fit = p.fits[f];
    const int k = fit.k, ps = 1 + 2 * (int)fit.ld;
    LbRegs r;
    if (STEP && tid < 64) lbfgs_load(r, states + f, 2 * k, false);
    if (ps <= 64) slice_sums<1>(p, fit, ps, part);
    else slice_sums<2>(p, fit, ps, part);
    __syncthreads();
    for (int idx = tid; idx < 2 * ps; idx += kCombineThreads) {
        const int sg = idx >= ps, cc = idx - sg * ps;
        double t = 0.0;
#pragma unroll
        for (int sl = 0; sl < kSlices; ++sl) t += part[sl][sg][cc];
        tot[sg][cc] = t;
    }
    __syncthreads();
    if (f == 0 && tid == 0) *p.item_counter = 0u;      // ready for the next launch
    if (tid >= 64) return;
    const double nd = (double)fit.n_data;
    const double sum_log = tot[0][0] * EventMath<float>::kLogScale;
    const double s_raw = tot[1][0];
    double nll = 0.0, c = 0.0;
    unsigned flags = 0;
    if (nd != 0.0) {
        const double S = s_raw / fit.n_gen;
        nll = -sum_log + nd * log(S);
        c = nd / s_raw;
        if (!isfinite(nll) || !(S > 0.0)) {
            nll = INFINITY;
            flags = 1;
        }
    }
    LbVec g;
#pragma unroll
    for (int u = 0; u < kLbfgsPer; ++u) {
        const int i = tid + 64 * u;
        g.e[u] = i < 2 * k ? 2.0 * (-tot[0][1 + i] + c * tot[1][1 + i]) : 0.0;
    }
    if constexpr (STEP) {
        lbfgs_advance(states + f, r, 2 * k, nll, g, c1, ftol, false, 0.0, prod);
    } else {
        double *out = p.out + (int64_t)f * kMultiOut;
        lb_store(out + 1, g, 2 * k, tid);
        if (tid == 0) {
            out[0] = nll;
            out[1 + 2 * k] = (double)flags;
        }
    }
}

}  // namespace

hipError_t launch_multi_eval(const MultiArgs &args, int blocks, hipStream_t stream) {
    hipLaunchKernelGGL(multi_stream_kernel, dim3(blocks), dim3(kMT), 0, stream, args);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(multi_combine_kernel<false>, dim3(args.n_fits), dim3(kCombineThreads), 0, stream, args, nullptr,
                       0.0, 0.0);
    return hipGetLastError();
}

hipError_t launch_multi_step(const MultiArgs &args, int blocks, LbfgsState *states, int m, double c1, double ftol,
                             hipStream_t stream) {
    if (m != kLbfgsHist) return hipErrorInvalidValue;
    hipLaunchKernelGGL(multi_stream_kernel, dim3(blocks), dim3(kMT), 0, stream, args);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(multi_combine_kernel<true>, dim3(args.n_fits), dim3(kCombineThreads), 0, stream, args, states, c1,
                       ftol);
    return hipGetLastError();
}

bool multi_ld_supported(int64_t ld) {
    return ld == 4 || ld == 6 || ld == 8 || ld == 12 || ld == 16 || ld == 24 || ld == 32 || ld == 48;
}

int64_t multi_layout_ld(int k) {
    static const int widths[] = {4, 6, 8, 12, 16, 24, 32, 48};
    for (int w : widths)
        if (w >= k) return w;
    return -1;
}

int multi_rows_per_tile(int64_t ld) {
    switch (ld) {
        case 4: return 32 * 4;
        case 6: return 32 * 2;
        case 8: return 16 * 4;
        case 12: return 16 * 2;
        case 16: return 8 * 4;
        case 24: return 16 * 2;
        case 32: return 4 * 4;
        case 48: return 8 * 2;
        default: return 0;
    }
}

}  // namespace pwa
