// Variant table, layout width and launch dispatch of the fused likelihood kernel.
#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "block_reduce.hpp"
#include "internal.hpp"

namespace pwa {

hipError_t stream_dispatch_f32_c1(int, int, int, const StreamArgs &, hipStream_t);
hipError_t stream_dispatch_f32_c2(int, int, int, const StreamArgs &, hipStream_t);
hipError_t stream_dispatch_f32_c3(int, int, int, const StreamArgs &, hipStream_t);
hipError_t stream_dispatch_f32_c4(int, int, int, const StreamArgs &, hipStream_t);
hipError_t stream_dispatch_f32_c8(int, int, int, const StreamArgs &, hipStream_t);
hipError_t stream_dispatch_f64_c1(int, int, int, const StreamArgs &, hipStream_t);
hipError_t stream_dispatch_f64_c2(int, int, int, const StreamArgs &, hipStream_t);
hipError_t stream_dispatch_f64_c3(int, int, int, const StreamArgs &, hipStream_t);
hipError_t stream_dispatch_f64_c4(int, int, int, const StreamArgs &, hipStream_t);

namespace {

// (C, U) pairs compiled per precision; L runs over powers of two with L * C <= 64.
struct CU {
    int C, U;
};
const CU kF32[] = {{1, 4}, {1, 8}, {2, 2}, {2, 4}, {3, 1}, {3, 2}, {4, 1}, {4, 2}, {8, 1}};
const CU kF64[] = {{1, 2}, {1, 4}, {2, 1}, {2, 2}, {3, 1}, {4, 1}};

struct Table {
    StreamCfg v[128];
    int n = 0;
    Table(const CU *cu, int ncu) {
        for (int i = 0; i < ncu; ++i)
            for (int L = 1; L <= 32; L <<= 1)
                if (L * cu[i].C <= 64) v[n++] = StreamCfg{L, cu[i].C, cu[i].U, 0};
    }
};

const Table &table(pwa_prec prec) {
    static const Table f32(kF32, sizeof kF32 / sizeof kF32[0]);
    static const Table f64(kF64, sizeof kF64 / sizeof kF64[0]);
    return prec == PWA_F32 ? f32 : f64;
}

}  // namespace

const StreamCfg *stream_variants(pwa_prec prec, int *count) {
    const Table &t = table(prec);
    *count = t.n;
    return t.v;
}

bool stream_cfg_available(pwa_prec prec, const StreamCfg &c) {
    const Table &t = table(prec);
    for (int i = 0; i < t.n; ++i)
        if (t.v[i].L == c.L && t.v[i].C == c.C && t.v[i].U == c.U) return true;
    return false;
}

int stream_layout_ld(pwa_prec prec, int k) {
    const Table &t = table(prec);
    int best = 1 << 30;
    for (int i = 0; i < t.n; ++i) {
        const int ld = t.v[i].L * t.v[i].C;
        if (ld >= k && ld < best) best = ld;
    }
    return best;
}

StreamCfg stream_default_cfg(pwa_prec prec, int ld) {
    // Preference: about 32 B per lane per row (fewer lanes per row means less
    // redundant per-event work), 64 B per lane per stage, one block per CU: its four
    // waves keep two stages each in flight, and every further block brings partials
    // and a ragged end.  256 against 1024 blocks, one evaluation: 20 MB of rows 19.7 /
    // 25.4 us at K = 16, 19.3 / 22.3 at 23; 60 MB 25.5 / 29.6 and 25.5 / 27.2; 180 MB
    // 42.4 / 49.8; 720 MB 129.9 / 132.2 (numbers between multiples of the CUs are worse).
    // At other widths and in FP64, these rules and those of stream_grid together against
    // 1024 blocks: K = 48 FP32, 20,000 rows 17.6 / 21.0 us, 300,000 33.4 / 38.6, 1.2 10^6
    // 88.6 / 94.1; K = 64 20.4 / 24.3, 40.6 / 48.2, 112 / 120; FP64 with half the rows
    // K = 2 14.3 / 16.8, 15.9 / 18.7, 17.6 / 22.3, K = 64 19.8 / 23.7, 42.6 / 47.9,
    // 116 / 122.
    const Table &t = table(prec);
    const int eb = prec == PWA_F32 ? 8 : 16;
    StreamCfg best{0, 0, 0, 1};
    int best_score = 1 << 30;
    for (int i = 0; i < t.n; ++i) {
        const StreamCfg &c = t.v[i];
        if (c.L * c.C != ld) continue;
        const int row_bytes = c.C * eb, stage_bytes = row_bytes * c.U;
        const int score = std::abs(row_bytes - 32) * 4 + std::abs(stage_bytes - 64);
        if (score < best_score) {
            best_score = score;
            best = StreamCfg{c.L, c.C, c.U, 1};
        }
    }
    return best;
}

// A block takes at least kLeastBlockBytes of rows, down to kLeastBlocks of them: with
// less, its partial costs more than it streams.  128 against 256 blocks: 4 MB of rows
// 16.2 / 17.3 us at K = 23, 7 MB 16.8 / 17.7, 12 MB 18.3 / 18.3, 20 MB 20.6 / 19.3; at
// 2 MB 64 blocks take 15.5, 128 15.8, 256 16.5 us.
constexpr int64_t kLeastBlockBytes = 48 << 10;
constexpr int64_t kLeastBlocks = 64;
// A sample keeps to the blocks whose partials the last block adds directly (block_reduce.hpp)
// up to this many bytes per block: 1 MB of rows 14.3 us instead of 15.7 at K = 23, 3 MB
// 15.1 / 16.5 at 23 and 15.1 / 16.7 at 14, 8 MB 15.8 / 18.0 at 8; at the limit the two meet.
constexpr int64_t kDirectBytes = 112 << 10;

void stream_grid(const StreamCfg &cfg, int64_t budget, int64_t row_bytes, int64_t n0, int64_t n1, int32_t nb[2]) {
    budget = std::min(budget, std::max(kLeastBlocks, (n0 + n1) * row_bytes / kLeastBlockBytes));
    const int64_t rows_per_block = (int64_t)stream_rows_per_wave(cfg) * (kStreamThreads / 64);
    const int64_t need[2] = {(n0 + rows_per_block - 1) / rows_per_block, (n1 + rows_per_block - 1) / rows_per_block};
    const int64_t direct = reduce_direct_blocks((int)(1 + 2 * cfg.L * cfg.C), kStreamThreads);
    const bool few = std::max(n0, n1) * row_bytes <= direct * kDirectBytes;
    if (few) budget = std::min(budget, 2 * direct);
    if (need[0] + need[1] <= budget) {
        nb[0] = (int32_t)(few ? std::min(need[0], direct) : need[0]);
        nb[1] = (int32_t)(few ? std::min(need[1], direct) : need[1]);
        return;
    }
    const double frac = (double)n0 / (double)(n0 + n1);
    int64_t b0 = (int64_t)std::llround(frac * (double)budget);
    if (n0 > 0) b0 = std::max<int64_t>(b0, 1);
    if (n1 > 0) b0 = std::min<int64_t>(b0, budget - 1);
    b0 = std::min(b0, need[0]);
    const int64_t b1 = std::min(budget - b0, need[1]);
    nb[0] = (int32_t)(few ? std::min(b0, direct) : b0);
    nb[1] = (int32_t)(few ? std::min(b1, direct) : b1);
}

hipError_t launch_stream(pwa_prec prec, const StreamCfg &c, int blocks, const StreamArgs &args,
                         hipStream_t stream) {
    // the kernel takes the row stride from its (L, C): the layout width
    if (!stream_cfg_available(prec, c) || blocks < 1 || args.ld != (int64_t)c.L * c.C) return hipErrorInvalidValue;
    if (prec == PWA_F32) {
        switch (c.C) {
            case 1: return stream_dispatch_f32_c1(c.L, c.U, blocks, args, stream);
            case 2: return stream_dispatch_f32_c2(c.L, c.U, blocks, args, stream);
            case 3: return stream_dispatch_f32_c3(c.L, c.U, blocks, args, stream);
            case 4: return stream_dispatch_f32_c4(c.L, c.U, blocks, args, stream);
            case 8: return stream_dispatch_f32_c8(c.L, c.U, blocks, args, stream);
            default: break;
        }
    } else {
        switch (c.C) {
            case 1: return stream_dispatch_f64_c1(c.L, c.U, blocks, args, stream);
            case 2: return stream_dispatch_f64_c2(c.L, c.U, blocks, args, stream);
            case 3: return stream_dispatch_f64_c3(c.L, c.U, blocks, args, stream);
            case 4: return stream_dispatch_f64_c4(c.L, c.U, blocks, args, stream);
            default: break;
        }
    }
    return hipErrorInvalidValue;
}

}  // namespace pwa
