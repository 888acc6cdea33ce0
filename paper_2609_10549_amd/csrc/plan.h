// Tile shape and K split of a launch whose tiles do not wait for one another's
// arrivals (plain GEMM, InterDecom sub-GEMMs, unfused baselines), from an
// estimate of its time. Host only.
#pragma once
#include <algorithm>

#include "kernel_params.h"

namespace compass {

struct Plan {
    int cfg;      // TileCfg
    int split;    // K slices per tile (1: whole)
};

// What may be split: the workspace's fp32 partial tiles, in bytes (0: nothing).
// A launch that reads part of its partial from other buffers can do so when
// the rows of its tiles divide `row_step`; with other tiles those rows are
// copied first, which takes `staging_us`.
struct PlanLimits {
    int num_cu;
    int slots_override;     // workgroups per launch (0: as many as the CUs hold)
    uint64_t split_bytes;
    int row_step = 0;
    double staging_us = 0.0;
};

constexpr int kMinSliceK = 512;     // K depth of a slice at least

// Microseconds on MI355X (bf16, N(0, 1) data), fitted to launches of 8 to 192
// stages of K = 64: a stage on one workgroup with most of the chip idle
// (`alone`), a stage of every workgroup with all CUs holding as many as they
// can (`full`: power bound for the large tiles, load bound for the small ones),
// the tile's prologue and epilogue, and the factor on the stages when rows of
// A and W do not start on 128-byte lines (K no multiple of 64: every row's
// load touches two lines).
struct TileCost { float alone, full, edge, ragged; };
constexpr TileCost kTileCosts[kTileCfgs] = {
    {0.984f, 1.365f, 6.9f, 1.05f},   // 256 x 256
    {0.385f, 0.914f, 1.3f, 1.40f},   // 128 x 128, two per CU
    {0.753f, 1.060f, 5.9f, 1.20f},   // 256 x 192
    {0.537f, 0.787f, 3.7f, 1.40f},   // 256 x 128
    {0.330f, 0.467f, 2.4f, 1.50f},   // 128 x 128 deep
    {0.319f, 0.768f, 1.4f, 1.50f},   // 128 x 64, two per CU
    {0.205f, 0.293f, 2.2f, 1.65f},   // 128 x 64 deep
    {0.137f, 0.418f, 2.8f, 1.35f},   // 64 x 64, two per CU
    {0.586f, 0.830f, 5.3f, 1.25f},   // 192 x 192
    {0.440f, 0.630f, 4.0f, 1.40f},   // 128 x 192
};

inline int slices_of(int K, int split, int *kslice) {
    *kslice = ((K + split - 1) / split + 63) / 64 * 64;
    return (K + *kslice - 1) / *kslice;
}

// Estimated time of M x N x K in tiles of `cfg`, K in `split` slices.
inline double plan_cost(int cfg, int split, int M, int N, int K, bool partial, const PlanLimits &lim) {
    const TileShape &ts = kTileShapes[cfg];
    const TileCost &tc = kTileCosts[cfg];
    const double area = (double)ts.rows * ts.cols;
    int kslice;
    const int sp = slices_of(K, split, &kslice);
    const long items = (long)((M + ts.rows - 1) / ts.rows) * ((N + ts.cols - 1) / ts.cols) * sp;
    const long slots = lim.slots_override > 0 ? lim.slots_override : (long)lim.num_cu * ts.wg_per_cu;
    const double stages = (std::min(kslice, K) + 63) / 64 * (K % 64 ? tc.ragged : 1.0);
    // the partial's read, and, split, the completing slice's wait for the
    // partial tiles' way through memory (uncached) and its sums over them
    const double edge = tc.edge + (partial ? 6.0 * area * ts.wg_per_cu / 65536 : 0.0) +
                        (sp > 1 ? (2.5 + sp * area * 4 / 65e3) * (items > lim.num_cu ? ts.wg_per_cu : 1) : 0.0);
    const long rounds = items / slots, rest = items % slots;
    double t = rounds * (stages * tc.full + edge);
    if (rest) {
        // a partly filled chip runs between the two stage times (the power
        // the busy CUs draw sets the clock of all), and with some CUs holding
        // two workgroups it ends with those
        const double x = rest > lim.num_cu ? std::max(0.9, (double)rest / slots) : (double)rest / slots;
        t += stages * (tc.alone + (tc.full - tc.alone) * x * x) + edge;
    }
    return lim.row_step % ts.rows ? t + lim.staging_us : t;
}

inline Plan plan_gemm(int M, int N, int K, bool partial, const PlanLimits &lim) {
    auto allowed = [&](int cfg, int split) {
        const TileShape &ts = kTileShapes[cfg];
        const long tm = (M + ts.rows - 1) / ts.rows, tiles = tm * ((N + ts.cols - 1) / ts.cols);
        if (tm > kMaxRowTiles) return false;
        if (split == 1) return true;
        const long slots = lim.slots_override > 0 ? lim.slots_override : (long)lim.num_cu * ts.wg_per_cu;
        // one round of slices (the workspace holds a launch's partial tiles)
        return ts.rows > 64 && K / split >= kMinSliceK && tiles <= kMaxSplitTiles && tiles * split <= slots &&
               (uint64_t)tiles * split * ts.rows * ts.cols * 4 <= lim.split_bytes;
    };
    Plan best{kTile128, 1};
    double tb = 1e30;
    for (int cfg = 0; cfg < kTileCfgs; ++cfg)
        for (int sp = 1; sp <= kMaxSplit; ++sp) {
            if (!allowed(cfg, sp)) continue;
            const double t = plan_cost(cfg, sp, M, N, K, partial, lim);
            if (t < tb) {
                tb = t;
                int kslice;
                best = {cfg, slices_of(K, sp, &kslice)};
            }
        }
    return best;
}

// Tile of a fused operator so small that tiles of at most 128 x 128 fit one
// round of workgroups; -1 when no such tile's do. Every tile then starts with
// the launch, and what follows the last arrival is one tile, so the estimate's
// cheapest is the shortest tail. (Larger tiles in one round wait for more of
// the arrivals and leave a longer tail: the MLP fc1 218 us in 256 x 256 tiles,
// 190 in two rounds of 256 x 128.)
//
// An AllGather whose 64 x 64 tiles have a CU each takes those: the estimate's
// costs are those of a busy chip, and below some 30 stages they put 128 x 64
// first, which in 19 sizes of K = 64 to 2048 was never the faster by more than
// 0.3 us (512 x 1024 x 512 over two ranks 20.8 us against 22.1, in 128 x 128
// 24.0; 1024 x 1024 x 1024 over four 30.8 against 32.6). With two of them on a
// CU they no longer are (1024 x 2048 x 512: 33.9 against 28.1). For a
// ReduceScatter, whose last sends follow the launch, either is within 1.5 %.
inline int plan_one_round(int M, int N, int K, bool partial, const PlanLimits &lim) {
    const long tiles64 = (long)((M + 63) / 64) * ((N + 63) / 64);
    if (!partial && tiles64 <= lim.num_cu && (lim.slots_override <= 0 || tiles64 <= lim.slots_override)) return kTile64;
    int best = -1;
    double tb = 1e30;
    for (int cfg = 0; cfg < kTileCfgs; ++cfg) {
        const TileShape &ts = kTileShapes[cfg];
        const long tm = (M + ts.rows - 1) / ts.rows, tiles = tm * ((N + ts.cols - 1) / ts.cols);
        const long slots = lim.slots_override > 0 ? lim.slots_override : (long)lim.num_cu * ts.wg_per_cu;
        if (tm > kMaxRowTiles || tiles > slots || ts.rows > 128 || ts.cols > 128) continue;
        const double t = plan_cost(cfg, 1, M, N, K, partial, lim);
        if (t < tb) {
            tb = t;
            best = cfg;
        }
    }
    return best;
}

// Whether the few-row kernel (skinny_kernel: 16 columns per workgroup, K dealt
// to its waves) beats the plan. Its stages take 0.06 us per 16 columns with up
// to 16 rows, 0.015 more per further 16 rows, a third more when its workgroups
// need several rounds (A's rows then compete with W for the caches); a plan
// takes at least W's way in at 5.5 TB/s. 48 x 3072 x 8192: 25.2 us whole in
// 64 x 64 tiles, 16.8 split in slices, 15.8 here; 8 x 12288 x 12288: 58.5
// against 49.4; but 64 x 12288 x 12288: 74.4 against 101.
inline bool skinny_faster(int M, int N, int K, bool partial, const Plan &pl, const PlanLimits &lim) {
    if (M > kSkinnyRows || N > (1 << 24)) return false;   // (the latter: threads of one launch below 2^32)
    const int mt = (M + 15) / 16;
    const long wgs = (N + 15) / 16, rounds = (wgs + lim.num_cu - 1) / lim.num_cu;
    const double stage = (0.045 + 0.015 * mt) * (rounds > 1 ? 1.33 : 1.0);
    const double skinny = rounds * (1.5 + (K + 63) / 64 * stage);
    const double tiles = std::max(plan_cost(pl.cfg, pl.split, M, N, K, partial, lim), (double)N * K * 2 / 5.5e6);
    return skinny < tiles;
}

}  // namespace compass
