// Host check of the launch plan (plan.h) and of the fixed work positions
// (kernel_params.h: static_position): over a grid of GEMM sizes, odd ones among
// them, the plan's row tiles fit the row-tile table, a split fits one round of
// workgroups, the split counters and the workspace, no slice is empty, no plan
// within these bounds has a lower estimate, the rounds of all workgroups take
// every work position once, and fused operators of one round get the tile that
// plan_one_round describes. The sizes given as
// arguments ("M,N,K,partial,cfg,split") must get that tile and split.
// Prints "ok <sizes>" or the first failure.
#include <cstdio>
#include <cstring>
#include <vector>

#define __host__
#define __device__
#include "plan.h"

using namespace compass;

static GemmParams params(int M, int N, int K, const Plan &pl, int num_cu) {
    GemmParams g;
    std::memset(&g, 0, sizeof g);
    const TileShape &ts = kTileShapes[pl.cfg];
    g.tiles_m = (M + ts.rows - 1) / ts.rows;
    g.tiles_n = (N + ts.cols - 1) / ts.cols;
    g.K = K;
    g.kslice = K;
    g.ksplit = 1;
    g.group_m = ts.rows == 256 ? 4 : 8;
    const int slots = num_cu * ts.wg_per_cu;
    if (pl.split > 1) g.ksplit = slices_of(K, pl.split, &g.kslice);
    g.grid = std::min(g.tiles_m * g.tiles_n * g.ksplit, slots);
    return g;
}

static bool check(int M, int N, int K, bool partial, const PlanLimits &lim, char *why) {
    const Plan pl = plan_gemm(M, N, K, partial, lim);
    if (pl.cfg < 0 || pl.cfg >= kTileCfgs || pl.split < 1 || pl.split > kMaxSplit) { std::sprintf(why, "plan %d/%d", pl.cfg, pl.split); return false; }
    const GemmParams g = params(M, N, K, pl, lim.num_cu);
    const TileShape &ts = kTileShapes[pl.cfg];
    if (g.tiles_m > kMaxRowTiles) { std::sprintf(why, "%d row tiles", g.tiles_m); return false; }
    const int tiles = g.tiles_m * g.tiles_n;
    if (pl.split > 1) {
        if (g.ksplit != pl.split) { std::sprintf(why, "%d slices for a plan of %d", g.ksplit, pl.split); return false; }
        if (ts.rows <= 64) { std::sprintf(why, "the smallest tile split"); return false; }
        if (tiles > kMaxSplitTiles || (long)tiles * g.ksplit > (long)lim.num_cu * ts.wg_per_cu ||
            (uint64_t)tiles * g.ksplit * ts.rows * ts.cols * 4 > lim.split_bytes) { std::sprintf(why, "split out of bounds"); return false; }
        if ((g.ksplit - 1) * g.kslice >= K || g.kslice % 64) { std::sprintf(why, "slice %d of K %d", g.kslice, K); return false; }
    }
    // the staging copies on top of the estimate for tiles they cannot do without
    PlanLimits bare = lim;
    bare.row_step = 0;
    auto cost_of = [&](int cfg, int sp) {
        return plan_cost(cfg, sp, M, N, K, partial, bare) +
               (lim.row_step && lim.row_step % kTileShapes[cfg].rows ? lim.staging_us : 0.0);
    };
    const double cost = cost_of(pl.cfg, pl.split);
    for (int cfg = 0; cfg < kTileCfgs; ++cfg)
        for (int sp = 1; sp <= kMaxSplit; ++sp) {
            const TileShape &o = kTileShapes[cfg];
            const long tm = (M + o.rows - 1) / o.rows, t = tm * ((N + o.cols - 1) / o.cols);
            if (tm > kMaxRowTiles) continue;
            if (sp > 1 && (o.rows <= 64 || K / sp < kMinSliceK || t > kMaxSplitTiles || t * sp > (long)lim.num_cu * o.wg_per_cu ||
                           (uint64_t)t * sp * o.rows * o.cols * 4 > lim.split_bytes))
                continue;
            const double c = cost_of(cfg, sp);
            if (c < cost * (1 - 1e-9)) { std::sprintf(why, "plan %d/%d at %.2f us, %d/%d at %.2f", pl.cfg, pl.split, cost, cfg, sp, c); return false; }
        }
    const int all = work_items(g);
    for (int fixed = 1; fixed <= 2; ++fixed) {
        GemmParams f = g;
        f.fixed = fixed;
        std::vector<int> by(all, -1);   // workgroup of each position
        for (int b = 0; b < f.grid; ++b)
            for (int j = 0; fixed == 1 || j < 2; ++j) {
                const int pos = static_position(f, b, j);
                if (pos < 0) break;
                if (pos >= all || by[pos] >= 0) { std::sprintf(why, "position %d of %d by workgroup %d round %d", pos, all, b, j); return false; }
                by[pos] = b;
            }
        if (fixed == 2 && all > f.grid) continue;   // (only launches of one round are dealt so)
        for (int p = 0; p < all; ++p) {
            if (by[p] < 0) { std::sprintf(why, "position %d of %d left out", p, all); return false; }
            // dealt group_m at a time over the XCDs, as long as the turns are full
            if (fixed == 2 && p < all / (kMaxQueues * f.group_m) * kMaxQueues * f.group_m &&
                by[p] % kMaxQueues != p / f.group_m % kMaxQueues) { std::sprintf(why, "position %d on XCD %d", p, by[p] % kMaxQueues); return false; }
        }
    }
    return true;
}

// The tile of a fused operator of one round: 64 x 64 for an AllGather whose
// tiles of that size have a CU each, else the lowest estimate among the tiles of
// at most 128 x 128 that fit.
static bool check_one_round(int M, int N, int K, bool partial, const PlanLimits &lim, char *why) {
    const int cfg = plan_one_round(M, N, K, partial, lim);
    auto tiles = [&](int c) {
        return (long)((M + kTileShapes[c].rows - 1) / kTileShapes[c].rows) * ((N + kTileShapes[c].cols - 1) / kTileShapes[c].cols);
    };
    auto fits = [&](int c) {
        const TileShape &ts = kTileShapes[c];
        return ts.rows <= 128 && ts.cols <= 128 && (M + ts.rows - 1) / ts.rows <= kMaxRowTiles &&
               tiles(c) <= (lim.slots_override > 0 ? lim.slots_override : (long)lim.num_cu * ts.wg_per_cu);
    };
    if (cfg >= 0 && !fits(cfg)) { std::sprintf(why, "one round in tile %d", cfg); return false; }
    if (!partial && fits(kTile64) && tiles(kTile64) <= lim.num_cu) {
        if (cfg != kTile64) std::sprintf(why, "tile %d, not 64 x 64 with a CU each", cfg);
        return cfg == kTile64;
    }
    for (int c = 0; c < kTileCfgs; ++c)
        if (fits(c) && (cfg < 0 || plan_cost(c, 1, M, N, K, partial, lim) < plan_cost(cfg, 1, M, N, K, partial, lim) * (1 - 1e-9))) {
            std::sprintf(why, "one round in tile %d, cheaper in %d", cfg, c);
            return false;
        }
    return true;
}

int main(int argc, char **argv) {
    const PlanLimits split{256, 0, 3ull * 256 * 256 * 256 * 4}, whole{256, 0, 0}, small{4, 0, 3ull * 4 * 256 * 256 * 4},
                     few{256, 24, 0}, stage128{256, 0, split.split_bytes, 128, 8.0}, stage192{256, 0, split.split_bytes, 192, 8.0};
    char why[256];
    int count = 0;
    const int Ms[] = {1, 15, 64, 65, 127, 129, 257, 640, 1000, 2049, 4096, 8191, 32768, 32769, 65536};
    const int Ns[] = {8, 72, 256, 776, 2048, 3080, 12288};
    const int Ks[] = {8, 64, 200, 512, 1032, 4096, 8192, 12296};
    for (int M : Ms)
        for (int N : Ns)
            for (int K : Ks)
                for (int p = 0; p < 2; ++p)
                    for (const PlanLimits &lim : {split, whole, small, stage128, stage192}) {
                        ++count;
                        if (!check(M, N, K, p, lim, why) || !check_one_round(M, N, K, p, lim, why)) {
                            std::printf("FAIL %d x %d x %d partial %d cus %d: %s\n", M, N, K, p, lim.num_cu, why);
                            return 1;
                        }
                    }
    for (const int *x : {(const int[]){512, 1024, 512}, (const int[]){1000, 1000, 520}, (const int[]){256, 256, 64}}) {
        for (const PlanLimits &lim : {split, few})
            if (!check_one_round(x[0], x[1], x[2], false, lim, why)) { std::printf("FAIL %d x %d x %d: %s\n", x[0], x[1], x[2], why); return 1; }
    }
    for (int i = 1; i < argc; ++i) {
        int M, N, K, p, cfg, sp;
        if (std::sscanf(argv[i], "%d,%d,%d,%d,%d,%d", &M, &N, &K, &p, &cfg, &sp) != 6) { std::printf("FAIL argument %s\n", argv[i]); return 1; }
        const Plan pl = plan_gemm(M, N, K, p, split);
        if (pl.cfg != cfg || pl.split != sp) { std::printf("FAIL %s: plan %d/%d\n", argv[i], pl.cfg, pl.split); return 1; }
    }
    std::printf("ok %d\n", count);
    return 0;
}
