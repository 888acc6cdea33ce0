// compass_gemm_noalloc: the plain GEMM of compass_gemm for callers that
// cannot allocate device memory (code under HIP graph capture, tight serving
// loops, harnesses that forbid allocation).
//
// The launch never splits K (that would need a partial-tile workspace) and
// its workgroups take their tiles by position, without tickets, so the kernel
// needs no scratch at all: no hipMalloc, no hipFree, no library
// initialisation, no memory shared between calls. The first call on a device
// looks up its architecture and CU count and keeps them.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>

#include "compass.h"
#include "internal.h"
#include "kernel_params.h"
#include "plan.h"

namespace compass {

hipError_t launch_gemm(const GemmParams &p, int cfg, bool rs, hipStream_t stream);
hipError_t launch_skinny(const SkinnyParams &p, hipStream_t stream);

namespace {

constexpr int kMaxDevices = 64;

int g_num_cu[kMaxDevices];   // 0: not looked up yet
std::mutex g_mu;

int hip_error(hipError_t e, const char *what) {
    return set_error(COMPASS_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

// The CU count of the current device, looked up on the first call on it.
int current_num_cu(int *out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_error(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return set_error(COMPASS_ERR_UNSUPPORTED, "device %d beyond %d", dev, kMaxDevices);
    std::lock_guard<std::mutex> lk(g_mu);
    if (g_num_cu[dev] == 0) {
        hipDeviceProp_t prop;
        if ((e = hipGetDeviceProperties(&prop, dev)) != hipSuccess) return hip_error(e, "hipGetDeviceProperties");
        if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
            return set_error(COMPASS_ERR_UNSUPPORTED, "device %d is %s, this library is built for gfx950", dev,
                             prop.gcnArchName);
        g_num_cu[dev] = prop.multiProcessorCount;
    }
    *out = g_num_cu[dev];
    return COMPASS_OK;
}

}  // namespace

int op_gemm_noalloc(int M, int N, int K, const void *A, const void *W, void *C, const float *P, void *stream) {
    if (M < 1 || N < 1 || K < 1 || K % 8 || N % 8)
        return set_error(COMPASS_ERR_INVALID, "need positive M, N, K with K, N multiples of 8");
    if (!A || !W || !C) return set_error(COMPASS_ERR_INVALID, "A, W and C are required");
    if ((M + 127) / 128 > kMaxRowTiles)
        return set_error(COMPASS_ERR_UNSUPPORTED, "M = %d above the %d rows of the tile table", M, kMaxRowTiles * 128);
    // the kernel addresses a tile's operands with 32-bit offsets from the
    // tile's first row (column of W): a 256-row tile spans at most
    // kTileSpanMax bytes of each
    if (256ull * (uint64_t)K * 2 > kTileSpanMax || (P && 256ull * (uint64_t)N * 4 > kTileSpanMax))
        return set_error(COMPASS_ERR_UNSUPPORTED, "K = %d, N = %d: a 256-row tile would span more than 1 GiB of A, W "
                                                  "or the partial", K, N);
    int num_cu = 0;
    int rc = current_num_cu(&num_cu);
    if (rc != COMPASS_OK) return rc;

    hipStream_t s = (hipStream_t)stream;
    // compass_gemm's choice among the plans that split no K
    const PlanLimits lim{num_cu, 0, 0};
    const Plan pl = plan_gemm(M, N, K, P != nullptr, lim);
    if (skinny_faster(M, N, K, P != nullptr, pl, lim)) {
        const hipError_t e = launch_skinny({(const uint16_t *)A, (const uint16_t *)W, (uint16_t *)C, P, M, N, K}, s);
        return e == hipSuccess ? COMPASS_OK : hip_error(e, "GEMM launch");
    }
    const int cfg = pl.cfg;
    GemmParams g;
    std::memset(&g, 0, sizeof g);
    const int bm = tile_rows(cfg), bn = tile_cols(cfg);
    g.A = (const uint16_t *)A;
    g.W = (const uint16_t *)W;
    g.C = (uint16_t *)C;
    g.P = P;
    g.M = M;
    g.N = N;
    g.K = K;
    g.lda = K;
    g.ldw = K;
    g.ldc = N;
    g.ldp = N;
    g.a_bytes = (uint64_t)M * (uint64_t)K * 2;
    g.w_bytes = (uint64_t)N * (uint64_t)K * 2;
    g.p_bytes = P ? (uint64_t)M * (uint64_t)N * 4 : 0u;
    g.c_bytes = (uint64_t)M * (uint64_t)N * 2;
    g.tiles_m = (M + bm - 1) / bm;
    g.tiles_n = (N + bn - 1) / bn;
    const int total = g.tiles_m * g.tiles_n;
    g.grid = std::max(1, std::min(total, num_cu * tile_wg_per_cu(cfg)));
    g.group_m = bm == 256 ? 4 : 8;
    g.fixed = 1;
    g.ksplit = 1;
    g.kslice = K;
    g.gate = kGateNone;
    for (int t = 0; t < g.tiles_m; ++t) g.rt_order[t] = (uint16_t)t;

    const hipError_t e = launch_gemm(g, cfg, P != nullptr, s);
    if (e != hipSuccess) return hip_error(e, "GEMM launch");
    return COMPASS_OK;
}

}  // namespace compass
