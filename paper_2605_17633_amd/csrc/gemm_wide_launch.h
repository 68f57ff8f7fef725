// Launches of gemm_wide_kernel.  The kernels of one epilogue are one source file (gemm_wide_*.hip), compiled side by side.
#pragma once

#include "gemm_wide.h"

struct GemmWideArgs {
    const bf16 *A, *W;
    const float *bias;
    bf16 *C;
    int M, N, K;
    GemmLd ld;
    GemmRowMap rm;
    GemmFold fold;
    hipStream_t st;
    WarmAhead *warm = nullptr;
    double us = 0.0;          // what the launch takes
};

// Tiles, in the order of their index in the dispatcher's time model (gemm.hip).
#define GEMM_WIDE_TILES(X)                                                                                     \
    X(0, 64, 64, 2) X(1, 96, 64, 2) X(2, 96, 96, 2) X(3, 64, 128, 2) X(4, 128, 128, 1) X(5, 128, 192, 1)         \
    X(6, 192, 128, 1) X(7, 256, 128, 1) X(8, 192, 192, 1) X(9, 192, 256, 1) X(10, 256, 192, 1) X(11, 256, 256, 1)
constexpr int GEMM_WIDE_COUNT = 12;

// Tiles that can write GemmParts, and tiles that can read them, a bit each.
#define X(id, bm, bn, wgk) | (unsigned)GemmWide<bm, bn, wgk>::WRITES_PARTS << id
constexpr unsigned GEMM_WIDE_WRITES_PARTS = 0 GEMM_WIDE_TILES(X);
#undef X
#define X(id, bm, bn, wgk) | (unsigned)GemmWide<bm, bn, wgk>::READS_PARTS << id
constexpr unsigned GEMM_WIDE_READS_PARTS = 0 GEMM_WIDE_TILES(X);
#undef X

template <int BM, int BN, int WGK, int EPI, bool WPACK, bool LNF, bool PARTS>
int gemm_wide_launch_tile(const GemmWideArgs &a)
{
    constexpr size_t lds = GemmWide<BM, BN, WGK>::lds_bytes;
    auto kern = gemm_wide_kernel<BM, BN, WGK, EPI, WPACK, LNF, PARTS>;
    // more than 64 KiB of LDS per workgroup needs the per-kernel opt-in (idempotent, host-side only)
    if (lds > 64 * 1024 &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return SSAM_EHIP;
    GemmTileRange tr = { ssam_div_up(a.M, BM), ssam_div_up(a.N, BN), 0, 0 };
    tr.tile_count = tr.tiles_m * tr.tiles_n;
    const int tiles = ssam_div_up(tr.tile_count, 8) * 8, fills = PARTS && LNF && EPI == SSAM_EPI_BIAS_SCATTER ? ssam_div_up(a.fold.fill.total_rows, GEMM_WIDE_FILL) : 0;
    const GemmWarm warm = a.warm ? a.warm->behind(tiles, fills, a.us) : GemmWarm{};
    hipLaunchKernelGGL(kern, dim3(tiles + fills + warm.groups), dim3(512), lds, a.st, a.A, a.W, a.bias, a.C, a.M, a.N, a.K, a.ld, tr, a.rm, a.fold, warm);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

template <int EPI, bool WPACK, bool LNF, bool PARTS = false>
int gemm_wide_launch(int tile, const GemmWideArgs &a)
{
    switch (tile) {
#define X(id, bm, bn, wgk) case id: if constexpr (!PARTS || (((LNF ? GEMM_WIDE_READS_PARTS : GEMM_WIDE_WRITES_PARTS) >> id) & 1)) return gemm_wide_launch_tile<bm, bn, wgk, EPI, WPACK, LNF, PARTS>(a); else return SSAM_EINVAL;
    GEMM_WIDE_TILES(X)
#undef X
    default: return SSAM_EINVAL;
    }
}
