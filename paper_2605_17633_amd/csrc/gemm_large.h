// Launches of the large tiles (gemm_kernel.h): whole rounds, and what is left over as smaller tiles or K ranges.  Included by the sources that instantiate them.
#pragma once

#include "gemm_kernel.h"

namespace {

struct SplitWs { void *ptr; size_t bytes; };

// How a launch of `total` large tiles over `slots` concurrent workgroups is cut: `rem` left-over large
// tiles go to a second launch of `subs` smaller tiles each (0: none, when the tiles do not fill one
// round, fill the last one exactly, fill more than half of it, or give every CU a workgroup), and that launch also cuts K into
// `parts` ranges (1: no) when a workspace is there, K is long and the left-over is small.  A problem of less
// than one round is treated as all left-over when cutting K gives it at least twice the workgroups.
struct TailPlan { int rem, parts; };

TailPlan plan_tail(int total, int slots, int nk, int subs, size_t sub_tile_bytes, const SplitWs &ws)
{
    TailPlan p = { total % slots, 1 };
    if (total < slots) {
        // not even one round of large tiles (small batches): a handful of workgroups would each walk all of K
        // alone.  With a workspace the whole problem runs as the left-over form instead: smaller tiles, K cut
        // into ranges, so that about 512 workgroups share it.
        const int n_all = total * subs;
        int parts = nk / 4;
        if (n_all > 0 && parts > 512 / n_all) parts = 512 / n_all;
        if (ws.ptr && parts >= 2 && (size_t)n_all * parts * sub_tile_bytes <= ws.bytes) {
            p.rem = total;
            p.parts = parts;
            return p;
        }
        p.rem = 0;
    }
    // A last round that is more than half full stays in the main launch.  So does one that gives every CU a
    // workgroup (tiles that run two per CU: a lone workgroup has the CU to itself and finishes in about 0.6 of
    // a full round's time, sooner than the same work as a second launch of smaller tiles).
    if (p.rem > slots / 2 || p.rem >= 256) p.rem = 0;
    if (p.rem == 0) return p;
    const int n_sub = p.rem * subs;
    int parts = nk / 4;                         // at least 4 slabs per workgroup
    if (parts > 256 / n_sub) parts = 256 / n_sub;
    if (ws.ptr && parts >= 4 && (size_t)n_sub * parts * sub_tile_bytes <= ws.bytes) p.parts = parts;
    return p;
}

template <int BM, int BN, int EPI, int SUB_M, int SUB_N, int WGM = 2, int WGN = 2, bool WPACK = false, bool LNF = false, bool PARTS = false>
int launch_range(const bf16 *A, const bf16 *W, const float *bias, bf16 *C, int M, int N, int K,
                 const GemmLd &ld, const GemmTileRange &tr, const GemmRowMap &rm, const GemmSplit &sp, const GemmFold &fold,
                 hipStream_t st)
{
    if (tr.tile_count <= 0) return SSAM_OK;
    constexpr size_t lds = gemm_lds_bytes<BM, BN, WGM, WGN, WPACK>();
    auto kern = gemm_bf16_nt_kernel<BM, BN, EPI, SUB_M, SUB_N, WGM, WGN, WPACK, LNF, PARTS>;
    // more than 64 KiB of LDS per workgroup needs the per-kernel opt-in (idempotent, host-side only)
    if (lds > 64 * 1024 &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return SSAM_EHIP;
    int per_xcd = ssam_div_up((long)tr.tile_count * SUB_M * SUB_N * sp.parts, 8);
    hipLaunchKernelGGL(kern, dim3(per_xcd * 8), dim3(64 * WGM * WGN), lds, st, A, W, bias, C, M, N, K, ld, tr, rm, sp, fold);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

// Whole rounds of BM x BN tiles, then the left-over tiles (when they would fill less than half a round)
// as TM x TN tiles, BM = SUB_M*TM, BN = SUB_N*TN.  slots = workgroups the chip runs at once with the large
// tile.  With a workspace, a long K and few left-over tiles, the left-over launch also cuts K (see the kernel).
template <int BM, int BN, int TM, int TN, int EPI, int WGM = 2, int WGN = 2, bool WPACK = false, bool LNF = false, bool PARTS = false>
int launch_split(const bf16 *A, const bf16 *W, const float *bias, bf16 *C, int M, int N, int K,
                 const GemmLd &ld, int slots, const GemmRowMap &rm, const SplitWs &ws, const GemmFold &fold, hipStream_t st)
{
    constexpr int SUB_M = BM / TM, SUB_N = BN / TN;
    const GemmSplit whole = { nullptr, 1 };
    GemmTileRange tr = { ssam_div_up(M, BM), ssam_div_up(N, BN), 0, 0 };
    const int total = tr.tiles_m * tr.tiles_n;
    const int nk = ssam_div_up(K, GEMM_BK);
    const TailPlan plan = plan_tail(total, slots, nk, SUB_M * SUB_N, (size_t)TM * TN * sizeof(float), ws);
    const int rem = plan.rem, parts = plan.parts;
    tr.tile_count = total - rem;
    if constexpr (WGM * WGN == 4 && WPACK) if (rem != 0 && tr.tile_count != 0) {
        // four-wave large tiles: whole rounds and left-over share one launch (see the fused kernel); a K-split
        // left-over is then finished by the reduce kernel as usual
        GemmTileRange tt = tr;
        tt.tile_begin = total - rem;
        tt.tile_count = rem;
        const int n_sub = rem * SUB_M * SUB_N;
        const int n_tail = ssam_div_up(n_sub * parts, 8) * 8, n_main = ssam_div_up(tr.tile_count, 8) * 8;
        constexpr size_t lds_main = gemm_lds_bytes<BM, BN, WGM, WGN, WPACK>(), lds_tail = gemm_lds_bytes<TM, TN, 2, 2, WPACK>();
        constexpr size_t lds = lds_main > lds_tail ? lds_main : lds_tail;
        static_assert(lds <= 64 * 1024, "the fused launch stays within the default LDS limit");
        if (parts > 1) {
            const GemmSplit sp = { (float *)ws.ptr, parts };
            hipLaunchKernelGGL((gemm_bf16_nt_fused_kernel<BM, BN, EPI, WGM, WGN, TM, TN, GEMM_EPI_PARTIAL, SUB_M, SUB_N, WPACK, LNF, PARTS>),
                               dim3(n_tail + n_main), dim3(256), lds, st, A, W, bias, C, M, N, K, ld, tr, tt, rm, sp, n_tail, fold);
            SSAM_CHECK_LAUNCH();
            constexpr int RPB = 256 / (TN / 8);
            hipLaunchKernelGGL((gemm_tail_reduce_kernel<TM, TN, EPI, SUB_M, SUB_N, LNF, PARTS>), dim3(n_sub * (TM / RPB)), dim3(256), 0, st,
                               (const float *)ws.ptr, parts, bias, C, M, N, K, ld, tt, rm, fold);
        } else {
            hipLaunchKernelGGL((gemm_bf16_nt_fused_kernel<BM, BN, EPI, WGM, WGN, TM, TN, EPI, SUB_M, SUB_N, WPACK, LNF, PARTS>),
                               dim3(n_tail + n_main), dim3(256), lds, st, A, W, bias, C, M, N, K, ld, tr, tt, rm, whole, n_tail, fold);
        }
        SSAM_CHECK_LAUNCH();
        return SSAM_OK;
    }
    int rc = launch_range<BM, BN, EPI, 1, 1, WGM, WGN, WPACK, LNF, PARTS>(A, W, bias, C, M, N, K, ld, tr, rm, whole, fold, st);
    if (rc != SSAM_OK || rem == 0) return rc;
    tr.tile_begin = total - rem;
    tr.tile_count = rem;
    const int n_sub = rem * SUB_M * SUB_N;
    if (parts > 1) {
        const GemmSplit sp = { (float *)ws.ptr, parts };
        rc = launch_range<TM, TN, GEMM_EPI_PARTIAL, SUB_M, SUB_N, 2, 2, WPACK, LNF, PARTS>(A, W, bias, C, M, N, K, ld, tr, rm, sp, fold, st);
        if (rc != SSAM_OK) return rc;
        constexpr int RPB = 256 / (TN / 8);
        hipLaunchKernelGGL((gemm_tail_reduce_kernel<TM, TN, EPI, SUB_M, SUB_N, LNF, PARTS>), dim3(n_sub * (TM / RPB)), dim3(256), 0, st,
                           (const float *)ws.ptr, parts, bias, C, M, N, K, ld, tr, rm, fold);
        SSAM_CHECK_LAUNCH();
        return SSAM_OK;
    }
    return launch_range<TM, TN, EPI, SUB_M, SUB_N, 2, 2, WPACK, LNF, PARTS>(A, W, bias, C, M, N, K, ld, tr, rm, whole, fold, st);
}

}  // namespace
