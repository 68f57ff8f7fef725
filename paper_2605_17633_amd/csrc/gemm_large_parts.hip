// The large tiles with a LayerNorm folded in whose row statistics come in pieces (GemmParts; rows of 1280): GELU with a gather (fc1), mapped store (qkv).  A source of their
// own: in the dispatcher's code object these seven kernels moved the small ones, and a block of ViT-B, 28 x 28, whose kernels were the same instruction for instruction, took 46.6 -> 46.9 to
// 47.1 us (of it fc1's ring 0.1); apart 46.75, 46.8 before there were any.
#include "gemm_large.h"
#include "gemm_wide_launch.h"

int ssam_gemm_large_parts_gelu(const GemmWideArgs &a, void *split_ws, size_t split_ws_bytes)
{
    return launch_split<128, 256, 128, 128, SSAM_EPI_BIAS_GELU, 1, 4, true, true, true>(a.A, a.W, a.bias, a.C, a.M, a.N, a.K, a.ld, 512, a.rm, SplitWs{ split_ws, split_ws_bytes }, a.fold, a.st);
}

// M a multiple of 128 and N of 256; padding rows of a.fold.fill behind the tiles.
int ssam_gemm_large_parts_scatter(const GemmWideArgs &a)
{
    constexpr size_t lds = gemm_lds_bytes<128, 256, 1, 4, true>();
    static_assert(lds <= 64 * 1024, "default LDS limit");
    const GemmTileRange tr = { a.M / 128, a.N / 256, 0, (a.M / 128) * (a.N / 256) };
    hipLaunchKernelGGL((gemm_bf16_nt_lnf_kernel<128, 256, SSAM_EPI_BIAS_SCATTER, 1, 4, true>), dim3(ssam_div_up(tr.tile_count, 8) * 8 + ssam_div_up(a.fold.fill.total_rows, GEMM_LNF_FILL)),
                       dim3(256), lds, a.st, a.A, a.W, a.bias, a.C, a.M, a.N, a.K, a.ld, tr, a.rm, a.fold);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}
