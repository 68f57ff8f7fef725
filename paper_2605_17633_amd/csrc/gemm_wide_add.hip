// The wide contraction (gemm_wide.h), bias, scattered and added to what is there.
#include "gemm_wide_launch.h"

int ssam_gemm_wide_add(int tile, bool packed, const GemmWideArgs &a)
{
    return packed ? gemm_wide_launch<SSAM_EPI_BIAS_SCATTER_ADD, true, false>(tile, a) : gemm_wide_launch<SSAM_EPI_BIAS_SCATTER_ADD, false, false>(tile, a);
}
