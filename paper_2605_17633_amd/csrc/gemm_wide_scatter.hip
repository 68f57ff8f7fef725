// The wide contraction (gemm_wide.h), bias, scattered.
#include "gemm_wide_launch.h"

int ssam_gemm_wide_scatter(int tile, bool packed, const GemmWideArgs &a)
{
    return packed ? gemm_wide_launch<SSAM_EPI_BIAS_SCATTER, true, false>(tile, a) : gemm_wide_launch<SSAM_EPI_BIAS_SCATTER, false, false>(tile, a);
}
