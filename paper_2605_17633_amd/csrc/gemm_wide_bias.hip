// The wide contraction (gemm_wide.h), bias epilogue.
#include "gemm_wide_launch.h"

int ssam_gemm_wide_bias(int tile, bool packed, const GemmWideArgs &a)
{
    return packed ? gemm_wide_launch<SSAM_EPI_BIAS, true, false>(tile, a) : gemm_wide_launch<SSAM_EPI_BIAS, false, false>(tile, a);
}
