// The wide contraction (gemm_wide.h), bias and GELU epilogue.
#include "gemm_wide_launch.h"

int ssam_gemm_wide_gelu(int tile, bool packed, const GemmWideArgs &a)
{
    return packed ? gemm_wide_launch<SSAM_EPI_BIAS_GELU, true, false>(tile, a) : gemm_wide_launch<SSAM_EPI_BIAS_GELU, false, false>(tile, a);
}
