// The wide contraction (gemm_wide.h) with a LayerNorm folded in whose row statistics come in pieces (GemmParts): mapped store (qkv), GELU with a gather (fc1); and the
// scatter-add that leaves such pieces (proj, fc2).
#include "gemm_wide_launch.h"

int ssam_gemm_wide_parts_scatter(int tile, const GemmWideArgs &a) { return gemm_wide_launch<SSAM_EPI_BIAS_SCATTER, true, true, true>(tile, a); }

int ssam_gemm_wide_parts_gelu(int tile, const GemmWideArgs &a) { return gemm_wide_launch<SSAM_EPI_BIAS_GELU, true, true, true>(tile, a); }

int ssam_gemm_wide_parts_add(int tile, const GemmWideArgs &a) { return gemm_wide_launch<SSAM_EPI_BIAS_SCATTER_ADD, true, false, true>(tile, a); }
