// The contraction of gemm_kernel.h, packed weights, for problems of at most one 32x32 tile per CU (a 28 x 28 grid, batch 1: 313
// kept rows x 768 columns): too few tiles for the rings of gemm_ring.h to give every CU a workgroup.
//
// What bounds such a problem is what one CU can pull from the L2, 50 to 60 bytes a ns (8 KB in 0.14 us here): all CUs have to pull.  A workgroup's tile
// is 32x32; its four waves cut K between them (wave w takes the k-steps w, w + 4, ...) and load their MFMA fragments straight
// into registers, DIRECT_DEPTH steps ahead, with no LDS and no barrier until the four partial tiles are added there, in wave
// order.  Packed weights only: with rows in both operands the half cache lines of the fragments cost what the width gains.
// Measured (us, weights that no cache holds, before = 64x64 ring): 313 x 768 x 3072 18.6 -> 10.6, 196 x 1024 x 4096 23.8 -> 12.8, 313 x 768 x 768
// 6.1 -> 4.9, 64 x 1280 x 1280 8.3 -> 7.0; with two tiles per CU the two are level (253 x 1152 x 1152 9.2 against 9.5).  Pairs of adjacent
// k-steps per wave: no faster.  Loads chosen between the operand and a chunk of zeros became FLAT loads that the compiler
// moved next to their use and waited for one by one: 313 x 768 x 3072 14.8 with the bias epilogue, 12.0 mapped.
#pragma once

#include "gemm_kernel.h"

constexpr int DIRECT_DEPTH = 6;

template <int EPI, bool LNF = false>
__global__ void __launch_bounds__(256, 2)
gemm_direct_kernel(const bf16 *__restrict__ A, const bf16 *__restrict__ W, const float *__restrict__ bias,
                   bf16 *C, int M, int N, int K, GemmLd ld, GemmTileRange tr, GemmRowMap rm, GemmFold fold)
{
    constexpr int DEPTH = DIRECT_DEPTH, T = 32, PS = T + 4;      // PS: floats per row of a partial tile
    __shared__ __attribute__((aligned(16))) float part[4][T * PS];
    const int bid = blockIdx.x, per_xcd = (tr.tile_count + 7) / 8, tl = (bid & 7) * per_xcd + (bid >> 3);
    if (tl >= tr.tile_count) return;
    int m0, n0;
    gemm_tile_origin(tr, tl, 0, 1, 1, T, T, m0, n0);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, quad = lane >> 4;

    const int nsteps = K / 32, n = (nsteps - wave + 3) / 4;         // this wave's k-steps: wave + 4*i, i < n
    const bf16 *pa[2], *pw[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        long arow = min(m0 + i * 16 + l16, M - 1);                          // rows past M repeat the last one, never stored
        if constexpr (LNF) if (fold.src) arow = fold.src[arow];
        pa[i] = A + arow * ld.a + quad * 8;
        pw[i] = W + (long)((n0 >> 4) + i) * nsteps * 512 + lane * 8;         // N is a multiple of 32
    }
    bf16x8 fa[DEPTH][2], fw[DEPTH][2];
    // k-step wave + 4*i into register set s; past the end of K the last step again, which is not multiplied: the loads carry
    // no predicate and stay where they are written (sched_barrier), so that each wait leaves the steps behind it in flight
    auto load = [&](int i, int s) {
        const int k = min(wave + 4 * i, nsteps - 1) * 32;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            fa[s][j] = *reinterpret_cast<const bf16x8 *>(pa[j] + k);
            fw[s][j] = *reinterpret_cast<const bf16x8 *>(pw[j] + (long)k * 16);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mul = [&](f32x4 (&acc)[2][2], int s) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[s][x], fw[s][y], acc[x][y], 0, 0, 0);
    };
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{ 0.f, 0.f, 0.f, 0.f };
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) load(s, s);
    int i = 0;
    for (; i + DEPTH < n; i += DEPTH) {          // turns of the register ring with steps behind them
#pragma unroll
        for (int s = 0; s < DEPTH; ++s) {
            mul(acc, s);
            load(i + s + DEPTH, s);
        }
    }
#pragma unroll
    for (int s = 0; s < DEPTH; ++s)              // the last turn, all of it requested
        if (i + s < n) mul(acc, s);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");       // see gemm_bf16_nt_body
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) part[wave][(x * 16 + 4 * quad + r) * PS + y * 16 + l16] = acc[x][y][r];
    __syncthreads();
    if (tid >= T * T / 8) return;                             // two waves finish 8 columns of a row each
    const int row = tid >> 2, cl = (tid & 3) * 8, m = m0 + row, ncol = n0 + cl;
    if (m >= M || ncol >= N) return;                          // N % 8 == 0
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; e += 4) {
        f32x4 s = *reinterpret_cast<const f32x4 *>(&part[0][row * PS + cl + e]);
#pragma unroll
        for (int w = 1; w < 4; ++w) s += *reinterpret_cast<const f32x4 *>(&part[w][row * PS + cl + e]);
        const f32x4 b = *reinterpret_cast<const f32x4 *>(bias + ncol + e);
        if constexpr (LNF) {
            const float2 t = fold.stats[m];
            const f32x4 c = *reinterpret_cast<const f32x4 *>(fold.colsum + ncol + e);
#pragma unroll
            for (int q = 0; q < 4; ++q) v[e + q] = s[q] * t.x + (t.y * c[q] + b[q]);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) v[e + q] = s[q] + b[q];
        }
    }
    if constexpr (EPI == SSAM_EPI_BIAS_GELU) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = gelu_erf(v[e]);
    }
    long dst = m;
    if constexpr (EPI == SSAM_EPI_BIAS_SCATTER_ADD || EPI == SSAM_EPI_BIAS_SCATTER) {
        const int b = m / rm.rows_per_batch, idx = rm.map[(long)b * rm.map_batch_stride + (m - b * rm.rows_per_batch)];
        if (idx < 0 || idx >= rm.dst_rows_per_batch) return;
        dst = (long)b * rm.dst_rows_per_batch + idx;
    }
    uint4 *out = reinterpret_cast<uint4 *>(C + dst * ld.c + ncol);
    if constexpr (EPI == SSAM_EPI_BIAS_SCATTER_ADD) {
        float o[8];
        unpack_bf16x8(*out, o);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += o[e];
    }
    *out = pack_bf16x8(v);
}
