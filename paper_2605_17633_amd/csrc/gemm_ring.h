// The contraction of gemm_kernel.h for problems that give a compute unit one to three workgroups (one image, a few
// hundred to a few thousand rows): same MFMA, same order of summation, another main loop.
//
// What bounds such a problem is the latency of a slab (memory -> LDS -> registers -> MFMA), not the matrix pipes: with
// one workgroup per CU and one slab of prefetch the loop of gemm_kernel.h takes 0.8 us per 128x128x64 slab, of which the
// MFMAs are 0.2.  Here
//   * tiles are small (128x128, 128x64, 64x64; four waves, 2 x 2), so that every CU has work and up to three workgroups
//     share it: one's barrier, LDS reads and epilogue are covered by the others;
//   * A and W go from memory straight into a ring of 2 or 3 slabs in LDS (16-byte loads with an LDS destination), which
//     costs no registers and no LDS write instructions; the ring stays below 64 KB, the reach of M0 as LDS address.
//     Rows are swizzled on the memory side: a lane requests the 16-byte chunk that belongs at its place in LDS, so that
//     the fragment reads are conflict-free; packed weights arrive as fragments already;
//   * K is never cut: no partial tiles in memory and no second launch to add them (4 us and more in a chain of kernels).
//   * what the epilogue reads is requested before the loop ends (gemm_bf16_nt_body's epilogue begins with it: there other
//     workgroups' main loops cover it).
// Past one round of workgroups the traffic from the L2 bounds it and the larger tiles of gemm_kernel.h are faster again: a slab of a
// 64x64 tile is 16 KB, and takes 0.31 us with one workgroup to a CU and 0.565 with three, 22 TB/s over the chip.
// Measured (us, weights that no cache holds, packed | row-major; before = the loop of gemm_kernel.h with its K-split launch):
//   784 x 2304 x 768 21.6 -> 8.9 | 23 -> 9.3; 1638 x 768 x 3072 26.2 -> 20.9 | 28.5 -> 22.3; 4096 x 768 x 768 15 -> 11.8 | 18.1 -> 12.5;
//   1638 x 3072 x 768 + GELU 20.4 -> 17.4 | 24.2 -> 18; 8192 x 576 x 2304 - | 48 -> 40.  Slabs of 32, four stages, wave priority, 256-row
//   tiles and a non-temporal hint on the mapped store gave nothing more.
// Blocks: ViT-B 28 x 28 windowed 88 -> 62 us; encoder ViT-B batch 1 1.57 -> 1.39 ms, row-major 800 x 800 batch 2 2.08 -> 1.80 ms.
#pragma once

#include "gemm_kernel.h"

template <int BM, int BN, int STAGES>
constexpr size_t gemm_ring_lds_bytes()
{
    size_t pipe = (size_t)STAGES * (BM + BN) * GEMM_BK * sizeof(bf16);
    size_t epi = (size_t)4 * 32 * (BN / 2 + 4) * sizeof(float);
    return pipe > epi ? pipe : epi;
}

// 16 bytes per lane from memory straight into LDS: lane l's land at byte lds + 16*l of the workgroup's LDS (lds
// wave-uniform, below 64 KB).  The compiler does not see the request: the caller waits for it (vmcnt).
__device__ __forceinline__ void gemm_load_lds16(uint32_t lds, const bf16 *src)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds), "v"(src) : "m0", "memory");
}

template <int BM, int BN, int STAGES, int EPI, bool WPACK, bool LNF = false>
__device__ __forceinline__ void
gemm_ring_body(const bf16 *__restrict__ A, const bf16 *__restrict__ W, const float *__restrict__ bias,
               bf16 *C, int M, int N, int K, const GemmLd &ld, const GemmTileRange &tr, const GemmRowMap &rm,
               int bid, const GemmFold &fold)
{
    constexpr int BK = GEMM_BK, WGM = 2, WGN = 2, WM = BM / WGM, WN = BN / WGN, MT16 = WM / 16, NT16 = WN / 16, KS = BK / 32;
    constexpr int CPR = BK / 8, RPI = 64 / CPR;                 // 16-byte chunks per row of a slab; rows per request
    constexpr int NA = BM * BK / 512 / 4, NW = BN * BK / 512 / 4, L = NA + NW;     // 1 KB requests per wave and slab
    static_assert(NA >= 1 && NW >= 1 && (size_t)STAGES * (BM + BN) * BK * 2 <= 64 * 1024, "ring within the reach of M0");
    static_assert((STAGES == 2 || STAGES == 3) && L < 64, "one wait per depth; vmcnt is 6 bits");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    bf16 *ring = reinterpret_cast<bf16 *>(smem);
    constexpr int STAGE = (BM + BN) * BK;                      // elements of a stage: A rows, then W

    const int per_xcd = (tr.tile_count + 7) / 8;
    const int tl = (bid & 7) * per_xcd + (bid >> 3);
    if (tl >= tr.tile_count) return;
    int m0, n0;
    gemm_tile_origin(tr, tl, 0, 1, 1, BM, BN, m0, n0);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave / WGN) * WM, wn = (wave % WGN) * WN;
    const int l16 = lane & 15, quad = lane >> 4;
    const int n = (K + BK - 1) / BK;

    const int rl = lane / CPR, cp = lane % CPR;
    auto swz = [](int row) { return (row >> 1) & 7; };
    const bf16 *ga[NA], *gw[NW];
    int ka[NA], kw[NW];                          // k of the lane's chunk inside a slab
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int row = (wave * NA + i) * RPI + rl, c = cp ^ swz(row);
        long arow = min(m0 + row, M - 1);
        if constexpr (LNF) if (fold.src) arow = fold.src[arow];
        ka[i] = c * 8;
        ga[i] = A + arow * ld.a + c * 8;
    }
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        if constexpr (WPACK) {
            // request f of a slab is fragment (column block f / KS, k-step f % KS): 1 KB in memory as in LDS
            const int f = wave * NW + i, nb = min((n0 >> 4) + f / KS, (N >> 4) - 1);
            kw[i] = (f % KS) * 32;
            gw[i] = W + ((long)nb * (K / 32) + f % KS) * 512 + lane * 8;
        } else {
            const int row = (wave * NW + i) * RPI + rl, c = cp ^ swz(row);
            kw[i] = c * 8;
            gw[i] = W + (long)min(n0 + row, N - 1) * ld.w + c * 8;
        }
    }
    const bf16 *zchunk = reinterpret_cast<const bf16 *>(gemm_zero_chunk);
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(__attribute__((address_space(3))) bf16 *)ring);
    const uint32_t lds_a = lds0 + wave * NA * 1024, lds_w = lds0 + BM * BK * 2 + wave * NW * 1024;

    auto request = [&](int kt, int st) {         // slab kt into stage st
        const long ko = (long)kt * BK, kow = WPACK ? (long)kt * KS * 512 : ko;
        const uint32_t so = (uint32_t)st * (STAGE * 2);
        if (ko + BK <= K) {
#pragma unroll
            for (int i = 0; i < NA; ++i) gemm_load_lds16(lds_a + so + i * 1024, ga[i] + ko);
#pragma unroll
            for (int i = 0; i < NW; ++i) gemm_load_lds16(lds_w + so + i * 1024, gw[i] + kow);
        } else {                                 // a ragged last slab reads zeros past K (K % 8 == 0)
#pragma unroll
            for (int i = 0; i < NA; ++i) gemm_load_lds16(lds_a + so + i * 1024, ko + ka[i] < K ? ga[i] + ko : zchunk);
#pragma unroll
            for (int i = 0; i < NW; ++i) gemm_load_lds16(lds_w + so + i * 1024, ko + kw[i] < K ? gw[i] + kow : zchunk);
        }
    };

    f32x4 acc[MT16][NT16];
#pragma unroll
    for (int i = 0; i < MT16; ++i)
#pragma unroll
        for (int j = 0; j < NT16; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;

#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s)
        if (s < n) request(s, s);

    const int fa0 = (wm + l16) * BK, fw0 = WPACK ? (wn / 16) * KS * 512 + lane * 8 : (wn + l16) * BK;
    const int sw = swz(l16);

    // a lane finishes 8 columns of RR rows in the epilogue (slice i, pass p: row wm + 32*i + RPP*p + er)
    constexpr int LPR = WN / 8, RPP = 64 / LPR, PASSES = 32 / RPP, MT = WM / 32, RR = MT * PASSES;
    constexpr int EPS = WN + 4;
    const int er = lane / LPR, ec = lane % LPR, ncol = n0 + wn + ec * 8;
    const bool col_ok = ncol < N;                // N % 8 == 0: a lane's 8 columns are all inside or all outside
    float bv[8], sv[LNF ? 8 : 1];
    auto load8 = [&](const float *src, float *d) {
        const float4 *p4 = reinterpret_cast<const float4 *>(src + (col_ok ? ncol : 0));
        const float4 x0 = p4[0], x1 = p4[1];
        d[0] = x0.x; d[1] = x0.y; d[2] = x0.z; d[3] = x0.w;
        d[4] = x1.x; d[5] = x1.y; d[6] = x1.z; d[7] = x1.w;
    };
    constexpr bool MAPPED = EPI == SSAM_EPI_BIAS_SCATTER_ADD || EPI == SSAM_EPI_BIAS_SCATTER;
    int drow[RR];                                // destination row, -1: not stored
    float2 rst[LNF ? RR : 1];
    auto slab = [&](int it, int st) {
        // this wave's requests for slab `it` have landed when no more than those of the slabs behind it are out
        if (STAGES == 2 || it == n - 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" :: "n"(L) : "memory");
        LDS_BARRIER();                           // every wave's have; and every wave is done reading the stage before
        if (it + STAGES - 1 < n) request(it + STAGES - 1, st == 0 ? STAGES - 1 : st - 1);
        const bf16 *as = ring + st * STAGE, *ws = as + BM * BK;
        bf16x8 af[KS][MT16], bw[KS][NT16];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
#pragma unroll
            for (int i = 0; i < MT16; ++i)
                af[s][i] = *reinterpret_cast<const bf16x8 *>(as + fa0 + i * 16 * BK + (((s * 4 + quad) ^ sw) << 3));
#pragma unroll
            for (int j = 0; j < NT16; ++j)
                bw[s][j] = *reinterpret_cast<const bf16x8 *>(WPACK ? ws + fw0 + (j * KS + s) * 512
                                                                   : ws + fw0 + j * 16 * BK + (((s * 4 + quad) ^ sw) << 3));
        }
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int i = 0; i < MT16; ++i)
#pragma unroll
                for (int j = 0; j < NT16; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[s][i], bw[s][j], acc[i][j], 0, 0, 0);
    };
    int st = 0, it = 0;
    for (; it < n - 2; ++it) {
        slab(it, st);
        st = st + 1 == STAGES ? 0 : st + 1;
    }
    // what the epilogue reads is requested two slabs before the end, so that the workgroup's tail is no chain of memory
    // round trips (map, then old values, then the stores); the waits in slab() then also cover these requests
    load8(bias, bv);
    if constexpr (LNF) load8(fold.colsum, sv);
#pragma unroll
    for (int q = 0; q < RR; ++q) {
        const int m = m0 + wm + (q / PASSES) * 32 + (q % PASSES) * RPP + er, mc = min(m, M - 1);
        if constexpr (MAPPED) {
            const int b = mc / rm.rows_per_batch, idx = rm.map[(long)b * rm.map_batch_stride + (mc - b * rm.rows_per_batch)];
            drow[q] = idx >= 0 && idx < rm.dst_rows_per_batch ? b * rm.dst_rows_per_batch + idx : -1;
        } else {
            drow[q] = m;
        }
        if (m >= M || !col_ok) drow[q] = -1;
        if constexpr (LNF) rst[q] = fold.stats[mc];
    }

    uint4 old[EPI == SSAM_EPI_BIAS_SCATTER_ADD ? RR : 1];
    if constexpr (EPI == SSAM_EPI_BIAS_SCATTER_ADD) {
#pragma unroll
        for (int q = 0; q < RR; ++q)             // a row that is not stored reads row 0 and drops the value
            old[q] = *reinterpret_cast<const uint4 *>(C + (long)max(drow[q], 0) * ld.c + (col_ok ? ncol : 0));
    }
#pragma unroll 1
    for (; it < n; ++it) {
        slab(it, st);
        st = st + 1 == STAGES ? 0 : st + 1;
    }
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");       // see gemm_bf16_nt_body
    __builtin_amdgcn_sched_barrier(0);
    LDS_BARRIER();                               // every wave is done with the ring: its LDS becomes the staging tiles
    float *stage = reinterpret_cast<float *>(smem) + wave * 32 * EPS;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
#pragma unroll
        for (int t = 0; t < 2; ++t)              // the slice's two 16-row tiles: lane (l16, quad) holds rows 4*quad + r
#pragma unroll
            for (int j = 0; j < NT16; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    stage[(t * 16 + 4 * quad + r) * EPS + j * 16 + l16] = acc[2 * i + t][j][r];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int q = i * PASSES + p;
            const float4 *s4 = reinterpret_cast<const float4 *>(stage + (p * RPP + er) * EPS + ec * 8);
            const float4 y0 = s4[0], y1 = s4[1];
            float v[8] = { y0.x, y0.y, y0.z, y0.w, y1.x, y1.y, y1.z, y1.w };
            if constexpr (LNF) {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = v[e] * rst[q].x + (rst[q].y * sv[e] + bv[e]);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] += bv[e];
            }
            if constexpr (EPI == SSAM_EPI_BIAS_GELU) {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = gelu_erf(v[e]);
            }
            if constexpr (EPI == SSAM_EPI_BIAS_SCATTER_ADD) {
                float o[8];
                unpack_bf16x8(old[q], o);
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] += o[e];
            }
            if (drow[q] >= 0) *reinterpret_cast<uint4 *>(C + (long)drow[q] * ld.c + ncol) = pack_bf16x8(v);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");      // the slice is read before the next one is staged
    }
}

template <int BM, int BN, int STAGES, int EPI, bool WPACK, bool LNF = false>
__global__ void __launch_bounds__(256, (gemm_ring_lds_bytes<BM, BN, STAGES>() <= 53 * 1024 ? 3 : 2))
gemm_ring_kernel(const bf16 *__restrict__ A, const bf16 *__restrict__ W, const float *__restrict__ bias,
                 bf16 *C, int M, int N, int K, GemmLd ld, GemmTileRange tr, GemmRowMap rm, GemmFold fold)
{
    gemm_ring_body<BM, BN, STAGES, EPI, WPACK, LNF>(A, W, bias, C, M, N, K, ld, tr, rm, (int)blockIdx.x, fold);
}
