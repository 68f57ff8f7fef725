// The contraction of gemm_kernel.h for problems of a few rounds of workgroups: one workgroup of eight waves to a CU, its tile as large
// as still gives (almost) every CU one.  Same MFMA; K in one chain, or in two below 128x128.
//
// What bounds such a problem is one workgroup's chain on its CU: the first slabs from HBM, what a CU can pull from the L2 (95 bytes a ns at best, 25 TB/s over
// the chip, measured with nothing else going on; a slab of a 64x64 tile is 16 KB for 0.05 us of matrix work and one of 256x192 56 KB for 0.64 us), and the epilogue.
// Over whole launches of ViT layers the counters show 23 to 51 bytes a ns and CU and the matrix pipes 15 to 36 % busy.  So
//   * tiles are as large as the problem allows, in many sizes (the dispatcher has their times): 4096 x 3072 x 1024 is 256 tiles of
//     256x192; rings of 64x64 tiles pull 3.4 times its bytes;
//   * the LDS of a CU, all of it, holds up to four slabs of A and W ahead of the MFMAs.  They come by 16-byte loads with an LDS destination
//     (M0 reaches all 160 KB), swizzled on the memory side so that fragment reads are conflict-free, in whole cache lines;
//   * the fragments of a k-step are read under the MFMAs of the one before, into the other set of registers, and the requests for a slab
//     go out behind the MFMAs that follow the barrier that freed its stage: one barrier a slab, in its middle where the waves are 2x4 or 4x2
//     over the tile, and nothing between two MFMAs that waits;
//   * eight waves: 4 of 128x128 read a third less LDS but a wave alone on its SIMD has nothing under its barriers (4096 x 4096 x 5120:
//     122 us against 116).  Below 128x128 the waves are 2x2 over the tile, each half of them takes half of every slab of K, and the halves
//     are added in LDS: half the fragment reads of 2x4 (1638 x 768 x 3072: 18.3 us with 4 waves, 15.3);
//   * W is operand a, so that a lane ends up with columns of one row of C, and W's rows are dealt to the MFMA tiles such that those of two
//     tiles are 8 consecutive columns: the epilogue goes from registers to memory by 16 bytes, through no LDS and past no barrier.  What
//     it reads is requested before the last slabs.
// Measured (us, weights that no cache holds, before = rings or large tiles; epilogues of a block):
//   4096 x 2304 x 768 22.9 -> 18.5 | 4096 x 3072 x 1024 31 -> 24 | 1638 x 3072 x 768 + GELU 17.8 -> 14.5 | 1638 x 768 x 3072 + scatter-add
//   21 -> 16.5 | 4096 x 1024 x 1024 + scatter-add 16.9 -> 13 | 2456 x 1280 x 5120 57 -> 38 (its K-split launch and reduce) | 8192 x 1280 x 1280
//   38 -> 28 | 8192 x 576 x 2304 row-major 36.5 -> 25.  Packed and row-major weights take the same time.
// Encoders, batch 1: ViT-B 1360 -> 1258 us, ViT-L 3051 -> 2674; with the row statistics left and read by these kernels instead of launches of their
// own (GemmParts) 1181 -> 1149 and 2517 -> 2424 on another card.  Steady state 1.29 us a slab of 256x256 (1.66 PFLOP/s).  Not faster: eight or
// six slabs ahead, requests in front of the k-step (10 % slower: they crowd out the fragment reads), wave priority, 128x192 tiles two to
// a CU, a persistent form whose next tile's slabs are requested under the epilogue (its waits then are for the stores too).
#pragma once

#include <type_traits>

#include "gemm_kernel.h"

// 16 bytes per lane from memory straight into LDS: lane l's, from sbase + its voff (bytes), land at byte lds + 16*l of the LDS
// (sbase, lds wave-uniform).  The compiler does not see the request: the caller waits for it (vmcnt).
__device__ __forceinline__ void gemm_load_lds16_s(uint32_t lds, uint32_t voff, const void *sbase)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(lds), "v"(voff), "s"(sbase) : "m0", "memory");
}

// 4 bytes per lane: lane l's, from src, land at byte lds + 4*l.
__device__ __forceinline__ void gemm_load_lds4(uint32_t lds, const int32_t *src)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" :: "s"(lds), "v"(src) : "m0", "memory");
}

template <int N> __device__ __forceinline__ void gemm_wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }

constexpr int GEMM_WIDE_SLABS = 5;           // the fewest slabs of K that are taken

// WGK = 2: the workgroup's eight waves are 2 x 2 over the tile times two halves of every slab of K; 1: 2 x 4 or 4 x 2 over the tile (128x128: 4 x 2, as
// many fragments read as 2 x 4, and waves with whole pieces of 64 columns; 48 shapes of all epilogues and layouts -3.0 to +2.3 %, on average -0.4, so that the
// time model's constants hold).
template <int BM, int BN, int WGK>
struct GemmWide {
    static constexpr int WGM = WGK == 1 && BM > BN - (BN == 128) ? 4 : 2, WGN = 8 / WGK / WGM, MT = BM / WGM / 16, NT = BN / WGN / 16;       // 16x16 MFMA tiles of a wave
    static constexpr bool EARLY = MT * NT < 32;         // registers and LDS for what the epilogue reads before the last slabs
    static constexpr int AB = BM * GEMM_BK * 2, WB = BN * GEMM_BK * 2;                          // bytes of a slab
    static constexpr int MAP = EARLY ? 1024 : 0, LDS = 160 * 1024 - MAP;                        // of the tile's row map, of the ring
    static constexpr int S = LDS / (AB + WB) < 4 ? LDS / (AB + WB) : 4;
    static constexpr int SW = S, SA = WGK == 1 && S < 4 && (S + 1) * AB + S * WB <= LDS ? S + 1 : S;      // slabs of W and of A in LDS
    static constexpr size_t ring = (size_t)SA * AB + (size_t)SW * WB, lds_bytes = ring + MAP;
    // 1 KB requests of a slab: A's, then W's; wave w takes w, w + 8, ...
    static constexpr int QA = BM / 8, QW = BN / 8, L = (QA + QW + 7) / 8, LREST = (QA + QW) % 8;
    static_assert(BM % (16 * WGM) == 0 && BN % (16 * WGN) == 0 && (WGK == 2 || (QA % 8 == 0 && QW % 8 == 0)), "whole MFMA tiles and requests");
    static_assert(GEMM_BK * 2 == GEMM_PARTS_LINE * 8 && GEMM_PARTS_MOST <= GEMM_PARTS_LINE + 4, "a row's pieces take the place of its part of a slab, the rest 32 bytes");
    static_assert(gemm_parts_pitch(GEMM_PARTS_LINE) >= GEMM_PARTS_LINE && gemm_parts_pitch(GEMM_PARTS_LINE + 1) >= GEMM_PARTS_LINE + 4, "and of no other row");
    static_assert(WGK == 1 || (size_t)BM * BN * 4 <= ring, "the halves are added in the ring's LDS");
    // Row statistics in pieces (GemmParts).  Waves that hold whole pieces of 64 columns, or halves of which the next wave has the other, can write them.
    static constexpr bool WRITES_PARTS = (NT * 16 == 32 && WGN % 2 == 0) || NT * 16 == 64;
    // Where A has stages of its own its rows' pieces can come as one more slab.  They are requested in iteration n - SA of n: that has to be one (SA <= the fewest
    // slabs), every slab of W has to be out by then (SA <= SW + 1), and the wait for the last slab has to come behind it (SA >= 3).
    static constexpr bool READS_PARTS = WGK == 1 && SA >= 3 && SA <= SW + 1 && SA <= GEMM_WIDE_SLABS;
};

constexpr int GEMM_WIDE_FILL = 16;

// Reads its share of the weights to come; nothing is kept.  Plain loads: with the non-temporal hint they do not stay in the memory-side cache (encoders 2 to 5 %
// slower than without any).  More than 32 KB in flight a CU delays the tiles beside it (16 loads a thread: ViT-L 2538 -> 2550 us, ViT-H 7728 -> 7750).
__device__ __forceinline__ void gemm_warm(const GemmWarm &warm, int group)
{
    constexpr uint32_t STEP = 512 * 16, U = 4;
    static_assert(GEMM_WARM_PIECE + U * 256 * STEP < 1ull << 32, "32-bit offsets past the end of a piece");
    const uint32_t stride = warm.groups * STEP;
    for (int s = 0; s < GEMM_WARM_AHEAD; ++s) {
        const uint32_t bytes = warm.bytes[s];
        for (uint32_t at = group * STEP + threadIdx.x * 16; at < bytes; at += U * stride) {
            u32x4 v[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) v[u] = *reinterpret_cast<const u32x4 *>(warm.at[s] + min(at + u * stride, bytes - 16));
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) asm volatile("" :: "v"(v[u]));
        }
    }
}

// Sum over the four quads of a wave's lanes.
__device__ __forceinline__ float gemm_quad_sum(float v)
{
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    const float s = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// PARTS: the row statistics of the folded LayerNorm come in pieces (GemmParts), or, of a scatter-add, it leaves such pieces.
// The pieces of a tile's rows are as large as a slab of A and come as one more, into the stage that the last slab but SA - 1 has freed: no registers, and
// under the products of the last slabs.  Loaded in front of the ring's first slabs they cost 4 us, as much as the launch they save.
// Of rows of 1280 (20 pieces) the last four come with the next slab's place: 4608 rows, density 0.2, 149.7 us a block with statistics launches, 147.8.  (No other width has more than 16
// pieces: a block that folds LN1 has 3 D in multiples of 256.)
template <int BM, int BN, int WGK, int EPI, bool WPACK, bool LNF, bool PARTS = false>
__global__ void __launch_bounds__(512, 1)
gemm_wide_kernel(const bf16 *__restrict__ A, const bf16 *__restrict__ W, const float *__restrict__ bias,
                 bf16 *C, int M, int N, int K, GemmLd ld, GemmTileRange tr, GemmRowMap rm, GemmFold fold, GemmWarm warm)
{
    using G = GemmWide<BM, BN, WGK>;
    constexpr bool READS = PARTS && LNF, LEAVES = PARTS && !LNF;
    static_assert((!READS || G::READS_PARTS) && (!LEAVES || (EPI == SSAM_EPI_BIAS_SCATTER_ADD && WPACK && G::WRITES_PARTS)), "the forms that read or leave pieces");
    constexpr int BK = GEMM_BK, WGN = G::WGN, MT = G::MT, NT = G::NT, NP = NT / 2, WM = MT * 16, WN = NT * 16;
    constexpr int SA = G::SA, SW = G::SW, L = G::L;
    constexpr bool MAPPED = EPI == SSAM_EPI_BIAS_SCATTER_ADD || EPI == SSAM_EPI_BIAS_SCATTER, ADD = EPI == SSAM_EPI_BIAS_SCATTER_ADD;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    // WGK == 1: SA slabs of A, then SW of W; 2: slab by slab, A then W
    constexpr int STRIDE_A = WGK == 1 ? G::AB : G::AB + G::WB, STRIDE_W = WGK == 1 ? G::WB : G::AB + G::WB, W0 = WGK == 1 ? SA * G::AB : G::AB;
    unsigned char *as = smem, *ws = smem + W0;

    const int per_xcd = (tr.tile_count + 7) / 8, bid = blockIdx.x;
    const int fills = READS && EPI == SSAM_EPI_BIAS_SCATTER ? (fold.fill.total_rows + GEMM_WIDE_FILL - 1) / GEMM_WIDE_FILL : 0;
    if (bid >= 8 * per_xcd + fills) {
        gemm_warm(warm, bid - 8 * per_xcd - fills);
        return;
    }
    if constexpr (READS && EPI == SSAM_EPI_BIAS_SCATTER) if (bid >= 8 * per_xcd) {
        // padding rows, GEMM_WIDE_FILL a workgroup, one after the other in a wave: on CUs that have no tile, or behind the first tiles that end.  After a
        // global block they are all that the statistics launch would be for (ViT-B, 64 x 64, batch 1: 192 tiles, 1110 -> 1093 us; ViT-L, 256 tiles: no change)
        for (int i = threadIdx.x >> 6; i < GEMM_WIDE_FILL; i += 8) fill_pad_row(fold.fill, (bid - 8 * per_xcd) * GEMM_WIDE_FILL + i);
        return;
    }
    const int tl = (bid & 7) * per_xcd + (bid >> 3);
    if (tl >= tr.tile_count) return;
    int m0, n0;
    gemm_tile_origin(tr, tl, 0, 1, 1, BM, BN, m0, n0);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave * WGK >> 3, wt = wave & (8 / WGK - 1), wm = wt / WGN * WM, wn = wt % WGN * WN;
    const int l16 = lane & 15, quad = lane >> 4;
    const int n = K / BK;

    // column of C (from the wave's first) of operand row l of its MFMA tile j: a lane then holds 8 consecutive columns of a pair of tiles
    auto perm = [](int j, int l) { return j < 2 * NP ? 32 * (j >> 1) + (l >> 2) * 8 + (j & 1) * 4 + (l & 3) : 16 * j + l; };

    using std::integral_constant;

    // ---- requests
    uint32_t off[L], dst[L], inc[L];
    const unsigned char *base[L];
    uint32_t poff[READS ? G::QA / 8 : 1];             // of the rows' pieces, which are requested as one more slab of A,
    uint32_t poff_rest = 0;                           // and of those past 128 bytes (rows of 1280), 32 bytes of 32 rows a request
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char *)smem);
    auto a_row = [&](int m) {
        if constexpr (!READS) return fold.src[m];
        const int t = fold.src[m];
        return m / fold.src_rows * fold.src_stride + ((unsigned)t < (unsigned)fold.src_stride ? t : 0);
    };
    auto is_a = [&](int i) { return WGK == 1 ? i < G::QA / 8 : i * 8 + wave < G::QA; };
#pragma unroll
    for (int i = 0; i < L; ++i) {
        const int f = i * 8 + wave;
        inc[i] = WPACK && !is_a(i) ? 2048 : BK * 2;
        if (is_a(i)) {
            const int row = f * 8 + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7), m = min(m0 + row, M - 1);
            const bool gather = LNF && fold.src;
            const int ar = gather ? a_row(m) : m - m0;
            off[i] = ((uint32_t)ar * (uint32_t)ld.a + c * 8) * 2;
            if constexpr (READS) poff[i] = (uint32_t)(gather ? ar : m) * (gemm_parts_pitch(fold.slots) * 8) + c * 16;
            base[i] = reinterpret_cast<const unsigned char *>(gather ? A : A + (long)m0 * ld.a);
            dst[i] = lds0 + f * 1024;
        } else {
            const int w = f - G::QA;
            if constexpr (WPACK) {
                const int h = w / (2 * NT), g = w % (2 * NT), combo = (g & 1) * 8 + (lane >> 3), lq = combo & 3;
                const bool pair = g < 4 * NP;            // half a pair of fragments, 64 of its 128 chunks, in whole cache lines
                const int qd = pair ? combo >> 2 : quad, s = pair ? (g >> 1) & 1 : g & 1;
                const int col = n0 + h * WN + (pair ? 32 * (g >> 2) + lq * 8 + (((lane >> 2) & 1) ^ (lq >> 1)) * 4 + (lane & 3) : 32 * NP + l16);
                const int nb = min(col >> 4, (N >> 4) - 1) - (n0 >> 4);
                off[i] = (uint32_t)((nb * (K / 32) + s) * 512 + (16 * qd + (col & 15)) * 8) * 2;
                base[i] = reinterpret_cast<const unsigned char *>(W + (long)(n0 >> 4) * (K / 32) * 512);
            } else {
                const int row = w * 8 + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7), h = row / WN, q = row % WN;
                const int col = min(n0 + h * WN + perm(q >> 4, q & 15), N - 1) - n0;
                off[i] = ((uint32_t)col * (uint32_t)ld.w + c * 8) * 2;
                base[i] = reinterpret_cast<const unsigned char *>(W + (long)n0 * ld.w);
            }
            dst[i] = lds0 + W0 + w * 1024;
        }
    }
    if constexpr (READS) if (fold.slots > GEMM_PARTS_LINE) {
        const int m = min(m0 + wave * 32 + (lane >> 1), M - 1);
        poff_rest = (uint32_t)(fold.src ? a_row(m) : m) * (gemm_parts_pitch(fold.slots) * 8) + GEMM_PARTS_LINE * 8 + (lane & 1) * 16;
    }
    const bool all = G::LREST == 0 || wave < G::LREST;              // this wave has an L-th request
    auto request = [&](int i, int sa, int sw) {
        if (G::LREST != 0 && i == L - 1 && !all) return;
        gemm_load_lds16_s(dst[i] + (WGK == 1 && i >= G::QA / 8 ? sw * STRIDE_W : sa * STRIDE_A), off[i], base[i]);
        base[i] += inc[i];
    };
    // waits until the slab before the last `rem` requested ones has landed; MAX: the most that rem can be
    auto wait_slabs = [&](int rem, auto max_) {
        constexpr int MAX = decltype(max_)::value;
        auto out = [&](auto slabs) {                // no more than the requests of `slabs` slabs still out (of W's at most MAX - (SA - SW))
            constexpr int s = decltype(slabs)::value, w = s < MAX - (SA - SW) ? s : MAX - (SA - SW);
            if constexpr (WGK == 1) gemm_wait_vm<G::QA / 8 * s + G::QW / 8 * w>();
            else if (G::LREST != 0 && !all) gemm_wait_vm<(L - 1) * s>();
            else gemm_wait_vm<L * s>();
        };
        // (behind the last slab only the rows' pieces are out)
        if (READS && rem < 1) { gemm_wait_vm<G::QA / 8>(); return; }
        if (rem >= MAX) out(integral_constant<int, MAX>{});
        else if (MAX > 2 && rem >= 2) out(integral_constant<int, 2>{});
        else if (MAX > 1 && rem >= 1) out(integral_constant<int, 1>{});
        else gemm_wait_vm<0>();
    };
    constexpr int LA = G::QA / 8, LW = G::QW / 8;   // WGK == 1: requests per wave of A and of W

    // ---- fragments: operand a = 16 columns of C (rows of W), operand b = 16 rows
    const uint32_t fa0 = (wm + l16) * 128 + ((quad ^ ((l16 >> 1) & 7)) << 4);
    const uint32_t fw0 = WPACK ? wt % WGN * NT * 2048 + ((quad * 4 + (l16 >> 2)) * 8 + (l16 >> 3) * 4 + (l16 & 3)) * 16
                               : (wn + l16) * 128 + ((quad ^ ((l16 >> 1) & 7)) << 4);
    bf16x8 fa[2][MT], fw[2][NT];
    f32x4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{ 0.f, 0.f, 0.f, 0.f };
    // read q of k-step s of a slab into set b, in the order its MFMAs want them
    auto read = [&](int q, int b, int s, int sa, int sw) {
        if (q == 0 || q > NT) {
            const int i = q == 0 ? 0 : q - NT;
            fa[b][i] = *reinterpret_cast<const bf16x8 *>(as + sa * STRIDE_A + (fa0 ^ (s * 64)) + i * 2048);
            return;
        }
        const int j = q - 1;
        const unsigned char *p = ws + sw * STRIDE_W;
        if constexpr (!WPACK) p += (fw0 ^ (s * 64)) + j * 2048;
        else if (j < 2 * NP) p += (fw0 ^ ((j & 1) * 64)) + (j >> 1) * 4096 + s * 2048;
        else p += wt % WGN * NT * 2048 + NP * 4096 + s * 1024 + lane * 16;
        fw[b][j] = *reinterpret_cast<const bf16x8 *>(p);
    };
    constexpr int NM = MT * NT, NR = MT + NT;
    auto mfma = [&](int m, int b) {
        const int i = m / NT, j = m % NT;
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[b][j], fa[b][i], acc[i][j], 0, 0, 0);
    };
    // ---- what the epilogue reads (group wk of two finishes rows i of its MTH, from wk * MTH on).  A wait for an ordinary load
    // would also wait for every request behind it, so the row map goes to LDS in front of the first slab; the rest is requested before
    // the last slabs
    constexpr bool EARLY = G::EARLY;
    constexpr int MTH = (MT + WGK - 1) / WGK, NB = NP * 2 + NT % 2;          // NB: groups of 4 columns
    const int ncol = n0 + wn + quad * 8, ncol1 = n0 + wn + 32 * NP + quad * 4;      // first column of pair 0, of the odd tile
    if constexpr (MAPPED && EARLY) {
        if (wave * 64 < BM) {
            const int m = min(m0 + wave * 64 + lane, M - 1), b = m / rm.rows_per_batch;
            gemm_load_lds4(lds0 + (uint32_t)G::ring + wave * 256, rm.map + (long)b * rm.map_batch_stride + (m - b * rm.rows_per_batch));
        }
    }
    int drow[MTH];                                // destination rows, -1: not stored
    auto load_rows = [&]() {
#pragma unroll
        for (int k = 0; k < MTH; ++k) {
            const int i = wk * MTH + k, row = wm + 16 * i + l16, m = m0 + row, mc = min(m, M - 1);
            if constexpr (MAPPED) {
                const int b = mc / rm.rows_per_batch;
                const int idx = EARLY ? reinterpret_cast<const int32_t *>(smem + G::ring)[row] : rm.map[(long)b * rm.map_batch_stride + (mc - b * rm.rows_per_batch)];
                drow[k] = idx >= 0 && idx < rm.dst_rows_per_batch ? b * rm.dst_rows_per_batch + idx : -1;
            } else {
                drow[k] = m;
            }
            if (m >= M || (MTH * WGK != MT && i >= MT)) drow[k] = -1;
        }
    };
    f32x4 bv[NB], sv[LNF ? NB : 1];
    float2 rst[LNF ? MTH : 1];
    constexpr int ROW = NP * 4 + NT % 2 * 2, AHEAD = !ADD ? 1 : ROW * MTH <= 32 ? MTH : 32 / ROW;      // rows whose old values are requested ahead
    uint4 old[ADD ? AHEAD : 1][NP > 0 ? NP : 1];
    uint2 old1[ADD ? AHEAD : 1];
    auto load_old = [&](int k) {
        const bf16 *row = C + (long)max(drow[k], 0) * ld.c;      // a row that is not stored reads row 0 and drops the value
#pragma unroll
        for (int p = 0; p < NP; ++p) old[k % AHEAD][p] = *reinterpret_cast<const uint4 *>(row + (ncol + 32 * p < N ? ncol + 32 * p : 0));
        if constexpr (NT % 2) old1[k % AHEAD] = *reinterpret_cast<const uint2 *>(row + (ncol1 < N ? ncol1 : 0));
    };
    auto load_epilogue = [&]() {
        load_rows();
        if constexpr (ADD) {
#pragma unroll
            for (int k = 0; k < AHEAD; ++k) load_old(k);
        }
        if constexpr (LNF && !READS) {
#pragma unroll
            for (int k = 0; k < MTH; ++k) rst[k] = fold.stats[min(m0 + wm + 16 * (wk * MTH + k) + l16, M - 1)];
        }
#pragma unroll
        for (int g = 0; g < NB; ++g) {
            int c = g < 2 * NP ? ncol + 32 * (g >> 1) + 4 * (g & 1) : ncol1;
            c = c < N ? c : 0;
            bv[g] = *reinterpret_cast<const f32x4 *>(bias + c);
            if constexpr (LNF) sv[g] = *reinterpret_cast<const f32x4 *>(fold.colsum + c);
        }
    };

    // ---- ring
    int sa = 0, sw = 0;                          // stages of slab t
    int pieces = 0, pieces_rest = 0;             // where in the ring the rows' pieces land
    if constexpr (WGK == 1) {
        // iteration t of the loop requests W of slab t + SW, then A of slab t + SA; here those of t = -SA .. -1
#pragma unroll
        for (int t = -SA; t < 0; ++t) {
            if (t + SW >= 0 && t + SW < n)
#pragma unroll
                for (int i = LA; i < L; ++i) request(i, 0, t + SW);
            if (t + SA < n)
#pragma unroll
                for (int i = 0; i < LA; ++i) request(i, t + SA, 0);
        }
        wait_slabs(n - 1, integral_constant<int, SA - 1>{});
        LDS_BARRIER();
#pragma unroll
        for (int q = 0; q < NR; ++q) read(q, 0, 0, 0, 0);
        auto slab = [&](int t, auto full) {
            constexpr bool FULL = decltype(full)::value;
            const int sa1 = sa + 1 == SA ? 0 : sa + 1, sw1 = sw + 1 == SW ? 0 : sw + 1;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                mfma(m, 0);
#pragma unroll
                for (int q = m * NR / NM; q < (m + 1) * NR / NM; ++q) read(q, 1, 1, sa, sw);
                __builtin_amdgcn_sched_barrier(0);
            }
            // slab t + 1 has landed when no more than the requests behind it are out; every wave has read all of slab t
            wait_slabs(FULL ? SA : n - 2 - t, integral_constant<int, SA - 2>{});
            LDS_BARRIER();
            if constexpr (FULL) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    mfma(m, 1);
#pragma unroll
                    for (int q = m * NR / NM; q < (m + 1) * NR / NM; ++q) read(q, 0, 0, sa1, sw1);
#pragma unroll
                    for (int q = m * L / NM; q < (m + 1) * L / NM; ++q) request(q < LW ? LA + q : q - LW, sa, sw);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                if (t + SW < n)
#pragma unroll
                    for (int i = LA; i < L; ++i) request(i, sa, sw);
                // into the first stage that takes no slab any more, behind every slab (what is waited for from here on counts on it)
                if constexpr (READS) {
                    if (t == n - SA) {
                        pieces = sa * STRIDE_A;
#pragma unroll
                        for (int i = 0; i < LA; ++i) gemm_load_lds16_s(dst[i] + pieces, poff[i], fold.parts);
                    } else if (t == n - SA + 1 && fold.slots > GEMM_PARTS_LINE) {       // (and the next; a request more than is counted on makes a wait longer, not shorter)
                        pieces_rest = sa * STRIDE_A;
                        if (wave < BM / 32) gemm_load_lds16_s(lds0 + pieces_rest + wave * 1024, poff_rest, fold.parts);
                    }
                }
                if (t + 1 < n)
#pragma unroll
                    for (int q = 0; q < NR; ++q) read(q, 0, 0, sa1, sw1);
#pragma unroll
                for (int m = 0; m < NM; ++m) mfma(m, 1);
            }
            sa = sa1;
            sw = sw1;
        };
        int t = 0;
        for (; t < n - SA; ++t) slab(t, std::true_type{});
        if (EARLY) load_epilogue();
#pragma unroll 1
        for (; t < n; ++t) slab(t, std::false_type{});
    } else {
        constexpr int S = SA;
#pragma unroll
        for (int t = 0; t < S; ++t)
            if (t < n)
#pragma unroll
                for (int i = 0; i < L; ++i) request(i, t, t);
        wait_slabs(n - 1, integral_constant<int, S - 1>{});
        LDS_BARRIER();
#pragma unroll
        for (int q = 0; q < NR; ++q) read(q, 0, wk, 0, 0);
        // slab t from set B; its stage, which every wave has read, takes slab t + S
        auto slab = [&](int t, auto set, auto full) {
            constexpr bool FULL = decltype(full)::value;
            constexpr int B = decltype(set)::value;
            const int s1 = sa + 1 == S ? 0 : sa + 1;
            wait_slabs(FULL ? S : n - 2 - t, integral_constant<int, S - 2>{});
            LDS_BARRIER();
            if constexpr (FULL) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    mfma(m, B);
#pragma unroll
                    for (int q = m * NR / NM; q < (m + 1) * NR / NM; ++q) read(q, B ^ 1, wk, s1, s1);
#pragma unroll
                    for (int q = m * L / NM; q < (m + 1) * L / NM; ++q) request(q, sa, sa);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                if (t + 1 < n)
#pragma unroll
                    for (int q = 0; q < NR; ++q) read(q, B ^ 1, wk, s1, s1);
#pragma unroll
                for (int m = 0; m < NM; ++m) mfma(m, B);
            }
            sa = s1;
        };
        int t = 0;
        for (; t < n - S; t += 2) {
            slab(t, integral_constant<int, 0>{}, std::true_type{});
            if (t + 1 >= n - S) break;
            slab(t + 1, integral_constant<int, 1>{}, std::true_type{});
        }
        t = n > S ? n - S : 0;
        if (EARLY) load_epilogue();
#pragma unroll 1
        for (; t < n; ++t) {
            if (t & 1) slab(t, integral_constant<int, 1>{}, std::false_type{});
            else slab(t, integral_constant<int, 0>{}, std::false_type{});
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");       // see gemm_bf16_nt_body
    __builtin_amdgcn_sched_barrier(0);

    if (!EARLY) load_epilogue();
    if constexpr (READS) {
        // a row's pieces over the four quads, its mean, then the squares about it (ln_stats_kernel's pieces in the same order)
        gemm_wait_vm<0>();
        LDS_BARRIER();
#pragma unroll
        for (int k = 0; k < MTH; ++k) {
            const int row = wm + 16 * k + l16;
            const unsigned char *at = as + pieces + row * 128;
            const bool rest = fold.slots > GEMM_PARTS_LINE;
            float2 v[GEMM_PARTS_LINE / 4], v_rest = make_float2(0.f, 0.f);
            float mean = 0.f, sq = 0.f;
#pragma unroll
            for (int i = 0; i < GEMM_PARTS_LINE / 4; ++i) {
                const int s = 4 * i + quad;
                v[i] = *reinterpret_cast<const float2 *>(at + (((s >> 1) ^ ((row >> 1) & 7)) << 4) + (s & 1) * 8);
                if (s < fold.slots) mean += v[i].x;
            }
            if (rest) {
                v_rest = *reinterpret_cast<const float2 *>(as + pieces_rest + row * 32 + quad * 8);
                if (GEMM_PARTS_LINE + quad < fold.slots) mean += v_rest.x;
            }
            mean = gemm_quad_sum(mean) / (float)fold.slots;
#pragma unroll
            for (int i = 0; i < GEMM_PARTS_LINE / 4; ++i)
                if (4 * i + quad < fold.slots) sq += gemm_piece_term(v[i], mean);
            if (rest && GEMM_PARTS_LINE + quad < fold.slots) sq += gemm_piece_term(v_rest, mean);
            const float inv = rsqrtf(gemm_quad_sum(sq) / (float)K + fold.eps);          // K: the rows' length
            rst[k] = make_float2(inv, -inv * mean);
        }
    }

    // ---- epilogue, straight from the accumulators: lane (l16, quad) holds row 16*i + l16, columns 8*quad .. + 7 of every pair of tiles
    f32x4 fin[MTH][NT];
    if constexpr (WGK == 2) {
        // the halves of K: either group sends the rows that the other one finishes
        f32x4 *x = reinterpret_cast<f32x4 *>(smem) + wt * (2 * MTH * NT * 64) + lane;
#pragma unroll
        for (int k = 0; k < MTH; ++k)
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const int hi = MTH + k < MT ? MTH + k : MT - 1;
                x[((wk ^ 1) * MTH + k) * NT * 64 + j * 64] = wk ? acc[k][j] : acc[hi][j];
                fin[k][j] = wk ? acc[hi][j] : acc[k][j];
            }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < MTH; ++k)
#pragma unroll
            for (int j = 0; j < NT; ++j) fin[k][j] += x[(wk * MTH + k) * NT * 64 + j * 64];
    } else {
#pragma unroll
        for (int k = 0; k < MTH; ++k)
#pragma unroll
            for (int j = 0; j < NT; ++j) fin[k][j] = acc[k][j];
    }
    auto finish = [&](float *v, int cnt, int k, int g) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (e >= cnt) break;
            const float b = bv[g + e / 4][e % 4];
            if constexpr (LNF) v[e] = v[e] * rst[k].x + (rst[k].y * sv[g + e / 4][e % 4] + b);
            else v[e] += b;
            if constexpr (EPI == SSAM_EPI_BIAS_GELU) v[e] = gelu_erf(v[e]);
        }
    };
    uint4 kept[LEAVES ? MTH : 1][LEAVES ? NP : 1];
#pragma unroll
    for (int k = 0; k < MTH; ++k) {
        bf16 *row = C + (long)drow[k] * ld.c;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = fin[k][2 * p + e / 4][e % 4];
            finish(v, 8, k, 2 * p);
            if constexpr (ADD) {
                float o[8];
                unpack_bf16x8(old[k % AHEAD][p], o);
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] += o[e];
            }
            const uint4 packed = pack_bf16x8(v);
            if (drow[k] >= 0 && ncol + 32 * p < N) *reinterpret_cast<uint4 *>(row + ncol + 32 * p) = packed;      // N % 8 == 0
            if constexpr (LEAVES) kept[k][p] = packed;
        }
        if constexpr (NT % 2) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = fin[k][NT - 1][e];
            finish(v, 4, k, 2 * NP);
            if constexpr (ADD) {
                v[0] += __uint_as_float(old1[k % AHEAD].x << 16); v[1] += __uint_as_float(old1[k % AHEAD].x & 0xffff0000u);
                v[2] += __uint_as_float(old1[k % AHEAD].y << 16); v[3] += __uint_as_float(old1[k % AHEAD].y & 0xffff0000u);
            }
            if (drow[k] >= 0 && ncol1 < N) *reinterpret_cast<uint2 *>(row + ncol1) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
        }
        if constexpr (ADD) if (k + AHEAD < MTH) load_old(k + AHEAD);
    }
    if constexpr (LEAVES) {
        // Pieces of the rows from the values as stored: sums of 8 columns, of columns 32 apart, over the quads (gemm_piece_sum8 and the same tree in
        // whatever writes pieces: a row's are the same bits whichever kernel wrote it last).  Waves of 32 columns have the next wave's from LDS.
        float *x = reinterpret_cast<float *>(smem) + lane;        // [2][wave][MTH][64]: the ring is done with
        auto over_row = [&](float (&s8)[MTH][NP], int turn) {
            if constexpr (WN == 32) {
                if (turn == 0) LDS_BARRIER();
#pragma unroll
                for (int k = 0; k < MTH; ++k) x[((turn * 8 + wave) * MTH + k) * 64] = s8[k][0];
                LDS_BARRIER();
            }
#pragma unroll
            for (int k = 0; k < MTH; ++k)
                s8[k][0] = gemm_quad_sum(s8[k][0] + (WN == 32 ? x[((turn * 8 + (wave ^ 1)) * MTH + k) * 64] : s8[k][NP - 1]));
        };
        float sum[MTH][NP], sq[MTH][NP];
#pragma unroll
        for (int k = 0; k < MTH; ++k)
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                float v[8];
                unpack_bf16x8(kept[k][p], v);
                sum[k][p] = gemm_piece_sum8(v);
            }
        over_row(sum, 0);
#pragma unroll
        for (int k = 0; k < MTH; ++k)
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                float v[8];
                unpack_bf16x8(kept[k][p], v);
                sq[k][p] = gemm_piece_squares8(v, sum[k][0] * (1.f / 64.f));
            }
        over_row(sq, 1);
        const int col = n0 + (wn & ~63), pitch = gemm_parts_pitch(fold.slots);
        if (WN == 32 && (wt & 1)) return;
#pragma unroll
        for (int k = 0; k < MTH; ++k)
            if (quad == 0 && drow[k] >= 0 && col < N) fold.parts[(long)drow[k] * pitch + (col >> 6)] = make_float2(sum[k][0] * (1.f / 64.f), sq[k][0]);
    }
}
