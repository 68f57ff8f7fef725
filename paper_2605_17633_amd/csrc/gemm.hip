// Dispatcher of the bf16 NT GEMM (qkv / proj / fc1 / fc2 of the SAM block).
#include <algorithm>

#include "gemm_direct.h"
#include "gemm_large.h"
#include "gemm_ring.h"
#include "gemm_wide_launch.h"

int ssam_gemm_wide_bias(int tile, bool packed, const GemmWideArgs &a);
int ssam_gemm_wide_gelu(int tile, bool packed, const GemmWideArgs &a);
int ssam_gemm_wide_add(int tile, bool packed, const GemmWideArgs &a);
int ssam_gemm_wide_scatter(int tile, bool packed, const GemmWideArgs &a);
int ssam_gemm_wide_ln_scatter(int tile, const GemmWideArgs &a);
int ssam_gemm_wide_ln_gelu(int tile, const GemmWideArgs &a);
int ssam_gemm_wide_parts_scatter(int tile, const GemmWideArgs &a);
int ssam_gemm_wide_parts_gelu(int tile, const GemmWideArgs &a);
int ssam_gemm_wide_parts_add(int tile, const GemmWideArgs &a);
int ssam_gemm_large_parts_gelu(const GemmWideArgs &a, void *split_ws, size_t split_ws_bytes);
int ssam_gemm_large_parts_scatter(const GemmWideArgs &a);

namespace {

const GemmFold no_fold = {};

template <int EPI, bool LNF = false>
int launch_tile_packed(int tile, const bf16 *A, const bf16 *W, const float *bias, bf16 *C, int M, int N, int K,
                       const GemmLd &ld, const GemmRowMap &rm, const SplitWs &ws, hipStream_t st, const GemmFold &fold = no_fold)
{
    switch (tile) {
    case 1: return launch_split<256, 256, 128, 128, EPI, 2, 4, true, LNF>(A, W, bias, C, M, N, K, ld, 256, rm, ws, fold, st);
    case 3: return launch_split<128, 128, 64, 128, EPI, 2, 2, true, LNF>(A, W, bias, C, M, N, K, ld, 512, rm, ws, fold, st);
    case 4: return launch_split<128, 256, 128, 128, EPI, 1, 4, true, LNF>(A, W, bias, C, M, N, K, ld, 512, rm, ws, fold, st);
    default: return SSAM_EUNSUPPORTED;
    }
}

template <int EPI>
int launch_tile(int tile, const bf16 *A, const bf16 *W, const float *bias, bf16 *C, int M, int N, int K,
                const GemmLd &ld, const GemmRowMap &rm, const SplitWs &ws, hipStream_t st)
{
    switch (tile) {
    case 1: return launch_split<256, 256, 128, 128, EPI, 2, 4>(A, W, bias, C, M, N, K, ld, 256, rm, ws, no_fold, st);
    case 2: return launch_split<256, 128, 128, 128, EPI>(A, W, bias, C, M, N, K, ld, 256, rm, ws, no_fold, st);
    case 3: return launch_split<128, 128, 64, 128, EPI>(A, W, bias, C, M, N, K, ld, 512, rm, ws, no_fold, st);
    case 4: return launch_split<128, 256, 128, 128, EPI, 1, 4>(A, W, bias, C, M, N, K, ld, 512, rm, ws, no_fold, st);   // same plan as packed
    default: return SSAM_EINVAL;
    }
}

// What launches of the large tiles take (see pick_ring), from the time that pick_tile orders them by.
double large_tile_us(int tile, double rounds_us, bool packed)
{
    if (tile == 3) return 0.2 + 1.18 * rounds_us;
    return packed ? 3.7 + 0.76 * rounds_us : 0.5 + rounds_us;
}

// The same for a problem that is all left-over with K cut (tm x tn tiles): its ranges, and its partial tiles, of which only rows
// that exist are written and read.
double all_split_us(int M, int N, int nk, int parts, int bn, int tm, int tn, bool packed)
{
    const double tiles = (double)ssam_div_up(M, tm) * ssam_div_up(N, bn) * (bn / tn);
    const double mb = tiles * parts * (M < tm ? M : tm) * tn * 4e-6;
    return (packed ? 6.7 : 7.0) + ssam_div_up(nk, parts) * (packed ? 0.84 : 1.10) + 0.37 * mb;
}

// Pick the tile by a time model in microseconds, fitted on MI355X to the ViT-H layer shapes: a round of
// workgroups costs nk * t_slab + t_epi.  The 256x256 tile (eight waves, one workgroup per CU) and the 128x256
// tile (four waves in a row, two workgroups per CU) give a wave the same 128x64 piece and move the same data
// per flop; with two independent workgroups per CU one's epilogue overlaps the other's main loop, which is worth
// 5 us a round behind the GELU epilogue and 1-2.5 us behind the others.  The 128x128 tile (two per CU) moves
// more data per flop and is for small problems.  The left-over launch costs a lone workgroup's walk over its
// K range, latency bound, plus the reduce.
int pick_tile(int M, int N, int K, int epilogue, const SplitWs &ws, bool packed, double &launch_us, int only = 0)
{
    struct Cand { int id, bm, bn, tm, tn, slots; double t_slab, t_epi[4]; };   // t_epi: bias, +GELU, scatter-add, scatter
    const Cand cands[4] = { { 1, 256, 256, 128, 128, 256, 1.73, { 5.1, 13.6, 13.5, 6.0 } },
                            { 2, 256, 128, 128, 128, 256, 1.15, { 4.0, 9.0, 9.5, 4.5 } },
                            { 3, 128, 128, 64, 128, 512, 1.10, { 3.5, 6.6, 6.8, 4.0 } },
                            { 4, 128, 256, 128, 128, 512, 1.71, { 5.0, 9.0, 11.5, 5.5 } } };
    const int nk = ssam_div_up(K, GEMM_BK);
    int best = 3;
    double best_time = 1e30;
    for (const Cand &c : cands) {
        if (c.id == 2) continue;    // 256x128 is never the fastest on these shapes: kept as a forced choice only
        if (only != 0 && c.id != only) continue;
        if (c.id == 4 && !packed) continue;   // with W in LDS a 128x256 workgroup needs 96 KB: one per CU, nothing overlaps
        const int subs = (c.bm / c.tm) * (c.bn / c.tn);
        const int total = ssam_div_up(M, c.bm) * ssam_div_up(N, c.bn);
        const TailPlan plan = plan_tail(total, c.slots, nk, subs, (size_t)c.tm * c.tn * sizeof(float), ws);
        const double round = nk * c.t_slab + c.t_epi[epilogue];
        const int in_main = total - plan.rem, last = in_main % c.slots;
        double t = (double)(in_main / c.slots) * round;
        if (last != 0) t += round * (c.slots > 256 && last * 2 <= c.slots ? 0.62 : 1.0);   // lone workgroups on their CUs
        if (plan.rem != 0) {
            const int n_sub = plan.rem * subs;
            t += plan.parts > 1 ? ssam_div_up(nk, plan.parts) * 0.9 + 11.0 : (nk * 0.75 + 5.0) * (1.0 + n_sub / 1024.0);
        }
        if (t >= best_time) continue;
        best_time = t;
        best = c.id;
        // t leaves the launch out and serves to order the tiles; what the launch takes:
        launch_us = plan.rem == total && plan.parts > 1 ? all_split_us(M, N, nk, plan.parts, c.bn, c.tm, c.tn, packed)
                                                        : large_tile_us(c.id, t, packed);
    }
    return best;
}

// The ring's tiles (gemm_ring.h) for a problem that they hold in one round of workgroups.  A launch takes t0 plus t_slab[k - 1] per
// slab of 64 when its busiest CU has k workgroups, with row-major and with packed weights.
struct RingTile { int bm, bn, slots; struct { double t0, t_slab; } us[2][3]; };
constexpr RingTile ring_tiles[3] = { { 128, 128, 2, { { { 3.6, 0.82 }, { 7.4, 0.79 }, {} }, { { 3.7, 0.73 }, { 6.9, 0.80 }, {} } } },
                                     { 128, 64, 3, { { { 2.6, 0.70 }, { 4.7, 0.70 }, { 6.2, 0.85 } }, { { 2.65, 0.65 }, { 4.3, 0.645 }, { 6.0, 0.78 } } } },
                                     { 64, 64, 3, { { { 2.7, 0.335 }, { 3.9, 0.385 }, { 4.5, 0.58 } }, { { 2.7, 0.31 }, { 3.7, 0.355 }, { 4.0, 0.565 } } } } };

constexpr int RING_DIRECT = 3;

// Index of the ring tile (or RING_DIRECT: gemm_direct.h) that is faster than the large tiles (launch_us; what is taken, on return), or -1.  whole_lines: the rows
// of row-major operands begin at multiples of 128 bytes; where they do not, a slab's 128-byte pieces of a row take two
// lines each and a CU with two or three workgroups 1.35 times as long (427 x 3824 x 4560: 54 us, large tiles 44).
// The estimates are fitted to 1200 shapes (M 8 to 8192, N 8 to 6144, K 8 to 6144: the layers of widths 576 to 1280, any sizes, few
// rows against a long K) with weights that no cache holds, as in a deep stack: those cost every form 0.2 us a megabyte on top
// of its estimate, the direct kernel 0.1, hence its credit.  Standard errors are 7-12 %.  What is taken is 0.9 % on
// average from the fastest form, and on 9 of the shapes slower than the large tiles by more than 3 %, 7 % at most; with it they
// are 25 % (row-major) and 31 % (packed) faster on average than with the large tiles alone.
int pick_ring(int M, int N, int K, bool packed, bool whole_lines, double &launch_us)
{
    const int nk = ssam_div_up(K, GEMM_BK);
    int best = -1;
    double best_us = launch_us;
    for (int i = 0; i < 3; ++i) {
        const RingTile &t = ring_tiles[i];
        const long tiles = (long)ssam_div_up(M, t.bm) * ssam_div_up(N, t.bn);
        if (tiles > 256L * t.slots) continue;
        const auto &u = t.us[packed][ssam_div_up(tiles, 256) - 1];
        const double us = u.t0 + nk * u.t_slab * (!whole_lines && !packed && tiles > 256 ? 1.35 : 1.0);
        if (us < best_us) { best_us = us; best = i; }
    }
    // at most one tile per CU
    if (packed && (long)ssam_div_up(M, 32) * (N / 32) <= 256 && 3.2 + nk * 0.14 - 0.2e-6 * N * K < best_us) {
        best = RING_DIRECT;
        best_us = 3.2 + nk * 0.14 - 0.2e-6 * N * K;
    }
    launch_us = best_us;
    return best;
}

// What the GELU epilogue adds to a ring's estimate, which is an average over the epilogues, by the columns x rows that its busiest CU finishes (two 128x128 tiles: 1.5 us).
// Only against the wide kernel, whose estimate has it, and of the tiles of 128 rows: 94 routed MLPs of 900 to 3500 rows that it moves are 2.4 % faster (none slower), 64x64 rings
// of 120 to 640 rows were 2 to 5 % faster than what it would move them to.  2500 x 3072 x 768 takes the ring 19.5 to 20.3 us, estimated as 16.9, and 256x128 17.8 with 56 CUs left to read weights ahead
// (encoders of ViT-B, two images of 50 x 50: 1256 -> 1236 us packed, 1253 -> 1235 row-major).  With gather and LN2 folded in: 25 routed MLPs of 1580 to 3270 rows
// (512 x 2048 to 1024 x 4096) 0.5 to 3.5 % faster, 26 stacks 1.1 % together (9 images of 30 x 30 of ViT-L's width, density 0.2 164.4 -> 158.0 us a block), none slower; same bits.
double ring_gelu_us(int ring, int M, int N, int epilogue)
{
    if (ring < 0 || ring >= RING_DIRECT || epilogue != SSAM_EPI_BIAS_GELU) return 0.0;
    const RingTile &t = ring_tiles[ring];
    if (t.bm < 128) return 0.0;
    return 1.5 / (2 * 128 * 128) * t.bm * t.bn * ssam_div_up((long)ssam_div_up(M, t.bm) * ssam_div_up(N, t.bn), 256);
}

// The wide kernel's tiles (gemm_wide.h).  A launch of r rounds (one workgroup per CU at a time) takes
// t0 + r * (t_round + t_slab per slab of 64, t_gelu and t_add behind those epilogues) + t_mb per megabyte of C.
// t_parts: what a round takes longer where it leaves row statistics in pieces (GemmParts), reads them, and reads them of gathered rows (measured with the tiles
// that can: D = 768 and 1024, half a round and a whole one, within 0.2 of these).
struct WideTile { int bm, bn; double t0, t_round, t_slab, t_gelu, t_add, t_mb, t_parts[3]; };
constexpr WideTile wide_tiles[GEMM_WIDE_COUNT] = {
    { 64, 64, 3.7, 0, 0.16, 0.262, 0, 0.326, { 0.3 } },
    { 96, 64, 0, 4.18, 0.207, 0.375, 0.03, 0.246, { 0.55 } },
    { 96, 96, 0, 4.66, 0.251, 0.336, 0.504, 0.223, {} },
    { 64, 128, 0, 4.27, 0.228, 0.614, 0.075, 0.354, { 0.25 } },
    { 128, 128, 1.14, 2.89, 0.382, 1.2, 0, 0.153, { 0.35, 0.45, 1.15 } },
    { 128, 192, 0.896, 4.09, 0.498, 1.31, 0, 0.205, { 0, 1.05, 1.75 } },
    { 192, 128, 0.478, 3.86, 0.505, 1.71, 0, 0.183, { 0.65, 0.75, 1.5 } },
    { 256, 128, 0.243, 4.64, 0.623, 2.1, 0, 0.2, { 0.95, 0.95, 2.25 } },
    { 192, 192, 0.697, 5.38, 0.668, 1.56, 0, 0.22, { 0, 1.35, 2.4 } },
    { 192, 256, 1.07, 4.83, 0.85, 3.16, 0, 0.197, { 1.8, 1.55, 2.55 } },
    { 256, 192, 0.964, 5, 0.838, 3.1, 0, 0.194, { 0, 1.05, 2.5 } },
    { 256, 256, 1.7, 4.96, 1.09, 4.28, 0, 0.207, { 2.1, 1.9, 3.4 } } };
enum PartsUse { PARTS_LEFT, PARTS_READ, PARTS_READ_GATHERED, PARTS_NONE };

// Index of the wide kernel's tile that is faster than the others' launch_us, or -1.  rows_a: rows of A where its rows are
// gathered.  The tiles below 128x128 add K in two chains instead of one, and are taken where that is faster than the others with either
// layout of the weights (both_us), so that packing a program's weights does not change its bits.
// The kernel takes whole slabs; below five of them its prologue is not earned back, and up to 32 rows packed weights have a kernel
// with tiles of 32 (31 x 3840 x 3648: 12.9 us, the direct kernel 10.9).  Its requests address memory by 32-bit offsets from the tile's
// first row, or from A's where rows are gathered.
// Rows that do not begin on 128 bytes (torn: operands of such rows) take two lines for a slab's 128 bytes, and two chains over K pull
// twice the bytes a flop of the large tiles: a slab takes 1.12 times as long for either operand and 1.36 for both in tiles below 128x128, 1.1 and 1.2
// above.  Charged with more, since the others lose less there (a K-split 1.04 for both): of 639 row-major shapes with both operands torn 114 were
// slower than without this kernel by more than 3 %, 84 % at most, with no such charge; 26, 13 % at most, with it, and 5 with one operand torn.
// Few rows against a long K: with weights that no cache holds a slab of the 64x64 tile takes HBM's latency over the four slabs in flight, 0.22 us
// where no other workgroup has fetched it (22 x 1088 x 3456 16.9 us, a K-split 14.1; 177 x 984 x 5120 26.4, 20.0).  With that charged from the 17th on, of 472 row-major
// shapes of 8 to 300 rows 25 are slower than without this kernel by more than 3 % (18 % at most; 47 and 32 % without the charge), of 384 of any 9 (6 %; 22, 23 %).
// Fitted to 1339 shapes (M 8 to 24576, N 128 to 5120, K 128 to 5376, all epilogues, both layouts, weights that no cache holds; those
// cost the others 0.2 us a megabyte on top of their estimates, which is left out here: with warm weights 784 x 2304 x 768 takes the ring
// 8.9 us and this kernel 9.5).  What is taken is 1 % on average from the fastest form, 10 % faster on average than
// without this kernel, and on 9 of the shapes slower than that by more than 3 %, 9 % at most (shapes of 5 to 8 us).  More than two rounds of packed problems
// are left to the large tiles, two workgroups to a CU, whose epilogues run under other workgroups' main loops (16384 x 1280 x 5120:
// 180 us against 185, 32768 x 3840 x 1280: 264 against 269); with row-major weights those are alone on their CU too, and four are fitted.
// parts: what the kernel does with row statistics in pieces, of the tiles that can; what that takes is not held against the others, who would have to wait for a
// launch, but where others_read: they read pieces too, and launch_us has it.  Left out there, fc1 of 1265 to 1536 rows (x 5120 x 1280) was left to the large tile for a margin that two rounds of
// 192x192 wanted, 1 to 6 % of a block slower (2 images of 40 x 40, density 0.4 135.8 us, 125.9 with 256x128), and qkv of 3328 to 5120 rows taken from it, 1 to 2.5 % (5 of 32 x 32, 0.6 200.7,
// 196.4).  launch_us: what is taken, on return.
int pick_wide(int M, int N, int K, int epilogue, const GemmLd &ld, bool packed, long rows_a, double &launch_us, double both_us, PartsUse parts = PARTS_NONE, bool others_read = false)
{
    const unsigned among = parts == PARTS_NONE ? ~0u : parts == PARTS_LEFT ? GEMM_WIDE_WRITES_PARTS : GEMM_WIDE_READS_PARTS;
    const int nk = K / GEMM_BK;
    if (K % GEMM_BK != 0 || nk < GEMM_WIDE_SLABS || (packed && M <= 32)) return -1;
    if ((long)256 * ld.a * 2 >= 1L << 31 || (rows_a + 1) * ld.a * 2 >= 1L << 32 || (long)256 * (packed ? K : ld.w) * 2 >= 1L << 31) return -1;
    const int torn = (ld.a % GEMM_BK != 0) + (!packed && ld.w % GEMM_BK != 0);
    int best = -1;
    double best_us = 1e30, best_parts = 0.0;
    for (int i = 0; i < GEMM_WIDE_COUNT; ++i) {
        if (!((among >> i) & 1)) continue;
        const WideTile &t = wide_tiles[i];
        const double slab = t.t_slab * (1.0 + torn * (t.bm * t.bn < 128 * 128 ? 0.3 : 0.15));
        const int rounds = ssam_div_up(ssam_div_up((long)ssam_div_up(M, t.bm) * ssam_div_up(N, t.bn), 8), 32);      // (see the kernel's XCDs)
        if (rounds > (packed ? 2 : 4)) continue;
        const double us = t.t0 + rounds * (t.t_round + nk * slab + (i == 0 && nk > 16 ? 0.06 * (nk - 16) : 0.0) + (epilogue == SSAM_EPI_BIAS_GELU ? t.t_gelu : epilogue == SSAM_EPI_BIAS_SCATTER_ADD ? t.t_add : 0.0))
                          + t.t_mb * (epilogue == SSAM_EPI_BIAS_SCATTER_ADD ? 4e-6 : 2e-6) * M * N;
        const double parts_us = parts == PARTS_NONE ? 0.0 : rounds * t.t_parts[parts];
        if (us + parts_us < best_us + best_parts) { best_us = us; best_parts = parts_us; best = i; }
    }
    const double others_us = best >= 0 && wide_tiles[best].bm * wide_tiles[best].bn < 128 * 128 && both_us < launch_us ? both_us : launch_us;
    if (best_us + (others_read ? best_parts : 0.0) >= 0.99 * others_us) return -1;
    launch_us = best_us + best_parts;
    return best;
}

// What the others take with the other layout of the weights (1e30: there is none).
double other_layout_us(int M, int N, int K, int epilogue, const SplitWs &ws, bool packed, bool whole_lines)
{
    if (!packed && N % 128 != 0) return 1e30;
    double us;
    pick_tile(M, N, K, epilogue, ws, !packed, us);
    const int ring = pick_ring(M, N, K, !packed, whole_lines, us);
    return us + ring_gelu_us(ring, M, N, epilogue);
}

template <int BM, int BN, int STAGES, int EPI, bool WPACK, bool LNF>
int launch_ring_tile(const bf16 *A, const bf16 *W, const float *bias, bf16 *C, int M, int N, int K,
                     const GemmLd &ld, const GemmRowMap &rm, const GemmFold &fold, hipStream_t st)
{
    constexpr size_t lds = gemm_ring_lds_bytes<BM, BN, STAGES>();
    static_assert(lds <= 64 * 1024, "default LDS limit");
    GemmTileRange tr = { ssam_div_up(M, BM), ssam_div_up(N, BN), 0, 0 };
    tr.tile_count = tr.tiles_m * tr.tiles_n;
    hipLaunchKernelGGL((gemm_ring_kernel<BM, BN, STAGES, EPI, WPACK, LNF>), dim3(ssam_div_up(tr.tile_count, 8) * 8), dim3(256), lds, st,
                       A, W, bias, C, M, N, K, ld, tr, rm, fold);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

template <int EPI, bool WPACK, bool LNF = false>
int launch_ring(int ring, const bf16 *A, const bf16 *W, const float *bias, bf16 *C, int M, int N, int K,
                const GemmLd &ld, const GemmRowMap &rm, const GemmFold &fold, hipStream_t st)
{
    if constexpr (WPACK) if (ring == RING_DIRECT) {
        GemmTileRange tr = { ssam_div_up(M, 32), N / 32, 0, 0 };
        tr.tile_count = tr.tiles_m * tr.tiles_n;
        hipLaunchKernelGGL((gemm_direct_kernel<EPI, LNF>), dim3(ssam_div_up(tr.tile_count, 8) * 8), dim3(256), 0, st, A, W, bias, C, M, N, K, ld, tr, rm, fold);
        SSAM_CHECK_LAUNCH();
        return SSAM_OK;
    }
    switch (ring) {
    case 0: return launch_ring_tile<128, 128, 2, EPI, WPACK, LNF>(A, W, bias, C, M, N, K, ld, rm, fold, st);
    case 1: return launch_ring_tile<128, 64, 2, EPI, WPACK, LNF>(A, W, bias, C, M, N, K, ld, rm, fold, st);
    default: return launch_ring_tile<64, 64, 3, EPI, WPACK, LNF>(A, W, bias, C, M, N, K, ld, rm, fold, st);
    }
}

template <int EPI, bool WPACK>
int launch_any(int tile, int ring, const bf16 *A, const bf16 *W, const float *bias, bf16 *C, int M, int N, int K,
               const GemmLd &ld, const GemmRowMap &rm, const SplitWs &ws, hipStream_t st)
{
    if (ring >= 0) return launch_ring<EPI, WPACK>(ring, A, W, bias, C, M, N, K, ld, rm, no_fold, st);
    if constexpr (WPACK) return launch_tile_packed<EPI>(tile, A, W, bias, C, M, N, K, ld, rm, ws, st);
    else return launch_tile<EPI>(tile, A, W, bias, C, M, N, K, ld, rm, ws, st);
}

// The kernel of a contraction: the wide kernel's tile, or (wide = -1) the ring, or (ring = -1) the large tile; what it takes, in microseconds.
struct Choice { int wide, tile, ring; double us; };

// Row statistics in more pieces than a row of a slab holds (D = 1280) are read by the large 128x256 tile too, in front of its first slab: 0.5 us a round of it,
// 1.2 of gathered rows (8192 x 3840 x 1280 69.0 -> 68.8 us, 32768 264.1 -> 268.7; 2456 x 5120 x 1280 40.0 -> 41.3).  It leaves none: 32768 x 1280 x 1280 103.9 -> 109.7,
// and at such sizes, at the power limit, ViT-H of 8 images was 0.8 % slower with its launches saved.
constexpr int LARGE_PARTS_TILE = 4;
bool large_reads_parts(int D) { return D / 64 > GEMM_PARTS_LINE; }
double large_parts_us(int M, int N, bool gathered) { return ssam_div_up((long)ssam_div_up(M, 128) * ssam_div_up(N, 256), 512) * (gathered ? 1.2 : 0.5); }

Choice choose(int M, int N, int K, int epilogue, const GemmLd &ld, const SplitWs &ws, bool packed, PartsUse parts = PARTS_NONE)
{
    Choice c;
    c.tile = pick_tile(M, N, K, epilogue, ws, packed, c.us);
    c.ring = pick_ring(M, N, K, packed, ld.a % GEMM_BK == 0 && ld.w % GEMM_BK == 0, c.us);
    c.us += ring_gelu_us(c.ring, M, N, epilogue);
    c.wide = pick_wide(M, N, K, epilogue, ld, packed, 0, c.us, other_layout_us(M, N, K, epilogue, ws, packed, ld.a % GEMM_BK == 0), parts);
    return c;
}

// How much faster the others may be than a tile that reads row statistics in pieces: fc1 of ViT-L at a density of 0.4 (1638 x 4096 x 1024) is 1 % faster on the
// large tiles by itself.
constexpr double PARTS_US = 3.0;

// The same for fc1 with gather and LayerNorm folded in.  parts: its row statistics come in pieces.  ring_gelu: see ring_gelu_us.
Choice choose_fold_gelu(int M, int N, int K, const GemmLd &ld, long rows_a, const SplitWs &ws, bool parts, bool ring_gelu = true)
{
    Choice c;
    if (parts && large_reads_parts(K)) {
        c.tile = pick_tile(M, N, K, SSAM_EPI_BIAS_GELU, ws, true, c.us, LARGE_PARTS_TILE);
        c.ring = -1;
        c.us += large_parts_us(M, N, true);
        c.wide = pick_wide(M, N, K, SSAM_EPI_BIAS_GELU, ld, true, rows_a, c.us, c.us, PARTS_READ_GATHERED, true);
        return c;
    }
    c.tile = pick_tile(M, N, K, SSAM_EPI_BIAS_GELU, ws, true, c.us);
    c.ring = pick_ring(M, N, K, true, true, c.us);
    c.us += parts ? PARTS_US : ring_gelu ? ring_gelu_us(c.ring, M, N, SSAM_EPI_BIAS_GELU) : 0.0;
    c.wide = pick_wide(M, N, K, SSAM_EPI_BIAS_GELU, ld, true, rows_a, c.us, c.us, parts ? PARTS_READ_GATHERED : PARTS_NONE);
    return c;
}

double folded_ln_us(int tiles, int K);

// And for qkv with a LayerNorm folded in.
Choice choose_ln(int M, int N, int K, const GemmLd &ld, bool parts)
{
    Choice c = { -1, 4, -1, folded_ln_us((M / 128) * (N / 256), K) };
    if (parts && large_reads_parts(K)) {
        c.us += large_parts_us(M, N, false);
        c.wide = pick_wide(M, N, K, SSAM_EPI_BIAS_SCATTER, ld, true, 0, c.us, c.us, PARTS_READ, true);
        return c;
    }
    c.ring = pick_ring(M, N, K, true, true, c.us);
    if (parts) c.us += PARTS_US;
    c.wide = pick_wide(M, N, K, SSAM_EPI_BIAS_SCATTER, ld, true, 0, c.us, c.us, parts ? PARTS_READ : PARTS_NONE);
    return c;
}

// The contractions of a block with both LayerNorms folded in that can read or leave pieces: qkv, proj, fc1, fc2.
struct BlockChoices { Choice c[4]; };

BlockChoices block_choices(int rows, int kept, int D, int Dm, bool parts, bool ring_gelu = true)
{
    alignas(16) static unsigned char some;
    // fc1 and fc2 with what the launch will have: the kernel that is found here has to be the one that is taken there
    const SplitWs whole = { &some, GEMM_SPLIT_WS_BYTES }, ws = { &some, parts ? gemm_split_beside_parts(rows, D) : GEMM_SPLIT_WS_BYTES };
    const PartsUse left = parts ? PARTS_LEFT : PARTS_NONE;
    return { { choose_ln(rows, 3 * D, D, GemmLd{ D, D, 3 * D }, parts),
               choose(rows, D, D, SSAM_EPI_BIAS_SCATTER_ADD, GemmLd{ D, D, D }, whole, true, left),
               choose_fold_gelu(kept, Dm, D, GemmLd{ D, D, Dm }, rows, ws, parts, ring_gelu),
               choose(kept, D, Dm, SSAM_EPI_BIAS_SCATTER_ADD, GemmLd{ Dm, Dm, D }, ws, true, left) } };
}

}  // namespace

// Row statistics in pieces (GemmParts) of the residual stream, [rows][D] of which `kept` go through the MLP, in blocks with packed weights and both
// LayerNorms folded in.  0: none; 1: proj leaves them and fc1 reads them; 3: fc2 leaves them too, and the next block's qkv reads those.  What leaves or reads
// them is the wide kernel (of rows of 1280 the large tile reads them too), where it is at least near the fastest by the tiles that can: what a contraction takes longer than without, leaving and reading included,
// goes against the launch saved.  A block by itself has a launch for qkv's statistics all the same, reads and leaves nothing there and takes the stack's tiles.
// LAUNCH_US: 90 folded stacks of widths 512, 768 and 1024 (512 to 10000 rows, densities 0.2 to 1) ran with each form.  With 4.6 to 5.5 all together are 231 us a
// block faster than without pieces (235 with the best form of each, 230 with pieces wherever tiles fit) and two are slower, by 1.1 us at most; with 3.4 212.  Larger
// ones lost without that charge: fc2 of ViT-B with 2760 kept rows (6 images of 48 x 48, density 0.2) went from 96x96 to 128x128, 25.2 -> 29.0 us, and dense or
// large stacks were up to 5 % slower than without.
int ssam_parts_form_of(int rows, int kept, int D, int Dm)
{
    if (D % 128 != 0 || D / 64 > GEMM_PARTS_MOST) return 0;
    // (what fc1 takes without is as LAUNCH_US was fitted.  With a ring's GELU charged there nine more stacks would have pieces, at a density of 0.2: seven of them were 0.2 % faster than with
    // the ring, less than the wide kernel without pieces is by itself)
    const BlockChoices with = block_choices(rows, kept, D, Dm, true), without = block_choices(rows, kept, D, Dm, false, false);
    constexpr double LAUNCH_US = 5.0;
    double gain[2] = { LAUNCH_US, LAUNCH_US };    // of the pieces between proj and fc1, and between fc2 and qkv
    const bool large = large_reads_parts(D);
    if (large) {
        // A launch over 32768 rows of 1280 takes 14.9 us, 16384 9.8, 13104 9.1, 8192 5.6.  73 folded stacks of ViT-H's width (1024 to 9600 rows, densities 0.2 to 1) are
        // 1.5 % faster than without pieces, -0.3 to 4.6 %; with 5 us for the smaller launches three more took pieces for fc1 alone, and lost 0.2 to 2 %.
        const double row_us = 2.0 * D / 7.2e6;
        gain[0] = std::max(4.0, 3.4 + kept * row_us);
        gain[1] = std::max(4.0, 3.4 + rows * row_us);
    }
    for (int i = 0; i < 4; ++i) gain[i == 0 || i == 3] -= with.c[i].wide < 0 && !(large && i % 2 == 0) ? 1e30 : with.c[i].us - without.c[i].us;
    // The estimates fall short where fc1 leaves the small tiles for one that reads twenty pieces, and of its largest launches.  With any gain at all, 115 shapes, nearly all with an MLP that is not
    // four times as wide (200 to 3500 kept rows with Dm 512 to 3840, 7000 and more with 7680), were 1.2 % slower with pieces than without as stacks (4.6 % at most; 23 faster, by 2.8 % at most) and
    // 3.2 % as blocks by themselves (7 % at most): 3 images of 16 x 16, dense, Dm = 1280 62.2 and 72.1 us a block without, 64.5 and 76.3 with.
    const double least = large && with.c[2].us - without.c[2].us > 4.5 ? 2.5 : 0.0;
    if (gain[1] > 0 && gain[0] + gain[1] > least) return 3;
    return gain[0] > 0 ? 1 : 0;
}

// The form, for tests, and the wide kernel's tiles of qkv, proj, fc1 and fc2 with it (-1: another kernel).  Host only; not part of the interface.
extern "C" int ssam_parts_form(int rows, int kept, int D, int Dm) { return ssam_parts_form_of(rows, kept, D, Dm); }

extern "C" int ssam_parts_tiles(int rows, int kept, int D, int Dm, int *tiles)
{
    const int form = ssam_parts_form_of(rows, kept, D, Dm);
    for (int i = 0; i < 4; ++i) tiles[i] = block_choices(rows, kept, D, Dm, form == 3 || (form == 1 && (i == 1 || i == 2))).c[i].wide;
    return form;
}

// And what the launches of fc1 and fc2 take with split_bytes of scratch (fc1 reads pieces in form 1 and 3, fc2 leaves them in form 3).
extern "C" void ssam_mlp_tiles(int rows, int kept, int D, int Dm, int form, size_t split_bytes, int *tiles)
{
    alignas(16) unsigned char some;
    const SplitWs ws = { &some, split_bytes };
    tiles[0] = choose_fold_gelu(kept, Dm, D, GemmLd{ D, D, Dm }, rows, ws, form != 0).wide;
    tiles[1] = choose(kept, D, Dm, SSAM_EPI_BIAS_SCATTER_ADD, GemmLd{ Dm, Dm, D }, ws, true, form == 3 ? PARTS_LEFT : PARTS_NONE).wide;
}

namespace {

struct WarmBudget { int groups; double bytes; };

// Weights are read ahead by one workgroup for each CU without a tile, where there are a few; each gets what it can read in the time of the last round, the only one
// that it has no tile in (bytes a microsecond; half of it leaves weights of ViT-B's 240 tiles unread: 2 % of an encoder).  With the whole launch's time the reading ended behind
// the tiles of two rounds and more: eight blocks of ViT-H without reading, with that, now: row-major, five images of 60 x 60, density 0.4 4662 | 4820 | 4629 us, three of 44 x 44, 0.6
// 2018 | 2067 | 1957, packed, four of 40 x 40, 0.5 1879 | 1959 | 1868; 70 stacks with such launches 0.9 % faster than with the whole launch's time.
// Workgroups of padding rows, 16 rows of qkv at that rate, have the idle CUs first; counted as tiles they made qkv of ViT-L behind a global block, 256 tiles and 51 of those, a launch of two
// rounds with 205 idle CUs: 31.3 -> 32.9 us.
// More than 64 workgroups bring weights from HBM no sooner, and where the cache has them they are in the tiles' way: of 129 stacks of up to 2048 rows the 43 of ViT-B, whose weights
// stay there, were 0.5 % slower than without reading with as many as there are CUs (1.7 % at most), and are 0.1 % slower (1.2) with 64, all of them 0.4 % faster than with more; with 48 some
// weights are left to their contraction (four of 45 stacks slower by 3 to 4 %), with 32 such stacks are 2.5 % slower.
// A block by itself reads nothing ahead: called again on other tokens it finds its weights in the cache, and reading them once more cost 50 such blocks of 60 to 9000 rows 1.2 % (4 % at most).
// Only a stack knows of weights that no cache holds by their turn (stacks put together from calls of single blocks, 14 of ViT-B or ViT-L, would be 3.4 % faster with it).
// A stack reads whatever its size, since it does not know whether its last call's weights are still there: 40 stacks of 34 to 157 MB of weights are 5.0 % faster with it where they are not
// (0.4 % slower at most), 61 such stacks called again and again, and nothing else in between, 0.4 % slower (2.8 % at most: three blocks of ViT-H, 3 images of 28 x 28); ViT-B's 170 MB 0.5 %
// faster, more 1.9 %.  The launch that reads is itself slower by up to 0.8 us (fc1 of ViT-L), which is in all of these.  Its reading workgroups hold up to 64 CUs, each with a tile's LDS, for as
// long as a last round takes: a second stream's kernels find these taken.
WarmBudget warm_budget(int blocks, int tiles, int fills, double us)
{
    constexpr int FEWEST = 8, MOST = 64;
    constexpr double RATE = 30e3, FILL_US = 3.0;
    const int rounds = ssam_div_up(tiles, 256), idle = rounds * 256 - tiles;
    if (blocks < 2 || idle < FEWEST) return {};
    const double time = us / rounds - FILL_US * ssam_div_up(fills, idle);
    if (time <= 0.0) return {};
    const int groups = std::min(idle, MOST);
    return { groups, groups * RATE * time };
}

}  // namespace

GemmWarm WarmAhead::behind(int tiles, int fills, double us)
{
    const WarmBudget b = warm_budget(blocks, tiles, fills, us);
    return b.groups ? take(b.groups, b.bytes) : GemmWarm{};
}

// Its workgroups and the most bytes that they read, of any weights.  Host only, for tests; not part of the interface.
extern "C" int ssam_warm_budget(int blocks, int tiles, int fills, double us, double *bytes)
{
    const WarmBudget b = warm_budget(blocks, tiles, fills, us);
    *bytes = b.bytes;
    return b.groups;
}

// What a launch of `groups` workgroups without a tile reads: weights of the next contractions, no more than most_bytes, none twice.
GemmWarm WarmAhead::take(int groups, double most_bytes)
{
    GemmWarm out = {};
    if (next <= now) { next = now + 1; done = 0; }
    for (int s = 0; s < GEMM_WARM_AHEAD && next <= now + GEMM_WARM_AHEAD && next < 4 * blocks; ++s) {
        const ssam_block_weights &b = w[next / 4];
        const size_t mlp = (size_t)2 * D * Dm[is_global && is_global[next / 4]], sizes[4] = { (size_t)6 * D * D, (size_t)2 * D * D, mlp, mlp };
        const void *at[4] = { b.wqkv, b.wproj, b.w1, b.w2 };
        size_t bytes = std::min(sizes[next % 4] - done, (size_t)GEMM_WARM_PIECE);
        if ((double)bytes > most_bytes) bytes = (size_t)most_bytes & ~(size_t)8191;
        if (bytes == 0 || !at[next % 4] || !ssam_aligned16(at[next % 4])) break;      // (the contraction itself refuses such weights)
        out.at[s] = (const unsigned char *)at[next % 4] + done;
        out.bytes[s] = (uint32_t)bytes;
        out.groups = groups;
        most_bytes -= (double)bytes;
        done += bytes;
        if (done < sizes[next % 4]) break;
        ++next;
        done = 0;
    }
    return out;
}

// The pieces that the launch of contraction `launch` reads ahead with `groups` workgroups, after those of every contraction before it: their addresses and
// bytes.  Returns their number.  For tests.
int WarmAhead::pieces(int launch, int groups, double most_bytes, const void **at, uint32_t *bytes)
{
    GemmWarm out = {};
    for (now = 0; now <= launch; ++now) out = take(groups, most_bytes);
    int k = 0;
    for (; k < GEMM_WARM_AHEAD && out.bytes[k]; ++k) { at[k] = out.at[k]; bytes[k] = out.bytes[k]; }
    return out.groups == groups || k == 0 ? k : SSAM_EINVAL;
}

// The same of blocks of one kind.  Host only, for tests; not part of the interface.
extern "C" int ssam_warm_pieces(const ssam_block_weights *weights, int n_blocks, int D, int Dm, int now, int groups, double most_bytes, const void **at, uint32_t *bytes)
{
    return WarmAhead{ weights, nullptr, n_blocks, D, { Dm, Dm } }.pieces(now, groups, most_bytes, at, bytes);
}

// parts (optional): row statistics that a scatter-add leaves; the caller has asked ssam_parts_form_of.  With no place for them (at = NULL) only its tile is taken.
int ssam_linear_impl(const void *A, const void *W, const float *bias, void *C, int M, int N, int K,
                     const GemmLd &ld, bool packed, int epilogue, const GemmRowMap &rm, int tile,
                     void *split_ws, size_t split_ws_bytes, hipStream_t st, const GemmParts &parts, WarmAhead *warm)
{
    const SplitWs ws = { split_ws, split_ws_bytes };
    const bf16 *a = (const bf16 *)A, *w = (const bf16 *)W;
    bf16 *c = (bf16 *)C;
    int ring = -1;
    if (tile == 0) {
        const Choice pick = choose(M, N, K, epilogue, ld, ws, packed, parts.slots ? PARTS_LEFT : PARTS_NONE);
        tile = pick.tile;
        ring = pick.ring;
        if (const int wide = pick.wide; wide >= 0) {
            GemmFold out;
            out.parts = parts.at;
            out.slots = parts.slots;
            const GemmWideArgs args = { a, w, bias, c, M, N, K, ld, rm, out, st, warm, pick.us };
            switch (epilogue) {
            case SSAM_EPI_BIAS: return ssam_gemm_wide_bias(wide, packed, args);
            case SSAM_EPI_BIAS_GELU: return ssam_gemm_wide_gelu(wide, packed, args);
            case SSAM_EPI_BIAS_SCATTER_ADD: return parts.at ? ssam_gemm_wide_parts_add(wide, args) : ssam_gemm_wide_add(wide, packed, args);
            case SSAM_EPI_BIAS_SCATTER: return ssam_gemm_wide_scatter(wide, packed, args);
            default: return SSAM_EINVAL;
            }
        }
    }
    if (parts.slots) return SSAM_EUNSUPPORTED;
    if (packed) {
        switch (epilogue) {
        case SSAM_EPI_BIAS: return launch_any<SSAM_EPI_BIAS, true>(tile, ring, a, w, bias, c, M, N, K, ld, rm, ws, st);
        case SSAM_EPI_BIAS_GELU: return launch_any<SSAM_EPI_BIAS_GELU, true>(tile, ring, a, w, bias, c, M, N, K, ld, rm, ws, st);
        case SSAM_EPI_BIAS_SCATTER_ADD: return launch_any<SSAM_EPI_BIAS_SCATTER_ADD, true>(tile, ring, a, w, bias, c, M, N, K, ld, rm, ws, st);
        case SSAM_EPI_BIAS_SCATTER: return launch_any<SSAM_EPI_BIAS_SCATTER, true>(tile, ring, a, w, bias, c, M, N, K, ld, rm, ws, st);
        default: return SSAM_EINVAL;
        }
    }
    switch (epilogue) {
    case SSAM_EPI_BIAS: return launch_any<SSAM_EPI_BIAS, false>(tile, ring, a, w, bias, c, M, N, K, ld, rm, ws, st);
    case SSAM_EPI_BIAS_GELU: return launch_any<SSAM_EPI_BIAS_GELU, false>(tile, ring, a, w, bias, c, M, N, K, ld, rm, ws, st);
    case SSAM_EPI_BIAS_SCATTER_ADD: return launch_any<SSAM_EPI_BIAS_SCATTER_ADD, false>(tile, ring, a, w, bias, c, M, N, K, ld, rm, ws, st);
    case SSAM_EPI_BIAS_SCATTER: return launch_any<SSAM_EPI_BIAS_SCATTER, false>(tile, ring, a, w, bias, c, M, N, K, ld, rm, ws, st);
    default: return SSAM_EINVAL;
    }
}

// fc1 of the routed MLP with gather and LN2 folded in (see GemmFold): rows src[m] of A, packed folded weights,
// GELU epilogue, any M; the kernel is picked as for the plain contraction of the same shape (choose_fold_gelu), but in one layout only.  rows_a: rows of A.
// With parts (see ssam_parts_form_of) there are no stats, and src holds the rows of every batch of src_rows: row m / src_rows * src_stride + src[m] of A.
int ssam_linear_fold_gelu_impl(const void *A, long rows_a, const int32_t *src, const float *stats, const void *Wfp, const float *colsum,
                               const float *bias_f, void *C, int M, int N, int K, const GemmLd &ld,
                               void *split_ws, size_t split_ws_bytes, hipStream_t st, const GemmParts &parts, int src_rows, int src_stride, WarmAhead *warm)
{
    const SplitWs ws = { split_ws, split_ws_bytes };
    const GemmFold fold = { reinterpret_cast<const float2 *>(stats), colsum, src, parts.at, parts.slots, parts.eps, src_rows, src_stride };
    const GemmRowMap none = { nullptr, 1, 0, 1 };
    const auto [wide, tile, ring, us] = choose_fold_gelu(M, N, K, ld, rows_a, ws, parts.at != nullptr);
    if (parts.at) {
        const GemmWideArgs args = { (const bf16 *)A, (const bf16 *)Wfp, bias_f, (bf16 *)C, M, N, K, ld, none, fold, st, warm, us };
        if (wide >= 0) return ssam_gemm_wide_parts_gelu(wide, args);
        return large_reads_parts(K) ? ssam_gemm_large_parts_gelu(args, split_ws, split_ws_bytes) : SSAM_EUNSUPPORTED;
    }
    if (wide >= 0)
        return ssam_gemm_wide_ln_gelu(wide, GemmWideArgs{ (const bf16 *)A, (const bf16 *)Wfp, bias_f, (bf16 *)C, M, N, K, ld, none, fold, st, warm, us });
    if (ring >= 0)
        return launch_ring<SSAM_EPI_BIAS_GELU, true, true>(ring, (const bf16 *)A, (const bf16 *)Wfp, bias_f, (bf16 *)C, M, N, K, ld, none, fold, st);
    return launch_tile_packed<SSAM_EPI_BIAS_GELU, true>(tile, (const bf16 *)A, (const bf16 *)Wfp, bias_f, (bf16 *)C, M, N, K, ld,
                                                        none, ws, st, fold);
}

// Time of its large tiles: 512 workgroups a round, a last round of at most half of them at 0.62 of a round's time (as in pick_tile).
namespace {

double folded_ln_us(int tiles, int K)
{
    const double round = (K / GEMM_BK) * 1.71 + 5.5;
    const int last = tiles % 512;
    return large_tile_us(4, (tiles / 512) * round + (last == 0 ? 0.0 : last <= 256 ? 0.62 * round : round), true);
}

}  // namespace

// The contraction with the LayerNorm of its A rows folded in (see GemmFold): 128x256 tiles, packed weights,
// mapped store; M a multiple of 128 and N of 256, so there are no left-over tiles.  parts: instead of stats; with at = NULL the same kernel that would read
// them with stats (of ssam_ln_stats_impl as from pieces: the same bits).  Padding rows of `fill` are written behind the tiles of whatever reads pieces.
int ssam_linear_ln_impl(const void *A, const float *stats, const void *Wfp, const float *colsum, const float *bias_f,
                        void *C, int M, int N, int K, const GemmLd &ld, const GemmRowMap &rm, hipStream_t st, const GemmParts &parts, const PadFill &fill, WarmAhead *warm)
{
    constexpr size_t lds = gemm_lds_bytes<128, 256, 1, 4, true>();
    static_assert(lds <= 64 * 1024, "default LDS limit");
    GemmTileRange tr = { M / 128, N / 256, 0, (M / 128) * (N / 256) };
    const GemmFold fold = { reinterpret_cast<const float2 *>(stats), colsum, nullptr, parts.at, parts.slots, parts.eps, 1, 0, fill };
    const auto [wide, tile, ring, us] = choose_ln(M, N, K, ld, parts.slots != 0);
    const GemmWideArgs args = { (const bf16 *)A, (const bf16 *)Wfp, bias_f, (bf16 *)C, M, N, K, ld, rm, fold, st, warm, us };
    if (parts.at) {
        if (wide >= 0) return ssam_gemm_wide_parts_scatter(wide, args);
        return large_reads_parts(K) ? ssam_gemm_large_parts_scatter(args) : SSAM_EUNSUPPORTED;
    }
    if (wide >= 0) return ssam_gemm_wide_ln_scatter(wide, args);
    if (ring >= 0)
        return launch_ring<SSAM_EPI_BIAS_SCATTER, true, true>(ring, (const bf16 *)A, (const bf16 *)Wfp, bias_f, (bf16 *)C, M, N, K, ld, rm, fold, st);
    const int per_xcd = ssam_div_up(tr.tile_count, 8);
    hipLaunchKernelGGL((gemm_bf16_nt_lnf_kernel<128, 256, SSAM_EPI_BIAS_SCATTER, 1, 4>), dim3(per_xcd * 8), dim3(256), lds, st,
                       (const bf16 *)A, (const bf16 *)Wfp, bias_f, (bf16 *)C, M, N, K, ld, tr, rm, fold);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

extern "C" int ssam_linear_ln(const void *x, int ldx, const float *stats, const void *Wfp, const float *colsum,
                              const float *bias_f, void *C, int ldc, int M, int N, int K,
                              const int32_t *row_map, int rows_per_batch, int map_batch_stride, int dst_rows_per_batch,
                              void *stream)
{
    if (!x || !stats || !Wfp || !colsum || !bias_f || !C || !row_map || M <= 0 || N <= 0 || K <= 0) return SSAM_EINVAL;
    if (!ssam_aligned16(x) || !ssam_aligned16(Wfp) || !ssam_aligned16(colsum) || !ssam_aligned16(bias_f) || !ssam_aligned16(C) ||
        ((uintptr_t)stats & 7))
        return SSAM_EINVAL;
    if (ldx < K || ldc < N || ldx % 8 || ldc % 8 || rows_per_batch <= 0 || map_batch_stride < 0 || dst_rows_per_batch <= 0) return SSAM_EINVAL;
    if (M % 128 != 0 || N % 256 != 0 || K % GEMM_BK != 0) return SSAM_EUNSUPPORTED;
    const GemmRowMap rm = { row_map, rows_per_batch, map_batch_stride, dst_rows_per_batch };
    return ssam_linear_ln_impl(x, stats, Wfp, colsum, bias_f, C, M, N, K, GemmLd{ ldx, K, ldc }, rm, (hipStream_t)stream, GemmParts{}, PadFill{}, nullptr);
}

// The wide kernel's tile of fc1 with gather and LN2 folded in, its row statistics from a launch, or -1: the ring or the large tiles.  Host only, for tests; not part of the interface.
extern "C" int ssam_fold_gelu_wide_form(int rows, int kept, int D, int Dm)
{
    alignas(16) unsigned char some;
    return choose_fold_gelu(kept, Dm, D, GemmLd{ D, D, Dm }, rows, SplitWs{ &some, GEMM_SPLIT_WS_BYTES }, false).wide;
}

// Which kernel a contraction takes where the wide kernel does not (tile 0; `folded`: ssam_linear_ln): the large tile's id, or 16 + the ring's index (16: 128x128,
// 17: 128x64, 18: 64x64, 19: the direct one).  Host only, for tests; not part of the interface.
extern "C" int ssam_linear_form(int M, int N, int K, int epilogue, int packed, int folded, size_t workspace_bytes)
{
    if (M <= 0 || N <= 0 || K <= 0 || epilogue < 0 || epilogue > SSAM_EPI_BIAS_SCATTER) return SSAM_EINVAL;
    double us = folded_ln_us((M / 128) * (N / 256), K);
    int tile = 4;
    if (!folded) {
        alignas(16) unsigned char some;
        tile = pick_tile(M, N, K, epilogue, SplitWs{ workspace_bytes ? &some : nullptr, workspace_bytes }, packed != 0, us);
    }
    const int ring = pick_ring(M, N, K, packed != 0 || folded != 0, K % GEMM_BK == 0, us);
    return ring >= 0 ? 16 + ring : tile;
}

// The wide kernel's tile that the same contraction takes instead (its index in wide_tiles), or -1; _ld: with rows of lda and ldw elements.
extern "C" int ssam_linear_wide_form_ld(int M, int N, int K, int epilogue, int packed, int folded, size_t workspace_bytes, int lda, int ldw)
{
    if (M <= 0 || N <= 0 || K <= 0 || epilogue < 0 || epilogue > SSAM_EPI_BIAS_SCATTER || lda < K || ldw < K) return -1;
    double us = folded_ln_us((M / 128) * (N / 256), K);
    alignas(16) unsigned char some;
    const SplitWs ws = { workspace_bytes ? &some : nullptr, workspace_bytes };
    const bool whole_lines = lda % GEMM_BK == 0 && ldw % GEMM_BK == 0;
    if (!folded) pick_tile(M, N, K, epilogue, ws, packed != 0, us);
    const int ring = pick_ring(M, N, K, packed != 0 || folded != 0, folded != 0 || whole_lines, us);
    if (!folded) us += ring_gelu_us(ring, M, N, epilogue);
    return pick_wide(M, N, K, epilogue, GemmLd{ lda, ldw, N }, packed != 0 || folded != 0, 0, us,
                     folded ? us : other_layout_us(M, N, K, epilogue, ws, packed != 0, lda % GEMM_BK == 0));
}

extern "C" int ssam_linear_wide_form(int M, int N, int K, int epilogue, int packed, int folded, size_t workspace_bytes)
{
    return ssam_linear_wide_form_ld(M, N, K, epilogue, packed, folded, workspace_bytes, K, K);
}

extern "C" size_t ssam_linear_workspace_bytes(void) { return GEMM_SPLIT_WS_BYTES; }

__global__ void __launch_bounds__(256)
pack_weight_kernel(const bf16 *__restrict__ W, int ldw, bf16 *__restrict__ Wp, int N, int K)
{
    // one thread per 16-byte chunk of the packed matrix: chunk id = ((nb*ksteps + s)*64 + lane); lane = 16*quad + l
    // holds row 16*nb + l, k = 32*s + 8*quad .. + 7: the operand-b fragment of the 16x16x32 MFMA
    const long id = (long)blockIdx.x * 256 + threadIdx.x;
    const int ksteps = K / 32;
    if (id >= (long)(N / 16) * ksteps * 64) return;
    const int lane = (int)(id & 63), l = lane & 15, quad = lane >> 4;
    const long cell = id >> 6;
    const int ks = (int)(cell % ksteps), nb = (int)(cell / ksteps);
    reinterpret_cast<u32x4 *>(Wp)[id] = *reinterpret_cast<const u32x4 *>(W + (long)(16 * nb + l) * ldw + 32 * ks + 8 * quad);
}

extern "C" int ssam_pack_weight(const void *W, int ldw, void *Wp, int N, int K, void *stream)
{
    if (!W || !Wp || N <= 0 || K <= 0 || ldw < K || ldw % 8) return SSAM_EINVAL;
    if (!ssam_aligned16(W) || !ssam_aligned16(Wp)) return SSAM_EINVAL;
    if (N % 16 != 0 || K % 32 != 0) return SSAM_EUNSUPPORTED;
    const long chunks = (long)N * K / 8;
    hipLaunchKernelGGL(pack_weight_kernel, dim3((unsigned)ssam_div_up(chunks, 256)), dim3(256), 0, (hipStream_t)stream,
                       (const bf16 *)W, ldw, (bf16 *)Wp, N, K);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

extern "C" int ssam_linear_ld(const void *A, int lda, const void *W, int ldw, int w_packed, const float *bias, void *C, int ldc,
                              int M, int N, int K, int epilogue, const int32_t *row_map, int rows_per_batch,
                              int map_batch_stride, int dst_rows_per_batch, int tile,
                              void *workspace, size_t workspace_bytes, void *stream)
{
    if (!A || !W || !bias || !C || M <= 0 || N <= 0 || K <= 0) return SSAM_EINVAL;
    if (!ssam_aligned16(A) || !ssam_aligned16(W) || !ssam_aligned16(bias) || !ssam_aligned16(C)) return SSAM_EINVAL;
    if (N % 8 != 0 || K % 8 != 0) return SSAM_EUNSUPPORTED;
    if (w_packed && (N % 128 != 0 || K % GEMM_BK != 0)) return SSAM_EUNSUPPORTED;
    if (lda < K || ldc < N || lda % 8 || ldc % 8 || (!w_packed && (ldw < K || ldw % 8))) return SSAM_EINVAL;
    if (workspace && !ssam_aligned16(workspace)) return SSAM_EINVAL;
    if (tile < 0 || tile > 4) return SSAM_EINVAL;
    if (w_packed && tile == 2) return SSAM_EUNSUPPORTED;
    GemmRowMap rm = { nullptr, 1, 0, 1 };
    if (epilogue == SSAM_EPI_BIAS_SCATTER_ADD || epilogue == SSAM_EPI_BIAS_SCATTER) {
        if (!row_map || rows_per_batch <= 0 || map_batch_stride < 0 || dst_rows_per_batch <= 0) return SSAM_EINVAL;
        rm = { row_map, rows_per_batch, map_batch_stride, dst_rows_per_batch };
    } else if (epilogue != SSAM_EPI_BIAS && epilogue != SSAM_EPI_BIAS_GELU) {
        return SSAM_EINVAL;
    }
    GemmLd ld = { lda, ldw, ldc };
    return ssam_linear_impl(A, W, bias, C, M, N, K, ld, w_packed != 0, epilogue, rm, tile, workspace, workspace ? workspace_bytes : 0,
                            (hipStream_t)stream, GemmParts{}, nullptr);
}

extern "C" int ssam_linear_tiled(const void *A, const void *W, const float *bias, void *C, int M, int N, int K,
                                 int epilogue, const int32_t *row_map, int rows_per_batch, int map_batch_stride,
                                 int dst_rows_per_batch, int tile, void *stream)
{
    return ssam_linear_ld(A, K, W, K, 0, bias, C, N, M, N, K, epilogue, row_map, rows_per_batch, map_batch_stride,
                          dst_rows_per_batch, tile, nullptr, 0, stream);
}

extern "C" int ssam_linear(const void *A, const void *W, const float *bias, void *C, int M, int N, int K,
                           int epilogue, const int32_t *row_map, int rows_per_batch, int map_batch_stride,
                           int dst_rows_per_batch, void *stream)
{
    return ssam_linear_ld(A, K, W, K, 0, bias, C, N, M, N, K, epilogue, row_map, rows_per_batch, map_batch_stride,
                          dst_rows_per_batch, 0, nullptr, 0, stream);
}
