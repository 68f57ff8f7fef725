// Stripe-Sort attention (App. A.1, Alg. 1) for gfx950: block-sparse, flash-style
// attention over the static A-shape tile mask, with SAM's decomposed 2-D
// relative-position bias fused in.  Tokens arrive in scan order; sigma maps a
// scan position to its spatial cell for the bias lookup.
//
// Formulation.  Scores are computed transposed, S^T = K Q^T, on the 32x32x16 bf16
// MFMA: the Q fragments (operand b) stay in registers for the whole problem, K
// rows come from LDS (operand a).  In the result layout every lane owns ONE
// query (column l & 31) and 16 of the 32 keys of a block, so the softmax row
// statistics are per-lane scalars: the row maximum needs a single exchange with
// lane l^32, the row sum none until the end.  exp(S^T) converted to bf16 is
// already in the operand-b layout of the second product O^T = V^T P^T.  Its
// operand-a fragments (8 keys of one feature column per lane, in the key order
// the result layout dictates: contraction slot e of half-wave hf of MFMA t <->
// key 16t + 8(e/4) + 4hf + (e&3)) come from the row-major V rows in LDS through
// the transposing LDS read of gfx950 (ds_read_b64_tr_b16: a 16-lane group reads
// 4 rows x 16 columns and every lane receives one column), so V is staged
// exactly like K and never transposed in memory.
// Key blocks (32 keys) are processed in chunks of one (window kernels) or as many as the register budget of
// two waves per SIMD allows (two to four; above 64 x 64): all score MFMAs of the chunk first, one max and, where the reference moves,
// one rescale of the running output per chunk, then all P V MFMAs; up to 64 x 64 the global kernel interleaves three blocks instead.
// Bias: per wave, U = Q R^T is formed once with the MFMA for both tables and kept in LDS as fp16, query-major.  A score gets
// its two entries as a product with the table in the scores' accumulator: of one 16-entry operand on orders whose
// blocks are patches, of the whole row of up to 64 entries a table on others (AttnPipe) or of 16 (windows,
// attn_window_step); above 64 x 64 by two look-ups.
// Memory requests are spread over a problem's / a tile's phases (see the prefetch
// macros): a wave whose loads do not fit the CU's request queues waits instead of
// computing, and a wait placed behind a branch or on a value that is used at once
// drains every load and store in flight.
//
// Three launch shapes:
//   window kernel, a wave to a query tile: one-wave workgroups, each walks the active key blocks of its tile by itself
//                  (few problems or tiles at d = 80, nearly all below);
//   window kernel, persistent (window_waves_most): workgroups looping over (window, head) problems, one
//                  wave per 32-query tile (= mask tile of 32), the window's whole K
//                  and V in LDS, the next problem's K and V prefetched into registers
//                  and its Q straight into LDS, in three pieces, the rel-pos tables
//                  resident in LDS;
//   global kernel: one workgroup per (128-query mask tile, image, head), 4 waves, two or
//                  more workgroups per CU; active key blocks go straight into rings in LDS, or, above
//                  64 x 64 off the patch path, active 128-key tiles through registers into LDS (K and V
//                  requested at different points).
#include <type_traits>

#include "common.h"

namespace {

constexpr float LOG2E = 1.4426950408889634f;

struct AttnParams {
    const bf16 *q, *k, *v;
    long row_stride;
    const bf16 *rel_h, *rel_w;
    const int32_t *sigma;
    long sigma_stride;      // elements between the sigma tables of consecutive groups; 0 = one shared table
    bf16 *out;
    const int32_t *out_rows;   // NULL: query p of group g goes to output row g*S+p; else to out_rows[g*S+p] (-1: dropped)
    int S, w, h, n_pre;
    float scale_log2e;
    uint32_t half_one;      // see bias_shift: 2^shift in fp16
    float table_one;        // and in fp32
    float table_inv;        // what turns a bias into an entry: 1 / (scale * 2^shift)
    int q_exp;              // windows: the scores are formed with q * 2^q_exp (see window_scale); scale is that of these scores
};

template <int D>
struct AttnCfg {
    static constexpr int KS = D / 16;            // k-steps of the score product
    static constexpr int DT = (D + 31) / 32;     // 32-row tiles of O^T
    static constexpr int KSTR = D + 8;           // row stride in LDS (elements): odd in 16-byte units
    static constexpr int CH = D / 8;             // 16-byte chunks per row
    // D = 16 mod 32: the last 32-row tile of O^T has 16 rows to spare and the LDS rows of V have 8 columns of
    // padding; with ones in that padding those rows come out of the P V product as the sum of the probabilities,
    // which the softmax then does not have to add up on the vector unit
    static constexpr bool ONES = D % 32 == 16;
};

// fill the padding columns of `rows` LDS rows of V with 1.0 (they are never written afterwards: tile stores cover
// the D real columns only)
template <int D>
__device__ __forceinline__ void set_ones_columns(bf16 *Vs, int rows, int tid, int nthreads)
{
    if constexpr (AttnCfg<D>::ONES) {
        const u32x4 ones = { 0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u };
        for (int p = tid; p < rows; p += nthreads) *reinterpret_cast<u32x4 *>(Vs + p * AttnCfg<D>::KSTR + D) = ones;
    }
}

// LDS is in order per wave: this keeps the compiler from reordering what its lanes exchange through it
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Per-wave softmax/output state for 32 queries (one per lane pair l, l^32).
template <int D>
struct WaveState {
    f32x16 o[AttnCfg<D>::DT];
    float m, l;
};

template <int D>
__device__ __forceinline__ void init_state(WaveState<D> &st)
{
#pragma unroll
    for (int dt = 0; dt < AttnCfg<D>::DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) st.o[dt][r] = 0.f;
    st.m = -INFINITY;
    st.l = 0.f;
}

// Bias table of the wave's 32 queries in the global kernel, query-major, fp16 (see GlbTab), divided by the softmax
// scale so that (score + row entry + column entry) * scale * log2e is the logit in log2 units.  General path:
//   tq[q*tstr + p]                            = q . rel_h[row(q)-p+w-1] / scale      (p = key row)
//   tq[q*tstr + wk + p]                       = q . rel_w[col(q)-p+w-1] / scale      (p = key column)
// Up to w = 64 wk is w rounded up to whole 32-entry operands (32 or 64), the entries past w zero, and tstr = 2*wk + 8: the 16 bytes
// of padding put the operand reads of 16 lanes on distinct banks.  Above, where entries are looked up one by one, wk is w
// rounded up to even and tstr = 2*wk + 4: 8 bytes of padding put the 32 lanes of a look-up (one entry, 32 queries) on
// distinct banks.  Patch path (w a power of two):
//   tq[q*tstr + (p&1)*hw + (p>>1)]            row entries,    tq[q*tstr + 2*hw + (p&1)*hw + (p>>1)]   column entries
// hw = w/2: even and odd rows (columns) are stored apart, so that rows two apart are neighbours: the 32-key
// blocks of the position-only Stripe-Sort order are 4 x 8 patches of stride 2 (see attn_patch_body), whose 4 row
// and 8 column entries are then contiguous.  tstr = 4*hw + 4: the 8 bytes of padding put the 32 lanes of a look-up
// (one entry, 32 queries) on distinct banks.  tq_lane: this lane's query row.  rel tables: rows of `rstr` elements.
//
// Range.  Where the bias is added as the product of a 0/1 matrix and the table (attn_window_step, AttnPipe) every entry
// meets every key, most of them as a zero, and an infinity would make NaNs of the query's whole row.  So
//   * entries past the range of fp16 become +-65504 (clamp_fp16), which as a logit is 65504 * scale, and
//   * with a small scale the table is 2^shift times smaller and the ones of that matrix, or what a looked-up entry is multiplied
//     by, are 2^shift: shift is the least that puts 65504 * 2^shift * scale past 128 (bias_shift), since exp(-128) is the "no
//     weight" that such a bias asks for.
inline int bias_shift(float scale)
{
    int n = 0;
    while (n < 15 && ldexpf(65504.f / 128.f * scale, n) < 1.f) ++n;
    return n;
}
// Windows.  An entry of 1 is scale * 2^n * log2 e units of a logit in powers of two, by the choice of n at least 1 (the range of such
// units: +-45400 as a logit) and below 512 (the spacing of the smallest entries is then 2^-15 of one; with n = 0 at a scale
// of 1e6 a bias of 0.01 was 0), and n is 0 where it can be, from a scale of 0.7 to 350.  Ones of fp16 hold 2^-14 to 2^15; past those, below
// a scale of 2e-5 and above 5e6, the rest goes into the queries, as a power of two that rounds nothing.
struct WindowScale { int shift, q_exp; };
inline WindowScale window_scale(float scale)
{
    const double unit = (double)scale * 1.4426950408889634;
    int e, n = 0;
    if (!(unit < HUGE_VAL)) return { 0, 0 };
    frexp(unit, &e);                       // unit = 2^(e - 1) up to 2^e
    if (e < 1) n = 1 - e;
    else if (e > 9) n = 9 - e;
    const int shift = n < -14 ? -14 : n > 15 ? 15 : n;
    return { shift, shift - n };
}
// bit 23 of the mode register: fp16 results past the range are clamped instead of rounded to infinity
__device__ __forceinline__ void clamp_fp16() { __builtin_amdgcn_s_setreg(1 | 23 << 6 | (1 - 1) << 11, 1); }

__host__ __device__ inline int glb_tstr(int w) { return 4 * ((w + 1) >> 1) + 4; }
// Entries per table of the operand form (AttnPipe), 0: look-ups.  Two images of 50 x 50, d = 80: 111 us by look-up, 88 by dense operands (sparse
// ones: see attn_onehot_body); of 72 x 72, where dense operands took 96 or 128 entries and their table a second workgroup's LDS: d = 64 264
// against 434, d = 80 428 against 500.
__host__ __device__ inline int glb_operand(int w) { return w <= 32 ? 32 : w <= 64 ? 64 : 0; }
__host__ __device__ inline int glb_wk(int w) { return glb_operand(w) ? glb_operand(w) : (w + 1) & ~1; }
__host__ __device__ inline int glb_general_tstr(int w) { return 2 * glb_wk(w) + 4; }        // of the look-ups

template <int D, typename TabT>
__device__ __forceinline__ void build_bias_rows(const bf16x8 *qf, const bf16 *rel_h, const bf16 *rel_w, int rstr,
                                                int w, int qrow, int qcol, TabT *tq_lane, float inv_scale)
{
    constexpr int KS = AttnCfg<D>::KS;
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    const int nrel = 2 * w - 1, wk = glb_wk(w);
    for (int p = w + half; p < wk; p += 2) tq_lane[p] = tq_lane[wk + p] = (TabT)0.f;      // (the two half-waves share a query)
    // operand a of slab mt: rows mt*32 + l32 of both tables; rows past the table re-read its last row (their
    // products are never stored), so every load is unconditional and a slab's 2*KS loads are in flight together
    bf16x8 cur[2][KS], nxt[2][KS];
    auto load_slab = [&](bf16x8 (&a)[2][KS], int mt) {
        const int mrow = min(mt * 32 + l32, nrel - 1);
#pragma unroll
        for (int tab = 0; tab < 2; ++tab)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                a[tab][ks] = *reinterpret_cast<const bf16x8 *>((tab ? rel_w : rel_h) + (long)mrow * rstr + ks * 16 + half * 8);
    };
    load_slab(cur, 0);
    for (int mt = 0; mt * 32 < nrel; ++mt) {
        // requested before this slab's products, used after them; past the last slab it re-reads the last row:
        // an unconditional request keeps the wait below counted (a branch here would force a full drain)
        load_slab(nxt, mt + 1);
#pragma unroll
        for (int tab = 0; tab < 2; ++tab) {
            f32x16 u;
#pragma unroll
            for (int r = 0; r < 16; ++r) u[r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) u = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur[tab][ks], qf[ks], u, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");          // MFMA passes done before u is read under predicates
            __builtin_amdgcn_sched_barrier(0);
            // entry of relative position m = mt*32 + 8*(r>>2) + 4*half + (r&3); positions past the table (m > 2w-2) would be negative ones
            const int p0 = (tab ? qcol : qrow) + (w - 1) - mt * 32 - 4 * half;
            TabT *dst = tq_lane + (tab ? wk : 0) + p0;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int d = 8 * (r >> 2) + (r & 3);
                if ((unsigned)(p0 - d) < (unsigned)w) dst[-d] = (TabT)(u[r] * inv_scale);
            }
        }
#pragma unroll
        for (int tab = 0; tab < 2; ++tab)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) cur[tab][ks] = nxt[tab][ks];
    }
}

typedef _Float16 WinTab;
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x16 __attribute__((ext_vector_type(16)));
// Bias operands of the window kernels (attn_window_step): entry p of the lane's query (p = key row, or 16 + key column) at
// tq[(l & 31) * WIN_OSTR + p], divided by the softmax scale (AttnParams::table_inv); those past w are zero.  A window has 2w-1 <= 32
// relative positions, so rel x Q^T is one MFMA tile per table.  It is stored the way it leaves the matrix core, query-major, and
// entry p read back as position q - p + w - 1: predicated stores of the entries to their places, as for larger grids, cost two to three times as much.
// rel(tab, ks): fragment ks of the lane's row l & 31 of rel_h (tab 0) or rel_w (1), elements 16*ks + 8*(l >> 5) .. + 7.
constexpr int WIN_TSTR = 36;             // row of a product: 8-byte stores aligned, and 32 lanes at one entry on distinct banks
constexpr int WIN_OSTR = 40;             // row of operands: 2 * 16 entries; reads of 16 bytes aligned, and 16 lanes on distinct banks
template <int D, typename Rel>
__device__ __forceinline__ void build_bias_operands_window(const bf16x8 *qf, Rel rel, int w, int qrow, int qcol, WinTab *tq, float inv_scale)
{
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    u32x4 keep, t[2];                    // this half-wave's entries 8*half .. + 7 that are below w
#pragma unroll
    for (int e = 0; e < 4; ++e) keep[e] = (8 * half + 2 * e < w ? 0xffffu : 0u) | (8 * half + 2 * e + 1 < w ? 0xffff0000u : 0u);
#pragma unroll
    for (int tab = 0; tab < 2; ++tab) {
        f32x16 u;
#pragma unroll
        for (int r = 0; r < 16; ++r) u[r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < AttnCfg<D>::KS; ++ks)
            u = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rel(tab, ks), qf[ks], u, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");          // MFMA passes done before u is read (as in build_bias_rows)
        __builtin_amdgcn_sched_barrier(0);
        WinTab *row = tq + l32 * WIN_TSTR;                            // u[4g + e] is rel row 8g + 4*half + e of query l32
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            f16x4 hv = { (_Float16)(u[4 * g] * inv_scale), (_Float16)(u[4 * g + 1] * inv_scale),
                         (_Float16)(u[4 * g + 2] * inv_scale), (_Float16)(u[4 * g + 3] * inv_scale) };
            *reinterpret_cast<f16x4 *>(row + 4 * half + 8 * g) = hv;
        }
        wave_lds_fence();
        // up to 15 entries in front of the row for p past w: LDS of this workgroup, and not kept
        const WinTab *at = row + ((tab ? qcol : qrow) + w - 1 - 8 * half);
        f16x8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = at[-e];
        t[tab] = __builtin_bit_cast(u32x4, v) & keep;
        wave_lds_fence();
    }
#pragma unroll
    for (int tab = 0; tab < 2; ++tab) *reinterpret_cast<u32x4 *>(tq + l32 * WIN_OSTR + tab * 16 + half * 8) = t[tab];
    wave_lds_fence();
}

// A chunk of nb (1..NB, wave-uniform) 32-key blocks against the wave's 32 queries.
//   Ks, Vs: LDS, row-major rows ([keys][KSTR]); blk[b]: index of the chunk's b-th block in them
//   krc:    LDS, per key two byte offsets into the query's table row, indexed like Ks: low half for the row part,
//           high half for the column part (see build_bias_rows)
//   key0[b]: scan position of the block's first key (for the S bound; RAGGED = the chunk crosses S)
//   tq_h, tq_w: where this lane's query starts in the row-part and column-part bias tables; a key's two
//           bias terms are read at tq_h + (low half of krc) and tq_w + (high half of krc), in bytes
// The tables hold bias / (scale * one) and the scores stay unscaled: logit = (s + (bh + bw) * one) * scale_log2e.
constexpr float ATTN_LAG = 8.f;

// Second half of a chunk step, the same for every way of forming the scores: s holds the chunk's logits before
// the multiplication by scale_log2e, mx their maximum over this lane's keys, in the same units.
// FULL: the chunk has all NB blocks (nb is not looked at: no per-block branches, no dummy scores)
template <int D, int NB, bool FULL>
__device__ __forceinline__ void attn_softmax_pv(WaveState<D> &st, f32x16 (&s)[NB], float mx, const bf16 *Vs,
                                                const int (&blk)[NB], int nb_, float scale_log2e)
{
    using C = AttnCfg<D>;
    const int nb = FULL ? NB : nb_;
    const int lane = threadIdx.x & 63, half = lane >> 5;
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    mx *= scale_log2e;
    // st.m is the exponent reference of the running sums, not the running maximum: it moves only when a chunk's
    // maximum exceeds it by more than 2^ATTN_LAG, so probabilities stay below 2^ATTN_LAG (all of a query's terms
    // carry the same power of two, which the final division removes) and the rescaling of the 32 x D accumulator
    // is skipped by the whole wave in most chunks.  First chunk: st.m = -inf, every lane moves, alpha = 0.
    const bool move = mx > st.m + ATTN_LAG;
    if (__builtin_amdgcn_ballot_w64(move) != 0) {
        const float mnew = move ? mx : st.m;
        const float alpha = __builtin_amdgcn_exp2f(st.m - mnew);
        st.m = mnew;
        if constexpr (!C::ONES) st.l *= alpha;
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) st.o[dt][r] *= alpha;
    }
    const float mref = st.m;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (b < nb) {
#pragma unroll
            for (int r = 0; r < 16; ++r) s[b][r] = __builtin_amdgcn_exp2f(fmaf(s[b][r], scale_log2e, -mref));
        }
    }
    // transposing read: lane li of a 16-lane group points at row (li >> 2), column chunk (li & 3) of a
    // 4-key x 16-feature block and receives the 4 keys of feature column li
    const int li = lane & 15, fblk = (lane >> 4) & 1;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (b < nb) {
            const bf16 *vblk = Vs + blk[b] * 32 * C::KSTR + (4 * half + (li >> 2)) * C::KSTR;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                bf16x8 p;
#pragma unroll
                for (int e = 0; e < 8; ++e) p[e] = (bf16)s[b][8 * t + e];
                if constexpr (!C::ONES) {
                    // the sum of what P V multiplies, the rounded probabilities, as with the ones columns: the rounding of a dominant
                    // one cancels (with sums of the unrounded ones the error is 1-2 % larger where one key dominates)
#pragma unroll
                    for (int e = 0; e < 8; e += 2) {
                        const bf16x2 pair = { p[e], p[e + 1] };
                        st.l = __builtin_amdgcn_fdot2_f32_bf16(pair, bf16x2{ (bf16)1.f, (bf16)1.f }, st.l, false);
                    }
                }
#pragma unroll
                for (int dt = 0; dt < C::DT; ++dt) {
                    int col = dt * 32 + 16 * fblk + 4 * (li & 3);
                    // feature columns past D re-read the last ones and their outputs are dropped; with ONES they are
                    // the ones columns D .. D+7, and their outputs are the sums of the probabilities
                    constexpr int CMAX = C::ONES ? D + 4 : D - 4;
                    col = col <= CMAX ? col : CMAX;
                    const bf16 *v0p = vblk + 16 * t * C::KSTR + col;
                    bf16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4 *)(v0p));
                    bf16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4 *)(v0p + 8 * C::KSTR));
                    bf16x8 a = { v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3] };
                    st.o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, p, st.o[dt], 0, 0, 0);
                }
            }
        }
    }
}

template <int D, int NB, bool RAGGED, typename TabT>
__device__ __forceinline__ void attn_chunk_step(WaveState<D> &st, const bf16x8 *qf, const bf16 *Ks, const bf16 *Vs,
                                                const uint32_t *krc, const int (&blk)[NB], const int (&key0)[NB], int nb,
                                                int S, float scale_log2e, const TabT *tq_h, const TabT *tq_w, float one)
{
    using C = AttnCfg<D>;
    static_assert(sizeof(TabT) == 2, "bias tables are fp16");
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    f32x16 s[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (b < nb) {
            const bf16 *kblk = Ks + blk[b] * 32 * C::KSTR + l32 * C::KSTR + half * 8;
            const f32x16 zero = { 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f };
#pragma unroll
            for (int ks = 0; ks < C::KS; ++ks) {
                bf16x8 a = *reinterpret_cast<const bf16x8 *>(kblk + ks * 16);
                s[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[ks], ks == 0 ? zero : s[b], 0, 0, 0);
            }
        }
    }
    // the score MFMAs sit behind wave-uniform branches (b < nb): wait their passes out before the reads
    // (the compiler's hazard handling is only relied upon within straight-line code; see the GEMM epilogue)
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    float mx = -INFINITY;                    // the chunk's own maximum
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (b < nb) {
            const unsigned char *tqh = reinterpret_cast<const unsigned char *>(tq_h);
            const unsigned char *tqw = reinterpret_cast<const unsigned char *>(tq_w);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if (RAGGED && key0[b] + 8 * g >= S) {      // all eight keys of this register group lie past S (wave-uniform)
#pragma unroll
                    for (int e = 0; e < 4; ++e) s[b][4 * g + e] = -INFINITY;
                    continue;
                }
                const u32x4 rc = *reinterpret_cast<const u32x4 *>(krc + blk[b] * 32 + 8 * g + 4 * half);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int r = 4 * g + e;
                    const uint32_t c = rc[e];
                    const float bh = (float)*reinterpret_cast<const TabT *>(tqh + (c & 0xffffu));
                    const uint32_t bw16 = *reinterpret_cast<const uint16_t *>(tqw + (c >> 16));
                    // the column part in one mixed-precision fma (fp16 operand widened inside the instruction)
                    float val = fmaf(bh, one, s[b][r]);
                    asm("v_fma_mix_f32 %0, %1, %3, %2 op_sel_hi:[1,0,0]" : "=v"(val) : "v"(bw16), "v"(val), "s"(one));
                    if (RAGGED) val = (key0[b] + 8 * g + 4 * half + e < S) ? val : -INFINITY;
                    s[b][r] = val;
                    mx = fmaxf(mx, val);
                }
            }
        }
    }
    attn_softmax_pv<D, NB, false>(st, s, mx, Vs, blk, nb, scale_log2e);
}

// Patches: scores of 32-key blocks that are 4 x 8 patches of stride 2 in the grid: key k of a block (bits c0 r1'.. in
// scan order: bit 0 and bits 2, 4 count columns, bits 1 and 3 rows, i.e. a Z-order walk) sits 2*rr(k) rows and 2*cc(k)
// columns from the block's first key.  That is how the position-only Stripe-Sort order (Sec. 4.1: Z-order, then the
// stripe interleave with G = 4, which collects the cells of one row and column parity) lays out a power-of-two grid.
// The decomposed bias of such a block is a product: B[k][q] = sum_f E[k][f] T[f][q] with E the 0/1 matrix that
// picks a key's row entry (f = rr) and column entry (f = 4 + cc) and T the 4 row and 8 column entries of every
// query, which are contiguous in the query's table row (build_bias_rows).  So the bias is ONE more MFMA (fp16
// operands, the same fp32 accumulator, issued first) and the vector unit does no look-ups and no additions.
// row and column steps (in units of 2 cells) of key k of a patch block from the block's first key
__device__ __forceinline__ int patch_rr(int k) { return ((k >> 1) & 1) | ((k >> 2) & 2); }
__device__ __forceinline__ int patch_cc(int k) { return (k & 1) | ((k >> 1) & 2) | ((k >> 2) & 4); }

// A block of 32 keys of a window, in any order, against the wave's 32 queries, with the decomposed bias as a product too: B[k][q] = sum_p E[k][p] T[p][q],
// where E has a one at the key's row and a one at its column and T is the query's table row, 16 entries each.  One sparse product (fp16
// operands, the same fp32 accumulator, issued last: its result cannot begin at a constant; see AttnPipe::describe): the lower half-wave makes the rows' part of E, the upper one the
// columns'.  Two look-ups per score instead cost 32 LDS reads and 80 vector instructions per block.
template <int D, bool RAGGED>
__device__ __forceinline__ void attn_window_step(WaveState<D> &st, const bf16x8 *qf, const bf16 *Ks, const bf16 *Vs, const uint32_t *krc, int blk, int key0,
                                                 int S, float scale_log2e, const _Float16 *tq_lane, uint32_t half_one)
{
    using C = AttnCfg<D>;
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    const uint32_t rc = krc[blk * 32 + l32], at = half ? rc >> 16 : rc & 0xffffu, i = at & 3u;               // row | column << 16
    const uint32_t one = i == 3 ? half_one << 16 : half_one, index = i == 3 ? 0xccccu : 0xccccu + i * 0x1111u;
    u32x4 e;
#pragma unroll
    for (int j = 0; j < 4; ++j) e[j] = at >> 2 == (uint32_t)j ? one : 0u;
    // operand b: entries 8 * half .. + 7 of the rows and of the columns; the same for every block, and read again all the same (kept in registers they spill)
    uint32_t fresh = 0;
    asm volatile("" : "+v"(fresh));
    const f16x8 lo = *reinterpret_cast<const f16x8 *>(tq_lane + fresh + half * 8), hi = *reinterpret_cast<const f16x8 *>(tq_lane + fresh + 16 + half * 8);
    const f16x16 t = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
    const f32x16 zero = { 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f };
    f32x16 s[1];
    const bf16 *kblk = Ks + blk * 32 * C::KSTR + l32 * C::KSTR + half * 8;
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks) {
        bf16x8 a = *reinterpret_cast<const bf16x8 *>(kblk + ks * 16);
        s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[ks], ks == 0 ? zero : s[0], 0, 0, 0);
    }
    s[0] = __builtin_amdgcn_smfmac_f32_32x32x32_f16(__builtin_bit_cast(f16x8, e), t, s[0], (int)index, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");          // MFMA passes done before the scores are read (as in attn_chunk_step)
    __builtin_amdgcn_sched_barrier(0);
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        if (RAGGED) s[0][r] = key0 + 8 * (r >> 2) + 4 * half + (r & 3) < S ? s[0][r] : -INFINITY;
        mx = fmaxf(mx, s[0][r]);
    }
    const int blks[1] = { blk };
    attn_softmax_pv<D, 1, true>(st, s, mx, Vs, blks, 1, scale_log2e);
}

template <int D>
__device__ __forceinline__ void load_q_frags(bf16x8 *qf, const bf16 *qrow)
{
    const int half = (threadIdx.x & 63) >> 5;
#pragma unroll
    for (int ks = 0; ks < AttnCfg<D>::KS; ++ks)
        qf[ks] = *reinterpret_cast<const bf16x8 *>(qrow + ks * 16 + half * 8);
}

// The wave's queries times 2^e (window_scale); what would overflow becomes the largest number, so that a zero key still gives 0.
template <int D>
__device__ __forceinline__ void scale_queries(bf16x8 *qf, int e)
{
    constexpr float MOST = 3.3895313892515355e38f;        // of bf16
#pragma unroll
    for (int ks = 0; ks < AttnCfg<D>::KS; ++ks)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float x = (float)qf[ks][i], y = ldexpf(x, e);
            if (fabsf(x) < INFINITY) qf[ks][i] = (bf16)fminf(fmaxf(y, -MOST), MOST);
        }
}

// Normalise the wave's 32 x D output tile and write it out.  The accumulators hold O^T (lane = query,
// registers = 4-feature groups); the tile goes through a per-wave LDS staging area ([32][STR] bf16) so
// that the global stores are 16 bytes per lane and cover whole rows.  `stage` may overlay LDS that only
// this wave used (its bias rows).  out_head: the output tensor at this head's columns; my_row: the output
// row of this lane's query (l & 31), negative = not stored (past S, or dropped by the row map).
template <int D, int STR = AttnCfg<D>::KSTR, bool ONES = AttnCfg<D>::ONES>
__device__ __forceinline__ void finish_and_store(WaveState<D> &st, bf16 *stage, bf16 *out_head, long out_stride, long my_row)
{
    using C = AttnCfg<D>;        // STR: row stride of the staging area in elements
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    // the last P V MFMAs may still be in flight and this point is reached through loop-exit branches:
    // wait their passes out explicitly before the accumulators are read (see the GEMM epilogue)
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    // ONES: row 16 + 4*half of the last tile of O^T is a ones column's output: the whole sum, in both half-waves
    const float l = ONES ? st.o[C::DT - 1][8] : st.l + __shfl_xor(st.l, 32, 64);
    const float inv = 1.0f / l;
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            int dd = dt * 32 + 8 * g + 4 * half;
            if (dd < D) {
                uint2 pk;
                pk.x = pack_bf16x2(st.o[dt][4 * g + 0] * inv, st.o[dt][4 * g + 1] * inv);
                pk.y = pack_bf16x2(st.o[dt][4 * g + 2] * inv, st.o[dt][4 * g + 3] * inv);
                *reinterpret_cast<uint2 *>(stage + l32 * STR + dd) = pk;
            }
        }
    wave_lds_fence();
    const int row_lo = (int)my_row, row_hi = (int)(my_row >> 32);
#pragma unroll
    for (int i = 0; i < (32 * C::CH + 63) / 64; ++i) {
        int id = lane + 64 * i, row = id / C::CH, c = id % C::CH;
        row = row < 32 ? row : 31;
        const long orow = ((long)__shfl(row_hi, row, 64) << 32) | (unsigned)__shfl(row_lo, row, 64);   // lane `row` holds query `row`
        if (id < 32 * C::CH && orow >= 0) {
            u32x4 v = *reinterpret_cast<const u32x4 *>(stage + row * STR + c * 8);
            *reinterpret_cast<u32x4 *>(out_head + orow * out_stride + c * 8) = v;
        }
    }
}

__device__ __forceinline__ uint32_t cell_row_col(int cell, int w)
{
    cell = min(max(cell, 0), w * w - 1);
    return (uint32_t)(cell / w) | ((uint32_t)(cell % w) << 16);
}

__device__ __forceinline__ uint32_t key_row_col(const int32_t *sigma, int p, int S, int w)
{
    return cell_row_col(sigma[p < S ? p : S - 1], w);
}

// per-wave LDS scratch of the global kernel: the bias table of its 32 queries (rows of tstr fp16), later overlaid by
// its output staging tile
template <int D>
__host__ __device__ inline int wave_scratch_bytes(int tstr)
{
    int bias = 32 * tstr * 2, stage = 32 * AttnCfg<D>::KSTR * 2;
    return ((bias > stage ? bias : stage) + 15) & ~15;
}

// ------------------------------------------------------------------ window kernel, persistent
// The bias as a product (two MFMAs a block, operands built once a tile) instead of 32 LDS look-ups and 80 vector instructions a block: 16 heads, d = 80,
// 800 problems 34.2 -> 32.4 us at r = 0.4, 51.1 -> 45.7 dense; 3200: 99.6 -> 96.5 and 154.8 -> 137.3.
// One sparse product instead of two dense ones: 3200 problems 98.4 -> 95.6 and 142.7 -> 138.6 on another card; a wave to a tile, d = 64, 1600 problems 38.3 -> 37.8.
inline int window_rel_rows(int w) { return ((2 * w - 1 + 31) / 32) * 32; }

// per-wave LDS landing area of the next problem's queries: the KS operand-b fragments of the wave's 32 queries
template <int D>
__host__ __device__ constexpr int window_q_bytes() { return AttnCfg<D>::KS * 1024; }

// LDS of a gfx950 compute unit.  A compile-time layout choice below is made for it; the launch itself checks the
// size the device reports.
constexpr long GFX950_LDS_BYTES = 160 * 1024;

// Row stride of the output staging tile: padded like the K and V rows (conflict-free 8-byte stores) when a
// 7-tile window then still fits the LDS, else the bare D (d = 80).
template <int D>
__host__ __device__ constexpr int window_stage_stride()
{
    constexpr int KSTR = AttnCfg<D>::KSTR, bias = 32 * WIN_OSTR * (int)sizeof(WinTab), stage = 32 * KSTR * 2;
    constexpr long total = 7L * window_q_bytes<D>() + 2L * 224 * KSTR * 2 + 2L * 32 * KSTR * 2 +
                           7L * (bias > stage ? bias : stage) + 224 * 4;
    return total <= GFX950_LDS_BYTES ? KSTR : D;
}

template <int D>
__host__ __device__ inline int window_scratch_bytes()
{
    int bias = 32 * WIN_OSTR * (int)sizeof(WinTab), stage = 32 * window_stage_stride<D>() * 2;
    return ((bias > stage ? bias : stage) + 15) & ~15;
}

template <int D>
size_t window_lds_bytes(int nqb, int w)
{
    int SP = nqb * 32;
    return (size_t)nqb * window_q_bytes<D>() + (size_t)2 * SP * AttnCfg<D>::KSTR * 2 +
           (size_t)2 * window_rel_rows(w) * AttnCfg<D>::KSTR * 2 + (size_t)nqb * window_scratch_bytes<D>() + (size_t)SP * 4;
}

constexpr int WIN_MAX_LOADS = 5;     // 16-byte K (and V) chunks per thread: 224 keys * 10 chunks / 448 threads

template <int D>
__global__ void __launch_bounds__(448)
attn_window_kernel(AttnParams P, int n_groups)
{
    using C = AttnCfg<D>;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int nqb = blockDim.x >> 6, SP = nqb * 32;
    const int nrel = 2 * P.w - 1, rrows = ((nrel + 31) / 32) * 32;      // nrel <= 32 (checked on the host)
    bf16 *Qs = reinterpret_cast<bf16 *>(smem);    // [nqb][KS][64 lanes][8]: query fragments, one problem ahead (first in LDS)
    bf16 *Ks = Qs + nqb * (window_q_bytes<D>() / 2);
    bf16 *Vs = Ks + SP * C::KSTR;
    bf16 *Rh = Vs + SP * C::KSTR;                 // rel-pos tables, zero-padded to rrows rows
    bf16 *Rw = Rh + rrows * C::KSTR;
    unsigned char *T = reinterpret_cast<unsigned char *>(Rw + rrows * C::KSTR);
    const int wsb = window_scratch_bytes<D>();
    uint32_t *krc = reinterpret_cast<uint32_t *>(T + nqb * wsb);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31;
    const int S = P.S;
    const int nloads = (SP * C::CH + blockDim.x - 1) / blockDim.x;     // <= WIN_MAX_LOADS (checked on the host)

    clamp_fp16();
    // problem-independent state: scan-order geometry and the rel-pos tables
    if (P.sigma_stride == 0)
        for (int p = tid; p < SP; p += blockDim.x) krc[p] = key_row_col(P.sigma, p, S, P.w);
    for (int id = tid; id < 2 * rrows * C::CH; id += blockDim.x) {
        int tab = id / (rrows * C::CH), rem = id % (rrows * C::CH), row = rem / C::CH, c = rem % C::CH;
        u32x4 v = { 0, 0, 0, 0 };
        if (row < nrel) v = *reinterpret_cast<const u32x4 *>((tab ? P.rel_w : P.rel_h) + (long)row * D + c * 8);
        *reinterpret_cast<u32x4 *>((tab ? Rw : Rh) + row * C::KSTR + c * 8) = v;
    }
    set_ones_columns<D>(Vs, SP, tid, (int)blockDim.x);
    const int q0 = wave * 32, qpos = q0 + l32;
    const int qclamp = qpos < S ? qpos : S - 1;
    uint32_t qrc = key_row_col(P.sigma, qclamp, S, P.w);
    WinTab *tq = reinterpret_cast<WinTab *>(T + wave * wsb);
    const int nact = P.n_pre + (wave >= P.n_pre ? 1 : 0);

    u32x4 rk[WIN_MAX_LOADS], rv[WIN_MAX_LOADS];
    bf16x8 qf[C::KS];
    int32_t row_next = -1;
    bf16 *q_mine = Qs + wave * (window_q_bytes<D>() / 2) + lane * 8;        // this lane's slot in fragment 0
    const uint32_t q_lds = __builtin_amdgcn_readfirstlane(
        (uint32_t)(size_t)(__attribute__((address_space(3))) bf16 *)(Qs + wave * (window_q_bytes<D>() / 2)));

    // The next problem's operands are requested in three pieces (K, V here, Q below) spread over the current problem's
    // phases: a CU keeps only so many cache-line requests in flight, and a wave that issues all of its loads
    // at once sits in the issue queue behind the other waves' loads instead of computing.
#define WIN_PREFETCH(prob_, WHAT)                                                                       \
    {                                                                                                   \
        __builtin_amdgcn_sched_barrier(0);                                                              \
        const int g_ = (prob_) / P.h, hd_ = (prob_) % P.h;                                              \
        const long base_ = (long)g_ * S * P.row_stride + (long)hd_ * D;                                 \
        /* K and V of a problem are read exactly once: non-temporal loads, so that they do not displace the      \
           residual stream and the attention output that the next kernels read (0.8 % of a ViT-H step) */         \
        if ((WHAT) & 3) {                                                                               \
            _Pragma("unroll") for (int i = 0; i < WIN_MAX_LOADS; ++i)                                   \
            {                                                                                           \
                int id = tid + i * (int)blockDim.x, key = id / C::CH, c = id % C::CH;                   \
                key = key < S ? key : S - 1; /* pad keys repeat the last row: finite values, masked */  \
                if (i < nloads && ((WHAT) & 1))                                                         \
                    rk[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(P.k + base_ + (long)key * P.row_stride + c * 8)); \
                if (i < nloads && ((WHAT) & 2))                                                         \
                    rv[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(P.v + base_ + (long)key * P.row_stride + c * 8)); \
            }                                                                                           \
        }                                                                                               \
        if (((WHAT) & 1) && P.out_rows != nullptr && qpos < S) row_next = P.out_rows[(long)g_ * S + qpos]; \
        __builtin_amdgcn_sched_barrier(0);                                                              \
    }
    // The queries of a problem do not pass through registers: 16-byte loads with an LDS destination drop fragment
    // ks of the wave's 32 queries into its landing area (lane l's 16 bytes at 16*l, the layout operand b wants)
    // while the problem before it is still in its chunk loop, which has no registers to spare for them.  The
    // compiler does not see these requests; the kernel waits for them itself before it reads the landing area.
    // The wait in front makes sure the LDS reads of the current fragments have returned.
#define WIN_PREFETCH_Q(prob_)                                                                           \
    {                                                                                                   \
        __builtin_amdgcn_sched_barrier(0);                                                              \
        const int g_ = (prob_) / P.h, hd_ = (prob_) % P.h;                                              \
        const bf16 *qsrc_ = P.q + (long)g_ * S * P.row_stride + (long)hd_ * D + (long)qclamp * P.row_stride + (lane >> 5) * 8; \
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                                              \
        _Pragma("unroll") for (int ks = 0; ks < C::KS; ++ks)                                            \
            asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off"                          \
                         :: "s"(q_lds + ks * 1024), "v"(qsrc_ + ks * 16) : "m0", "memory");             \
        __builtin_amdgcn_sched_barrier(0);                                                              \
    }

    // Problems are dealt so that the heads of one window run on one XCD (workgroup b sits on XCD b & 7):
    // a head's rows are 2*D bytes at a stride of the packed row, so neighbouring heads share cache lines,
    // and those are then fetched into one L2 instead of eight.  XCD x takes windows x, x+8, ..., heads fastest.
    const int xcd = blockIdx.x & 7, nslots = ((int)gridDim.x - xcd + 7) >> 3;
    auto local_problem = [&](int lp) { int g = xcd + 8 * (lp / P.h); return g < n_groups ? g * P.h + lp % P.h : -1; };
    int lp = blockIdx.x >> 3;
    int prob = local_problem(lp);
    if (prob >= 0) {
        WIN_PREFETCH_Q(prob)
        WIN_PREFETCH(prob, 3)
    }
    for (; prob >= 0; lp += nslots, prob = local_problem(lp)) {
        const int grp = prob / P.h, head = prob % P.h;
        long my_row = -1;                         // output row of this lane's query (a mapped row was requested a problem ahead)
        if (qpos < S) my_row = P.out_rows ? (long)row_next : (long)grp * S + qpos;
        LDS_BARRIER();                            // every wave is done with the previous problem's LDS (output stores stay in flight)
#pragma unroll
        for (int i = 0; i < WIN_MAX_LOADS; ++i) {
            int id = tid + i * (int)blockDim.x, key = id / C::CH, c = id % C::CH;
            if (i < nloads && id < SP * C::CH) {
                *reinterpret_cast<u32x4 *>(Ks + key * C::KSTR + c * 8) = rk[i];
                *reinterpret_cast<u32x4 *>(Vs + key * C::KSTR + c * 8) = rv[i];
            }
        }
        if (P.sigma_stride != 0) {                // per-group order: this window's own sigma
            const int32_t *sg = P.sigma + (long)grp * P.sigma_stride;
            for (int p = tid; p < SP; p += blockDim.x) krc[p] = key_row_col(sg, p, S, P.w);
            qrc = key_row_col(sg, qclamp, S, P.w);
        }
        // this problem's queries were sent to LDS during the previous problem (WIN_PREFETCH_Q): wait for every
        // outstanding request of this wave (the K and V registers above have been waited for already; what else is
        // in flight is the previous problem's output stores) before reading them
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
        for (int ks = 0; ks < C::KS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8 *>(q_mine + ks * 512);
        const int next = local_problem(lp + nslots);
        if (next >= 0) WIN_PREFETCH(next, 1)
        WinTab *tq_lane = tq + l32 * WIN_OSTR;
        build_bias_operands_window<D>(qf, [&](int tab, int ks) {
            return *reinterpret_cast<const bf16x8 *>((tab ? Rw : Rh) + l32 * C::KSTR + (lane >> 5) * 8 + ks * 16);
        }, P.w, (int)(qrc & 0xffffu), (int)(qrc >> 16), tq, P.table_inv);
        LDS_BARRIER();
        if (next >= 0) WIN_PREFETCH(next, 2)

        WaveState<D> st;
        init_state<D>(st);
        // active key tiles of query tile `wave`: the dense prefix, then the diagonal
        for (int a = 0; a < nact; ++a) {
            const int blk = a < P.n_pre ? a : wave, key0 = blk * 32;
            // only the last 32-key tile of the window can cross S
            if (key0 + 32 > S) attn_window_step<D, true>(st, qf, Ks, Vs, krc, blk, key0, S, P.scale_log2e, tq_lane, P.half_one);
            else attn_window_step<D, false>(st, qf, Ks, Vs, krc, blk, key0, S, P.scale_log2e, tq_lane, P.half_one);
            // after the second tile (the only one, when there is one): early enough to cover the request's
            // latency with the last tile and the output stores on the tiles that have three, and not in the same
            // burst as the K or the V requests
            if (a == (nact > 1 ? 1 : 0) && next >= 0) WIN_PREFETCH_Q(next)
        }
        finish_and_store<D, window_stage_stride<D>()>(st, reinterpret_cast<bf16 *>(tq), P.out + (long)head * D, (long)P.h * D, my_row);
    }
}

// ------------------------------------------------------------------ window kernel, a wave to a query tile
// One workgroup = one wave = one 32-query tile: the active key blocks one after the other through LDS of its own, the next one
// in registers, no barriers.  The persistent kernel above stages a problem's K and V once for its seven waves, but with one workgroup
// to a CU it is bound by latency where there are few problems (set-up, tables, requests and seven waves' barriers in a chain, 15 us) and by its seven
// tiles on four SIMDs and its nearly empty last round where there are more.  Here everything up to the first key block is requested
// at once, twelve waves share a CU (eight at d = 80), and the tiles of a problem, which run next to each other on one XCD, find each other's K and V
// in its L2.  us, persistent kernel with look-ups -> this one, cold inputs, 14 x 14, r = 0.4: d = 64, 64 problems 15.9 -> 7.5, 400 18.1 -> 13.2,
// 800 30.2 -> 24.0, 1600 48.9 -> 41.8, 3200 86.3 -> 79.5 (4.0 TB/s of q, k, v and output); dense, 3200 140 -> 125; d = 32, 2400 54.6 -> 38.9; d = 16 49.2 -> 29.0.
// Two blocks ahead, which leaves registers for two waves a SIMD, is slower (d = 64, 1600 problems 44.2 -> 47.8).
template <int D, bool ANY>
struct WinWave {
    using C = AttnCfg<D>;
    static constexpr int AHEAD = D <= 32 ? 2 : 1;         // key blocks requested ahead, in registers
    static constexpr int LOADS = C::CH / 2;               // 16-byte chunks of a block's K (and V) per lane
    static constexpr int KV = 32 * C::KSTR;               // elements of a block of K or V in LDS
    static constexpr int WAVES = D <= 64 && !ANY ? 3 : 2; // per SIMD: the register budget
    static size_t lds_bytes(int nact) { return (size_t)2 * KV * 2 + 32 * WIN_OSTR * sizeof(WinTab) + (size_t)nact * 32 * 4; }
};

// Problems (window, head) prob0 .. prob0 + n_problems - 1.  ANY: for rows of a window that need 64-bit byte offsets and for scales that the
// queries take a part of.
template <int D, bool ANY>
__global__ void __launch_bounds__(64, (WinWave<D, ANY>::WAVES))
attn_window_kernel_waves(AttnParams P, int prob0, int n_problems, int T)
{
    using C = AttnCfg<D>;
    using G = WinWave<D, ANY>;
    using Offset = std::conditional_t<ANY, uint64_t, uint32_t>;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    bf16 *Ks = reinterpret_cast<bf16 *>(smem), *Vs = Ks + G::KV;          // one block of keys
    WinTab *tq = reinterpret_cast<WinTab *>(Vs + G::KV);
    uint32_t *krc = reinterpret_cast<uint32_t *>(tq + 32 * WIN_OSTR);      // cells of every active block, in the order of the list
    // the tiles of a problem, and runs of problems, on one XCD (workgroup b sits on XCD b & 7)
    const int per_xcd = (n_problems + 7) >> 3, slot = (int)(blockIdx.x >> 3), qt = slot % T;
    int prob = (int)(blockIdx.x & 7) * per_xcd + slot / T;
    if (prob >= n_problems) return;
    prob += prob0;
    const int grp = prob / P.h, head = prob % P.h;
    clamp_fp16();
    const int lane = threadIdx.x, l32 = lane & 31, half = lane >> 5, S = P.S;
    const int nact = P.n_pre + (qt >= P.n_pre ? 1 : 0);
    const int qpos = qt * 32 + l32, qclamp = min(qpos, S - 1);
    const int32_t *sg = P.sigma + (long)grp * P.sigma_stride;
    const long base = (long)grp * S * P.row_stride + (long)head * D;
    const unsigned char *kbase = reinterpret_cast<const unsigned char *>(P.k + base), *vbase = reinterpret_cast<const unsigned char *>(P.v + base);
    const Offset rs2 = (Offset)P.row_stride * 2u;
    auto block_at = [&](int a) { return a < P.n_pre ? a : qt; };

    // everything up to the first key blocks is requested at once, in the order in which it is wanted
    constexpr int PAIRS = 4;                       // pairs of active blocks: at most 7 blocks (S <= 224)
    int32_t qcell = sg[qclamp], cell[PAIRS];
#pragma unroll
    for (int i = 0; i < PAIRS; ++i) cell[i] = sg[min(block_at(min(2 * i + half, nact - 1)) * 32 + l32, S - 1)];      // (behind a branch each would be waited for by itself)
    const long row_at = (long)grp * S + qclamp;
    const int32_t row_mapped = *(P.out_rows ? P.out_rows + row_at : sg + qclamp);      // without a map: read, not used
    bf16x8 qf[C::KS], rel[2][C::KS];
    load_q_frags<D>(qf, P.q + base + (long)qclamp * P.row_stride);
#pragma unroll
    for (int tab = 0; tab < 2; ++tab)              // rows past the table repeat its last one: never looked up
        load_q_frags<D>(rel[tab], (tab ? P.rel_w : P.rel_h) + min(l32, 2 * P.w - 2) * D);
    u32x4 rk[G::AHEAD][G::LOADS], rv[G::AHEAD][G::LOADS];
    auto load_block = [&](u32x4 (&k)[G::LOADS], u32x4 (&v)[G::LOADS], int a) {
        const int key0 = block_at(a) * 32;
#pragma unroll
        for (int i = 0; i < G::LOADS; ++i) {
            const int id = lane + 64 * i;          // pad keys repeat the last row: finite values, masked
            const Offset at = (Offset)min(key0 + id / C::CH, S - 1) * rs2 + id % C::CH * 16;
            k[i] = *reinterpret_cast<const u32x4 *>(kbase + at);
            v[i] = *reinterpret_cast<const u32x4 *>(vbase + at);
        }
    };
#pragma unroll
    for (int u = 0; u < G::AHEAD; ++u)
        load_block(rk[u], rv[u], min(u, nact - 1));
    __builtin_amdgcn_sched_barrier(0);
    const long my_row = qpos < S ? (P.out_rows ? (long)row_mapped : row_at) : -1;

    set_ones_columns<D>(Vs, 32, lane, 64);
    const uint32_t qrc = cell_row_col(qcell, P.w);
#pragma unroll
    for (int i = 0; i < PAIRS; ++i)
        if (2 * i + half < nact) krc[64 * i + lane] = cell_row_col(cell[i], P.w);
    WinTab *tq_lane = tq + l32 * WIN_OSTR;
    build_bias_operands_window<D>(qf, [&](int tab, int ks) { return rel[tab][ks]; }, P.w, (int)(qrc & 0xffffu), (int)(qrc >> 16), tq, P.table_inv);
    if constexpr (ANY) if (P.q_exp != 0) scale_queries<D>(qf, P.q_exp);

    WaveState<D> st;
    init_state<D>(st);
    for (int a0 = 0; a0 < nact; a0 += G::AHEAD) {
#pragma unroll
        for (int u = 0; u < G::AHEAD; ++u) {
            const int a = a0 + u;
            if (a >= nact) break;
            wave_lds_fence();
#pragma unroll
            for (int i = 0; i < G::LOADS; ++i) {
                const int id = lane + 64 * i, at = id / C::CH * C::KSTR + id % C::CH * 8;
                *reinterpret_cast<u32x4 *>(Ks + at) = rk[u][i];
                *reinterpret_cast<u32x4 *>(Vs + at) = rv[u][i];
            }
            wave_lds_fence();
            if (a + G::AHEAD < nact) load_block(rk[u], rv[u], a + G::AHEAD);
            const int key0 = block_at(a) * 32;
            if (key0 + 32 > S) attn_window_step<D, true>(st, qf, Ks, Vs, krc + 32 * a, 0, key0, S, P.scale_log2e, tq_lane, P.half_one);
            else attn_window_step<D, false>(st, qf, Ks, Vs, krc + 32 * a, 0, key0, S, P.scale_log2e, tq_lane, P.half_one);
        }
    }
    wave_lds_fence();
    finish_and_store<D>(st, Ks, P.out + (long)head * D, (long)P.h * D, my_row);
}

// ------------------------------------------------------------------ global kernel
constexpr int GLB_TILE = 128;
// Bias rows of the global kernel are held as fp16 (11 significant bits on log2e * q.r, below the bf16
// rounding of the probabilities that feed the second product): at w = 64 that brings a workgroup to
// 78 KB of LDS, so two workgroups share a CU and one hides the other's LDS, MFMA and barrier latency.
typedef _Float16 GlbTab;

// ---- patch path
// One workgroup = one 128-query tile, four waves of 32 queries: a pipeline of 32-key blocks.
// Scores, softmax and P V of a block depend on each other, and with a tile of 128 keys at a time between two barriers the matrix,
// vector and LDS pipes were all 35-50 % busy.  So
//   * a wave works on three blocks at once: while the vector unit takes the exponentials of block b, one MFMA behind every
//     few of those instructions forms the scores of block b + 1 and adds P V of block b - 1;
//   * K and V blocks go from memory straight into two rings of four blocks in LDS, by twos, two blocks ahead (no registers, no LDS
//     writes).  Such loads fill LDS in lane order, so rows are packed without padding and the 16-byte
//     chunks of a row are swizzled on the memory side: the reads of K are conflict-free, as with padding;
//   * one barrier for two blocks, no more: four waves that wait for each other were what bound a loop with a barrier a block, alone on their CU (1300
//     cycles a block, now 920) as with another workgroup's.  Fewer instructions, operands read further ahead, wider spread requests or a deeper ring changed nothing
//     there.  64 x 64, d = 80 | 64, us: 16 images of 16 heads, r = 0.4 802 | 660 -> 742 | 608; 1 image 53.7 | 44 -> 50 | 41; 8 heads of d = 80 39.5 -> 31.9;
//     d = 32, 8 images 247 -> 225.  At large batches what is left is power: the clock falls to 1.8 GHz with the matrix pipes 45 % busy;
//   * where the exponent reference moves in block b, the output is rescaled in front of block b + 1, behind P V of block b - 1, whose probabilities are still
//     in units of the reference before.  (Moving it by whole powers of two would allow rescaling those probabilities instead,
//     but then a query's largest probability is no longer exactly 1 and is rounded to bf16 like the others: up to 19 % more
//     error where one key dominates.)
// WK != 0: any order (attn_onehot_body), the bias by products with the whole table row of a query, WK entries each of rows and columns.
template <int D, int WK>
struct AttnPipe {
    using C = AttnCfg<D>;
    static constexpr int SLOT = 32 * D * 2;                       // bytes of a block of K or V
    static constexpr int RING = 4 * SLOT;                         // bytes of a ring
    static constexpr int SEG = WK / 32;                           // sparse products of a block's bias and table
    static constexpr int NQ = WK ? C::KS + 2 * SEG : 1 + C::KS, NP = 2 * C::DT;          // MFMAs of a block's scores and of its P V
    static constexpr int LOADS = C::CH / 2;                       // 1 KB requests of a block of K or V
    static constexpr int AHEAD = 3, FR = 4;                       // operand fragments are read three MFMAs ahead

    // chunk c of row `row` sits at chunk position c ^ swz(row).  K: 16 rows at one chunk then touch 16 distinct 16-byte banks.  V: a transposing
    // read takes 64 bytes of each of 8 rows, and of rows of 128 bytes every other pair has them in the other half
    static __device__ __forceinline__ int swz(int row, bool v)
    {
        if (C::CH == 8) return v ? (row << 1) & 4 : (row >> 1) & 7;
        return C::CH == 4 ? (row >> 2) & 3 : (row >> 3) & 1;
    }

    WaveState<D> &st;
    const bf16x8 *qf;
    const unsigned char *lds, *tq_lane;
    float scale_log2e;
    f16x8 efrag;
    int ka[C::KS], va[C::CH == 8 ? 2 : 1][2];   // byte offsets: this lane's K chunks in a block, its V reads (rows +0 and +8), by column tile where rows have 8 chunks
    uint32_t bo;                     // table offsets of the block whose scores are formed next (patches)
    f16x16 t[2][WK ? SEG : 1];       // the lane's query's table entries: 32 * segment + 8 * half .. + 7 and 16 more on (any order)
    int cell, w;                     // cell of this lane's key in the block whose scores are formed next, side of the grid
    uint32_t per_w, half_one;        // 2^20 / w rounded up; the one of the bias products
    int group[2];                    // that key's row and column: which four entries, less this half-wave's first four
    uint32_t one[2], index[2];       //   the dword that holds the one, and which of the four it is
    int limit;                       // keys of the block whose softmax is taken that exist
    float start;                     // maximum of block 1's scores
    f32x16 s[2];
    bf16x8 p[2][2], frag[FR];
    float most;                      // the reference moves past this
    float alpha;                     // it moved by this factor in the block before (moved, wave-uniform)
    bool moved;

    // operand I of the interleaved sequence of a step with scores (HQ) and / or P V (HP): spread evenly, scores first
    static constexpr int q_before(int k) { return NQ <= NP + 1 ? (k + 1) / 2 : (k * NQ + NQ + NP - 1) / (NQ + NP); }
    template <bool HQ, bool HP> static constexpr bool is_q(int k) { return HQ && (!HP || q_before(k + 1) > q_before(k)); }
    template <bool HQ, bool HP> static constexpr int idx(int k) { return !HQ || !HP ? k : is_q<HQ, HP>(k) ? q_before(k) : k - q_before(k); }

    // Row and column of the next block's key for the bias products.  A table of 32 entries is one sparse product: the one is in the
    // first of the two values kept of its four entries, or in the second where it is the last of them.
    __device__ __forceinline__ void describe()
    {
        const int half = (threadIdx.x & 63) >> 5;
        const uint32_t cl = min(max(cell, 0), w * w - 1), r = __umul24(cl, per_w) >> 20;
#pragma unroll
        for (int tab = 0; tab < 2; ++tab) {
            const uint32_t at = tab ? cl - r * w : r, i = at & 3u;
            group[tab] = (int)(at >> 2) - 4 * half;
            one[tab] = i == 3 ? half_one << 16 : half_one;
            index[tab] = (i == 3 ? 0xccccu : 0xccccu + i * 0x1111u);
        }
    }

    template <bool HQ, bool HP, int K>
    __device__ __forceinline__ void load(int k_slot, int v_slot)
    {
        if constexpr (K < (HQ ? NQ : 0) + (HP ? NP : 0)) {
            constexpr int i = idx<HQ, HP>(K);
            bf16x8 &f = frag[K % FR];
            if constexpr (!is_q<HQ, HP>(K)) {
                constexpr int t = i / C::DT, dt = i % C::DT;
                bf16x4 v[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int at = va[C::CH == 8 ? dt : 0][u] + v_slot + t * 16 * D * 2 + (C::CH == 8 ? 0 : dt * 64);
                    v[u] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4 *)(lds + at));
                }
                f = bf16x8{ v[0][0], v[0][1], v[0][2], v[0][3], v[1][0], v[1][1], v[1][2], v[1][3] };
            } else if constexpr (WK != 0) {
                if constexpr (i < C::KS) {
                    f = *reinterpret_cast<const bf16x8 *>(lds + k_slot + ka[i]);
                } else {
                    constexpr int tab = (i - C::KS) / SEG, seg = (i - C::KS) % SEG;
                    u32x4 e;
#pragma unroll
                    for (int j = 0; j < 4; ++j) e[j] = group[tab] == 8 * seg + j ? one[tab] : 0u;
                    f = __builtin_bit_cast(bf16x8, e);
                }
            } else if constexpr (i == 0) {
                // operand b of the bias product: f = 8*half + e; f 0..3 the block's rows, 4..11 its columns, 12..15 meet
                // zeros of E (finite values: the upper half-wave reads columns twice)
                const f16x4 t1 = *reinterpret_cast<const f16x4 *>(tq_lane + (bo & 0xffffu));
                const f16x4 t2 = *reinterpret_cast<const f16x4 *>(tq_lane + (bo >> 16));
                f = __builtin_bit_cast(bf16x8, f16x8{ t1[0], t1[1], t1[2], t1[3], t2[0], t2[1], t2[2], t2[3] });
            } else {
                f = *reinterpret_cast<const bf16x8 *>(lds + k_slot + ka[i - 1]);
            }
        }
    }

    // PAR: parity of the block whose softmax this step is (the scores formed are the other parity's, so is the P V)
    template <bool HQ, bool HP, int PAR, int K>
    __device__ __forceinline__ void mfma()
    {
        constexpr int i = idx<HQ, HP>(K);
        const bf16x8 &f = frag[K % FR];
        if constexpr (!is_q<HQ, HP>(K)) {
            st.o[i % C::DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, p[PAR ^ 1][i / C::DT], st.o[i % C::DT], 0, 0, 0);
        } else if constexpr (WK != 0) {
            const f32x16 zero = { 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f };
            if constexpr (i < C::KS) {
                s[PAR ^ 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, qf[i], i == 0 ? zero : s[PAR ^ 1], 0, 0, 0);
            } else {
                constexpr int tab = (i - C::KS) / SEG, seg = (i - C::KS) % SEG;
                s[PAR ^ 1] = __builtin_amdgcn_smfmac_f32_32x32x32_f16(__builtin_bit_cast(f16x8, f), t[tab][seg], s[PAR ^ 1], (int)index[tab], 0, 0);
            }
        } else if constexpr (i == 0) {
            const f32x16 zero = { 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f };
            s[PAR ^ 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(efrag, __builtin_bit_cast(f16x8, f), zero, 0, 0, 0);
        } else {
            s[PAR ^ 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, qf[i - 1], s[PAR ^ 1], 0, 0, 0);
        }
    }

    template <int PAR, int J, int J1>
    __device__ __forceinline__ void exp_pairs(float mref)         // probabilities 2*J .. 2*J1 - 1
    {
        if constexpr (J < J1) {
            const float e0 = __builtin_amdgcn_exp2f(fmaf(s[PAR][2 * J], scale_log2e, -mref));
            const float e1 = __builtin_amdgcn_exp2f(fmaf(s[PAR][2 * J + 1], scale_log2e, -mref));
            u32x4 w = __builtin_bit_cast(u32x4, p[PAR][J / 4]);
            const uint32_t pair = pack_bf16x2(e0, e1);
            w[J % 4] = pair;
            // the sum of what P V multiplies, the rounded probabilities, as with the ones columns: one instruction, and the rounding of
            // a dominant one cancels
            st.l = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), bf16x2{ (bf16)1.f, (bf16)1.f }, st.l, false);
            p[PAR][J / 4] = __builtin_bit_cast(bf16x8, w);
            exp_pairs<PAR, J + 1, J1>(mref);
        }
    }

    template <bool HQ, bool HP, int PAR, bool SM, int K>
    __device__ __forceinline__ void steps(int k_slot, int v_slot, float mref)
    {
        constexpr int n = (HQ ? NQ : 0) + (HP ? NP : 0);
        if constexpr (K < n) {
            if constexpr (WK != 0 && HQ && K == 0 && C::KS >= 4) describe();
            load<HQ, HP, K + AHEAD>(k_slot, v_slot);
            mfma<HQ, HP, PAR, K>();
            if constexpr (SM) exp_pairs<PAR, 8 * K / n, 8 * (K + 1) / n>(mref);       // spread evenly behind the MFMAs
            __builtin_amdgcn_sched_barrier(0);
            steps<HQ, HP, PAR, SM, K + 1>(k_slot, v_slot, mref);
        }
    }

    template <bool HQ, bool HP>
    __device__ __forceinline__ void begin(int k_slot, int v_slot)
    {
        if constexpr (WK != 0 && HQ && C::KS < 4) describe();             // (else under the first products)
        load<HQ, HP, 0>(k_slot, v_slot);
        load<HQ, HP, 1>(k_slot, v_slot);
        load<HQ, HP, 2>(k_slot, v_slot);
    }

    // addresses of this lane's operands, state of the softmax
    __device__ __forceinline__ void addresses()
    {
        const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5, li = lane & 15, fblk = (lane >> 4) & 1;
        moved = false;
        alpha = 1.f;
        most = -INFINITY;
#pragma unroll
        for (int ks = 0; ks < C::KS; ++ks) ka[ks] = l32 * D * 2 + ((2 * ks + half) ^ swz(l32, false)) * 16;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            // transposing read: lane li of a 16-lane group points at row (li >> 2) of its 4 keys, column chunk (li & 3) of 4
            // features of its 16; feature columns past D are whatever lies there in LDS, and their outputs are dropped
            const int row = 8 * u + 4 * half + (li >> 2), f0 = (C::ONES && D == 16 ? 0 : 16 * fblk) + 4 * (li & 3);
#pragma unroll
            for (int dt = 0; dt < (C::CH == 8 ? 2 : 1); ++dt)
                va[dt][u] = RING + row * D * 2 + (((4 * dt + (f0 >> 3)) ^ swz(row, true)) << 4) + (f0 & 7) * 2;
        }
    }

    // the output in units of the present reference, if that moved in the block before
    __device__ __forceinline__ void rescale()
    {
        if (!moved) return;
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");          // P V MFMAs may be in flight (as in finish_and_store)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) st.o[dt][r] *= alpha;
    }

    // softmax of block b (parity PAR) with, behind it, the scores of b + 1 (HQ) and P V of b - 1 (HP)
    template <bool HQ, bool HP, int PAR>
    __device__ __forceinline__ void block(int k_slot, int v_slot)
    {
        begin<HQ, HP>(k_slot, v_slot);
        if (WK != 0 && __builtin_expect(limit < 32, 0)) {          // keys past the end
            const int half = (threadIdx.x & 63) >> 5;
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");      // the scores' MFMAs may be in flight
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < 16; ++r) s[PAR][r] = 8 * (r >> 2) + 4 * half + (r & 3) < limit ? s[PAR][r] : -INFINITY;
        }
        float mx = fmaxf(s[PAR][0], s[PAR][1]);
#pragma unroll
        for (int r = 2; r < 16; ++r) mx = fmaxf(mx, s[PAR][r]);
        if constexpr (WK != 0 && !HP) mx = fmaxf(mx, start);                               // the first block
        const bool any = __builtin_amdgcn_ballot_w64(mx * scale_log2e > most) != 0;        // over this half-wave's keys
        if (__builtin_expect(any || moved, 0)) {
            rescale();                                  // P V of the block before is in the output: what moved there
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * scale_log2e;
            const bool move = mx > most;                // see attn_softmax_pv
            alpha = 1.f;
            moved = any;
            if (move) {
                alpha = __builtin_amdgcn_exp2f(st.m - mx);
                st.m = mx;
                most = mx + ATTN_LAG;
            }
            st.l *= alpha;
        }
        __builtin_amdgcn_sched_barrier(0);
        // ahead of the other workgroup's requests, maxima and barriers (1 % at batch 16, 5 % when a launch is one round)
        __builtin_amdgcn_s_setprio(1);
        steps<HQ, HP, PAR, true, 0>(k_slot, v_slot, st.m);
        __builtin_amdgcn_s_setprio(0);
    }
};

// Requests of a wave for the rings of a workgroup: waves 0 and 1 bring K, 2 and 3 V, a block each: lane l of request i the chunk that
// belongs at 16-byte place 64 * i + l.  RAGGED: rows past S repeat the last one (their scores are masked).
template <int D, bool RAGGED, bool SHORT = false>
struct AttnRequests {
    using Pipe = AttnPipe<D, 0>;
    static constexpr int CH = AttnCfg<D>::CH, SLOT = Pipe::SLOT, LOADS = Pipe::LOADS;
    static_assert(2 * Pipe::RING <= 64 * 1024, "the rings are filled through M0");
    const unsigned char *kvbase;
    uint32_t rs2, lds0, src_off[LOADS];
    int S, n_pre, qt, nblk, wave;
    bool is_v;

    __device__ __forceinline__ AttnRequests(const AttnParams &P, int qt_, long base, unsigned char *smem)
        : rs2((uint32_t)P.row_stride * 2u), S(P.S), n_pre(P.n_pre), qt(qt_), nblk(blocks(P, qt_)),
          wave(__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))), is_v(wave >= 2)
    {
        kvbase = reinterpret_cast<const unsigned char *>((is_v ? P.v : P.k) + base);
        lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char *)smem) + (is_v ? Pipe::RING : 0);
        int l64 = threadIdx.x & 63;
        asm volatile("" : "+v"(l64));             // (else rows and chunks are kept for finish_and_store, which has the same, through the loops)
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int place = i * 64 + l64, row = place / CH, pos = place % CH;
            src_off[i] = (uint32_t)row * rs2 + (uint32_t)(pos ^ Pipe::swz(row, is_v)) * 16u;
        }
    }
    // Blocks of the active tiles; with SHORT two of the last one, where no more than two have keys (sides that are 4 mod 8 have 16 keys in their last tile).  Its other
    // two, masked, cost 12 x 12, 256 problems, r = 0.5 1.9 us at d = 64 (14.3 -> 12.4; tiles of 128 keys between two barriers took 13.0), 16 problems of
    // 28 x 28, dense, 21.4 -> 20.1.
    __device__ __forceinline__ static int blocks(const AttnParams &P, int qt)
    {
        const int n = (P.n_pre + (qt >= P.n_pre ? 1 : 0)) * (GLB_TILE / 32);
        if (!SHORT) return n;
        const int last = max(qt, P.n_pre - 1) * GLB_TILE;       // first key of the last active tile
        return P.S - last <= 64 ? n - 2 : n;
    }
    __device__ __forceinline__ int key0(int blk) const       // scan position of the first key of the workgroup's block blk
    {
        const int a = blk >> 2;
        return __builtin_amdgcn_readfirstlane((a < n_pre ? a : qt) * GLB_TILE + (blk & 3) * 32);
    }
    // this wave's operand of a block, into slot blk % 4 of its ring
    __device__ __forceinline__ void operator()(int blk) const
    {
        if (blk >= nblk) return;
        const int first = key0(blk);
        const uint32_t at = lds0 + __builtin_amdgcn_readfirstlane((blk & 3) * SLOT);
        if (RAGGED && first + 32 > S) {
            int l64 = threadIdx.x & 63;
            asm volatile("" : "+v"(l64));
#pragma unroll
            for (int i = 0; i < LOADS; ++i) {
                const int place = i * 64 + l64, row = place / CH, pos = place % CH;
                send(at + i * 1024, (uint32_t)min(first + row, S - 1) * rs2 + (uint32_t)(pos ^ Pipe::swz(row, is_v)) * 16u, kvbase);
            }
            return;
        }
        const unsigned char *src = kvbase + (size_t)(uint32_t)first * rs2;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) send(at + i * 1024, src_off[i], src);
    }
    __device__ __forceinline__ static void send(uint32_t at, uint32_t off, const unsigned char *src)
    {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(at), "v"(off), "s"(src) : "m0", "memory");
    }
    __device__ __forceinline__ void first() const            // K(0), K(1), V(0), K(2)
    {
        if (wave != 3) (*this)(wave & 1);
        if (wave == 0) (*this)(2);
    }
};

// The blocks of a workgroup through its pipe; K(0), K(1), V(0) and K(2) have landed, or are waited for with what `arrived` waits for.
// Blocks b and b + 1 (b even) form the scores of b + 1 and b + 2 and add P V of b - 1 and b: what they read was requested two blocks ago.  Every
// wave is done with K(b - 1) and K(b) and with V(b - 3) and V(b - 2): they make room for K(b + 3), K(b + 4), V(b + 1) and V(b + 2).
// nblk is a multiple of four, with TWO_MORE two more: every slot read is a constant, in the instructions.
// ahead(): in front of it all; arrived(): behind the wait for all that was requested; one(b), two(b): in front of blocks b and b + 1.
template <bool TWO_MORE, class Pipe, class Request, class Ahead, class Arrived, class One, class Two>
__device__ __forceinline__ void attn_pipe_run(Pipe &pipe, const Request &request, int nblk, Ahead ahead, Arrived arrived, One one, Two two)
{
    constexpr int SLOT = Pipe::SLOT;
    ahead();
    pipe.template begin<true, false>(0, 0);
    pipe.template steps<true, false, 1, false, 0>(0, 0, 0.f);       // scores of block 0
    auto pair = [&](auto odd_, auto first_, auto last_, int b) {
        constexpr int K0 = decltype(odd_)::value ? 2 : 0;        // b % 4
        constexpr bool FIRST = decltype(first_)::value, LAST = decltype(last_)::value;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        arrived();
        LDS_BARRIER();
        request(b + (request.is_v ? 1 : 3) + (request.wave & 1));
        one(b);
        pipe.template block<true, !FIRST, 0>((K0 + 1) % 4 * SLOT, (K0 + 3) % 4 * SLOT);
        two(b);
        pipe.template block<!LAST, true, 1>((K0 + 2) % 4 * SLOT, K0 * SLOT);
    };
    using std::true_type;
    using std::false_type;
    if constexpr (TWO_MORE) {
        // the last pair is the other one
        if (nblk == 2) {
            pair(false_type{}, true_type{}, true_type{}, 0);
        } else {
            pair(false_type{}, true_type{}, false_type{}, 0);
            for (int b = 2; b < nblk - 4; b += 4) {
                pair(true_type{}, false_type{}, false_type{}, b);
                pair(false_type{}, false_type{}, false_type{}, b + 2);
            }
            pair(true_type{}, false_type{}, false_type{}, nblk - 4);
            pair(false_type{}, false_type{}, true_type{}, nblk - 2);
        }
    } else {
        pair(false_type{}, true_type{}, false_type{}, 0);
        for (int b = 2; b < nblk - 2; b += 4) {
            pair(true_type{}, false_type{}, false_type{}, b);
            pair(false_type{}, false_type{}, false_type{}, b + 2);
        }
        pair(true_type{}, false_type{}, true_type{}, nblk - 2);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // V of the last block was requested in front of the block before it
    LDS_BARRIER();
    constexpr int last_v = TWO_MORE ? SLOT : 3 * SLOT;
    pipe.rescale();
    pipe.template begin<false, true>(0, last_v);
    pipe.template steps<false, true, 0, false, 0>(0, last_v, 0.f);   // P V of the last block (parity 1)
}

// LDS of the patch path: K ring, V ring (below 64 KB: the reach of M0 as LDS address), the waves' check results, table offsets
// of every block for either half-wave, the waves' bias tables
inline __host__ __device__ int patch_blocks_bytes(int n_blocks) { return (n_blocks * 8 + 15) & ~15; }
template <int D>
inline __host__ __device__ size_t patch_lds_bytes(int w, int n_blocks)
{
    return (size_t)2 * AttnPipe<D, 0>::RING + 16 + patch_blocks_bytes(n_blocks) + (size_t)4 * wave_scratch_bytes<D>(glb_tstr(w));
}

// The bias table (layout of build_bias_rows) of a wave whose 32 queries are a patch: rows qr0 .. qr0 + 6 and columns
// qc0 .. qc0 + 14 in steps of two, so that only w + 6 and w + 14 relative positions occur, and away from both ends every one of
// them is an entry of every query: one conversion and one store per entry (the general form spends
// nine vector instructions on one; at 64 x 64 the tables took 107 us of 850, now 65).
template <int D>
__device__ __forceinline__ void build_bias_rows_patch(const bf16x8 *qf, const bf16 *rel_h, const bf16 *rel_w, int w, int lgw, int qrow, int qcol,
                                                      int qr0, int qc0, GlbTab *tq_lane, float inv_scale)
{
    constexpr int KS = AttnCfg<D>::KS;
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    const int nrel = 2 * w - 1, hw = w >> 1;
    bf16x8 cur[2][KS], nxt[2][KS];
    auto load_slab = [&](bf16x8 (&a)[2][KS], int mt) {
#pragma unroll
        for (int tab = 0; tab < 2; ++tab) {
            const bf16 *src = (tab ? rel_w : rel_h) + min((tab ? qc0 : qr0) + mt * 32 + l32, nrel - 1) * D + half * 8;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) a[tab][ks] = *reinterpret_cast<const bf16x8 *>(src + ks * 16);
        }
    };
    load_slab(cur, 0);
    for (int mt = 0; mt * 32 < w + 14; ++mt) {
        load_slab(nxt, mt + 1);
#pragma unroll
        for (int tab = 0; tab < 2; ++tab) {
            f32x16 u;
#pragma unroll
            for (int r = 0; r < 16; ++r) u[r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) u = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur[tab][ks], qf[ks], u, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");          // MFMA passes done before u is read under branches
            __builtin_amdgcn_sched_barrier(0);
            // entry r of the lane is relative position q0 + mt*32 + 8*(r>>2) + 4*half + (r&3), i.e. key row p = p0 - 8*(r>>2) - (r&3)
            const int spread = tab ? 14 : 6, p0 = (tab ? qcol - qc0 : qrow - qr0) + w - 1 - mt * 32 - 4 * half;
            GlbTab *row = tq_lane + (tab ? 2 * hw : 0);
            GlbTab *ev = row + ((p0 & 1) << (lgw - 1)) + (p0 >> 1);              // where p0 lies; p0 - 2 is one entry in front of it
            GlbTab *od = row + (((p0 - 1) & 1) << (lgw - 1)) + ((p0 - 1) >> 1);  // where p0 - 1 lies
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int d0 = mt * 32 + 8 * g;                                  // the group's first relative position less q0
                if (d0 > w - 1 + spread) continue;                               // no query has these (wave-uniform, as below)
                if (d0 >= spread && d0 + 7 < w) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) ((e & 1) ? od : ev)[-4 * g - (e >> 1)] = (GlbTab)(u[4 * g + e] * inv_scale);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if ((unsigned)(p0 - 8 * g - e) < (unsigned)w) ((e & 1) ? od : ev)[-4 * g - (e >> 1)] = (GlbTab)(u[4 * g + e] * inv_scale);
                }
            }
        }
#pragma unroll
        for (int tab = 0; tab < 2; ++tab)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) cur[tab][ks] = nxt[tab][ks];
    }
}

// The patch path of a workgroup.  Any table is legal input, so the cells of every key it will visit (its own queries among
// them) are looked at first, under the latency of the first K, V and Q requests: false = some block is not a patch, nothing has
// been stored, and the caller takes the general path.  w is a power of two, 16 or more: S is a multiple of the tile.
template <int D>
__device__ __forceinline__ bool attn_patch_body(const AttnParams &P, int qt, int grp, int head, unsigned char *smem)
{
    using C = AttnCfg<D>;
    using Pipe = AttnPipe<D, 0>;
    constexpr int END = 2 * Pipe::RING;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, half = lane >> 5;
    const int lgw = 31 - __builtin_clz(P.w), nact = P.n_pre + (qt >= P.n_pre ? 1 : 0), nblk = nact * (GLB_TILE / 32);
    int *ok_words = reinterpret_cast<int *>(smem + END);
    uint32_t *bo_tab = reinterpret_cast<uint32_t *>(smem + END + 16);
    const int tstr = glb_tstr(P.w);
    unsigned char *Tb = smem + END + 16 + patch_blocks_bytes(nblk);
    GlbTab *tq = reinterpret_cast<GlbTab *>(Tb + wave * wave_scratch_bytes<D>(tstr));

    const long base = (long)grp * P.S * P.row_stride + (long)head * D;
    AttnRequests<D, false> request(P, qt, base, smem);
    request.first();

    const int qpos = qt * GLB_TILE + wave * 32 + l32;
    bf16x8 qf[C::KS];
    load_q_frags<D>(qf, P.q + base + (long)qpos * P.row_stride);
    const int32_t *sg = P.sigma + (long)grp * P.sigma_stride;
    const int qcell = sg[qpos];
    long my_row = (long)grp * P.S + qpos;         // output row of this lane's query
    if (P.out_rows) my_row = P.out_rows[my_row];

    // A key passes if it sits where the patch anchored at its block's first key puts it (inside the grid) and, for a block's
    // first key, the block's 4 row and 8 column entries start at 8- and 16-byte boundaries of a table row.
    bool ok = true;
    constexpr int BATCH = 8;                                            // cells per thread per pass: 16 tiles a pass
    for (int a = 0; a < nact; a += 2 * BATCH) {
        int cell[BATCH];
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {                               // the loads of a pass are in flight together
            const int a1 = min(a + 2 * j + (tid >> 7), nact - 1);       // this thread's tile (past the end: the last one again)
            cell[j] = sg[(a1 < P.n_pre ? a1 : qt) * GLB_TILE + (tid & 127)];
        }
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            const int a1 = min(a + 2 * j + (tid >> 7), nact - 1);
            const int c0 = __shfl(cell[j], lane & 32, 64);              // cell of the block's first key
            const int k = tid & 31, r0 = c0 >> lgw, cl0 = c0 & (P.w - 1);
            ok = ok && c0 >= 0 && r0 + 6 < P.w && cl0 + 14 < P.w && cell[j] == c0 + ((2 * patch_rr(k)) << lgw) + 2 * patch_cc(k);
            if (k == 0) {
                const uint32_t hw = (uint32_t)P.w >> 1, esz = sizeof(GlbTab);
                const uint32_t row = esz * ((r0 & 1) * hw + (r0 >> 1)), col = esz * (2 * hw + (cl0 & 1) * hw + (cl0 >> 1));
                ok = ok && (row & 7u) == 0 && (col & 15u) == 0;
                uint32_t *bo = bo_tab + 2 * (a1 * (GLB_TILE / 32) + ((tid & 127) >> 5));
                bo[0] = row | col << 16;                                // of the lower half-wave and the upper one (see load)
                bo[1] = (col + 8) | col << 16;
            }
        }
    }
    const bool wave_ok = __builtin_amdgcn_ballot_w64(!ok) == 0;
    if (lane == 0) ok_words[wave] = wave_ok;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the first blocks have landed
    __syncthreads();
    if ((ok_words[0] & ok_words[1] & ok_words[2] & ok_words[3]) == 0) {
        __syncthreads();                          // the words are part of another region from here on
        return false;
    }

    const int qrow = qcell >> lgw, qcol = qcell & (P.w - 1);
    GlbTab *tq_lane = tq + l32 * tstr;            // this lane's query row of the wave's bias table
    build_bias_rows_patch<D>(qf, P.rel_h, P.rel_w, P.w, lgw, qrow, qcol, __builtin_amdgcn_readfirstlane(qrow), __builtin_amdgcn_readfirstlane(qcol),
                             tq_lane, P.table_inv);
    WaveState<D> st;
    init_state<D>(st);

    Pipe pipe{ st, qf, smem, reinterpret_cast<const unsigned char *>(tq_lane), P.scale_log2e };
    // operand a of the bias product: lane (key l32, half) holds E[l32][8*half + e]
    const int rr = patch_rr(l32), cc = patch_cc(l32);
    const _Float16 one = __builtin_bit_cast(_Float16, (uint16_t)P.half_one);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int f = 8 * half + e;
        pipe.efrag[e] = (f < 4 ? rr == f : (f < 12 ? cc == f - 4 : false)) ? one : (_Float16)0.f;
    }
    pipe.addresses();

    pipe.bo = bo_tab[half];
    uint32_t bo1 = bo_tab[2 + half], bo2 = bo_tab[4 + half], next1, next2;
    attn_pipe_run<false>(pipe, request, nblk, [&]() {}, [&]() {},
        [&](int b) {
            pipe.bo = bo1;
            next1 = bo_tab[2 * min(b + 3, nblk - 1) + half], next2 = bo_tab[2 * min(b + 4, nblk - 1) + half];
        },
        [&](int) { pipe.bo = bo2; bo1 = next1; bo2 = next2; });
    finish_and_store<D, C::KSTR, false>(st, reinterpret_cast<bf16 *>(tq), P.out + (long)head * D, (long)P.h * D, my_row);
    return true;
}

// Any order, any S, up to 64 x 64 (WK = 32 or 64 entries a table): the pipeline of the patch path, whose bias is one product of the patch's
// entries, with the whole table row of a query instead, as in attn_window_step: B[k][q] = sum_p E[k][p] T[p][q], E a one at the key's row
// and a one at its column.  Three quarters of E's groups of four are known zeros and no group has two ones, so it is a structured-sparse operand: a
// 32x32x32 sparse product takes the time of a dense 32x32x16 one (15.6 ns against 15.4 on a SIMD, measured), four a block instead of eight at 64 entries, and a
// lane makes 16 dwords of E for a block, two instructions each.  T stays in registers, as its operands b.
// Tiles of 128 keys between two barriers with the dense products -> this, us: 2 images of 12 heads, 50 x 50, d = 64, r = 0.5 68.4 -> 54.3; content order of 64 x 64: 8 images
// of 16 heads, d = 80, r = 0.4 583 -> 482, 4 of d = 64 dense 577 -> 448, 1 of 12 heads 74 -> 60; 8 images of 32 x 32 40.1 -> 33.3, 4 of 20 x 20 16.8 -> 15.2.  What bounds it
// now: at large batches vector instructions issue in 61 % of the cycles (137 a block and wave), matrix pipes 39 % busy.
template <int D, int WK>
inline __host__ __device__ size_t onehot_lds_bytes()
{
    return (size_t)2 * AttnPipe<D, WK>::RING + (size_t)4 * wave_scratch_bytes<D>(2 * WK + 8);
}

template <int D, int WK, bool SHORT>
__device__ __forceinline__ void attn_onehot_body(const AttnParams &P, int qt, int grp, int head, unsigned char *smem)
{
    using C = AttnCfg<D>;
    using Pipe = AttnPipe<D, WK>;
    constexpr int TSTR = 2 * WK + 8;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), l32 = lane & 31, half = lane >> 5;
    const int S = P.S;
    GlbTab *tq = reinterpret_cast<GlbTab *>(smem + 2 * Pipe::RING + wave * wave_scratch_bytes<D>(TSTR));
    const long base = (long)grp * S * P.row_stride + (long)head * D;
    AttnRequests<D, true, SHORT> request(P, qt, base, smem);
    request.first();

    const int qpos = qt * GLB_TILE + wave * 32 + l32, qclamp = min(qpos, S - 1);
    bf16x8 qf[C::KS];
    load_q_frags<D>(qf, P.q + base + (long)qclamp * P.row_stride);
    const int32_t *sg = P.sigma + (long)grp * P.sigma_stride;
    const uint32_t qrc = key_row_col(sg, qclamp, S, P.w);
    const int nblk = request.nblk;
    auto cell_of = [&](int b) { return sg[min(request.key0(min(b, nblk - 1)) + l32, S - 1)]; };
    int cell0 = cell_of(0), cell1 = cell_of(1), cell2 = cell_of(2);
    GlbTab *tq_lane = tq + l32 * TSTR;            // this lane's query row of the wave's bias table
    build_bias_rows<D, GlbTab>(qf, P.rel_h, P.rel_w, D, P.w, (int)(qrc & 0xffffu), (int)(qrc >> 16), tq_lane, P.table_inv);
    wave_lds_fence();
    WaveState<D> st;
    init_state<D>(st);
    Pipe pipe{ st, qf, smem, nullptr, P.scale_log2e };
    pipe.w = P.w;
    pipe.per_w = ((1u << 20) + P.w - 1) / P.w;          // exact for cells below 4096: the error is below 4096 / 2^20 of a row
    pipe.half_one = P.half_one;
    pipe.addresses();
#pragma unroll
    for (int tab = 0; tab < 2; ++tab)
#pragma unroll
        for (int seg = 0; seg < Pipe::SEG; ++seg) {
            // operand b of the sparse product: a half-wave holds entries 8 * half .. + 7 and 16 + 8 * half .. + 7
            const f16x8 lo = *reinterpret_cast<const f16x8 *>(tq_lane + tab * WK + 32 * seg + 8 * half);
            const f16x8 hi = *reinterpret_cast<const f16x8 *>(tq_lane + tab * WK + 32 * seg + 8 * half + 16);
            pipe.t[tab][seg] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
        }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the first blocks have landed
    asm volatile("" : "+v"(cell0), "+v"(cell1), "+v"(cell2));
    LDS_BARRIER();
    int next1 = cell1, next2 = cell2;
    auto run = [&](auto two_more) {
        attn_pipe_run<decltype(two_more)::value>(pipe, request, nblk,
            [&]() {
                // The exponent reference begins as the maximum over two blocks (one more block's scores): the likelier a query's largest probability is
                // exactly 1, the smaller the error.  With that of the first alone it is 1 to 6 % larger.  Keys past the end repeat the last one here.
                pipe.cell = cell1;
                pipe.template begin<true, false>(Pipe::SLOT, 0);
                pipe.template steps<true, false, 0, false, 0>(Pipe::SLOT, 0, 0.f);
                float mx = pipe.s[1][0];
#pragma unroll
                for (int r = 1; r < 16; ++r) mx = fmaxf(mx, pipe.s[1][r]);
                pipe.start = mx;
                pipe.cell = cell0;
            },
            [&]() { asm volatile("" : "+v"(next1), "+v"(next2)); },        // the compiler's own wait for them is here, where nothing else is out
            [&](int b) {
                pipe.cell = next1;
                cell2 = next2;
                next1 = cell_of(b + 3);
                next2 = cell_of(b + 4);
                pipe.limit = S - request.key0(b);
            },
            [&](int b) {
                pipe.cell = cell2;
                pipe.limit = S - request.key0(b + 1);
            });
        long my_row = -1;                             // output row of this lane's query (not looked up before: no registers)
        if (qpos < S) {
            my_row = (long)grp * S + qpos;
            if (P.out_rows) my_row = P.out_rows[my_row];
        }
        finish_and_store<D, C::KSTR, false>(st, reinterpret_cast<bf16 *>(tq), P.out + (long)head * D, (long)P.h * D, my_row);
    };
    if (SHORT && (nblk & 2)) run(std::bool_constant<SHORT>{});
    else run(std::false_type{});
}

// Above 64 x 64: tiles of 128 keys through registers into LDS, the bias by look-ups (attn_chunk_step).  NB: key blocks per
// softmax chunk, as many as the register budget of two waves per SIMD allows.
template <int D, int NB>
__device__ __forceinline__ void attn_global_body(const AttnParams &P, int qt, int grp, int head, unsigned char *smem)
{
    using C = AttnCfg<D>;
    constexpr int LOADS = GLB_TILE * C::CH / 256;       // 16-byte chunks per thread per operand
    static_assert(GLB_TILE * C::CH % 256 == 0, "tile chunks must divide over the workgroup");
    const int wk = glb_wk(P.w), tstr = glb_general_tstr(P.w);
    bf16 *Ks = reinterpret_cast<bf16 *>(smem);
    bf16 *Vs = Ks + GLB_TILE * C::KSTR;
    unsigned char *Tb = reinterpret_cast<unsigned char *>(Vs + GLB_TILE * C::KSTR);
    const int wsb = wave_scratch_bytes<D>(tstr);
    uint32_t *krc = reinterpret_cast<uint32_t *>(Tb + 4 * wsb);    // [128] per key

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31;
    const int S = P.S;
    const long base = (long)grp * S * P.row_stride + (long)head * D;

    const int qpos = qt * GLB_TILE + wave * 32 + l32;
    const int qclamp = qpos < S ? qpos : S - 1;
    bf16x8 qf[C::KS];
    load_q_frags<D>(qf, P.q + base + (long)qclamp * P.row_stride);
    const int32_t *sg = P.sigma + (long)grp * P.sigma_stride;
    const uint32_t qrc = key_row_col(sg, qclamp, S, P.w);
    GlbTab *tq = reinterpret_cast<GlbTab *>(Tb + wave * wsb);
    GlbTab *tq_lane = tq + l32 * tstr;            // this lane's query row of the wave's bias table

    const int nact = P.n_pre + (qt >= P.n_pre ? 1 : 0);
    u32x4 rk[LOADS], rv[LOADS];
    int rcell = 0;
    // this (image, head)'s K and V: a uniform base and 32-bit byte offsets (S * row_stride * 2 < 2^31, checked on the host)
    const unsigned char *kbase = reinterpret_cast<const unsigned char *>(P.k + base);
    const unsigned char *vbase = reinterpret_cast<const unsigned char *>(P.v + base);
    const uint32_t rs2 = (uint32_t)P.row_stride * 2u;

    // WHAT: 1 = K and the keys' cells, 2 = V; the two halves are requested at different points of the
    // current tile's work so that the waves do not queue up behind each other's loads.
#define ATTN_LOAD_TILE(kt_, WHAT)                                                                       \
    {                                                                                                   \
        __builtin_amdgcn_sched_barrier(0);                                                              \
        const int key0_ = (kt_) * GLB_TILE;                                                             \
        _Pragma("unroll") for (int i = 0; i < LOADS; ++i)                                               \
        {                                                                                               \
            const int id = tid + i * 256, kl = id / C::CH, c = id - kl * C::CH;                         \
            /* keys past S repeat the last row (masked in the scores); 32-bit byte offset from a uniform base */ \
            const uint32_t off_ = (uint32_t)min(key0_ + kl, S - 1) * rs2 + (uint32_t)c * 16u;           \
            if ((WHAT) & 1) rk[i] = *reinterpret_cast<const u32x4 *>(kbase + off_);                     \
            if ((WHAT) & 2) rv[i] = *reinterpret_cast<const u32x4 *>(vbase + off_);                     \
        }                                                                                               \
        if (((WHAT) & 1) && tid < GLB_TILE)                                                             \
            rcell = sg[min(key0_ + tid, S - 1)]; /* used at the LDS store, not before */                \
        __builtin_amdgcn_sched_barrier(0);                                                              \
    }
#define ATTN_STORE_TILE()                                                                               \
    {                                                                                                   \
        _Pragma("unroll") for (int i = 0; i < LOADS; ++i)                                               \
        {                                                                                               \
            int id = tid + i * 256, key = id / C::CH, c = id % C::CH;                                   \
            *reinterpret_cast<u32x4 *>(Ks + key * C::KSTR + c * 8) = rk[i];                             \
            *reinterpret_cast<u32x4 *>(Vs + key * C::KSTR + c * 8) = rv[i];                             \
        }                                                                                               \
        if (tid < GLB_TILE) krc[tid] = 2 * cell_row_col(rcell, P.w) + ((uint32_t)wk << 17); \
    }

    ATTN_LOAD_TILE(0 < P.n_pre ? 0 : qt, 3)       // in flight while the bias rows are formed
    set_ones_columns<D>(Vs, GLB_TILE, tid, 256);
    build_bias_rows<D, GlbTab>(qf, P.rel_h, P.rel_w, D, P.w, (int)(qrc & 0xffffu), (int)(qrc >> 16), tq_lane, P.table_inv);

    WaveState<D> st;
    init_state<D>(st);
    for (int a = 0; a < nact; ++a) {
        const int kt = a < P.n_pre ? a : qt;
        LDS_BARRIER();                         // every wave is done with the previous tile
        ATTN_STORE_TILE()
        LDS_BARRIER();
        const int kt_next = a + 1 < P.n_pre ? a + 1 : qt;
        if (a + 1 < nact) ATTN_LOAD_TILE(kt_next, NB < GLB_TILE / 32 ? 1 : 3)     // one step per tile: nothing to put V between
        // the softmax / MFMA phase goes ahead of the other workgroup's tile traffic (loads, LDS stores, barriers)
        __builtin_amdgcn_s_setprio(1);
        const int nblk = min(GLB_TILE / 32, (S - kt * GLB_TILE + 31) / 32);     // blocks wholly past the end are skipped ...
#pragma unroll
        for (int c0 = 0; c0 < GLB_TILE / 32; c0 += NB) {
            if (c0 >= nblk) break;
            int blk[NB], key0[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) { blk[b] = c0 + b; key0[b] = kt * GLB_TILE + 32 * (c0 + b); }
            const bool ragged = key0[NB - 1] + 32 > S;                          // ... but for one in a chunk with a block that is not: masked
            const int nb = min(NB, nblk - c0);
            if (ragged) attn_chunk_step<D, NB, true, GlbTab>(st, qf, Ks, Vs, krc, blk, key0, nb, S, P.scale_log2e, tq_lane, tq_lane, P.table_one);
            else attn_chunk_step<D, NB, false, GlbTab>(st, qf, Ks, Vs, krc, blk, key0, nb, S, P.scale_log2e, tq_lane, tq_lane, P.table_one);
            if (NB < GLB_TILE / 32 && c0 == 0 && a + 1 < nact) ATTN_LOAD_TILE(kt_next, 2)
        }
        __builtin_amdgcn_s_setprio(0);
    }
    long my_row = -1;                             // output row of this lane's query (not looked up before: no registers)
    if (qpos < S) {
        my_row = (long)grp * S + qpos;
        if (P.out_rows) my_row = P.out_rows[my_row];
    }
    finish_and_store<D>(st, reinterpret_cast<bf16 *>(tq), P.out + (long)head * D, (long)P.h * D, my_row);
#undef ATTN_LOAD_TILE
#undef ATTN_STORE_TILE
}

template <int D>
size_t global_lds_bytes(int w)
{
    // K and V tile, the four waves' bias tables, per key (or per block) table offsets
    if (glb_operand(w)) return glb_operand(w) == 32 ? onehot_lds_bytes<D, 32>() : onehot_lds_bytes<D, 64>();
    return (size_t)2 * GLB_TILE * AttnCfg<D>::KSTR * 2 + (size_t)4 * wave_scratch_bytes<D>(glb_general_tstr(w)) + (size_t)GLB_TILE * 4;
}

// TRY_PATCH: the instantiation for a shared position-only order on a power-of-two grid (attn_patch_body, and one of the
// others where a block is not a patch).  !TRY_PATCH: those only.  SHORT: any order, of the last tile two blocks (see AttnRequests::blocks).
// d = 16 with tables of 32: four workgroups to a CU, for which registers nearly suffice by themselves (135): with three 28 x 28, 8 images of 16 heads, r = 0.4
// took 25.0 us instead of 21.0, 32 x 32 in position order 26.4 instead of 22.5, both longer than tiles of 128 keys between two barriers.
template <int D, bool TRY_PATCH, int WK, bool SHORT = false>
__global__ void __launch_bounds__(256, D == 16 && WK == 32 && !SHORT ? 4 : 2)
attn_global_kernel(AttnParams P, int T, int n_gh)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    // the query tiles of one (image, head) run on one XCD (workgroup b sits on XCD b & 7), whose L2 then
    // serves the re-reads of that problem's K and V tiles
    int qt = (blockIdx.x >> 3) % T;
    const int gh = ((blockIdx.x >> 3) / T) * 8 + (blockIdx.x & 7);
    if (gh >= n_gh) return;
    const int grp = gh / P.h, head = gh % P.h;
    clamp_fp16();                                               // (here and not at the table: nothing moves across it)
    if constexpr (TRY_PATCH) {
        if (attn_patch_body<D>(P, qt, grp, head, smem)) return;
        asm volatile("" : "+s"(qt));                            // nothing of what follows is computed in front of the patch path
    }
    if constexpr (WK != 0) attn_onehot_body<D, WK, SHORT>(P, qt, grp, head, smem);
    else attn_global_body<D, (D <= 64 ? 4 : 2)>(P, qt, grp, head, smem);
}

// CU count and LDS bytes per CU of the current device, asked once per device (host-side queries, no allocation)
struct DeviceShape { int cus; size_t lds; };
inline int device_shape(DeviceShape &out)
{
    static DeviceShape cache[64] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return SSAM_EHIP;
    if (cache[dev].cus == 0) {
        int cus = 0, lds = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return SSAM_EHIP;
        if (hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess || lds <= 0) return SSAM_EHIP;
        cache[dev].lds = (size_t)lds;
        cache[dev].cus = cus;                    // written last: a racing first call finds 0 and asks again
    }
    out = cache[dev];
    return SSAM_OK;
}

template <int D>
int launch_window_waves(const AttnParams &P, long n_problems, int nqb, hipStream_t st)
{
    const int nact = P.n_pre < nqb ? P.n_pre + 1 : nqb;
    const bool any = P.q_exp != 0 || (unsigned long)(P.S - 1) * P.row_stride * 2 + 2 * D > 0xffffffffUL;
    auto kern = any ? attn_window_kernel_waves<D, true> : attn_window_kernel_waves<D, false>;
    constexpr long MOST = 1L << 22;                       // a launch has fewer than 2^32 threads
    for (long p0 = 0; p0 < n_problems; p0 += MOST) {
        const int n = (int)(n_problems - p0 < MOST ? n_problems - p0 : MOST);
        hipLaunchKernelGGL(kern, dim3(8 * ssam_div_up(n, 8) * nqb), dim3(64), (WinWave<D, false>::lds_bytes(nact)), st, P, (int)p0, n, nqb);
    }
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

// The most problems that go to a wave a tile; above, staging a problem's K and V once for all of its tiles wins.  us, wave a tile | persistent.
//   d = 80: K and V of three blocks ahead of eight waves no longer fit beside Q in what a CU can request (14 x 14, 1600 problems 58.5 | 55, dense 90 | 77); few
//           problems leave the persistent workgroups' second round half empty (r = 0.4, 400 problems 18.6 | 19.5, 464 21.5 | 19.9; dense, 352 26.2 | 26.4,
//           400 27.5 | 26.6; one window of 16 heads, which the persistent kernel keeps on one XCD, 8 | 52).  With fewer tiles a workgroup has
//           fewer waves for the same requests, and wins later (r = 0.4: 12 x 12, 800 problems 24.5 | 30, 2400 62 | 65.5, dense, 4000 129 | 127.5; 10 x 10,
//           1600 32 | 36, 4800 85 | 85, r = 1 104 | 114; 9 x 9, 800 15.6 | 17.1, 3200 42.6 | 40.2) or never (8 x 8, 3200 30 | 42)
//   d = 64: four tiles, one to a SIMD, are the persistent kernel's best case; it wins where the tiles request K and V more than 2.5 times over (10 x 10, r = 0.4,
//           2048 28.4 | 28, 3200 41.5 | 39, 6400 78 | 71; 11 x 11, r = 0.75, 6400 100 | 91.5; r = 0.4, twice over, 3200 43.4 | 44.5)
//   below:  never (10 x 10, 6400 problems, r = 0.6, d = 32 58.7 | 75.6)
template <int D>
long window_waves_most(int nqb, int nact, int S, int cus)
{
    constexpr long ALL = 1L << 60;
    if (D == 64) return nqb == 4 && 4 * 32 * nact > 2.5 * S ? 8L * cus : ALL;
    switch (nqb) {
    case 1: case 2: return ALL;
    case 3: return 4L * cus;
    case 4: return 16L * cus;
    case 5: return 12L * cus;
    default: return (nact <= 5 ? 25L : 22L) * cus / 16;
    }
}

template <int D>
int launch_attention(const AttnParams &P, int groups, int mask_block, hipStream_t st)
{
    DeviceShape ds;
    if (int rc = device_shape(ds); rc != SSAM_OK) return rc;
    if (mask_block == 32) {
        const int nqb = ssam_div_up(P.S, 32), n_problems = groups * P.h;
        if (2 * P.w - 1 > 32) return SSAM_EUNSUPPORTED;       // a table is one 32-row MFMA tile, its entries one 16-entry operand
        if constexpr (D < 64) {
            return launch_window_waves<D>(P, n_problems, nqb, st);
        } else {
            const int nact = P.n_pre < nqb ? P.n_pre + 1 : nqb;
            if (P.q_exp != 0 || n_problems <= window_waves_most<D>(nqb, nact, P.S, ds.cus)) return launch_window_waves<D>(P, n_problems, nqb, st);
            size_t lds = window_lds_bytes<D>(nqb, P.w);
            if (lds > ds.lds) return SSAM_EUNSUPPORTED;
            // the queries of the next problem land in LDS through loads whose LDS address is a 16-bit immediate-free M0
            // offset: their landing area is first in LDS and must end below 64 KB
            if ((size_t)nqb * window_q_bytes<D>() > 64 * 1024) return SSAM_EUNSUPPORTED;
            auto kern = attn_window_kernel<D>;
            if (lds > 64 * 1024 &&
                hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
                return SSAM_EHIP;
            if (ssam_div_up((long)nqb * 32 * AttnCfg<D>::CH, nqb * 64) > WIN_MAX_LOADS) return SSAM_EUNSUPPORTED;
            // persistent workgroups: as many as fit on the device's CUs at once for this LDS footprint
            int per_cu = (int)(ds.lds / lds);
            if (per_cu < 1) per_cu = 1;
            if (per_cu > 4) per_cu = 4;
            int grid = n_problems < ds.cus * per_cu ? n_problems : ds.cus * per_cu;
            hipLaunchKernelGGL(kern, dim3(grid), dim3(nqb * 64), lds, st, P, groups);
        }
    } else {
        int T = ssam_div_up(P.S, GLB_TILE);
        size_t lds = global_lds_bytes<D>(P.w);
        // a shared table on a power-of-two grid of 16 x 16 or more can be the position-only order whose blocks are
        // patches; the kernel checks every tile, so any table is still handled correctly
        const bool patch = P.sigma_stride == 0 && P.w >= 16 && (P.w & (P.w - 1)) == 0;
        if (patch) {
            const size_t need = patch_lds_bytes<D>(P.w, (P.n_pre < T ? P.n_pre + 1 : T) * (GLB_TILE / 32));
            lds = need > lds ? need : lds;
        }
        if (lds > ds.lds) return SSAM_EUNSUPPORTED;
        const int wk = glb_operand(P.w);
        // SHORT takes registers: at d = 16 and 32 a CU holds fewer workgroups (36 x 36, 16 images, d = 32 108 | 124 us)
        const int rest = P.S % GLB_TILE;          // keys of the last tile
        const bool short_end = rest > 0 && rest <= 64 && (D >= 64 || (long)T * groups * P.h <= 2L * ds.cus);
        auto kern = wk == 32 && short_end ? attn_global_kernel<D, false, 32, true>
                  : wk == 64 && short_end ? attn_global_kernel<D, false, 64, true>
                  : wk == 32 ? (patch ? attn_global_kernel<D, true, 32> : attn_global_kernel<D, false, 32>)
                  : wk == 64 ? (patch ? attn_global_kernel<D, true, 64> : attn_global_kernel<D, false, 64>)
                             : (patch ? attn_global_kernel<D, true, 0> : attn_global_kernel<D, false, 0>);
        if (lds > 64 * 1024 &&
            hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
            return SSAM_EHIP;
        hipLaunchKernelGGL(kern, dim3((unsigned)((long)T * ssam_div_up(groups * P.h, 8) * 8)), dim3(256), lds, st, P, T, groups * P.h);
    }
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

}  // namespace

extern "C" int ssam_sparse_attention(const void *q, const void *k, const void *v, long row_stride,
                                     const void *rel_h, const void *rel_w, const int32_t *sigma,
                                     long sigma_group_stride, void *out, const int32_t *out_rows,
                                     int groups, int S, int w, int h, int d, int mask_block, double r,
                                     float scale, void *stream)
{
    if (!q || !k || !v || !rel_h || !rel_w || !sigma || !out) return SSAM_EINVAL;
    if (groups <= 0 || S <= 0 || w <= 0 || h <= 0 || d <= 0 || !(r > 0.0) || r > 1.0) return SSAM_EINVAL;
    if (sigma_group_stride != 0 && sigma_group_stride < S) return SSAM_EINVAL;
    if (w * w != S || row_stride < (long)h * d || row_stride % 8 != 0) return SSAM_EINVAL;
    if (!ssam_aligned16(q) || !ssam_aligned16(k) || !ssam_aligned16(v) || !ssam_aligned16(rel_h) ||
        !ssam_aligned16(rel_w) || !ssam_aligned16(out))
        return SSAM_EINVAL;
    if (mask_block == 32) {
        if (S > 224) return SSAM_EUNSUPPORTED;
    } else if (mask_block == 128) {
        if (S > 16384 || (long)ssam_div_up(S, 128) * ((long)groups * h + 7) > 0x7fffffffL) return SSAM_EUNSUPPORTED;
        if ((long)S * row_stride * 2 > 0x7fffffffL) return SSAM_EUNSUPPORTED;      // the kernel's 32-bit byte offsets within a group
    } else {
        return SSAM_EUNSUPPORTED;
    }
    if (w > 128) return SSAM_EUNSUPPORTED;
    AttnParams P;
    P.q = (const bf16 *)q; P.k = (const bf16 *)k; P.v = (const bf16 *)v;
    P.row_stride = row_stride;
    P.rel_h = (const bf16 *)rel_h; P.rel_w = (const bf16 *)rel_w;
    P.sigma = sigma;
    P.sigma_stride = sigma_group_stride;
    P.out = (bf16 *)out;
    P.out_rows = out_rows;
    P.S = S; P.w = w; P.h = h;
    P.n_pre = ssam_prefix_tiles(ssam_div_up(S, mask_block), r);
    if (!(scale > 0.f)) return SSAM_EINVAL;      // the bias tables hold bias / scale
    int shift = bias_shift(scale);
    P.q_exp = 0;
    if (mask_block == 32) {
        const WindowScale ws = window_scale(scale);
        shift = ws.shift;
        P.q_exp = ws.q_exp;
        scale = ldexpf(scale, -ws.q_exp);
    }
    P.scale_log2e = scale * LOG2E;
    P.half_one = 0x3c00u + ((uint32_t)shift << 10);
    P.table_one = ldexpf(1.f, shift);
    P.table_inv = ldexpf(1.f / scale, -shift);
    hipStream_t st = (hipStream_t)stream;
    switch (d) {
    case 64: return launch_attention<64>(P, groups, mask_block, st);
    case 80: return launch_attention<80>(P, groups, mask_block, st);
    case 32: return launch_attention<32>(P, groups, mask_block, st);
    case 16: return launch_attention<16>(P, groups, mask_block, st);
    default: return SSAM_EUNSUPPORTED;
    }
}
