// Composition of the structured-sparse encoder block: Stripe-Sort attention half
// (Sec. 4.1, App. A.1) and Residual-Consistency MLP half (Sec. 4.2), and the
// stack of blocks that shares one keep-set (Sec. 1, Sec. 4.1 "performed once").
// Host code only: every step is a kernel of this library enqueued on the
// caller's stream; intermediate tensors live in the caller's workspace.
#include "gemm_kernel.h"

int ssam_linear_impl(const void *A, const void *W, const float *bias, void *C, int M, int N, int K,
                     const GemmLd &ld, bool packed, int epilogue, const GemmRowMap &rm, int tile,
                     void *split_ws, size_t split_ws_bytes, hipStream_t st, const GemmParts &parts = GemmParts{}, WarmAhead *warm = nullptr);
int ssam_parts_form_of(int rows, int kept, int D, int Dm);

int ssam_compact_slots(const int32_t *table, int table_batch_stride, int B, int Nout, int N,
                       int32_t *real_slot, int32_t *real_spatial, int32_t *slot_row, int32_t *pad_slot, hipStream_t st);
int ssam_ln_gather_impl(const void *x, const int32_t *idx, int idx_batch_stride, const float *gamma, const float *beta, float eps, void *y,
                        int B, int Nin, int Nout, int D, const PadFill &fill, void *stream);
int ssam_select_and_tables(const float *scores, int32_t *keep_idx, int B, int N, int K, const BlockTables &local, const BlockTables &global, hipStream_t st);
int ssam_invert_table(const int32_t *table, int table_batch_stride, int B, int Nout, int N, int32_t *inv, hipStream_t st);
int ssam_linear_ln_impl(const void *A, const float *stats, const void *Wfp, const float *colsum, const float *bias_f,
                        void *C, int M, int N, int K, const GemmLd &ld, const GemmRowMap &rm, hipStream_t st, const GemmParts &parts, const PadFill &fill, WarmAhead *warm);

int ssam_linear_fold_gelu_impl(const void *A, long rows_a, const int32_t *src, const float *stats, const void *Wfp, const float *colsum,
                               const float *bias_f, void *C, int M, int N, int K, const GemmLd &ld,
                               void *split_ws, size_t split_ws_bytes, hipStream_t st, const GemmParts &parts, int src_rows, int src_stride, WarmAhead *warm);
int ssam_ln_stats_impl(const void *x, float *stats, long rows, int D, float eps, const int32_t *idx, int idx_batch_stride,
                       int Nin, int Nout, int32_t *src, const PadFill &fill, hipStream_t st, int slots);

namespace {

inline size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }

struct BlockGeom {
    int S, w, nW, Nout, N, d;
};

bool block_geom(const ssam_block_cfg *c, BlockGeom &g)
{
    if (!c || c->B <= 0 || c->g <= 0 || c->D <= 0 || c->heads <= 0 || c->Dm <= 0 || c->ws < 0) return false;
    if (c->D % c->heads != 0 || c->K <= 0 || c->K > c->g * c->g) return false;
    g.N = c->g * c->g;
    g.w = c->ws > 0 ? c->ws : c->g;
    g.S = g.w * g.w;
    int nws = (c->g + g.w - 1) / g.w;
    g.nW = nws * nws;
    g.Nout = g.nW * g.S;
    g.d = c->D / c->heads;
    return true;
}

// gathered LN2 rows, hidden activations, then the K-split scratch of the fc2 contraction
size_t mlp_core_bytes(int B, int K, int D, int Dm)
{
    return align256((size_t)B * K * D * 2) + align256((size_t)B * K * Dm * 2);
}

size_t mlp_ws_bytes(int B, int K, int D, int Dm) { return mlp_core_bytes(B, K, D, Dm) + GEMM_SPLIT_WS_BYTES; }

// Tables that let the dense contractions of a windowed block skip the padding slots (see
// compact_slots_kernel): real_slot, real_spatial [B][N], slot_row [B][Nout], pad_slot [B][Nout-N].
struct PadTables {
    int32_t *real_slot, *real_spatial, *slot_row, *pad_slot;
};

size_t pad_tables_bytes(int B, const BlockGeom &g)
{
    if (g.Nout == g.N) return 0;
    return align256((size_t)B * g.N * 4) * 2 + align256((size_t)B * g.Nout * 4) + align256((size_t)B * (g.Nout - g.N) * 4);
}

PadTables carve_pad_tables(unsigned char *p, int B, const BlockGeom &g)
{
    PadTables t;
    t.real_slot = (int32_t *)p;
    p += align256((size_t)B * g.N * 4);
    t.real_spatial = (int32_t *)p;
    p += align256((size_t)B * g.N * 4);
    t.slot_row = (int32_t *)p;
    p += align256((size_t)B * g.Nout * 4);
    t.pad_slot = (int32_t *)p;
    return t;
}

// Tables of a block that depend only on its gather table, kept behind everything a block writes so that a stack
// builds them once: the padding tables (windowed blocks with padding), then slot_of [B][N], the scan-order slot of
// every token (the inverse of the gather table; the folded-LN1 qkv contraction walks the tokens in memory order
// and stores each row to its slot).
size_t block_tables_bytes(int B, const BlockGeom &g) { return pad_tables_bytes(B, g) + align256((size_t)B * g.N * 4); }

int32_t *slot_of_table(unsigned char *tables, int B, const BlockGeom &g) { return (int32_t *)(tables + pad_tables_bytes(B, g)); }

// slots: some block folds its LayerNorm into the qkv contraction and reads slot_of
BlockTables block_tables(const ssam_block_cfg *cfg, const BlockGeom &g, const int32_t *gather_table, unsigned char *tables, bool slots)
{
    const int per_image = cfg->content_order != 0;
    BlockTables t = { gather_table, per_image ? g.Nout : 0, g.Nout, per_image ? cfg->B : 1 };
    if (g.Nout != g.N) {
        const PadTables pt = carve_pad_tables(tables, cfg->B, g);
        t.real_slot = pt.real_slot;
        t.real_spatial = pt.real_spatial;
        t.slot_row = pt.slot_row;
        t.pad_slot = pt.pad_slot;
    }
    if (slots) t.slot_of = slot_of_table(tables, cfg->B, g);
    return t;
}

int build_block_tables(const ssam_block_cfg *cfg, const BlockGeom &g, const int32_t *gather_table, unsigned char *tables, bool slots, hipStream_t st)
{
    const BlockTables t = block_tables(cfg, g, gather_table, tables, slots);
    if (t.real_slot) {
        int rc = ssam_compact_slots(t.table, t.table_batch_stride, cfg->B, g.Nout, g.N, t.real_slot, t.real_spatial, t.slot_row, t.pad_slot, st);
        if (rc != SSAM_OK) return rc;
    }
    if (!t.slot_of) return SSAM_OK;
    return ssam_invert_table(t.table, t.table_batch_stride, t.slot_images, g.Nout, g.N, t.slot_of, st);
}

}  // namespace

extern "C" size_t ssam_routed_mlp_workspace_bytes(int B, int K, int D, int Dm)
{
    if (B <= 0 || K <= 0 || D <= 0 || Dm <= 0) return 0;
    return mlp_ws_bytes(B, K, D, Dm);
}

// colsum1 != NULL: gather and LN2 folded into fc1 (w1 the packed folded weight, b1 the folded bias; ln_g, ln_b unused)
// parts: row statistics of x in pieces, read by fc1 instead of a statistics launch; left: what fc2 does with them (see ssam_linear_impl); split_bytes: what is
// left of the K-split scratch beside them
static int routed_mlp_impl(void *x, const int32_t *keep_idx, const float *ln_g, const float *ln_b, float eps,
                           const void *w1, const float *b1, const void *w2, const float *b2, bool packed,
                           int B, int N, int D, int Dm, int K,
                           void *workspace, size_t workspace_bytes, void *stream, const float *colsum1 = nullptr, const GemmParts &parts = GemmParts{},
                           const GemmParts &left = GemmParts{}, WarmAhead *warm = nullptr, size_t split_bytes = GEMM_SPLIT_WS_BYTES)
{
    const bool fold = colsum1 != nullptr;
    if (!x || !keep_idx || (!fold && (!ln_g || !ln_b)) || !w1 || !b1 || !w2 || !b2 || !workspace) return SSAM_EINVAL;
    if (fold && (!packed || !ssam_aligned16(colsum1) || !ssam_aligned16(b1))) return SSAM_EINVAL;
    if (B <= 0 || N <= 0 || D <= 0 || Dm <= 0 || K <= 0 || K > N) return SSAM_EINVAL;
    if (!ssam_aligned16(workspace)) return SSAM_EINVAL;
    if (D % 8 != 0 || Dm % 8 != 0) return SSAM_EUNSUPPORTED;
    if (packed && (D % 128 != 0 || Dm % 128 != 0)) return SSAM_EUNSUPPORTED;
    if (workspace_bytes < mlp_ws_bytes(B, K, D, Dm)) return SSAM_EWORKSPACE;
    unsigned char *ws = (unsigned char *)workspace;
    void *a2 = ws;
    void *hid = ws + align256((size_t)B * K * D * 2);
    void *split = ws + mlp_core_bytes(B, K, D, Dm);
    hipStream_t st = (hipStream_t)stream;
    int rc;
    if (warm) warm->now += 1;
    if (fold && parts.at) {
        rc = ssam_linear_fold_gelu_impl(x, (long)B * N, keep_idx, nullptr, w1, colsum1, b1, hid, B * K, Dm, D, GemmLd{ D, D, Dm }, split, split_bytes, st, parts, K, N, warm);
    } else if (fold) {
        // the region of the normalised rows holds only their statistics and the rows of x they are (8 + 4 bytes a row)
        float *stats = (float *)a2;
        int32_t *src = (int32_t *)(stats + 2 * (size_t)B * K);
        rc = ssam_ln_stats_impl(x, stats, (long)B * K, D, eps, keep_idx, K, N, K, src, PadFill{}, st, 0);
        if (rc != SSAM_OK) return rc;
        rc = ssam_linear_fold_gelu_impl(x, (long)B * N, src, stats, w1, colsum1, b1, hid, B * K, Dm, D, GemmLd{ D, D, Dm }, split, split_bytes, st, GemmParts{}, 1, 0, warm);
    } else {
        rc = ssam_ln_gather(x, keep_idx, K, ln_g, ln_b, eps, a2, B, N, K, D, stream);
        if (rc != SSAM_OK) return rc;
        GemmRowMap none = { nullptr, 1, 0, 1 };
        rc = ssam_linear_impl(a2, w1, b1, hid, B * K, Dm, D, GemmLd{ D, D, Dm }, packed, SSAM_EPI_BIAS_GELU, none, 0, split, split_bytes, st, GemmParts{}, warm);
    }
    if (rc != SSAM_OK) return rc;
    GemmRowMap scatter = { keep_idx, K, K, N };
    if (warm) warm->now += 1;
    return ssam_linear_impl(hid, w2, b2, x, B * K, D, Dm, GemmLd{ Dm, Dm, D }, packed, SSAM_EPI_BIAS_SCATTER_ADD, scatter, 0,
                            split, split_bytes, st, left, warm);
}

extern "C" int ssam_routed_mlp(void *x, const int32_t *keep_idx, const float *ln_g, const float *ln_b, float eps,
                               const void *w1, const float *b1, const void *w2, const float *b2,
                               int B, int N, int D, int Dm, int K,
                               void *workspace, size_t workspace_bytes, void *stream)
{
    return routed_mlp_impl(x, keep_idx, ln_g, ln_b, eps, w1, b1, w2, b2, false, B, N, D, Dm, K, workspace, workspace_bytes, stream);
}

extern "C" int ssam_routed_mlp_packed(void *x, const int32_t *keep_idx, const float *ln_g, const float *ln_b, float eps,
                                      const void *w1p, const float *b1, const void *w2p, const float *b2,
                                      int B, int N, int D, int Dm, int K,
                                      void *workspace, size_t workspace_bytes, void *stream)
{
    return routed_mlp_impl(x, keep_idx, ln_g, ln_b, eps, w1p, b1, w2p, b2, true, B, N, D, Dm, K, workspace, workspace_bytes, stream);
}

extern "C" int ssam_routed_mlp_folded(void *x, const int32_t *keep_idx, float eps,
                                      const void *w1fp, const float *colsum1, const float *b1f, const void *w2p, const float *b2,
                                      int B, int N, int D, int Dm, int K,
                                      void *workspace, size_t workspace_bytes, void *stream)
{
    if (!colsum1) return SSAM_EINVAL;
    return routed_mlp_impl(x, keep_idx, nullptr, nullptr, eps, w1fp, b1f, w2p, b2, true, B, N, D, Dm, K, workspace, workspace_bytes, stream, colsum1);
}

// everything but the padding tables, which sit behind it (so that no step of either half overwrites them
// and a stack of blocks can build them once)
static size_t attn_half_bytes(const ssam_block_cfg *cfg, const BlockGeom &g)
{
    size_t rows = (size_t)cfg->B * g.Nout;
    return align256(rows * cfg->D * 2) + align256(rows * 3 * cfg->D * 2) + GEMM_SPLIT_WS_BYTES;
}

static size_t block_core_bytes(const ssam_block_cfg *cfg, const BlockGeom &g)
{
    // the two halves do not share memory: the padding slots of the qkv tensor can then keep their contents from
    // block to block (see fold_kv_bias)
    return attn_half_bytes(cfg, g) + mlp_ws_bytes(cfg->B, cfg->K, cfg->D, cfg->Dm);
}

extern "C" size_t ssam_encoder_block_workspace_bytes(const ssam_block_cfg *cfg)
{
    BlockGeom g;
    if (!block_geom(cfg, g)) return 0;
    return block_core_bytes(cfg, g) + block_tables_bytes(cfg->B, g);
}

// Form of the row statistics (ssam_parts_form_of) and the scratch in which fc1 and fc2 may cut K: the kernels of the longer rows do so beside the pieces that lie in
// the same scratch (a single block likewise: the same cuts, the same bits).
struct PartsPlan { int form; size_t split_bytes; };

static PartsPlan parts_plan(int rows, int kept, int D, int Dm)
{
    const size_t beside = gemm_split_beside_parts(rows, D);
    const int form = beside ? ssam_parts_form_of(rows, kept, D, Dm) : 0;
    return { form, form ? beside : GEMM_SPLIT_WS_BYTES };
}

// The same.  Host only, for tests; not part of the interface.
extern "C" int ssam_parts_plan(int rows, int kept, int D, int Dm, size_t *split_bytes)
{
    const PartsPlan plan = parts_plan(rows, kept, D, Dm);
    *split_bytes = plan.split_bytes;
    return plan.form;
}

// tables: this block's block_tables_bytes region; tables_ready: a stack has built it already
// parts_ready (a block of a stack): the row statistics of x in pieces (GemmParts) are up to date, on entry from the block before.  They lie at the end of the
// workspace's bytes in front of the tables, the K-split scratch of the MLP; a stack's blocks all have the same end.  proj writes every row, and with it its
// pieces, which fc1 reads; where the next block's qkv reads them too (ssam_parts_form_of: 3) fc2 keeps them up to date and nothing uses that scratch, else they
// are done with when fc2, which may use it, begins; where D > 1024 fc1 and fc2 use what is in front of them.
static int encoder_block_impl(void *x, const ssam_block_weights *w, const ssam_block_cfg *cfg,
                              const int32_t *gather_table, const int32_t *sigma, const int32_t *keep_idx,
                              void *workspace, size_t workspace_bytes, void **qkv_events, unsigned char *tables,
                              bool tables_ready, bool *pad_rows_zero, bool *parts_ready, WarmAhead *warm, void *stream)
{
    BlockGeom g;
    if (!x || !w || !gather_table || !sigma || !keep_idx || !workspace || !block_geom(cfg, g)) return SSAM_EINVAL;
    if (!(cfg->r > 0.0) || cfg->r > 1.0) return SSAM_EINVAL;
    if (!ssam_aligned16(workspace) || !ssam_aligned16(x)) return SSAM_EINVAL;
    if (cfg->D % 128 != 0 || cfg->Dm % 128 != 0) return SSAM_EUNSUPPORTED;
    if (!tables) {
        if (workspace_bytes < ssam_encoder_block_workspace_bytes(cfg)) return SSAM_EWORKSPACE;
        workspace_bytes = block_core_bytes(cfg, g);
        tables = (unsigned char *)workspace + workspace_bytes;
    }
    const int B = cfg->B, D = cfg->D;
    const int rows = B * g.Nout;                               // slots of the scan-order layout (with padding)
    const bool padded = g.Nout != g.N;
    const int crows = B * g.N;                                 // rows the dense contractions multiply (real tokens)
    unsigned char *ws = (unsigned char *)workspace;
    void *u = ws;                                             // LN1(x) in scan order; later the attention output
    void *qkv = ws + align256((size_t)rows * D * 2);
    unsigned char *split = ws + align256((size_t)rows * D * 2) + align256((size_t)rows * 3 * D * 2);   // K-split scratch of the left-over launches
    hipStream_t st = (hipStream_t)stream;
    const int per_image = cfg->content_order != 0;             // tables carry a leading [B] dimension
    const bf16 *qp = (const bf16 *)qkv;
    const bool packed = w->packed != 0;
    GemmRowMap none = { nullptr, 1, 0, 1 };
    int rc;
    const bool fold = w->fold_ln1 != 0;
    const bool kv_shift = w->fold_kv_bias != 0;
    if (fold) {
        if (!packed || !w->qkv_colsum || !w->bqkv_folded) return SSAM_EINVAL;
        if (crows % 128 != 0 || (3 * D) % 256 != 0) return SSAM_EUNSUPPORTED;
    }
    if (kv_shift && (!fold || !w->bproj_folded)) return SSAM_EINVAL;
    const float *bproj = kv_shift ? w->bproj_folded : w->bproj;
    const size_t parts_bytes = gemm_parts_bytes(crows, D);
    const auto [form, split_bytes] = fold && w->fold_ln2 != 0 ? parts_plan(crows, B * cfg->K, D, cfg->Dm) : PartsPlan{ 0, GEMM_SPLIT_WS_BYTES };
    const GemmParts parts = form ? GemmParts{ (float2 *)((unsigned char *)workspace + (workspace_bytes & ~(size_t)255) - parts_bytes), D / 64, cfg->eps } : GemmParts{};
    const GemmParts whole = form == 3 ? parts : GemmParts{}, tile_only = { nullptr, whole.slots, cfg->eps };       // (in a single block: a stack's blocks are then the same bits)
    const bool have_parts = whole.at && parts_ready && *parts_ready;
    if (parts_ready) *parts_ready = whole.at != nullptr;
    if (!tables_ready) {
        rc = build_block_tables(cfg, g, gather_table, tables, fold, st);
        if (rc != SSAM_OK) return rc;
    }
    // The padding slots hold the qkv of a zero row: the bias, or, with the key and value biases taken out of the contraction,
    // zeros in the columns attention reads (k, v), which then need writing only when something else has used the memory
    // since.  The LayerNorm's launch writes them, or the contraction's where it needs none.
    PadFill fill = {};
    if (padded && !(kv_shift && pad_rows_zero && *pad_rows_zero))
        fill = { (bf16 *)qkv, 3L * D, kv_shift ? nullptr : w->bqkv, 3 * D, carve_pad_tables(tables, B, g).pad_slot, g.Nout - g.N, g.Nout, B * (g.Nout - g.N) };
    if (pad_rows_zero) *pad_rows_zero = padded && kv_shift;         // (an unpadded block's qkv tensor lies over the windowed blocks' one)
    if (fold) {
        // LN1 folded into the qkv contraction: only the statistics of every token are taken here (parked at the
        // start of u, which nothing else uses before attention writes its output there); the contraction reads
        // the tokens where they lie and stores every row to its scan-order slot
        float *stats = (float *)u;
        if (!have_parts) {
            rc = ssam_ln_stats_impl(x, stats, crows, D, cfg->eps, nullptr, 0, 0, 0, nullptr, fill, st, whole.slots);
            if (rc != SSAM_OK) return rc;
        }
        if (qkv_events && qkv_events[0] && hipEventRecord((hipEvent_t)qkv_events[0], st) != hipSuccess) return SSAM_EHIP;
        GemmRowMap to_slot = { slot_of_table(tables, B, g), g.N, per_image ? g.N : 0, g.Nout };
        rc = ssam_linear_ln_impl(x, stats, w->wqkv, w->qkv_colsum, w->bqkv_folded, qkv, crows, 3 * D, D, GemmLd{ D, D, 3 * D }, to_slot, st, have_parts ? whole : tile_only, have_parts ? fill : PadFill{}, warm);
        if (rc != SSAM_OK) return rc;
    }

    if (!padded) {
        if (!fold) {
            rc = ssam_ln_gather(x, gather_table, per_image ? g.Nout : 0, w->ln1_g, w->ln1_b, cfg->eps, u, B, g.N, g.Nout, D, stream);
            if (rc != SSAM_OK) return rc;
            if (qkv_events && qkv_events[0] && hipEventRecord((hipEvent_t)qkv_events[0], st) != hipSuccess) return SSAM_EHIP;
            rc = ssam_linear_impl(u, w->wqkv, w->bqkv, qkv, rows, 3 * D, D, GemmLd{ D, D, 3 * D }, packed, SSAM_EPI_BIAS, none, 0, split, GEMM_SPLIT_WS_BYTES, st, GemmParts{}, warm);
            if (rc != SSAM_OK) return rc;
        }
        if (qkv_events && qkv_events[1] && hipEventRecord((hipEvent_t)qkv_events[1], st) != hipSuccess) return SSAM_EHIP;
        rc = ssam_sparse_attention(qp, qp + D, qp + 2 * D, 3L * D, w->rel_h, w->rel_w, sigma, per_image ? g.S : 0, u, nullptr,
                                   B * g.nW, g.S, g.w, cfg->heads, g.d, cfg->mask_block, cfg->r,
                                   1.0f / sqrtf((float)g.d), stream);
        if (rc != SSAM_OK) return rc;
        warm->now += 1;
        GemmRowMap back = { gather_table, g.Nout, per_image ? g.Nout : 0, g.N };
        rc = ssam_linear_impl(u, w->wproj, bproj, x, rows, D, D, GemmLd{ D, D, D }, packed, SSAM_EPI_BIAS_SCATTER_ADD, back, 0, split, GEMM_SPLIT_WS_BYTES, st, parts, warm);
        if (rc != SSAM_OK) return rc;
    } else {
        // Windows with padding: the padding slots are zero rows after LN1, so their qkv rows are the bias and
        // their attention outputs are dropped.  LN1 gathers the N real tokens of every image into a compact
        // [B*N][D] matrix in scan order, the qkv contraction runs on those rows and scatters them to their
        // slots (the padding slots were filled above), attention writes only the real queries (compact
        // again), and the proj contraction scatters them back to spatial order.
        const PadTables pt = carve_pad_tables(tables, B, g);
        if (!fold) {
            rc = ssam_ln_gather_impl(x, pt.real_spatial, g.N, w->ln1_g, w->ln1_b, cfg->eps, u, B, g.N, g.N, D, fill, stream);
            if (rc != SSAM_OK) return rc;
            if (qkv_events && qkv_events[0] && hipEventRecord((hipEvent_t)qkv_events[0], st) != hipSuccess) return SSAM_EHIP;
            GemmRowMap to_slot = { pt.real_slot, g.N, g.N, g.Nout };
            rc = ssam_linear_impl(u, w->wqkv, w->bqkv, qkv, crows, 3 * D, D, GemmLd{ D, D, 3 * D }, packed, SSAM_EPI_BIAS_SCATTER, to_slot, 0, split, GEMM_SPLIT_WS_BYTES, st, GemmParts{}, warm);
            if (rc != SSAM_OK) return rc;
        }
        if (qkv_events && qkv_events[1] && hipEventRecord((hipEvent_t)qkv_events[1], st) != hipSuccess) return SSAM_EHIP;
        rc = ssam_sparse_attention(qp, qp + D, qp + 2 * D, 3L * D, w->rel_h, w->rel_w, sigma, per_image ? g.S : 0, u, pt.slot_row,
                                   B * g.nW, g.S, g.w, cfg->heads, g.d, cfg->mask_block, cfg->r,
                                   1.0f / sqrtf((float)g.d), stream);
        if (rc != SSAM_OK) return rc;
        warm->now += 1;
        GemmRowMap back = { pt.real_spatial, g.N, g.N, g.N };
        rc = ssam_linear_impl(u, w->wproj, bproj, x, crows, D, D, GemmLd{ D, D, D }, packed, SSAM_EPI_BIAS_SCATTER_ADD, back, 0, split, GEMM_SPLIT_WS_BYTES, st, parts, warm);
        if (rc != SSAM_OK) return rc;
    }
    const size_t attn_bytes = attn_half_bytes(cfg, g);
    if (w->fold_ln2 != 0) {
        if (!packed || !w->fc1_colsum || !w->b1_folded) return SSAM_EINVAL;
        return routed_mlp_impl(x, keep_idx, nullptr, nullptr, cfg->eps, w->w1, w->b1_folded, w->w2, w->b2, true,
                               B, g.N, D, cfg->Dm, cfg->K, ws + attn_bytes, mlp_ws_bytes(B, cfg->K, D, cfg->Dm), stream, w->fc1_colsum, parts, parts_ready ? whole : tile_only, warm, split_bytes);
    }
    return routed_mlp_impl(x, keep_idx, w->ln2_g, w->ln2_b, cfg->eps, w->w1, w->b1, w->w2, w->b2, packed,
                           B, g.N, D, cfg->Dm, cfg->K, ws + attn_bytes, mlp_ws_bytes(B, cfg->K, D, cfg->Dm), stream, nullptr, GemmParts{}, GemmParts{}, warm);
}

extern "C" int ssam_encoder_block(void *x, const ssam_block_weights *w, const ssam_block_cfg *cfg,
                                  const int32_t *gather_table, const int32_t *sigma, const int32_t *keep_idx,
                                  void *workspace, size_t workspace_bytes, void *stream)
{
    const int Dm = cfg ? cfg->Dm : 0;
    WarmAhead warm = { w, nullptr, 1, cfg ? cfg->D : 0, { Dm, Dm } };
    return encoder_block_impl(x, w, cfg, gather_table, sigma, keep_idx, workspace, workspace_bytes, nullptr, nullptr, false, nullptr, nullptr, &warm, stream);
}

extern "C" size_t ssam_encoder_workspace_bytes(const ssam_block_cfg *cfg_local, const ssam_block_cfg *cfg_global)
{
    // what either kind of block writes, then the tables of the windowed blocks, then those of the global blocks
    BlockGeom gl, gg;
    const bool l = cfg_local && block_geom(cfg_local, gl), g = cfg_global && block_geom(cfg_global, gg);
    if ((cfg_local && !l) || (cfg_global && !g)) return 0;
    size_t core = 0, tables = 0;
    if (l) { core = block_core_bytes(cfg_local, gl); tables += block_tables_bytes(cfg_local->B, gl); }
    if (g) { size_t c = block_core_bytes(cfg_global, gg); core = c > core ? c : core; tables += block_tables_bytes(cfg_global->B, gg); }
    const ssam_block_cfg *c = cfg_local ? cfg_local : cfg_global;
    size_t s = c ? align256(ssam_score_tokens_workspace_bytes(c->B, c->g, c->g)) : 0;
    return (core > s ? core : s) + tables;
}

// Either configuration may be missing where no block is of its kind.
static WarmAhead warm_of_stack(const ssam_block_weights *weights, const uint8_t *is_global, int n_blocks, const ssam_block_cfg *cfg_local, const ssam_block_cfg *cfg_global)
{
    const ssam_block_cfg *c0 = cfg_local ? cfg_local : cfg_global;
    return { weights, is_global, n_blocks, c0->D, { cfg_local ? cfg_local->Dm : 0, cfg_global ? cfg_global->Dm : 0 } };
}

// What the launch of contraction `now` of a stack reads ahead (WarmAhead::pieces).  Host only, for tests; not part of the interface.
extern "C" int ssam_warm_pieces_of_stack(const ssam_block_weights *weights, const uint8_t *is_global, int n_blocks, const ssam_block_cfg *cfg_local, const ssam_block_cfg *cfg_global,
                                         int now, int groups, double most_bytes, const void **at, uint32_t *bytes)
{
    return warm_of_stack(weights, is_global, n_blocks, cfg_local, cfg_global).pieces(now, groups, most_bytes, at, bytes);
}

extern "C" int ssam_encoder_forward(void *x, const ssam_block_weights *weights, const uint8_t *is_global, int n_blocks,
                                    const ssam_block_cfg *cfg_local, const ssam_block_cfg *cfg_global,
                                    int32_t *window_table, int32_t *sigma_window,
                                    int32_t *global_table, int32_t *sigma_global,
                                    float *scores, int32_t *keep_idx,
                                    void *workspace, size_t workspace_bytes, void **qkv_events, void *stream)
{
    if (!x || !weights || !is_global || n_blocks <= 0 || !scores || !keep_idx || !workspace) return SSAM_EINVAL;
    bool any_local = false, any_global = false, slots_local = false, slots_global = false;
    for (int i = 0; i < n_blocks; ++i) {
        (is_global[i] ? any_global : any_local) = true;
        if (weights[i].fold_ln1 != 0) (is_global[i] ? slots_global : slots_local) = true;
    }
    if ((any_local && (!cfg_local || !window_table || !sigma_window)) ||
        (any_global && (!cfg_global || !global_table || !sigma_global)))
        return SSAM_EINVAL;
    const ssam_block_cfg *c0 = any_local ? cfg_local : cfg_global;
    if (any_local && any_global &&
        (cfg_local->B != cfg_global->B || cfg_local->g != cfg_global->g || cfg_local->D != cfg_global->D ||
         cfg_local->K != cfg_global->K))
        return SSAM_EINVAL;
    if (workspace_bytes < ssam_encoder_workspace_bytes(any_local ? cfg_local : nullptr, any_global ? cfg_global : nullptr))
        return SSAM_EWORKSPACE;
    if (any_local && any_global && (cfg_local->content_order != 0) != (cfg_global->content_order != 0)) return SSAM_EINVAL;
    int rc = ssam_score_tokens(x, scores, c0->B, c0->g, c0->g, c0->D, workspace, workspace_bytes, stream);
    if (rc != SSAM_OK) return rc;
    if (c0->content_order != 0) {                 // Sec. 4.1: the content-aware order is taken once, from these scores
        const int G = c0->stripe;
        if (G <= 0) return SSAM_EINVAL;
        if (any_local) {
            rc = ssam_build_content_tables(scores, c0->B, c0->g, cfg_local->ws, G, window_table, sigma_window, stream);
            if (rc != SSAM_OK) return rc;
        }
        if (any_global) {
            rc = ssam_build_content_tables(scores, c0->B, c0->g, cfg_global->ws, G, global_table, sigma_global, stream);
            if (rc != SSAM_OK) return rc;
        }
    }
    // the tables of either kind of block are the same for every block of that kind: built once, behind everything
    // the blocks write
    BlockGeom gl, gg;
    size_t core = 0;
    if (any_local) { if (!block_geom(cfg_local, gl)) return SSAM_EINVAL; core = block_core_bytes(cfg_local, gl); }
    if (any_global) {
        if (!block_geom(cfg_global, gg)) return SSAM_EINVAL;
        size_t c = block_core_bytes(cfg_global, gg);
        core = c > core ? c : core;
    }
    {
        size_t sc = align256(ssam_score_tokens_workspace_bytes(c0->B, c0->g, c0->g));
        core = core > sc ? core : sc;
    }
    unsigned char *tables_local = (unsigned char *)workspace + core;
    unsigned char *tables_global = tables_local + (any_local ? block_tables_bytes(cfg_local->B, gl) : 0);
    rc = ssam_select_and_tables(scores, keep_idx, c0->B, c0->g * c0->g, c0->K,
                                any_local ? block_tables(cfg_local, gl, window_table, tables_local, slots_local) : BlockTables{},
                                any_global ? block_tables(cfg_global, gg, global_table, tables_global, slots_global) : BlockTables{}, (hipStream_t)stream);
    if (rc != SSAM_OK) return rc;
    bool pad_rows_zero = false;                 // the padding slots of the windowed blocks' qkv tensor hold zeros
    bool parts_ready = false;                   // and the row statistics of x in pieces are up to date
    WarmAhead warm = warm_of_stack(weights, is_global, n_blocks, any_local ? cfg_local : nullptr, any_global ? cfg_global : nullptr);
    for (int i = 0; i < n_blocks; ++i) {
        warm.now = 4 * i;
        void **ev = qkv_events ? qkv_events + 2 * i : nullptr;
        rc = is_global[i]
                 ? encoder_block_impl(x, &weights[i], cfg_global, global_table, sigma_global, keep_idx, workspace, core, ev, tables_global, true, &pad_rows_zero, &parts_ready, &warm, stream)
                 : encoder_block_impl(x, &weights[i], cfg_local, window_table, sigma_window, keep_idx, workspace, core, ev, tables_local, true, &pad_rows_zero, &parts_ready, &warm, stream);
        if (rc != SSAM_OK) return rc;
    }
    return SSAM_OK;
}
