// HBM-bound kernels: row gather / scatter in scan order (Sec. 4.1), fused
// LayerNorm + gather, token scores (Eq. 1) and keep-set selection (Sec. 4.2).
// Every global access is a 16-byte vector per lane along the feature axis.
#include "common.h"

namespace {

// ---------------------------------------------------------------- permute
__global__ void __launch_bounds__(256)
permute_kernel(const uint4 *__restrict__ x, const int32_t *__restrict__ idx, uint4 *__restrict__ y,
               int B, int Nin, int Nout, int chunks)
{
    long total = (long)B * Nout * chunks;
    long stride = (long)gridDim.x * blockDim.x;
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
        int c = (int)(i % chunks);
        long row = i / chunks;
        int p = (int)(row % Nout);
        int b = (int)(row / Nout);
        int src = idx[p];
        uint4 v = make_uint4(0, 0, 0, 0);
        if (src >= 0 && src < Nin) v = x[((long)b * Nin + src) * chunks + c];
        y[i] = v;
    }
}

__global__ void __launch_bounds__(256)
unpermute_kernel(const uint4 *__restrict__ y, const int32_t *__restrict__ idx, uint4 *x,
                 const uint4 *residual, int B, int Nx, int Ny, int chunks)
{
    long total = (long)B * Ny * chunks;
    long stride = (long)gridDim.x * blockDim.x;
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
        int c = (int)(i % chunks);
        long row = i / chunks;
        int p = (int)(row % Ny);
        int b = (int)(row / Ny);
        int dst = idx[p];
        if (dst < 0 || dst >= Nx) continue;
        long o = ((long)b * Nx + dst) * chunks + c;
        uint4 v = y[i];
        if (residual) {
            float a[8], r[8];
            unpack_bf16x8(v, a);
            unpack_bf16x8(residual[o], r);
#pragma unroll
            for (int e = 0; e < 8; ++e) a[e] += r[e];
            v = pack_bf16x8(a);
        }
        x[o] = v;
    }
}

// ---------------------------------------------------------------- LN + gather
// One wave per output row; the row lives in registers (MAXC 16-byte chunks per
// lane), two-pass statistics in fp32.
template <int MAXC>
__global__ void __launch_bounds__(256)
ln_gather_kernel(const uint4 *__restrict__ x, const int32_t *__restrict__ idx, int idx_batch_stride,
                 const float *__restrict__ gamma, const float *__restrict__ beta, float eps,
                 uint4 *__restrict__ y, int B, int Nin, int Nout, int chunks, PadFill fill, int ln_blocks)
{
    int lane = threadIdx.x & 63;
    long row = (long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if ((int)blockIdx.x >= ln_blocks) {
        fill_pad_row(fill, ((int)blockIdx.x - ln_blocks) * 4 + (threadIdx.x >> 6));
        return;
    }
    if (row >= (long)B * Nout) return;
    int p = (int)(row % Nout), b = (int)(row / Nout);
    int src = idx[(long)b * idx_batch_stride + p];
    uint4 *yrow = y + row * chunks;
    if (src < 0 || src >= Nin) {
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            int c = lane + 64 * i;
            if (c < chunks) yrow[c] = make_uint4(0, 0, 0, 0);
        }
        return;
    }
    const uint4 *xrow = x + ((long)b * Nin + src) * chunks;
    // every load of the row is requested before the first is used, without predicates (a chunk index past the
    // row re-reads its last chunk and is masked in the arithmetic): behind `c < chunks` each load would be
    // waited for on its own, one memory round trip after the other
    uint4 raw[MAXC];
    float4 g0[MAXC], g1[MAXC], b0[MAXC], b1[MAXC];
#pragma unroll
    for (int i = 0; i < MAXC; ++i) raw[i] = xrow[min(lane + 64 * i, chunks - 1)];
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
        const int c = min(lane + 64 * i, chunks - 1);
        const float4 *g4 = reinterpret_cast<const float4 *>(gamma) + 2 * c;
        const float4 *b4 = reinterpret_cast<const float4 *>(beta) + 2 * c;
        g0[i] = g4[0]; g1[i] = g4[1]; b0[i] = b4[0]; b1[i] = b4[1];
    }
    float v[MAXC][8];
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
        unpack_bf16x8(raw[i], v[i]);
        if (lane + 64 * i < chunks) {
#pragma unroll
            for (int e = 0; e < 8; ++e) s += v[i][e];
        }
    }
    int D = chunks * 8;
    float mean = wave_sum(s) / (float)D;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
        if (lane + 64 * i < chunks) {
#pragma unroll
            for (int e = 0; e < 8; ++e) { float t = v[i][e] - mean; q += t * t; }
        }
    }
    float inv = rsqrtf(wave_sum(q) / (float)D + eps);
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
        int c = lane + 64 * i;
        if (c < chunks) {
            float gg[8] = { g0[i].x, g0[i].y, g0[i].z, g0[i].w, g1[i].x, g1[i].y, g1[i].z, g1[i].w };
            float bb[8] = { b0[i].x, b0[i].y, b0[i].z, b0[i].w, b1[i].x, b1[i].y, b1[i].z, b1[i].w };
            float o[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (v[i][e] - mean) * inv * gg[e] + bb[e];
            yrow[c] = pack_bf16x8(o);
        }
    }
}

// ---------------------------------------------------------------- LN statistics only
// The statistics half of the LayerNorm above, for a contraction that has the normalisation folded in:
// one wave per row, stats[row] = { rstd, -rstd * mean } (same two-pass fp32 arithmetic as ln_gather_kernel).
// With `idx` (the kept tokens of the routed MLP, [B][idx_batch_stride] positions inside an image of Nin rows) the
// statistics are those of the gathered rows, Nout per image, and src[row] receives the row of x that was read, for
// the contraction that gathers the same rows; an index outside [0, Nin) reads the image's first row (its result is
// dropped by the scatter that follows).
// slots != 0: the statistics are put together from the row's pieces of 64 columns, in the order of a contraction that reads pieces (GemmParts): the same bits.
template <int MAXC>
__global__ void __launch_bounds__(256)
ln_stats_kernel(const uint4 *__restrict__ x, float2 *__restrict__ stats, long rows, int chunks, float eps,
                const int32_t *__restrict__ idx, int idx_batch_stride, int Nin, int Nout, int32_t *__restrict__ src,
                PadFill fill, int ln_blocks, int slots)
{
    int lane = threadIdx.x & 63;
    long row = (long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if ((int)blockIdx.x >= ln_blocks) {
        fill_pad_row(fill, ((int)blockIdx.x - ln_blocks) * 4 + (threadIdx.x >> 6));
        return;
    }
    if (row >= rows) return;
    long xr = row;
    if (idx) {
        const int b = (int)(row / Nout), p = (int)(row - (long)b * Nout);
        int t = idx[(long)b * idx_batch_stride + p];
        if (t < 0 || t >= Nin) t = 0;
        xr = (long)b * Nin + t;
        if (lane == 0) src[row] = (int32_t)xr;
    }
    const uint4 *xrow = x + xr * chunks;
    uint4 raw[MAXC];
#pragma unroll
    for (int i = 0; i < MAXC; ++i) raw[i] = xrow[min(lane + 64 * i, chunks - 1)];
    float v[MAXC][8];
#pragma unroll
    for (int i = 0; i < MAXC; ++i) unpack_bf16x8(raw[i], v[i]);
    int D = chunks * 8;
    if constexpr (MAXC * 8 <= (GEMM_PARTS_MOST + 7) / 8 * 8) if (slots) {
        // piece (lane >> 3) + 8 * i, in its eight lanes: sums of columns 32 apart first
        float2 own[MAXC], other[MAXC];           // other: piece s ^ 4
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            float ps = gemm_piece_sum8(v[i]);
            ps += __shfl_xor(ps, 4, 64);
            ps += __shfl_xor(ps, 1, 64);
            ps += __shfl_xor(ps, 2, 64);
            const float pm = ps * (1.f / 64.f);
            float pq = gemm_piece_squares8(v[i], pm);
            pq += __shfl_xor(pq, 4, 64);
            pq += __shfl_xor(pq, 1, 64);
            pq += __shfl_xor(pq, 2, 64);
            own[i] = make_float2(pm, pq);
            other[i] = make_float2(__shfl_xor(pm, 32, 64), __shfl_xor(pq, 32, 64));
        }
        // pieces 4 * k + quad one after the other, then the four quads
        const int quad = (lane >> 3) & 3;
        const bool upper = lane >= 32;
        float2 piece[2 * MAXC];
#pragma unroll
        for (int k = 0; k < 2 * MAXC; ++k) piece[k] = upper == (k % 2 == 1) ? own[k / 2] : other[k / 2];
        auto over_quads = [](float t) { t += __shfl_xor(t, 8, 64); return t + __shfl_xor(t, 16, 64); };
        float mean = 0.f, sq = 0.f;
#pragma unroll
        for (int k = 0; k < 2 * MAXC; ++k)
            if (4 * k + quad < slots) mean += piece[k].x;
        mean = over_quads(mean) / (float)slots;
#pragma unroll
        for (int k = 0; k < 2 * MAXC; ++k)
            if (4 * k + quad < slots) sq += gemm_piece_term(piece[k], mean);
        const float inv = rsqrtf(over_quads(sq) / (float)D + eps);
        if (lane == 0) stats[row] = make_float2(inv, -inv * mean);
        return;
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
        if (lane + 64 * i < chunks) {
#pragma unroll
            for (int e = 0; e < 8; ++e) s += v[i][e];
        }
    }
    float mean = wave_sum(s) / (float)D;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
        if (lane + 64 * i < chunks) {
#pragma unroll
            for (int e = 0; e < 8; ++e) { float t = v[i][e] - mean; q += t * t; }
        }
    }
    float inv = rsqrtf(wave_sum(q) / (float)D + eps);
    if (lane == 0) stats[row] = make_float2(inv, -inv * mean);
}

// Weight side of the fold: one wave per output channel n.
//   Wf[n][k] = bf16(W[n][k] * gamma[k]);  colsum[n] = sum_k Wf[n][k] (the stored values);  bias_f[n] = bias[n] + sum_k beta[k] W[n][k]
__global__ void __launch_bounds__(256)
fold_ln_weight_kernel(const bf16 *__restrict__ W, int ldw, const float *__restrict__ bias, const float *__restrict__ gamma,
                      const float *__restrict__ beta, bf16 *__restrict__ Wf, float *__restrict__ colsum,
                      float *__restrict__ bias_f, int N, int K)
{
    int lane = threadIdx.x & 63;
    int n = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (n >= N) return;
    float cs = 0.f, bs = 0.f;
    for (int c = lane; c < K / 8; c += 64) {
        float w[8], o[8];
        unpack_bf16x8(*reinterpret_cast<const uint4 *>(W + (long)n * ldw + c * 8), w);
#pragma unroll
        for (int e = 0; e < 8; ++e) { o[e] = w[e] * gamma[c * 8 + e]; bs += beta[c * 8 + e] * w[e]; }
        uint4 packed = pack_bf16x8(o);
        *reinterpret_cast<uint4 *>(Wf + (long)n * K + c * 8) = packed;
        unpack_bf16x8(packed, o);
#pragma unroll
        for (int e = 0; e < 8; ++e) cs += o[e];
    }
    cs = wave_sum(cs);
    bs = wave_sum(bs);
    if (lane == 0) { colsum[n] = cs; bias_f[n] = bias[n] + bs; }
}

// Key and value biases taken out of the qkv contraction (softmax over keys does not see a term that is the same
// for every key, and the probabilities of a query sum to one): one wave per output channel.
//   bias_out[n] = bias_in[n] - (n >= D ? bqkv[n] : 0)   n < 3D;   bproj_out[j] = bproj[j] + sum_c wproj[j][c] bqkv[2D + c]
__global__ void __launch_bounds__(256)
fold_kv_bias_kernel(const float *__restrict__ bias_in, const float *__restrict__ bqkv, const bf16 *__restrict__ wproj,
                    const float *__restrict__ bproj, float *__restrict__ bias_out, float *__restrict__ bproj_out, int D)
{
    int lane = threadIdx.x & 63;
    int n = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (n >= 3 * D) return;
    if (lane == 0) bias_out[n] = bias_in[n] - (n >= D ? bqkv[n] : 0.f);
    if (n < D) {
        float acc = 0.f;
        for (int c = lane; c < D / 8; c += 64) {
            float w[8];
            unpack_bf16x8(*reinterpret_cast<const uint4 *>(wproj + (long)n * D + c * 8), w);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc += w[e] * bqkv[2 * D + c * 8 + e];
        }
        acc = wave_sum(acc);
        if (lane == 0) bproj_out[n] = bproj[n] + acc;
    }
}

// inv[b][table[b][p]] = p for every slot p that holds a token (table entries < 0 are padding)
__device__ __forceinline__ void invert_slot(int id, const int32_t *__restrict__ table, int table_batch_stride, int Nout, int N, int32_t *__restrict__ inv, int total)
{
    if (id >= total) return;
    int b = id / Nout, p = id - b * Nout;
    int s = table[(long)b * table_batch_stride + p];
    if (s >= 0 && s < N) inv[(long)b * N + s] = p;
}

__global__ void __launch_bounds__(256)
invert_table_kernel(const int32_t *__restrict__ table, int table_batch_stride, int Nout, int N, int32_t *__restrict__ inv, int total)
{
    invert_slot(blockIdx.x * 256 + threadIdx.x, table, table_batch_stride, Nout, N, inv, total);
}

// ---------------------------------------------------------------- scores
// channel sum of every token: one wave per token
__global__ void __launch_bounds__(256)
channel_sum_kernel(const uint4 *__restrict__ x, float *__restrict__ csum, long tokens, int chunks)
{
    int lane = threadIdx.x & 63;
    long t = (long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (t >= tokens) return;
    const uint4 *row = x + t * chunks;
    float s = 0.f;
    for (int c = lane; c < chunks; c += 64) {
        float f[8];
        unpack_bf16x8(row[c], f);
        s += ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
    }
    s = wave_sum(s);
    if (lane == 0) csum[t] = s;
}

// gradient magnitude of a cell from its eight neighbours
__device__ __forceinline__ float sobel(float a00, float a01, float a02, float a10, float a12, float a20, float a21, float a22)
{
    const float gx = (a02 - a00) + 2.f * (a12 - a10) + (a22 - a20);
    const float gy = (a20 - a00) + 2.f * (a21 - a01) + (a22 - a02);
    return sqrtf(gx * gx + gy * gy);
}

// Sobel magnitude with zero padding on the channel-sum map
__global__ void __launch_bounds__(256)
sobel_kernel(const float *__restrict__ csum, float *__restrict__ scores, int B, int gh, int gw)
{
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    long n = (long)gh * gw;
    if (i >= (long)B * n) return;
    int b = (int)(i / n), cell = (int)(i % n), row = cell / gw, col = cell % gw;
    const float *c = csum + (long)b * n;
    auto at = [&](int rr, int cc) -> float {
        return (rr < 0 || rr >= gh || cc < 0 || cc >= gw) ? 0.f : c[rr * gw + cc];
    };
    float a00 = at(row - 1, col - 1), a01 = at(row - 1, col), a02 = at(row - 1, col + 1);
    float a10 = at(row, col - 1), a12 = at(row, col + 1);
    float a20 = at(row + 1, col - 1), a21 = at(row + 1, col), a22 = at(row + 1, col + 1);
    scores[i] = sobel(a00, a01, a02, a10, a12, a20, a21, a22);
}

// Both in one launch, for few tokens: a workgroup scores 4 x 4 cells from the channel sums of 6 x 6, three of them to a wave with all of their
// loads in flight.  The sums are those of channel_sum_kernel, bit for bit; every row is read 2.25 times, most of that from the caches.
constexpr int SCORE_TILE = 4, SCORE_HALO = SCORE_TILE + 2, SCORE_PER_WAVE = 3, SCORE_THREADS = SCORE_HALO * SCORE_HALO / SCORE_PER_WAVE * 64;
template <int MAXC>
__global__ void __launch_bounds__(SCORE_THREADS)
score_kernel(const uint4 *__restrict__ x, float *__restrict__ scores, int gh, int gw, int chunks)
{
    __shared__ float cs[SCORE_HALO * SCORE_HALO];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r0 = (int)blockIdx.y * SCORE_TILE - 1, c0 = (int)blockIdx.x * SCORE_TILE - 1;
    const long base = (long)blockIdx.z * gh * gw;
    uint4 raw[SCORE_PER_WAVE][MAXC];
#pragma unroll
    for (int u = 0; u < SCORE_PER_WAVE; ++u) {
        const int t = wave * SCORE_PER_WAVE + u, row = min(max(r0 + t / SCORE_HALO, 0), gh - 1), col = min(max(c0 + t % SCORE_HALO, 0), gw - 1);
        const uint4 *src = x + (base + (long)row * gw + col) * chunks;
#pragma unroll
        for (int i = 0; i < MAXC; ++i) raw[u][i] = src[min(lane + 64 * i, chunks - 1)];
    }
#pragma unroll
    for (int u = 0; u < SCORE_PER_WAVE; ++u) {
        const int t = wave * SCORE_PER_WAVE + u, row = r0 + t / SCORE_HALO, col = c0 + t % SCORE_HALO;
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            float f[8];
            unpack_bf16x8(raw[u][i], f);
            if (lane + 64 * i < chunks) s += ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
        }
        s = wave_sum(s);
        if (lane == 0) cs[t] = row >= 0 && row < gh && col >= 0 && col < gw ? s : 0.f;
    }
    __syncthreads();
    const int rr = threadIdx.x / SCORE_TILE, cc = threadIdx.x % SCORE_TILE;
    if (rr >= SCORE_TILE || r0 + 1 + rr >= gh || c0 + 1 + cc >= gw) return;
    const float *c = cs + rr * SCORE_HALO + cc;                     // the cell's upper left neighbour
    constexpr int H = SCORE_HALO;
    scores[base + (long)(r0 + 1 + rr) * gw + c0 + 1 + cc] = sobel(c[0], c[1], c[2], c[H], c[H + 2], c[2 * H], c[2 * H + 1], c[2 * H + 2]);
}

// Up to 28 MB of tokens: there the second launch costs more than the rows read twice (us, one launch | two, from a loop of calls: 4096 x 768
// 6.6 | 9.3, the rate of the calls; 8192 x 1280, 21 MB, 7.4 | 9.2; 16384 x 768, 25 MB, 8.6 | 9.3; 16384 x 1024, 34 MB, 9.8 | 9.4; 65536 x 1280 39.8 | 32.4).
// And up to 1024 workgroups, whose twelve waves each take 3.7 ns of the launch: small images and thin grids have many of few cells (64 images of 14 x 14 x 768, 1024 of
// them, 8.3 | 7.5 to 9.4; 22 of 28 x 28 9.8 | the same; 3000 of 2 x 2 15.0 | 7.9; 256 x 256 x 144, 4096, 18.7 | 10.8; 20000 single tokens 74.8 | 7.6).  Far within the 65536 that the device
// states for the grid's z (images) and y (rows of tiles).
bool score_in_one_launch(int B, int gh, int gw, int D)
{
    return (long)B * gh * gw * D * 2 <= 28000000 && D <= 2048 && (long)B * ssam_div_up(gh, SCORE_TILE) * ssam_div_up(gw, SCORE_TILE) <= 1024;
}

// csum: where the channel sums of the form with two launches go
int launch_score(const void *x, float *scores, int B, int gh, int gw, int D, float *csum, hipStream_t st)
{
    const long tokens = (long)B * gh * gw;
    const int chunks = D / 8;
    if (score_in_one_launch(B, gh, gw, D)) {
        const dim3 grid(ssam_div_up(gw, SCORE_TILE), ssam_div_up(gh, SCORE_TILE), B);
        auto kern = chunks <= 128 ? score_kernel<2> : chunks <= 192 ? score_kernel<3> : score_kernel<4>;
        hipLaunchKernelGGL(kern, grid, dim3(SCORE_THREADS), 0, st, (const uint4 *)x, scores, gh, gw, chunks);
        SSAM_CHECK_LAUNCH();
        return SSAM_OK;
    }
    hipLaunchKernelGGL(channel_sum_kernel, dim3(ssam_div_up(tokens, 4)), dim3(256), 0, st, (const uint4 *)x, csum, tokens, chunks);
    SSAM_CHECK_LAUNCH();
    hipLaunchKernelGGL(sobel_kernel, dim3(ssam_div_up(tokens, 256)), dim3(256), 0, st, (const float *)csum, scores, B, gh, gw);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

// ---------------------------------------------------------------- select
// Order-preserving key: larger float <=> larger unsigned.  NaN -> -inf, -0 -> +0.
__device__ __forceinline__ uint32_t score_key(float s)
{
    uint32_t u = __float_as_uint(s);
    if ((u & 0x7fffffffu) > 0x7f800000u) u = 0xff800000u;   // NaN ranks as -inf
    if (u == 0x80000000u) u = 0u;                            // -0.0 == +0.0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// exclusive prefix sum of one flag per thread over the block; returns the
// thread's offset and (through total) the block total.  scratch: 16 ints.
__device__ __forceinline__ int block_exclusive_count(bool flag, int *scratch, int &total)
{
    int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long ballot = __ballot(flag);
    int before = __popcll(ballot & ((1ull << lane) - 1ull));
    if (lane == 0) scratch[wave] = __popcll(ballot);
    __syncthreads();
    int base = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < SEL_THREADS / 64; ++w) {
        int c = scratch[w];
        if (w < wave) base += c;
        sum += c;
    }
    __syncthreads();
    total = sum;
    return base + before;
}

// inclusive prefix sum over the lanes of a wave
template <typename T>
__device__ __forceinline__ T wave_inclusive_sum(T v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const T up = __shfl_up(v, o, 64);
        if (lane >= o) v += up;
    }
    return v;
}

// One workgroup per image: three passes of a radix select (11, 11 and 10 bits) find the key of the K-th largest score,
// then one scan over the workgroup places every index with a larger key and the lowest-index ties in ascending index
// order.  One CU works alone here, so what counts is the length of the serial chain: the keys are read once and kept in
// registers (ITEMS consecutive ones per thread; 16-byte loads), a pass is a histogram in LDS and a scan of its bins by
// all threads (4096 scores: 32 -> 6.7 us, 0.4 of it by clearing the bins of all passes under the first load; 16384: 45 -> 13; 65536: 151 -> 50; four 8-bit passes over memory with a serial
// walk of the bins and two barriers for every 1024 scores of the compaction before).  With ITEMS = 64 (more than 16384 scores) a
// thread's 128 registers do not hold its keys and all the rest: 42 of them go through scratch (16400 scores: 34 us).
constexpr int SEL_BINS = 2048;
template <int ITEMS>
__device__ __forceinline__ void select_image(const float *__restrict__ s, int32_t *__restrict__ out, int N, int K)
{
    __shared__ alignas(16) int hist[3][SEL_BINS];         // cleared by 16-byte stores
    __shared__ unsigned long long scratch[SEL_THREADS / 64];
    __shared__ uint32_t sh_prefix;
    __shared__ int sh_remaining;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int first = tid * ITEMS;
    for (int i = tid; i < 3 * SEL_BINS / 4; i += SEL_THREADS) reinterpret_cast<int4 *>(hist)[i] = make_int4(0, 0, 0, 0);      // under the latency of the scores

    uint32_t key[ITEMS];                        // past N: 0, below the key of every score
    if (first + ITEMS <= N && (reinterpret_cast<uintptr_t>(s) & 15) == 0) {
#pragma unroll
        for (int i = 0; i < ITEMS; i += 4) {
            const float4 v = *reinterpret_cast<const float4 *>(s + first + i);
            key[i] = score_key(v.x); key[i + 1] = score_key(v.y); key[i + 2] = score_key(v.z); key[i + 3] = score_key(v.w);
        }
    } else {
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) key[i] = first + i < N ? score_key(s[first + i]) : 0u;
    }

    __syncthreads();
    uint32_t prefix = 0, prefix_mask = 0;
    int remaining = K;   // how many of the keys matching the prefix are still to be taken
    constexpr int SHIFT[3] = { 21, 10, 0 }, BITS[3] = { 11, 11, 10 };
#pragma unroll
    for (int pass = 0; pass < 3; ++pass) {
        const uint32_t mask = (1u << BITS[pass]) - 1u;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (first + i < N && (key[i] & prefix_mask) == prefix) atomicAdd(&hist[pass][(key[i] >> SHIFT[pass]) & mask], 1);
        __syncthreads();
        // thread t holds bins 2t and 2t + 1 counted from the top: the bin in which the running count reaches `remaining`
        const int b0 = SEL_BINS - 1 - 2 * tid, b1 = b0 - 1;
        const int c0 = hist[pass][b0], c1 = hist[pass][b1];
        const int incl = wave_inclusive_sum(c0 + c1);
        if (lane == 63) scratch[wave] = (unsigned)incl;
        __syncthreads();
        int above = incl - (c0 + c1);
#pragma unroll
        for (int w = 0; w < SEL_THREADS / 64; ++w) above += w < wave ? (int)scratch[w] : 0;
        const bool in0 = above < remaining && above + c0 >= remaining, in1 = above + c0 < remaining && above + c0 + c1 >= remaining;
        if (in0 || in1) {                       // exactly one thread
            sh_prefix = prefix | ((uint32_t)(in0 ? b0 : b1) << SHIFT[pass]);
            sh_remaining = remaining - above - (in0 ? 0 : c0);
        }
        __syncthreads();
        prefix = sh_prefix;
        remaining = sh_remaining;
        prefix_mask |= mask << SHIFT[pass];
    }
    // prefix = key of the K-th largest element; `remaining` ties are taken, lowest index first
    const uint32_t threshold = prefix;
    uint32_t gt = 0, eq = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        gt += first + i < N && key[i] > threshold;
        eq += first + i < N && key[i] == threshold;
    }
    const unsigned long long mine = ((unsigned long long)gt << 32) | eq;
    const unsigned long long incl = wave_inclusive_sum(mine);
    __syncthreads();                            // the last pass has read scratch
    if (lane == 63) scratch[wave] = incl;
    __syncthreads();
    unsigned long long before = incl - mine;
#pragma unroll
    for (int w = 0; w < SEL_THREADS / 64; ++w) before += w < wave ? scratch[w] : 0ull;
    int ties = (int)(before & 0xffffffffu);
    int pos = (int)(before >> 32) + min(ties, remaining);
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const bool tie = key[i] == threshold;
        if (first + i < N && (key[i] > threshold || (tie && ties < remaining))) {
            if (pos < K) out[pos] = first + i;
            ++pos;
        }
        ties += first + i < N && tie;
    }
}

template <int ITEMS>
__global__ void __launch_bounds__(SEL_THREADS)
select_kernel(const float *__restrict__ scores, int32_t *__restrict__ keep, int N, int K)
{
    select_image<ITEMS>(scores + (long)blockIdx.x * N, keep + (long)blockIdx.x * K, N, K);
}

}  // namespace

// ---------------------------------------------------------------- entry points
static bool movers_args_ok(const void *a, const void *b, const void *c, int B, int n1, int n2, int D)
{
    return a && b && c && ssam_aligned16(a) && ssam_aligned16(c) && B > 0 && n1 > 0 && n2 > 0 && D > 0 && D % 8 == 0;
}

static int mover_grid(long total_chunks)
{
    long blocks = (total_chunks + 255) / 256;
    return (int)(blocks < 1 ? 1 : (blocks > 256L * 32 ? 256L * 32 : blocks));
}

// ---------------------------------------------------------------- padding compaction
// SAM pads the grid up to a multiple of the window; padding slots are zero rows after LN1, so their
// qkv rows equal the bias and their attention outputs are dropped.  One workgroup per image walks the
// gather table (slot -> spatial index, -1 = padding) in slot order and writes
//   real_slot[b][c]    the slot of the c-th real token (c-th row of the compact activations)
//   real_spatial[b][c] its spatial index
//   slot_row[b][s]     b*N + c for a real slot (the compact row), -1 for padding
//   pad_slot[b][i]     the i-th padding slot
// so that the dense contractions run on the N real rows only.
__device__ __forceinline__ void compact_image(int b, const int32_t *__restrict__ table, int table_batch_stride, int Nout, int N,
                                              int32_t *__restrict__ real_slot, int32_t *__restrict__ real_spatial,
                                              int32_t *__restrict__ slot_row, int32_t *__restrict__ pad_slot)
{
    __shared__ int scratch[SEL_THREADS / 64];
    const int npad = Nout - N;
    const int32_t *t = table + (long)b * table_batch_stride;
    int base = 0;
    for (int s0 = 0; s0 < Nout; s0 += SEL_THREADS) {
        const int s = s0 + threadIdx.x;
        const int v = s < Nout ? t[s] : -1;
        const bool real = s < Nout && v >= 0 && v < N;
        int total;
        const int c = base + block_exclusive_count(real, scratch, total);
        if (s < Nout) {
            if (real) {
                if (c < N) {
                    real_slot[(long)b * N + c] = s;
                    real_spatial[(long)b * N + c] = v;
                }
                slot_row[(long)b * Nout + s] = c < N ? b * N + c : -1;
            } else {
                const int pc = s - c;
                if (pc < npad) pad_slot[(long)b * npad + pc] = s;
                slot_row[(long)b * Nout + s] = -1;
            }
        }
        base += total;
    }
}

__global__ void __launch_bounds__(SEL_THREADS)
compact_slots_kernel(const int32_t *__restrict__ table, int table_batch_stride, int Nout, int N,
                     int32_t *__restrict__ real_slot, int32_t *__restrict__ real_spatial,
                     int32_t *__restrict__ slot_row, int32_t *__restrict__ pad_slot)
{
    compact_image(blockIdx.x, table, table_batch_stride, Nout, N, real_slot, real_spatial, slot_row, pad_slot);
}

// What a stack needs in front of its first block beside the scores, in one launch: the keep-set (a workgroup an image), then of either kind of block the
// compaction of its slots (a workgroup an image) and the inverse of its gather table (a workgroup 1024 slots).  None waits for another, each leaves the chip all but
// idle, and in a chain each took 4.6 to 7.4 us however small: ViT-B, 64 x 64, one image 23.1 us in four launches, 7.9 in one.
template <int ITEMS>
__global__ void __launch_bounds__(SEL_THREADS)
select_and_tables_kernel(const float *__restrict__ scores, int32_t *__restrict__ keep, int B, int N, int K, BlockTables local, BlockTables global)
{
    int i = blockIdx.x;
    if (i < B) {
        select_image<ITEMS>(scores + (long)i * N, keep + (long)i * K, N, K);
        return;
    }
    i -= B;
    auto tables = [&](const BlockTables &t, int j) {
        if (t.real_slot && j < B) compact_image(j, t.table, t.table_batch_stride, t.Nout, N, t.real_slot, t.real_spatial, t.slot_row, t.pad_slot);
        else invert_slot((j - (t.real_slot ? B : 0)) * SEL_THREADS + threadIdx.x, t.table, t.table_batch_stride, t.Nout, N, t.slot_of, t.slot_images * t.Nout);
    };
    const int n = local.workgroups(B);
    if (i < n) tables(local, i);
    else tables(global, i - n);
}

// ---------------------------------------------------------------- content-aware order
// The cells of an attention group are ranked by (score descending, cell index ascending; padding cells last), then the
// stripe interleave sigma[g*(S/G)+t] = pi[t*G+g] (Sec. 4.1) places rank t*G+g at scan position g*(S/G)+t.
// Sort key of cell i of the group at (wr, wc): ascending keys are descending scores.
__device__ __forceinline__ uint32_t content_key(const float *sc, int g, int w, int wr, int wc, int i)
{
    const int row = wr * w + i / w, col = wc * w + i % w;
    return ~score_key(row < g && col < g ? sc[row * g + col] : -INFINITY);
}

__device__ __forceinline__ void content_place(int cell, int rank, int g, int w, int wr, int wc, int G, long base,
                                              int32_t *__restrict__ gather_table, int32_t *__restrict__ sigma)
{
    const int S = w * w, pos = (rank % G) * (S / G) + rank / G;
    const int row = wr * w + cell / w, col = wc * w + cell % w;
    sigma[base + pos] = cell;
    gather_table[base + pos] = (row < g && col < g) ? row * g + col : -1;
}

// Rank by counting: a cell's rank is the number of cells of its group that come before it.  Quadratic in the group, but
// every cell is independent of the others: RANK_LANES neighbouring lanes share one cell, each against its part of the keys
// (all keys of the group in LDS, 32 bits each), and a group spreads over as many workgroups as it has runs of blockDim /
// RANK_LANES cells; the sort below has one workgroup per group and a chain of log^2 barriers (64 x 64 grid: 40 -> 7.0 us; 7.6 with the keys loaded one by one).  Equal keys are told apart by their
// index: a key before the cell counts if it is <= the cell's, i.e. < mine + 1 (no key is the largest 32-bit number), a key
// behind it if it is < mine.  The four cells of a wave lie in one aligned run of four keys, so which of the two holds is
// the same for the whole wave except in the step that contains that run.
constexpr int RANK_LANES = 16, RANK_STEP = 4 * RANK_LANES;
__device__ __forceinline__ int count_below(const uint4 &k, uint32_t t) { return (k.x < t) + (k.y < t) + (k.z < t) + (k.w < t); }

__global__ void __launch_bounds__(1024)
content_rank_kernel(const float *__restrict__ scores, int g, int w, int nws, int G, int runs,
                    int32_t *__restrict__ gather_table, int32_t *__restrict__ sigma)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint32_t *keys = reinterpret_cast<uint32_t *>(smem);
    const int S = w * w, nW = nws * nws;
    const int group = blockIdx.x / runs, run = blockIdx.x - group * runs;
    const int b = group / nW, win = group - b * nW, wr = win / nws, wc = win - wr * nws;
    const float *sc = scores + (long)b * g * g;
    const int padded = (S + RANK_STEP - 1) / RANK_STEP * RANK_STEP;      // past S: the largest number, counted by nobody
    if (w == g && (S & 3) == 0 && (reinterpret_cast<uintptr_t>(sc) & 15) == 0) {
        // four loads of 16 bytes in flight at a time
        const float4 *s4 = reinterpret_cast<const float4 *>(sc);
        for (int i0 = threadIdx.x; i0 < padded / 4; i0 += 4 * blockDim.x) {
            float4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = s4[min(i0 + u * (int)blockDim.x, S / 4 - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + u * (int)blockDim.x;
                const uint4 k = make_uint4(~score_key(v[u].x), ~score_key(v[u].y), ~score_key(v[u].z), ~score_key(v[u].w));
                if (i < padded / 4) reinterpret_cast<uint4 *>(keys)[i] = i < S / 4 ? k : make_uint4(~0u, ~0u, ~0u, ~0u);
            }
        }
    } else if (w == g) {
        for (int i = threadIdx.x; i < padded; i += blockDim.x) keys[i] = i < S ? ~score_key(sc[i]) : ~0u;
    } else {
        for (int i = threadIdx.x; i < padded; i += blockDim.x) keys[i] = i < S ? content_key(sc, g, w, wr, wc, i) : ~0u;
    }
    __syncthreads();
    const int cell = run * (blockDim.x / RANK_LANES) + threadIdx.x / RANK_LANES, part = threadIdx.x % RANK_LANES;
    const int four = __builtin_amdgcn_readfirstlane(cell & ~3), step = four / RANK_STEP * RANK_STEP;
    const uint32_t mine = keys[min(cell, S - 1)];
    const uint4 *kp = reinterpret_cast<const uint4 *>(keys) + part;
    int before = 0;
#pragma unroll 4
    for (int j = 0; j < step; j += RANK_STEP) before += count_below(kp[j / 4], mine + 1);
    if (step < padded) {
        const uint4 k = kp[step / 4];
        const int j = step + part * 4;
        before += (k.x < mine + (j < cell)) + (k.y < mine + (j + 1 < cell)) + (k.z < mine + (j + 2 < cell)) + (k.w < mine + (j + 3 < cell));
    }
#pragma unroll 4
    for (int j = step + RANK_STEP; j < padded; j += RANK_STEP) before += count_below(kp[j / 4], mine);
#pragma unroll
    for (int o = RANK_LANES / 2; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
    if (part == 0 && cell < S) content_place(cell, before, g, w, wr, wc, G, (long)group * S, gather_table, sigma);
}

// One workgroup per (image, window): a bitonic sort of 64-bit (key, cell) pairs in LDS.
// P = the power of two >= S that is sorted; entries S..P-1 carry the largest key.
__global__ void __launch_bounds__(1024)
content_tables_kernel(const float *__restrict__ scores, int g, int w, int nws, int G, int P,
                      int32_t *__restrict__ gather_table, int32_t *__restrict__ sigma)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned long long *keys = reinterpret_cast<unsigned long long *>(smem);
    const int S = w * w, nW = nws * nws;
    const int b = blockIdx.x / nW, win = blockIdx.x % nW;
    const int wr = win / nws, wc = win % nws;
    const float *sc = scores + (long)b * g * g;
    for (int i = threadIdx.x; i < P; i += blockDim.x)
        keys[i] = i < S ? ((unsigned long long)content_key(sc, g, w, wr, wc, i) << 32) | (unsigned)i : ~0ull;
    __syncthreads();
    for (int k = 2; k <= P; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int t = threadIdx.x; t < P / 2; t += blockDim.x) {
                const int i = 2 * t - (t & (j - 1));            // index with bit j clear
                const int p = i | j;
                const unsigned long long a = keys[i], c = keys[p];
                const bool up = (i & k) == 0;
                if ((a > c) == up) { keys[i] = c; keys[p] = a; }
            }
            __syncthreads();
        }
    for (int rk = threadIdx.x; rk < S; rk += blockDim.x)
        content_place((int)(keys[rk] & 0xffffffffu), rk, g, w, wr, wc, G, (long)blockIdx.x * S, gather_table, sigma);
}

extern "C" int ssam_permute(const void *x, const int32_t *idx, void *y, int B, int Nin, int Nout, int D, void *stream)
{
    if (!movers_args_ok(x, idx, y, B, Nin, Nout, D)) return SSAM_EINVAL;
    int chunks = D / 8;
    hipLaunchKernelGGL(permute_kernel, dim3(mover_grid((long)B * Nout * chunks)), dim3(256), 0, (hipStream_t)stream,
                       (const uint4 *)x, idx, (uint4 *)y, B, Nin, Nout, chunks);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

extern "C" int ssam_unpermute(const void *y, const int32_t *idx, void *x, const void *residual,
                              int B, int Nx, int Ny, int D, void *stream)
{
    if (!movers_args_ok(y, idx, x, B, Nx, Ny, D)) return SSAM_EINVAL;
    if (residual && !ssam_aligned16(residual)) return SSAM_EINVAL;
    int chunks = D / 8;
    hipLaunchKernelGGL(unpermute_kernel, dim3(mover_grid((long)B * Ny * chunks)), dim3(256), 0, (hipStream_t)stream,
                       (const uint4 *)y, idx, (uint4 *)x, (const uint4 *)residual, B, Nx, Ny, chunks);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

// fill: padding rows written by the same launch
int ssam_ln_gather_impl(const void *x, const int32_t *idx, int idx_batch_stride,
                              const float *gamma, const float *beta, float eps, void *y,
                              int B, int Nin, int Nout, int D, const PadFill &fill, void *stream)
{
    if (!movers_args_ok(x, idx, y, B, Nin, Nout, D) || !gamma || !beta || idx_batch_stride < 0) return SSAM_EINVAL;
    if (!ssam_aligned16(gamma) || !ssam_aligned16(beta)) return SSAM_EINVAL;
    if (D > 2048) return SSAM_EUNSUPPORTED;
    int chunks = D / 8;
    long rows = (long)B * Nout;
    const int ln_blocks = ssam_div_up(rows, 4);
    dim3 grid(ln_blocks + ssam_div_up(fill.total_rows, 4)), block(256);
    hipStream_t st = (hipStream_t)stream;
    if (chunks <= 128)
        hipLaunchKernelGGL(ln_gather_kernel<2>, grid, block, 0, st, (const uint4 *)x, idx, idx_batch_stride,
                           gamma, beta, eps, (uint4 *)y, B, Nin, Nout, chunks, fill, ln_blocks);
    else if (chunks <= 192)
        hipLaunchKernelGGL(ln_gather_kernel<3>, grid, block, 0, st, (const uint4 *)x, idx, idx_batch_stride,
                           gamma, beta, eps, (uint4 *)y, B, Nin, Nout, chunks, fill, ln_blocks);
    else
        hipLaunchKernelGGL(ln_gather_kernel<4>, grid, block, 0, st, (const uint4 *)x, idx, idx_batch_stride,
                           gamma, beta, eps, (uint4 *)y, B, Nin, Nout, chunks, fill, ln_blocks);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

extern "C" int ssam_ln_gather(const void *x, const int32_t *idx, int idx_batch_stride,
                              const float *gamma, const float *beta, float eps, void *y,
                              int B, int Nin, int Nout, int D, void *stream)
{
    return ssam_ln_gather_impl(x, idx, idx_batch_stride, gamma, beta, eps, y, B, Nin, Nout, D, PadFill{}, stream);
}

extern "C" size_t ssam_score_tokens_workspace_bytes(int B, int gh, int gw)
{
    if (B <= 0 || gh <= 0 || gw <= 0) return 0;
    return (size_t)B * gh * gw * sizeof(float);
}

extern "C" int ssam_score_tokens(const void *x, float *scores, int B, int gh, int gw, int D,
                                 void *workspace, size_t workspace_bytes, void *stream)
{
    if (!x || !scores || !workspace || B <= 0 || gh <= 0 || gw <= 0 || D <= 0 || D % 8 != 0) return SSAM_EINVAL;
    if (!ssam_aligned16(x) || !ssam_aligned16(workspace)) return SSAM_EINVAL;
    if (workspace_bytes < ssam_score_tokens_workspace_bytes(B, gh, gw)) return SSAM_EWORKSPACE;
    return launch_score(x, scores, B, gh, gw, D, (float *)workspace, (hipStream_t)stream);
}

// ---- ssam_score_tokens for callers that cannot allocate: the channel-sum map lives in a file-scope device array.
// In host code the array's name is only a stand-in; its device address is looked up once per device and kept.
static __device__ __align__(256) float scratch[SSAM_SCORE_TOKENS_STATIC_MAX_TOKENS];

namespace {
constexpr int kMaxDevices = 64;
float *scratch_ptr[kMaxDevices];        // device address of `scratch` on each GPU this process has used it on

int scratch_on_current_device(float **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SSAM_EHIP;
    float *p = __atomic_load_n(&scratch_ptr[dev], __ATOMIC_ACQUIRE);
    if (!p) {                           // first call on this device (racing first calls resolve the same address)
        void *sym = nullptr;
        if (hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch)) != hipSuccess || !sym) return SSAM_EHIP;
        p = (float *)sym;
        __atomic_store_n(&scratch_ptr[dev], p, __ATOMIC_RELEASE);
    }
    *out = p;
    return SSAM_OK;
}
}  // namespace

// Launches that the scores of such an input take.  Host only, for tests; not part of the interface.
extern "C" int ssam_score_form(int B, int gh, int gw, int D) { return score_in_one_launch(B, gh, gw, D) ? 1 : 2; }

extern "C" int ssam_score_tokens_static(const void *x, float *scores, int B, int gh, int gw, int D, void *stream)
{
    if (!x || !scores || B <= 0 || gh <= 0 || gw <= 0 || D <= 0 || D % 8 != 0) return SSAM_EINVAL;
    if (!ssam_aligned16(x)) return SSAM_EINVAL;
    const long tokens = (long)B * gh * gw;
    if (tokens > SSAM_SCORE_TOKENS_STATIC_MAX_TOKENS) return SSAM_EWORKSPACE;
    float *csum = nullptr;
    int rc = scratch_on_current_device(&csum);
    if (rc != SSAM_OK) return rc;
    // channel_sum_kernel writes the sum of every token it is given and sobel_kernel reads only those, so nothing
    // in the array has to start at zero and what an earlier (larger) call left behind is never read
    return launch_score(x, scores, B, gh, gw, D, csum, (hipStream_t)stream);
}

extern "C" int ssam_select_tokens(const float *scores, int32_t *keep_idx, int B, int N, int K, void *stream)
{
    if (!scores || !keep_idx || B <= 0 || N <= 0 || K <= 0 || K > N) return SSAM_EINVAL;
    if (N > 65536) return SSAM_EUNSUPPORTED;
    const hipStream_t st = (hipStream_t)stream;
    if (N <= 4 * SEL_THREADS) hipLaunchKernelGGL(select_kernel<4>, dim3(B), dim3(SEL_THREADS), 0, st, scores, keep_idx, N, K);
    else if (N <= 16 * SEL_THREADS) hipLaunchKernelGGL(select_kernel<16>, dim3(B), dim3(SEL_THREADS), 0, st, scores, keep_idx, N, K);
    else hipLaunchKernelGGL(select_kernel<64>, dim3(B), dim3(SEL_THREADS), 0, st, scores, keep_idx, N, K);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

// Threads of a counting workgroup: no more waves than the group has cells for.
static int rank_threads(int S) { return S > 8192 ? 1024 : S >= 512 / RANK_LANES ? 512 : ssam_div_up(S, 64 / RANK_LANES) * 64; }

// Whether counting beats the sort, from their measured times (us, 233 pairs of a side w and a number of groups; chosen wrongly by
// more than 7 % only where both take 2.5 to 5 us).  The sort takes a latency that grows with its network, the same for up to 256
// groups, and then the chip's throughput; counting takes 3 us, 2.2 for every 1000 workgroups of 512 threads (its keys, loaded by
// each of a group's `runs` workgroups) and 75 for every 2^30 pairs of cells:
//   groups of 14 x 14: 25 3.6 by counting, 9.4 sorted; 200 7.1, 9.4; 400 10.9, 10.3; 1600 34, 12; 12800 235, 48
//   of 8 x 8: 25 3.3, 6.1; 800 6.4, 6.3; 12800 57, 17       of 64 x 64: 1 7.5, 40; 16 30, 41; 25 45, 41; 200 289, 41
static bool rank_by_counting(long groups, int S)
{
    int lg = 1;
    while ((1 << lg) < S) ++lg;
    const double P = 1 << lg, steps = lg * (lg + 1) / 2;
    const double sort_us = 2.3 + steps * (0.17 + 8e-5 * P) + (groups > 256 ? (groups - 256) * (2.5e-4 + 3.8e-7 * P * steps) : 0.0);
    const int threads = rank_threads(S), runs = ssam_div_up(S, threads / RANK_LANES);
    const double count_us = 3.0 + 4e-4 * S + groups * (4.4e-6 * runs * threads + 7e-8 * S * S);
    return count_us < sort_us;
}

// 1 if the tables of `groups` groups of w x w cells are made by counting, 0 if by the sort.  For tests; not part of the interface.
extern "C" int ssam_content_tables_form(long groups, int w) { return rank_by_counting(groups, w * w); }

extern "C" int ssam_build_content_tables(const float *scores, int B, int g, int ws, int G,
                                         int32_t *gather_table, int32_t *sigma, void *stream)
{
    if (!scores || !gather_table || !sigma || B <= 0 || g <= 0 || ws < 0 || G <= 0) return SSAM_EINVAL;
    const int w = ws > 0 ? ws : g;
    if (w > 128) return SSAM_EUNSUPPORTED;
    const int S = w * w, nws = (g + w - 1) / w;
    if (S % G != 0) return SSAM_EINVAL;
    const long groups = (long)B * nws * nws;
    int P = 2;
    while (P < S) P <<= 1;
    if (rank_by_counting(groups, S)) {
        const int threads = rank_threads(S), runs = ssam_div_up(S, threads / RANK_LANES);
        const size_t lds = (size_t)ssam_div_up(S, RANK_STEP) * RANK_STEP * sizeof(uint32_t);       // <= 64 KiB (w <= 128)
        hipLaunchKernelGGL(content_rank_kernel, dim3((unsigned)(groups * runs)), dim3(threads), lds, (hipStream_t)stream,
                           scores, g, w, nws, G, runs, gather_table, sigma);
        SSAM_CHECK_LAUNCH();
        return SSAM_OK;
    }
    const int threads = P / 2 < 1024 ? (P / 2 < 64 ? 64 : P / 2) : 1024;
    const size_t lds = (size_t)P * sizeof(unsigned long long);
    if (lds > 64 * 1024 &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(content_tables_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return SSAM_EHIP;
    hipLaunchKernelGGL(content_tables_kernel, dim3(B * nws * nws), dim3(threads), lds, (hipStream_t)stream,
                       scores, g, w, nws, G, P, gather_table, sigma);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

// internal (block composition): see compact_slots_kernel
int ssam_compact_slots(const int32_t *table, int table_batch_stride, int B, int Nout, int N,
                       int32_t *real_slot, int32_t *real_spatial, int32_t *slot_row, int32_t *pad_slot, hipStream_t st)
{
    hipLaunchKernelGGL(compact_slots_kernel, dim3(B), dim3(SEL_THREADS), 0, st, table, table_batch_stride, Nout, N,
                       real_slot, real_spatial, slot_row, pad_slot);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

// statistics of rows idx[b][p] of image b (idx == NULL: of every row in order), slots (D / 64 of at most GEMM_PARTS_MOST, or 0): see ln_stats_kernel
int ssam_ln_stats_impl(const void *x, float *stats, long rows, int D, float eps, const int32_t *idx, int idx_batch_stride,
                       int Nin, int Nout, int32_t *src, const PadFill &fill, hipStream_t st, int slots)
{
    if (!x || !stats || rows <= 0 || D <= 0 || D % 8 != 0) return SSAM_EINVAL;
    if (!ssam_aligned16(x) || ((uintptr_t)stats & 7)) return SSAM_EINVAL;
    if (idx && (!src || Nin <= 0 || Nout <= 0 || (long)(rows / Nout) * Nin > 0x7fffffffL)) return SSAM_EINVAL;
    if (D > 2048) return SSAM_EUNSUPPORTED;
    int chunks = D / 8;
    const int ln_blocks = ssam_div_up(rows, 4);
    dim3 grid((unsigned)(ln_blocks + ssam_div_up(fill.total_rows, 4))), block(256);
    if (chunks <= 128)
        hipLaunchKernelGGL(ln_stats_kernel<2>, grid, block, 0, st, (const uint4 *)x, (float2 *)stats, rows, chunks, eps, idx, idx_batch_stride, Nin, Nout, src, fill, ln_blocks, slots);
    else if (chunks <= 192)
        hipLaunchKernelGGL(ln_stats_kernel<3>, grid, block, 0, st, (const uint4 *)x, (float2 *)stats, rows, chunks, eps, idx, idx_batch_stride, Nin, Nout, src, fill, ln_blocks, slots);
    else
        hipLaunchKernelGGL(ln_stats_kernel<4>, grid, block, 0, st, (const uint4 *)x, (float2 *)stats, rows, chunks, eps, idx, idx_batch_stride, Nin, Nout, src, fill, ln_blocks, slots);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

extern "C" int ssam_ln_stats(const void *x, float *stats, long rows, int D, float eps, void *stream)
{
    return ssam_ln_stats_impl(x, stats, rows, D, eps, nullptr, 0, 0, 0, nullptr, PadFill{}, (hipStream_t)stream, 0);
}

extern "C" int ssam_fold_ln_weight(const void *W, int ldw, const float *bias, const float *gamma, const float *beta,
                                   void *Wf, float *colsum, float *bias_f, int N, int K, void *stream)
{
    if (!W || !bias || !gamma || !beta || !Wf || !colsum || !bias_f || N <= 0 || K <= 0 || ldw < K || ldw % 8) return SSAM_EINVAL;
    if (!ssam_aligned16(W) || !ssam_aligned16(Wf)) return SSAM_EINVAL;
    if (K % 8 != 0) return SSAM_EUNSUPPORTED;
    hipLaunchKernelGGL(fold_ln_weight_kernel, dim3(ssam_div_up(N, 4)), dim3(256), 0, (hipStream_t)stream,
                       (const bf16 *)W, ldw, bias, gamma, beta, (bf16 *)Wf, colsum, bias_f, N, K);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

// internal (block composition): see invert_table_kernel
int ssam_invert_table(const int32_t *table, int table_batch_stride, int B, int Nout, int N, int32_t *inv, hipStream_t st)
{
    const int total = B * Nout;
    hipLaunchKernelGGL(invert_table_kernel, dim3(ssam_div_up(total, 256)), dim3(256), 0, st, table, table_batch_stride, Nout, N, inv, total);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

// internal (stack composition): ssam_select_tokens and the tables of both kinds of block, in one launch
int ssam_select_and_tables(const float *scores, int32_t *keep_idx, int B, int N, int K, const BlockTables &local, const BlockTables &global, hipStream_t st)
{
    if (!scores || !keep_idx || B <= 0 || N <= 0 || K <= 0 || K > N) return SSAM_EINVAL;
    if (N > 65536) return SSAM_EUNSUPPORTED;
    // (a selection over more scores spills and takes 34 us: launches of their own)
    if (N > 16 * SEL_THREADS) {
        int rc = ssam_select_tokens(scores, keep_idx, B, N, K, st);
        for (const BlockTables *t : { &local, &global }) {
            if (rc == SSAM_OK && t->real_slot) rc = ssam_compact_slots(t->table, t->table_batch_stride, B, t->Nout, N, t->real_slot, t->real_spatial, t->slot_row, t->pad_slot, st);
            if (rc == SSAM_OK && t->slot_of) rc = ssam_invert_table(t->table, t->table_batch_stride, t->slot_images, t->Nout, N, t->slot_of, st);
        }
        return rc;
    }
    const dim3 grid(B + local.workgroups(B) + global.workgroups(B));
    auto kern = N <= 4 * SEL_THREADS ? select_and_tables_kernel<4> : select_and_tables_kernel<16>;
    hipLaunchKernelGGL(kern, grid, dim3(SEL_THREADS), 0, st, scores, keep_idx, B, N, K, local, global);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}

extern "C" int ssam_fold_kv_bias(const float *bias_in, const float *bqkv, const void *wproj, const float *bproj,
                                 float *bias_out, float *bproj_out, int D, void *stream)
{
    if (!bias_in || !bqkv || !wproj || !bproj || !bias_out || !bproj_out || D <= 0) return SSAM_EINVAL;
    if (!ssam_aligned16(wproj)) return SSAM_EINVAL;
    if (D % 8 != 0) return SSAM_EUNSUPPORTED;
    hipLaunchKernelGGL(fold_kv_bias_kernel, dim3(ssam_div_up(3 * D, 4)), dim3(256), 0, (hipStream_t)stream,
                       bias_in, bqkv, (const bf16 *)wproj, bproj, bias_out, bproj_out, D);
    SSAM_CHECK_LAUNCH();
    return SSAM_OK;
}
