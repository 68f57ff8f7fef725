// Internal helpers shared by the HIP sources of libssam (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ssam.h"

typedef __bf16 bf16;
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

#define SSAM_WAVE 64

// Workgroup barrier that orders LDS traffic only: unlike __syncthreads() it does not drain the
// global-memory counter, so prefetches of later K slabs stay in flight across it.
#define LDS_BARRIER()                                                         \
    do {                                                                      \
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");       \
        __builtin_amdgcn_s_barrier();                                         \
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");       \
    } while (0)

// Rows of a windowed block's qkv tensor that hold no token (padding slots): rows_per_batch * b + pad_slot[b][i] of C, i < npad,
// become bf16(bias) (NULL: zeros).  They are written by extra workgroups of the block's LayerNorm launch, or of its qkv contraction.
struct PadFill {
    bf16 *C;
    long ldc;
    const float *bias;
    int n_cols;
    const int32_t *pad_slot;
    int npad, rows_per_batch, total_rows;      // total_rows = B * npad; 0: none
};

constexpr int SEL_THREADS = 1024;             // threads of a workgroup that selects, compacts or inverts, and slots of a table that it inverts

// Tables of one kind of block that depend only on its gather table [image][Nout]: see compact_slots_kernel (real_slot = NULL: no padding) and
// invert_table_kernel (slot_of = NULL: not wanted; slot_images: 1 if all images share the table).
struct BlockTables {
    const int32_t *table;
    int table_batch_stride, Nout, slot_images;
    int32_t *real_slot, *real_spatial, *slot_row, *pad_slot, *slot_of;
    __host__ __device__ int workgroups(int B) const { return (real_slot ? B : 0) + (slot_of ? (slot_images * Nout + SEL_THREADS - 1) / SEL_THREADS : 0); }
};

#define SSAM_CHECK_LAUNCH()                                   \
    do {                                                      \
        if (hipGetLastError() != hipSuccess) return SSAM_EHIP; \
    } while (0)

static inline bool ssam_aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

static inline int ssam_div_up(long a, long b) { return (int)((a + b - 1) / b); }

// Number of dense prefix tiles of the A-shape mask (Alg. 1): floor(r*T), with a
// 1e-6 guard against r*T falling just below an integer, clamped to [0, T].
static inline int ssam_prefix_tiles(int T, double r)
{
    long n = (long)__builtin_floor(r * (double)T + 1e-6);
    if (n < 0) n = 0;
    if (n > T) n = T;
    return (int)n;
}

__device__ __forceinline__ float bf16_bits_to_float(uint32_t hi16) { return __uint_as_float(hi16 << 16); }

// 8 bf16 packed in a uint4 -> 8 floats
__device__ __forceinline__ void unpack_bf16x8(const uint4 &v, float *f)
{
    f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
    f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
    f[4] = __uint_as_float(v.z << 16); f[5] = __uint_as_float(v.z & 0xffff0000u);
    f[6] = __uint_as_float(v.w << 16); f[7] = __uint_as_float(v.w & 0xffff0000u);
}

// two floats -> two bf16 (round to nearest even) packed low|high
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    bf16x2 v = { (__bf16)lo, (__bf16)hi };
    return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ uint4 pack_bf16x8(const float *f)
{
    return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]),
                      pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
}

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// one padding row (see PadFill): a wave, 16 bytes per lane.  A launch of its own took 5 us of every unfolded block with padding
// (ViT-B, 50 x 50 tokens, batch 2) and after every global block of a folded stack; behind the LayerNorm, or behind the qkv contraction's tiles, it is hidden.
__device__ __forceinline__ void fill_pad_row(const PadFill &f, int r)
{
    if (r >= f.total_rows) return;
    const int b = r / f.npad, i = r - b * f.npad, lane = threadIdx.x & 63;
    bf16 *dst = f.C + ((long)b * f.rows_per_batch + f.pad_slot[(long)b * f.npad + i]) * f.ldc;
    for (int c = lane * 8; c < f.n_cols; c += 64 * 8) {
        if (f.bias == nullptr) {
            *reinterpret_cast<uint4 *>(dst + c) = make_uint4(0, 0, 0, 0);
            continue;
        }
        const float4 *b4 = reinterpret_cast<const float4 *>(f.bias + c);
        float4 x0 = b4[0], x1 = b4[1];
        float v[8] = { x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w };
        *reinterpret_cast<uint4 *>(dst + c) = pack_bf16x8(v);
    }
}

constexpr int GEMM_PARTS_LINE = 16;           // pieces of a row's statistics (GemmParts) in 128 bytes, a row of a slab of 64 bf16
constexpr int GEMM_PARTS_MOST = 20;           // the most: rows of 1280
// pieces from one row to the next: what a reader requests of a row, whatever their number, lies inside it (128 bytes, and above 16 pieces 32 more)
__host__ __device__ constexpr int gemm_parts_pitch(int slots) { return slots > GEMM_PARTS_LINE ? GEMM_PARTS_MOST : GEMM_PARTS_LINE; }

// Of 8 columns of a piece of a row's statistics (GemmParts): their sum, their squared deviations from the piece's mean.  In this order wherever pieces are written.
__device__ __forceinline__ float gemm_piece_sum8(const float *v)
{
    float s = v[0];
#pragma unroll
    for (int e = 1; e < 8; ++e) s += v[e];
    return s;
}
__device__ __forceinline__ float gemm_piece_squares8(const float *v, float mean)
{
    float q = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) { const float t = v[e] - mean; q = fmaf(t, t, q); }
    return q;
}

// What a piece adds to the squared deviations from the row's mean.
__device__ __forceinline__ float gemm_piece_term(float2 piece, float mean)
{
    const float d = piece.x - mean;
    return fmaf(64.f * d, d, piece.y);
}

// { rstd, -rstd * mean } of a row of K from its pieces, by one thread: pieces 4 * k + quad one after the other, then the four quads, as in ln_stats_kernel.
__device__ __forceinline__ float2 gemm_row_stats(const float2 *row, int slots, int K, float eps)
{
    float4 two[GEMM_PARTS_MOST / 2];
#pragma unroll
    for (int i = 0; i < GEMM_PARTS_MOST / 2; ++i) two[i] = reinterpret_cast<const float4 *>(row)[min(i, slots / 2 - 1)];
    float s[4] = { 0.f, 0.f, 0.f, 0.f };
#pragma unroll
    for (int i = 0; i < GEMM_PARTS_MOST; ++i)
        if (i < slots) s[i % 4] += i % 2 ? two[i / 2].z : two[i / 2].x;
    const float mean = ((s[0] + s[1]) + (s[2] + s[3])) / (float)slots;
#pragma unroll
    for (int q = 0; q < 4; ++q) s[q] = 0.f;
#pragma unroll
    for (int i = 0; i < GEMM_PARTS_MOST; ++i)
        if (i < slots) s[i % 4] += gemm_piece_term(i % 2 ? make_float2(two[i / 2].z, two[i / 2].w) : make_float2(two[i / 2].x, two[i / 2].y), mean);
    const float inv = rsqrtf(((s[0] + s[1]) + (s[2] + s[3])) / (float)K + eps);
    return make_float2(inv, -inv * mean);
}

// erf GELU, 0.5 t (1 + erf(t / sqrt 2)) = max(t, 0) - 0.5 |t| erfc(|t| / sqrt 2).  erfc by the rational approximation 7.1.26 of
// Abramowitz & Stegun, erfc(x) = (a1 u + ... + a5 u^5) exp(-x^2), u = 1 / (1 + p x) for x >= 0; absolute error below
// 1.5e-7, far under the bf16 rounding of the stored activation.  One reciprocal and one exp2 per element, eleven full-rate
// instructions (the form with erf took fourteen, and lost the small results of t << 0 in 1 + erf).
// At infinity u is 0, and |t| u is formed by the multiplication in which 0 * inf is 0 (for every finite t it gives the bits of the ordinary
// one): +inf gives +inf, -inf its limit 0, a NaN stays one.  fminf(|t|, 16) instead is an instruction more, 0.3 % of the ViT-B and ViT-L encoders.
// The assembly names poly so that it never follows the reciprocal directly: a transcendental's result needs a wait state before its use,
// which the compiler does not insert for assembly.
__device__ __forceinline__ float gelu_erf(float t)
{
    const float a = fabsf(t);
    const float u = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.70710678118654752440f, a, 1.0f));
    float poly = fmaf(0.5f * 1.061405429f, u, -0.5f * 1.453152027f);
    poly = fmaf(poly, u, 0.5f * 1.421413741f);
    poly = fmaf(poly, u, -0.5f * 0.284496736f);
    poly = fmaf(poly, u, 0.5f * 0.254829592f);
    const float s = a * 0.84932180028801904272f;               // sqrt(log2(e) / 2)
    const float e = __builtin_amdgcn_exp2f(-s * s);
    float au;
    asm("v_mul_legacy_f32 %0, |%1|, %2" : "=v"(au) : "v"(t), "v"(u), "v"(poly));
    return fmaf(-au * poly, e, fmaxf(t, 0.0f));
}
