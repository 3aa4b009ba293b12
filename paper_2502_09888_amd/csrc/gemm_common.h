// Device-side pieces shared by the projection kernels (gemm_bf16.hip, gemm_small_bf16.hip): operand types,
// the GELU of the feed-forward epilogue and the stores of a staged 32 x 64 output block.
#pragma once
#include "gemm.h"
#include "lanes.h"

#include <type_traits>
#include <utility>

namespace climber {
namespace gemm {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>), unrolled at compile time
template <int... Is, class F>
static __device__ __forceinline__ void static_for_impl(std::integer_sequence<int, Is...>, F &&f)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
static __device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// exact-erf GELU, erf by the rational/exponential formula 7.1.26 of Abramowitz & Stegun
// (|error| <= 1.5e-7, far below the bf16 rounding of the result).  With a = |x|, z = a/sqrt(2),
// t = 1/(1 + p z) and h = (1 - erf z)/2 = (poly(t)/2) t exp(-z^2):
//   GELU(x) = x (1 + erf(x/sqrt 2))/2 = max(x, 0) - a h        (x >= 0: x - x h;  x < 0: x h)
// which needs no sign select; the constants carry the factors 1/2, 1/sqrt(2) and log2(e)/2.
// (A polynomial for log2 of the normal tail would take two instructions and the reciprocal less, and
// the same absolute error; but its relative error is ten times as large where x < -4, above the bf16 rounding:
// 2e-2 against 3.6e-3 in (-6, -5).)
// In stages, for a kernel that deals them out between its matrix instructions (x, t, p: carried from stage to stage).
constexpr int kGeluStages = 11;
template <int STAGE>
static __device__ __forceinline__ void gelu_stage(float &x, float &t, float &p)
{
    if constexpr (STAGE == 0) t = fmaf(__builtin_fabsf(x), 0.3275911f * 0.70710678118654752f, 1.f);
    else if constexpr (STAGE == 1) t = __builtin_amdgcn_rcpf(t);
    else if constexpr (STAGE == 2) p = fmaf(0.5f * 1.061405429f, t, 0.5f * -1.453152027f);
    else if constexpr (STAGE == 3) p = fmaf(p, t, 0.5f * 1.421413741f);
    else if constexpr (STAGE == 4) p = fmaf(p, t, 0.5f * -0.284496736f);
    else if constexpr (STAGE == 5) p = fmaf(p, t, 0.5f * 0.254829592f);
    else if constexpr (STAGE == 6) p = p * t;
    else if constexpr (STAGE == 7) t = (x * x) * -0.72134752044448170f;
    else if constexpr (STAGE == 8) t = __builtin_amdgcn_exp2f(t);
    else if constexpr (STAGE == 9) p = p * t;
    else x = fmaf(-__builtin_fabsf(x), p, fmaxf(x, 0.f));
}
static __device__ __forceinline__ float gelu_erf(float x)
{
    float t, p;
    static_for<kGeluStages>([&](auto s) __attribute__((always_inline)) { gelu_stage<decltype(s)::value>(x, t, p); });
    return x;
}

// x^2 + y^2 + z^2 + w^2, one fixed order (the row sums of squares are the same bits whoever forms them)
static __device__ __forceinline__ float sumsq4(float x, float y, float z, float w)
{
    return fmaf(w, w, fmaf(z, z, fmaf(x, x, y * y)));
}

// A lane's part of a 32 x 32 block of fp32 rows, as its accumulators hold it: x = row l32 of the block, from column
// 4 (lane / 32) on.
static __device__ __forceinline__ void load_block(f32x16 &v, const float *x)
{
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const float4 q = *(const float4 *)(x + 8 * g);
        v[4 * g] = q.x, v[4 * g + 1] = q.y, v[4 * g + 2] = q.z, v[4 * g + 3] = q.w;
    }
}
static __device__ __forceinline__ void store_block(float *x, const f32x16 &v)
{
#pragma unroll
    for (int g = 0; g < 4; ++g) *(float4 *)(x + 8 * g) = float4{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
}

// 1/sqrt(mean(x^2) + eps) of one row from its partial sums of squares
static __device__ __forceinline__ float row_scale(const RowNormIn &nin, int64_t row)
{
    float ss = 0.f;
    if (nin.n_part == 8) {
        const float4 u = *(const float4 *)(nin.ss + row * 8), v = *(const float4 *)(nin.ss + row * 8 + 4);
        ss = ((u.x + u.y) + (u.z + u.w)) + ((v.x + v.y) + (v.z + v.w));
    } else {
        for (int q = 0; q < nin.n_part; ++q) ss += nin.ss[row * nin.n_part + q];
    }
    return 1.f / sqrtf(ss * nin.inv_d + nin.eps);
}

// The user that a block of 32 rows of the direct cache write belongs to: first row, padded and valid
// length -- by arithmetic in uniform batches, from the cache's tables (wave-uniform loads) in ragged ones.
struct CacheUser { int t0, l_pad, l_valid; };
static __device__ __forceinline__ CacheUser cache_user(const QkvToCache &qc, int row)
{
    CacheUser u;
    if (qc.l_pad > 0) {
        u.t0 = row / qc.l_pad * qc.l_pad, u.l_pad = qc.l_pad, u.l_valid = qc.l_valid;
    } else {
        const int b = qc.seg[row >> 6];
        u.t0 = qc.tok_off[b];
        u.l_pad = qc.tok_off[b + 1] - u.t0;
        u.l_valid = qc.hist_len[b];
    }
    return u;
}

// Direct cache write of a 32 x 64 block (32 tokens of one user, one head of the queries, keys or values;
// rows of `tr` are PITCH bytes apart, slots past the valid length already zero).  Of its four parts of 1 KiB
// [p0, p1) are stored, so that several waves can share a block.
template <int PITCH>
static __device__ __forceinline__ void store_block_to_cache(const uint8_t *tr, const QkvToCache &qc, const CacheUser &u,
                                                            int row_base, int col_base, int M, void *C, int64_t ldc,
                                                            int lane, int p0, int p1)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const int l32 = lane & 31, hf = lane >> 5;
    const int which = qc.which0 + col_base / qc.d, h = (col_base % qc.d) / 64;
    if (row_base >= M) return;
    const int kb = (row_base - u.t0) / 32;
    uint8_t *blk = qc.layer_base + ((size_t)u.t0 * qc.H + (size_t)h * u.l_pad) * 256 + (size_t)kb * 8192;
    if (which == 0) {        // query rows
#pragma unroll
        for (int it = p0; it < p1; ++it) {
            const int id = it * 64 + lane, r = id / 8, cc = id % 8;
            if (row_base + r < M)
                *(uint4 *)((__bf16 *)C + (int64_t)(row_base + r) * ldc + h * 64 + cc * 8) =
                    *(const uint4 *)(tr + r * PITCH + cc * 16);
        }
    } else if (which == 1) {  // K fragments: chunk (s, lane) = K[lane % 32][16 s + 8 (lane / 32) ..]
#pragma unroll
        for (int s4 = p0; s4 < p1; ++s4)
            *(uint4 *)(blk + (s4 * 64 + lane) * 16) = *(const uint4 *)(tr + l32 * PITCH + (2 * s4 + hf) * 16);
    } else {                  // V^T chunks by LDS transpose reads (see hist_fused_bf16.hip)
        const int G = lane >> 4, i16 = lane & 15;
#pragma unroll
        for (int part = p0; part < p1; ++part) {
            const int gg = part >> 1, db = part & 1;
            s16x4 hv[2];
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const int r = 16 * gg + 8 * hh + 4 * (G >> 1) + (i16 >> 2);
                const int cb = 64 * db + 32 * (G & 1) + 8 * (i16 & 3);
                hv[hh] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4 *)(tr + r * PITCH + cb));
            }
            const s16x8 both = __builtin_shufflevector(hv[0], hv[1], 0, 1, 2, 3, 4, 5, 6, 7);
            *(uint4 *)(blk + 4096 + (part * 64 + lane) * 16) = __builtin_bit_cast(uint4, both);
        }
    }
}

// bytes of a staged row of a wave's WN*32 columns: padded by 16 to spread the rows over the banks
template <int EPI, int WN>
constexpr int epilogue_pitch() { return WN * 32 * (EPI == EPI_RESID_F32 ? 4 : 2) + 16; }

// Epilogue of a wave's WM x WN blocks of 32 x 32.  The operands are fed to the MFMAs as (W fragment, A
// fragment), so a block accumulator is the transposed product: the lane holds C[row0 + 32i + l32][col_base +
// 32j + 8g + 4hf + 0..3] for g = r/4 -- four consecutive columns of ONE row.  The wave turns 32 rows x (WN*32)
// columns around in its own corner `tr` of the (idle) LDS (32 rows of epilogue_pitch bytes) and stores whole
// rows, 16 bytes per lane.  rs: scale of the lane's row of every block row (RMSNorm folded in).
// A residual row is added to the finished sum of products, one rounding of it; as the accumulators' start value it
// would have every partial sum rounded at the residual's magnitude (3 to 11 times the error).
template <int EPI, int WM, int WN>
static __device__ __forceinline__ void wave_epilogue(f32x16 (&acc)[WM][WN], const float (&rs)[WM], const CacheUser (&user)[WM],
                                                     uint8_t *tr, int row0, int col_base, int lane, int M, int N, void *C,
                                                     int64_t ldc, const float *resid, int64_t ldr, const RowNormOut &nout,
                                                     int tiled, const QkvToCache &qc)
{
    const int l32 = lane & 31, hf = lane >> 5;
    constexpr bool F32 = EPI == EPI_RESID_F32;
    constexpr int CW = WN * 32;                       // columns of the wave's block
    constexpr int kElem = F32 ? 4 : 2;
    constexpr int kPitch = epilogue_pitch<EPI, WN>();  // bytes per staged row
    constexpr int kChunksPerRow = CW * kElem / 16;
    constexpr int kIters = 32 * kChunksPerRow / 64;   // 16-byte pieces per lane and block row
    // Residual rows of block row i, all requested before anything waits for them (a load placed
    // after a store would make the wait for it drain the stores as well: one memory round trip per
    // 16 bytes).  Block row i + 1 is requested before block row i is stored.
    float4 rsd[2][F32 ? kIters : 1];
    auto load_resid = [&](int i, float4 *buf) __attribute__((always_inline)) {
        if constexpr (F32) {
#pragma unroll
            for (int it = 0; it < kIters; ++it) {
                const int id = it * 64 + lane, r = id / kChunksPerRow, cc = id % kChunksPerRow;
                const int row = min(row0 + 32 * i + r, M - 1);
                buf[it] = *(const float4 *)(resid + (int64_t)row * ldr + col_base + cc * 4);
            }
        }
    };
    load_resid(0, rsd[0]);
    // direct cache write: slots past a user's valid length hold zeros
    bool zero_row[WM];
#pragma unroll
    for (int i = 0; i < WM; ++i)
        zero_row[i] = EPI == EPI_STORE_BF16 && qc.layer_base &&
                      row0 + 32 * i - user[i].t0 + l32 >= user[i].l_valid;
#pragma unroll
    for (int i = 0; i < WM; ++i) {
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int col = 32 * j + 8 * g + 4 * hf;
                if (F32) {
                    float4 v = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
                    *(float4 *)(tr + l32 * kPitch + col * 4) = v;
                } else {
                    __attribute__((aligned(8))) __bf16 v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float x = acc[i][j][4 * g + e] * rs[i];
                        v[e] = (__bf16)(EPI == EPI_GELU_BF16 ? gelu_erf(x) : EPI == EPI_RELU_BF16 ? fmaxf(x, 0.f) : x);
                    }
                    if (EPI == EPI_STORE_BF16 && zero_row[i]) v[0] = v[1] = v[2] = v[3] = (__bf16)0.f;
                    *(uint2 *)(tr + l32 * kPitch + col * 2) = *(const uint2 *)v;
                }
            }
        if (i + 1 < WM) load_resid(i + 1, rsd[(i + 1) & 1]);
        const int row_base = row0 + 32 * i;
        if (EPI == EPI_STORE_BF16 && qc.layer_base) {
            // the wave's 32 x 64 block is one head of the queries, keys or values of 32 tokens of one
            // user (padded lengths are multiples of 64)
            static_assert(EPI != EPI_STORE_BF16 || CW == 64, "a wave's block = one head");
            store_block_to_cache<kPitch>(tr, qc, user[i], row_base, col_base, M, C, ldc, lane, 0, 4);
            continue;
        }
#pragma unroll
        for (int it = 0; it < kIters; ++it) {
            const int id = it * 64 + lane, r = id / kChunksPerRow, cc = id % kChunksPerRow;
            const int row = row_base + r;
            uint4 val = *(const uint4 *)(tr + r * kPitch + cc * 16);
            if (F32) {
                const int col = col_base + cc * 4;
                const float4 rd = rsd[i & 1][it];
                float4 o = *(const float4 *)&val;
                o.x += rd.x; o.y += rd.y; o.z += rd.z; o.w += rd.w;
                if (row < M) {
                    *(float4 *)((float *)C + (int64_t)row * ldc + col) = o;
                    if (nout.ss) {
                        bf16x4 ob;
                        ob[0] = (__bf16)o.x; ob[1] = (__bf16)o.y; ob[2] = (__bf16)o.z; ob[3] = (__bf16)o.w;
                        *(bf16x4 *)((__bf16 *)nout.xb + (int64_t)row * nout.ldb + col) = ob;
                    }
                }
                if (nout.ss) {  // sums of squares of 64-column slices of the row: 16 lanes each
                    static_assert(!F32 || kChunksPerRow % 16 == 0, "a 64-column slice = 16 lanes of one row");
                    const float sq = row_sum16(sumsq4(o.x, o.y, o.z, o.w));
                    if ((cc & 15) == 0 && row < M)
                        nout.ss[(int64_t)row * (N / 64) + (col_base + cc * 4) / 64] = sq;
                }
            } else if (EPI == EPI_GELU_BF16 && (tiled & kTiledC)) {
                // piece `it` = (16-row group it / 2, k-tile it % 2) of the block; a lane takes the chunk
                // that the consuming projection's copy puts at its place in LDS
                static_assert(EPI != EPI_GELU_BF16 || (CW == 64 && kIters == 4), "block = 2 x 2 pieces");
                const int rr = 16 * (it >> 1) + (lane >> 2), c = (lane & 3) ^ ((lane >> 4) & 3);
                val = *(const uint4 *)(tr + rr * kPitch + ((it & 1) * 4 + c) * 16);
                if (row_base + rr < M)
                    *(uint4 *)((uint8_t *)C + ((int64_t)((row_base >> 4) + (it >> 1)) * (N / 32) +
                                               (col_base >> 5) + (it & 1)) * 1024 + lane * 16) = val;
            } else if (row < M) {
                *(uint4 *)((__bf16 *)C + (int64_t)row * ldc + col_base + cc * 8) = val;
            }
        }
    }
}

}  // namespace gemm
}  // namespace climber
