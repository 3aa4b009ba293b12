// The fused QKV projection of rows that lie in LDS (f_QKV of Eq. (3), Climber, arXiv 2502.09888), shared by the kernel
// that starts a stack from its input rows (gemm_resident_bf16.hip) and by the layer tail, whose output rows are the next
// layer's input (layer_tail_bf16.hip).  A wave takes units of 64 columns (one head's queries, keys or values) and all
// rows of the tile: weight fragments stream from L2 into registers, R k-steps ahead across units, row fragments come out
// of LDS, and nothing is shared on the way out, so there is no barrier.  Per output element the products are summed as in
// gemm_bf16.hip (k ascending, one accumulator, the same MFMA): same bits.
//
// On the way out a unit goes through no LDS either.
//   Keys: the operands enter the MFMA as (weights, rows), a lane's accumulators are 4-column pieces of ONE row, and one
//     exchange between the half-waves makes them the 16-byte chunks of the cache's key fragments.
//   Values: as (rows, weights): a lane's accumulators are 4-row pieces of one column, which is what the V^T chunks are made
//     of (the row scale then belongs to the register, not to the lane).
//   Rows: as keys, then two more exchanges between lanes 16 and 8 apart, after which a store writes 8 whole rows of 128 bytes.
#pragma once
#include "gemm_common.h"

namespace climber {
namespace gemm {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The rows of a tile in LDS, K columns of bf16: 16-byte chunk c of row r at slot c ^ (r % 16) of its group of 16.
template <int K>
struct LdsRows {
    static constexpr int kPitch = K * 2;
    static __device__ __forceinline__ uint32_t base(int l32, int hf) { return (uint32_t)(l32 * kPitch + ((hf ^ (l32 & 15)) << 4)); }
    static __device__ __forceinline__ bf16x8 frag(const uint8_t *rows, uint32_t base, int step, int i)
    {
        return *(const bf16x8 *)(rows + ((base ^ ((step & 7) << 5)) + (step >> 3) * 256 + i * 32 * kPitch));
    }
};

// fragment e (column block e % 2, k-step e / 2) of unit `unit`, packed weights at byte `at` of w
template <int K>
static __device__ __forceinline__ u32x4 unit_frag(__amdgpu_buffer_rsrc_t w, int at, int unit, int e, int lane)
{
    return __builtin_amdgcn_raw_buffer_load_b128(w, lane * 16, at + (2 * unit + e % 2) * (K / 16 * 1024) + e / 2 * 1024, 0);
}

static __device__ __forceinline__ uint32_t pack2(float x, float y)
{
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
    bf16x2 v;
    v[0] = (__bf16)x, v[1] = (__bf16)y;
    return __builtin_bit_cast(uint32_t, v);
}

// acc = the tile's rows times the 64 columns of `unit`, as (rows, weights) if V, else (weights, rows).  `ring` holds the unit's
// first 2 R fragments, at the end, if MORE, those of `next`; a_base: LdsRows::base of the lane.
template <int K, int RB, int R, bool V, bool MORE = true>
static __device__ __forceinline__ void unit_product(f32x16 (&acc)[RB][2], const uint8_t *rows, __amdgpu_buffer_rsrc_t w, int w_at, u32x4 (&ring)[2 * R],
                                                    uint32_t a_base, int unit, int next, int lane)
{
    constexpr int S = K / 16;
    static_assert(S % R == 0 && S / R >= 2, "");
    uint32_t base = a_base;
    asm("" : "+v"(base));
    bf16x8 fa[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) fa[i] = LdsRows<K>::frag(rows, base, 0, i);
    auto steps = [&](int s0, auto first_tag, auto last_tag) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_tag)::value, LAST = decltype(last_tag)::value;
        static_for<R>([&](auto t_tag) __attribute__((always_inline)) {
            constexpr int t = decltype(t_tag)::value;
            __builtin_amdgcn_sched_barrier(0);
            static_for<2 * RB>([&](auto n_tag) __attribute__((always_inline)) {
                constexpr int i = decltype(n_tag)::value / 2, j = decltype(n_tag)::value % 2;
                const bf16x8 wf = __builtin_bit_cast(bf16x8, ring[2 * t + j]);
                const f32x16 c = FIRST && t == 0 ? f32x16{} : acc[i][j];
                acc[i][j] = V ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], wf, c, 0, 0, 0)
                              : __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, fa[i], c, 0, 0, 0);
                if constexpr (j == 1 && !(LAST && t == R - 1)) fa[i] = LdsRows<K>::frag(rows, base, s0 + t + 1, i);
                if constexpr (i == RB - 1 && (MORE || !LAST))
                    ring[2 * t + j] = LAST ? unit_frag<K>(w, w_at, next, 2 * t + j, lane) : unit_frag<K>(w, w_at, unit, 2 * (s0 + R + t) + j, lane);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    };
    steps(0, std::true_type{}, std::false_type{});
#pragma unroll 1
    for (int s0 = R; s0 + R < S; s0 += R) steps(s0, std::false_type{}, std::false_type{});
    steps(S - R, std::false_type{}, std::true_type{});
}

// rows of a row block's accumulators (weights, rows) as chunks, times rs: x[2 j + a] = columns 32 j + 16 a + 8 (lane / 32) .. + 7 of row lane % 32
static __device__ __forceinline__ void row_chunks(const f32x16 (&acc)[2], float rs, bool zero, u32x4 (&x)[4])
{
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            uint32_t y[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                y[e] = pack2(acc[j][8 * a + 2 * e] * rs, acc[j][8 * a + 2 * e + 1] * rs);
                if (zero) y[e] = 0;
            }
            const auto p = __builtin_amdgcn_permlane32_swap(y[0], y[2], false, false);
            const auto q = __builtin_amdgcn_permlane32_swap(y[1], y[3], false, false);
            x[2 * j + a] = u32x4{p[0], q[0], p[1], q[1]};
        }
}

// chunks -> whole rows: x[n] = chunk row_chunk(lane) of row 8 n + lane % 8
static __device__ __forceinline__ void whole_rows(u32x4 (&x)[4])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        uint32_t y[4];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const auto p = __builtin_amdgcn_permlane16_swap(x[2 * j][e], x[2 * j + 1][e], false, false);
            y[j] = p[0], y[2 + j] = p[1];
        }
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int x0 = (int)y[2 * m], x1 = (int)y[2 * m + 1];
            x[2 * m][e] = (uint32_t)__builtin_amdgcn_update_dpp(x0, x1, 0x128, 0xf, 0xc, false);      // row_ror:8
            x[2 * m + 1][e] = (uint32_t)__builtin_amdgcn_update_dpp(x1, x0, 0x128, 0xf, 0x3, false);
        }
    }
}
static __device__ __forceinline__ int row_chunk(int lane) { return 4 * ((lane >> 3) & 1) + 2 * ((lane >> 4) & 1) + (lane >> 5); }

// Units u, u + step, ... below `end` of the rows m0 .. m0 + 32 RB - 1 (RB even; scale: a factor per row in LDS).  `ring` holds the
// first 2 R fragments of unit u.  CACHE: the rows go to the cache, which holds all of them (user: of every 64), else to
// out.rows, from row out.n_cached on, as far as there are any (below M).
template <int K, int RB, int R, bool CACHE>
static __device__ __forceinline__ void qkv_units(const uint8_t *rows, const float *scale, __amdgpu_buffer_rsrc_t w, int w_at,
                                                 u32x4 (&ring)[2 * R], int u, int step, int end, const QkvOut &out,
                                                 const CacheUser (&user)[(RB + 1) / 2], int m0, int M, int lane)
{
    const int l32 = lane & 31, hf = lane >> 5;
    const uint32_t a_base = LdsRows<K>::base(l32, hf);
    f32x16 acc[RB][2];
    const int chunk = row_chunk(lane);
#pragma unroll 1
    for (; u < end; u += step) {
        const int next = u + step < end ? u + step : u, col = u * 64, d = out.qc.d;
        const int which = CACHE ? col / d : 0, h = CACHE ? col % d / 64 : 0;
        auto block = [&](int i) __attribute__((always_inline)) {  // the cache block of row block i
            const CacheUser &b = user[i / 2];
            return out.qc.layer_base + ((size_t)b.t0 * out.qc.H + (size_t)h * b.l_pad) * 256 + (size_t)((m0 + 32 * i - b.t0) / 32) * 8192 + lane * 16;
        };
        if (CACHE && which == 2) {
            unit_product<K, RB, R, true>(acc, rows, w, w_at, ring, a_base, u, next, lane);
#pragma unroll
            for (int i = 0; i < RB; ++i) {
                if (m0 + 32 * i >= M) break;
                const int valid = user[i / 2].l_valid - (m0 + 32 * i - user[i / 2].t0);  // rows of the block that count
                uint8_t *to = block(i) + 4096;
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    float rs[8];
                    *(float4 *)rs = *(const float4 *)(scale + 32 * i + 16 * g + 4 * hf);
                    *(float4 *)(rs + 4) = *(const float4 *)(scale + 32 * i + 16 * g + 8 + 4 * hf);
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        u32x4 x;
#pragma unroll
                        for (int e = 0; e < 8; e += 2)
                            x[e / 2] = pack2(acc[i][j][8 * g + e] * rs[e], acc[i][j][8 * g + e + 1] * rs[e + 1]);
                        if (valid < 32) {
#pragma unroll
                            for (int e = 0; e < 8; e += 2) {
                                const int r = 16 * g + 8 * (e >> 2) + 4 * hf + (e & 3);
                                x[e / 2] = r + 1 < valid ? x[e / 2] : r < valid ? x[e / 2] & 0xffff : 0;
                            }
                        }
                        *(u32x4 *)(to + (g * 2 + j) * 1024) = x;
                    }
                }
            }
        } else {
            unit_product<K, RB, R, false>(acc, rows, w, w_at, ring, a_base, u, next, lane);
#pragma unroll
            for (int i = 0; i < RB; ++i) {
                const int r0 = m0 + 32 * i;
                if (r0 >= M) break;
                u32x4 x[4];
                row_chunks(acc[i], scale[32 * i + l32], CACHE && r0 + l32 - user[i / 2].t0 >= user[i / 2].l_valid, x);
                if (which == 1) {
                    uint8_t *to = block(i);
#pragma unroll
                    for (int n = 0; n < 4; ++n) *(u32x4 *)(to + n * 1024) = x[n];
                } else {
                    whole_rows(x);
                    __bf16 *to = CACHE ? (__bf16 *)out.q + (int64_t)r0 * out.ld_q + h * 64 : (__bf16 *)out.rows + (int64_t)(r0 - out.n_cached) * out.ld_rows + col;
                    const int64_t ld = CACHE ? out.ld_q : out.ld_rows;
#pragma unroll
                    for (int n = 0; n < 4; ++n)
                        if (CACHE || r0 + 8 * n + (lane & 7) < M) *(u32x4 *)(to + (8 * n + (lane & 7)) * ld + chunk * 8) = x[n];
                }
            }
        }
    }
}

}  // namespace gemm
}  // namespace climber
