// bf16 MFMA GEMM for few rows: the projections (f_QKV and f_FFN of Eq. (3), Climber, arXiv 2502.09888) of
// a request or a small batch, where the macro tiles of gemm_bf16.hip leave most of the chip idle and the
// time is the latency of a workgroup's serial chain of k-tiles.
//
// A wave owns a 32 x 32 block of C and its whole K; two waves side by side (64 columns, what the epilogues need:
// one head, one 64-column slice of the row sums of squares) form a workgroup.  Nothing is shared through LDS on
// the way in: every wave loads its operand fragments from global memory (L2) straight into registers, D k-steps
// ahead (2*D KiB in flight per wave, more than the latency of L2 times what the wave consumes), so the k-loop has
// no barrier and no wait for other waves.  Weights come in fragment order (1 KiB per load); a fragment of A is 16
// bytes from each of 32 rows, or 1 KiB of the tiled layout.  Bound by the loads: two fragments of 1 KiB per MFMA
// and wave at the 64 bytes per clock of a CU's vector cache, i.e. 64 clocks per k-step of a workgroup.  FFN down
// (N = 512, K = 2048) at 200 / 1024 rows: 8.1 / 9.1 us against 19.4 / 20.0 with 128 x 128 tiles; attention output
// (N = K = 512) 5.0 / 5.4 against 9.4 / 9.8 (about 3.5 us of each are the launch itself).
// Per output element the products are summed in the same order as in gemm_bf16.hip (k ascending, one
// accumulator, the same MFMA): the two kernels give the same bits, so a row's result does not depend on how many
// rows a launch has.
#include "gemm_common.h"
#include "lanes.h"

namespace climber {
namespace {

using namespace gemm;

template <int EPI, int D>
__global__ __launch_bounds__(128) void gemm_small_kernel(
    const __bf16 *A, int64_t lda, const __bf16 *Wp, int M, int N, int K, void *C, int64_t ldc, const float *resid,
    int64_t ldr, const RowNormIn nin, const RowNormOut nout, const int tiled, const QkvToCache qc, const int by_cols)
{
    constexpr bool F32 = EPI == EPI_RESID_F32;
    constexpr int kPitch = epilogue_pitch<EPI, 2>();
    __shared__ __attribute__((aligned(16))) uint8_t tr[32 * kPitch];

    const int tid = threadIdx.x, lane = tid & 63, wn = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    // Tile of this workgroup.  Launch indices equal modulo 8 run on one XCD (one L2): the tiles are dealt so
    // that an XCD sees an eighth of the larger operand and all of the smaller one.
    const int n_ct = N / 64, n_rt = (M + 31) / 32;
    int ct, rt;
    {
        const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
        if (by_cols) {
            rt = j % n_rt, ct = j / n_rt * 8 + xcd;
        } else {
            ct = j % n_ct, rt = j / n_ct * 8 + xcd;
        }
        if (ct >= n_ct || rt >= n_rt) return;
    }
    const int m0 = rt * 32, n0 = ct * 64;
    const int S = K / 16;  // k-steps; a multiple of D

    const int row = m0 + l32;
    const bool a_tiled = tiled & kTiledA;
    const int a_step = a_tiled ? 512 : 32;  // elements per two k-steps
    const __bf16 *a_src;
    int a_odd;                              // distance from an even k-step's fragment to the odd one's
    if (a_tiled) {
        const int r = row & 15, x = r >> 2;
        a_src = A + (int64_t)min(row >> 4, (M - 1) >> 4) * (K / 32) * 512 + r * 32 + (hf ^ x) * 8;
        a_odd = (((2 + hf) ^ x) - (hf ^ x)) * 8;
    } else {
        a_src = A + (int64_t)min(row, M - 1) * lda + 8 * hf;
        a_odd = 16;
    }
    const __bf16 *w_src = Wp + ((int64_t)(n0 / 32 + wn) * S * 64 + lane) * 8;

    bf16x8 fa[D], fw[D];
    auto load = [&](int s, int slot) __attribute__((always_inline)) {
        fw[slot] = *(const bf16x8 *)(w_src + (int64_t)s * 512);
        fa[slot] = *(const bf16x8 *)(a_src + (int64_t)(s >> 1) * a_step + (slot & 1 ? a_odd : 0));
    };
#pragma unroll
    for (int s = 0; s < D; ++s) load(s, s);

    // what the epilogue needs of global memory is requested behind the first operands: the partial sums of
    // squares of the input rows (the lane's accumulators belong to row l32 of the tile), or the residual rows
    const bool scaled = !F32 && nin.ss, ss_fast = scaled && (nin.n_part == 8 || nin.n_part == 4);
    float4 raw_ss[2] = {};
    if (ss_fast) {
        const float *p = nin.ss + (int64_t)min(row, M - 1) * nin.n_part;
        raw_ss[0] = *(const float4 *)p;
        raw_ss[1] = *(const float4 *)(p + (nin.n_part == 8 ? 4 : 0));
    }
    float4 rsd[4];
    if constexpr (F32) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int id = (4 * wn + it) * 64 + lane, r = id >> 4, cc = id & 15;
            rsd[it] = *(const float4 *)(resid + (int64_t)min(m0 + r, M - 1) * ldr + n0 + cc * 4);
        }
    }
    CacheUser user{0, 64, 0};
    const bool to_cache = EPI == EPI_STORE_BF16 && qc.layer_base;
    if (to_cache) user = cache_user(qc, __builtin_amdgcn_readfirstlane(min(m0, M - 32)));

    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    for (int s0 = 0; s0 + D < S; s0 += D) {
#pragma unroll
        for (int s = 0; s < D; ++s) {
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[s], fa[s], acc, 0, 0, 0);
            load(s0 + D + s, s);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int s = 0; s < D; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[s], fa[s], acc, 0, 0, 0);

    // Epilogue (as wave_epilogue): the lane holds C[m0 + l32][n0 + 32 wn + 8g + 4hf + 0..3]; both waves stage
    // their halves of the 64 columns, then each stores half of the block.
    float rs = 1.f;
    if (ss_fast) {
        const float4 u = raw_ss[0], v = raw_ss[1];
        const float ss = nin.n_part == 8 ? ((u.x + u.y) + (u.z + u.w)) + ((v.x + v.y) + (v.z + v.w))
                                         : ((u.x + u.y) + u.z) + u.w;
        rs = 1.f / sqrtf(ss * nin.inv_d + nin.eps);
    } else if (scaled) {
        rs = row_scale(nin, min(row, M - 1));
    }
    const bool zero_row = to_cache && row - user.t0 >= user.l_valid;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int col = 32 * wn + 8 * g + 4 * hf;
        if (F32) {
            *(float4 *)(tr + l32 * kPitch + col * 4) = float4{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
        } else {
            __attribute__((aligned(8))) __bf16 v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = acc[4 * g + e] * rs;
                v[e] = (__bf16)(EPI == EPI_GELU_BF16 ? gelu_erf(x) : EPI == EPI_RELU_BF16 ? fmaxf(x, 0.f) : x);
            }
            if (zero_row) v[0] = v[1] = v[2] = v[3] = (__bf16)0.f;
            *(uint2 *)(tr + l32 * kPitch + col * 2) = *(const uint2 *)v;
        }
    }
    __syncthreads();
    if constexpr (F32) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int id = (4 * wn + it) * 64 + lane, r = id >> 4, cc = id & 15, out = m0 + r, col = n0 + cc * 4;
            float4 o = *(const float4 *)(tr + r * kPitch + cc * 16);
            const float4 rd = rsd[it];
            o.x += rd.x; o.y += rd.y; o.z += rd.z; o.w += rd.w;
            if (out < M) {
                *(float4 *)((float *)C + (int64_t)out * ldc + col) = o;
                if (nout.ss) {
                    bf16x4 ob;
                    ob[0] = (__bf16)o.x; ob[1] = (__bf16)o.y; ob[2] = (__bf16)o.z; ob[3] = (__bf16)o.w;
                    *(bf16x4 *)((__bf16 *)nout.xb + (int64_t)out * nout.ldb + col) = ob;
                }
            }
            if (nout.ss) {  // sum of squares of the row's 64-column slice: 16 lanes
                const float sq = row_sum16(sumsq4(o.x, o.y, o.z, o.w));
                if (cc == 0 && out < M) nout.ss[(int64_t)out * (N / 64) + n0 / 64] = sq;
            }
        }
    } else if (to_cache) {
        store_block_to_cache<kPitch>(tr, qc, user, m0, n0, M, C, ldc, lane, 2 * wn, 2 * wn + 2);
    } else {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int it = 2 * wn + half;
            if (EPI == EPI_GELU_BF16 && (tiled & kTiledC)) {
                // piece `it` = (16-row group it / 2, k-tile it % 2) of the block
                const int rr = 16 * (it >> 1) + (lane >> 2), c = (lane & 3) ^ ((lane >> 4) & 3);
                if (m0 + rr < M)
                    *(uint4 *)((uint8_t *)C + ((int64_t)((m0 >> 4) + (it >> 1)) * (N / 32) + (n0 >> 5) + (it & 1)) * 1024 +
                               lane * 16) = *(const uint4 *)(tr + rr * kPitch + ((it & 1) * 4 + c) * 16);
            } else {
                const int id = it * 64 + lane, r = id >> 3, cc = id & 7;
                if (m0 + r < M)
                    *(uint4 *)((__bf16 *)C + (int64_t)(m0 + r) * ldc + n0 + cc * 8) =
                        *(const uint4 *)(tr + r * kPitch + cc * 16);
            }
        }
    }
}

template <int EPI>
hipError_t launch_small(const GemmArgs &g, hipStream_t s)
{
    const int n_ct = g.N / 64, n_rt = (g.M + 31) / 32;
    const int by_cols = g.M < g.N && n_ct % 8 == 0;
    const unsigned grid = by_cols ? (unsigned)n_ct * n_rt : (unsigned)((n_rt + 7) / 8 * 8) * n_ct;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(128), 0, s, (const __bf16 *)g.A, g.lda, (const __bf16 *)g.W, g.M, g.N, g.K,
                           g.C, g.ldc, g.resid, g.ldr, g.nin, g.nout, g.tiled, g.qc, by_cols);
        return hipGetLastError();
    };
    return g.K % 256 == 0 ? go(gemm_small_kernel<EPI, 16>) : go(gemm_small_kernel<EPI, 8>);
}

}  // namespace

hipError_t gemm_small_bf16(int epi, const GemmArgs &g, hipStream_t s)
{
    if (g.N % 64 != 0 || g.K % 128 != 0) return hipErrorInvalidValue;
    switch (epi) {
    case EPI_STORE_BF16: return launch_small<EPI_STORE_BF16>(g, s);
    case EPI_GELU_BF16: return launch_small<EPI_GELU_BF16>(g, s);
    case EPI_RESID_F32: return launch_small<EPI_RESID_F32>(g, s);
    case EPI_RELU_BF16: return launch_small<EPI_RELU_BF16>(g, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace climber
