// bf16 MFMA GEMM for few rows: the projections (f_QKV and f_FFN of Eq. (3), Climber, arXiv 2502.09888) of
// a request or a small batch, where the macro tiles of gemm_bf16.hip leave most of the chip idle and the
// time is the latency of a workgroup's serial chain of k-tiles.
//
// A workgroup has 64 columns (what the epilogues need: one head, one 64-column slice of the row sums of squares) of 16 or 32 rows
// and their whole K; each of its four waves 16 columns, whose weights go straight from L2 into registers, 16 k-tiles of 32 ahead (in
// fragment order, 1 KiB a load: a quarter of the workgroup's, nobody's twice).  The rows come by way of LDS, 256 k at a time with a barrier
// each, the loads of the next but one in flight.  Bound by the loads, at the 64 bytes per clock of a CU's vector cache: 4 KiB of weights
// and 1 or 2 of rows per k-tile, so 16 rows cost a workgroup 5/6 of what 32 do and are taken while there are CUs for twice the workgroups.  (Beside them
// LDS: bank conflicts of 133 to 176 % of its active cycles, by the rows' places, which are the tiled layout's and suit reads of 32 x 32 x 16.)
// One request (1000 behaviours, 200 candidates, four layers, d_model 512) 216 us; with two waves of 32 columns a workgroup, each with its own
// fragments of all 32 rows (8 KiB per k-tile, 56 workgroups for 200 rows x 512), 244.  Score of 16 rows 86.6 / 110.9, 128 92.6 / 123.5, 256 101
// / 126, 640 127 / 135; d_model 256 72.3 / 79.8, 81.8 / 89.8, 82.4 / 91.1, 88.4 / 98.9.  32 k-tiles ahead: 0.99.
// Per output element the products are summed in the same order as in gemm_bf16.hip (k ascending, one
// accumulator; an instruction of 16 x 16 x 32 sums as two of 32 x 32 x 16 do, one after the other): the two kernels give the same
// bits, so a row's result does not depend on how many rows a launch has.
#include "gemm_common.h"
#include "lanes.h"

namespace climber {
namespace {

using namespace gemm;

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

constexpr int NW = 4;

// RB blocks of 16 rows a workgroup; K in chunks of C k-tiles of 32, of which U are a turn of the loop and of the weights' ring.
// IN: the rows are a call's inputs in place of bf16 rows with their sums.  Their sums of squares are formed here, in the order of row_prep_kernel, and of
// bf16 rows the fp32 copy goes to x32, 64 columns by each of the first K / 64 workgroups of a row block; fp32 rows are rounded on their way into
// LDS: instead of a launch before, 2 to 2.5 us.  K of 256 or 512.
enum { kSummed = 0, kGivenBf16 = 1, kGivenF32 = 2 };
template <int EPI, int RB, int C, int U, int IN>
__global__ __launch_bounds__(NW * 64, 2) void gemm_small_kernel(
    const __bf16 *A, int64_t lda, const __bf16 *Wp, int M, int N, int K, void *Cout, int64_t ldc, const float *resid,
    int64_t ldr, const RowNormIn nin, const RowNormOut nout, const int tiled, const QkvToCache qc, const int by_cols, float *x32)
{
    constexpr bool F32 = EPI == EPI_RESID_F32, OWN = IN != kSummed;
    constexpr int X = IN == kGivenF32 ? 2 : 1;  // loads per lane and piece
    constexpr int kPitch = epilogue_pitch<EPI, 2>(), kRows = 16 * RB, R = C * U, P = RB * C / NW, kBuf = RB * C * 1024, L = C < 4 ? C : 4;
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * kBuf + kRows * kPitch];
    uint8_t *const tr = lds + 2 * kBuf;
    __shared__ float parts[OWN ? NW : 1][RB][64][2], scale[kRows];
    static_assert(!OWN || (C == 8 && EPI == EPI_STORE_BF16), "");

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l15 = lane & 15, kq = lane >> 4;
    // Tile of this workgroup.  Launch indices equal modulo 8 run on one XCD (one L2): the tiles are dealt so
    // that an XCD sees an eighth of the larger operand and all of the smaller one.
    const int n_ct = N / 64, n_rt = (M + kRows - 1) / kRows;
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
    const int m0 = rt * kRows, n0 = ct * 64;
    const int T = K / 32, n = T / C;  // k-tiles, chunks (a multiple of U)

    // Rows: pieces of 16 rows x 32 k, 1 KiB, in LDS as the tiled layout has them (chunk c of row r at place c ^ r / 4 % 4 of the row's 64 bytes);
    // of a chunk's, one after the other's to each wave.
    const uint8_t *a_src[P];
    const int a_step = (tiled & kTiledA) ? 1024 : 64 * X;  // bytes per k-tile
#pragma unroll
    for (int i = 0; i < P; ++i) {
        const int p = NW * i + wave, g = p / C, kt = p % C;
        if (tiled & kTiledA)
            a_src[i] = (const uint8_t *)A + ((int64_t)min((m0 >> 4) + g, (M - 1) >> 4) * T + kt) * 1024 + lane * 16;
        else
            a_src[i] = (const uint8_t *)A + ((int64_t)min(m0 + 16 * g + (lane >> 2), M - 1) * lda + kt * 32 + ((lane & 3) ^ (lane >> 4)) * 8) * (2 * X);
    }
    auto fetch = [&](int ch, u32x4 (&x)[P][X]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < P; ++i)
#pragma unroll
            for (int e = 0; e < X; ++e) x[i][e] = *(const u32x4 *)(a_src[i] + (int64_t)ch * (C * a_step) + 16 * e);
    };
    auto put = [&](int buf, const u32x4 (&x)[P][X]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < P; ++i) {
            uint8_t *const to = lds + buf * kBuf + (NW * i + wave) * 1024 + lane * 16;
            if constexpr (IN == kGivenF32) {
                bf16x8 v;
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = (__bf16)__uint_as_float(x[i][e >> 2][e & 3]);
                *(bf16x8 *)to = v;
            } else {
                *(u32x4 *)to = x[i][0];
            }
        }
    };
    // Weights: 16 columns x 32 k of two neighbouring fragments of 32 columns x 16 k
    const __bf16 *w_src = Wp + ((int64_t)(n0 / 32 + (wave >> 1)) * 2 * T + (kq >> 1)) * 512 + ((kq & 1) * 32 + (wave & 1) * 16 + l15) * 8;
    bf16x8 ring[R];
    auto weights = [&](int t) __attribute__((always_inline)) { return *(const bf16x8 *)(w_src + (int64_t)t * 1024); };

    u32x4 x0[P][X], x1[P][X];
    fetch(0, x0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < R; ++t) {
        ring[t] = weights(t);
        if (t + 1 == C) fetch(min(1, n - 1), x1);
        __builtin_amdgcn_sched_barrier(0);
    }

    // what the epilogue needs of global memory is requested behind the first operands: the partial sums of
    // squares of the input rows (the lane's accumulators belong to rows l15 of the blocks), or the residual rows
    const bool scaled = !F32 && !OWN && nin.ss, ss_fast = scaled && (nin.n_part == 8 || nin.n_part == 4);
    float4 raw_ss[RB][2] = {};
    if (ss_fast) {
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const float *p = nin.ss + (int64_t)min(m0 + 16 * i + l15, M - 1) * nin.n_part;
            raw_ss[i][0] = *(const float4 *)p;
            raw_ss[i][1] = *(const float4 *)(p + (nin.n_part == 8 ? 4 : 0));
        }
    }
    float4 rsd[RB];
    if constexpr (F32) {
#pragma unroll
        for (int i = 0; i < RB; ++i)
            rsd[i] = *(const float4 *)(resid + (int64_t)min(m0 + 16 * i + (tid >> 4), M - 1) * ldr + n0 + l15 * 4);
    }
    CacheUser user{0, 64, 0};
    const bool to_cache = EPI == EPI_STORE_BF16 && RB == 2 && qc.layer_base;
    if (to_cache) user = cache_user(qc, __builtin_amdgcn_readfirstlane(min(m0, M - 32)));

    auto barrier = []() __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    put(0, x0);
    put(1, x1);
    if constexpr (OWN) {
        // row_prep_kernel adds the squares of four columns c and c + 256, then of column groups 32, 16, 8, 4, 2 and 1 apart: k-tiles 8 apart (the next chunk),
        // 4 (the wave's next), 2 and 1 (other waves), and the row's other places
#pragma unroll
        for (int g = 0; g < RB; ++g)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                float v[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    auto sum = [&](const u32x4 (&x)[X]) __attribute__((always_inline)) {
                        if constexpr (IN == kGivenF32) {
                            const u32x4 f = x[e];
                            return sumsq4(__uint_as_float(f[0]), __uint_as_float(f[1]), __uint_as_float(f[2]), __uint_as_float(f[3]));
                        } else {
                            const uint32_t a = x[0][2 * e], b = x[0][2 * e + 1];
                            return sumsq4(__uint_as_float(a << 16), __uint_as_float(a & 0xffff0000u), __uint_as_float(b << 16), __uint_as_float(b & 0xffff0000u));
                        }
                    };
                    v[i] = sum(x0[2 * g + i]);
                    if (U == 2) v[i] += sum(x1[2 * g + i]);
                }
                parts[wave][g][lane][e] = v[0] + v[1];
            }
    }
    barrier();
    if constexpr (OWN) {
        if (wave < RB) {
            float v[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                auto of = [&](int w) __attribute__((always_inline)) { return parts[w][wave][lane][e]; };
                v[e] = (of(0) + of(2)) + (of(1) + of(3));
                v[e] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[e]), 0x4E, 0xf, 0xf, false));  // quad_perm [2,3,0,1]
                v[e] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[e]), 0xB1, 0xf, 0xf, false));  // quad_perm [1,0,3,2]
            }
            const float ss = v[0] + v[1];
            if ((lane & 3) == 0) scale[16 * wave + (lane >> 2)] = 1.f / sqrtf(ss * nin.inv_d + nin.eps);
        }
    }
    f32x4 acc[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int a_at = l15 * 64 + (kq ^ (l15 >> 2)) * 16;
    auto turn = [&](int ch0, auto last_tag) __attribute__((always_inline)) {
        constexpr bool last = decltype(last_tag)::value;
        static_for<U>([&](auto u_tag) __attribute__((always_inline)) {
            constexpr int u = decltype(u_tag)::value;
            const int ch = ch0 + u;
            const uint8_t *a = lds + (U == 2 ? u : ch & 1) * kBuf + a_at;
            if constexpr (!last || u + 2 < U) fetch(min(ch + 2, n - 1), x0);
            bf16x8 f[L][RB];
#pragma unroll
            for (int t = 0; t < L; ++t)
#pragma unroll
                for (int i = 0; i < RB; ++i) f[t][i] = *(const bf16x8 *)(a + (i * C + t) * 1024);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < C; ++t) {
#pragma unroll
                for (int i = 0; i < RB; ++i) {
                    acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ring[u * C + t], f[t % L][i], acc[i], 0, 0, 0);
                    if (t + L < C) f[t % L][i] = *(const bf16x8 *)(a + (i * C + t + L) * 1024);
                }
                if constexpr (!last) ring[u * C + t] = weights(ch * C + t + R);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (!last || u + 2 < U) {
                barrier();  // the chunk's rows are read, its buffer is the next but one's
                put(U == 2 ? u : ch & 1, x0);
            } else if constexpr (u + 1 < U) {
                barrier();
            }
        });
    };
    int ch = 0;
    if constexpr (!OWN)  // (these K are one turn)
#pragma unroll 1
        for (; ch + U < n; ch += U) turn(ch, std::false_type{});
    turn(ch, std::true_type{});

    if constexpr (OWN) {
        if (IN == kGivenBf16 && ct < K / 64) {
#pragma unroll
            for (int i = 0; i < RB; ++i) {
                const int r = tid >> 4, cc = l15, kt = 2 * ct + (cc >> 3), out = m0 + 16 * i + r;
                const bf16x4 v = *(const bf16x4 *)(lds + (kt / C) * kBuf + (i * C + kt % C) * 1024 + r * 64 + (((cc >> 1) & 3) ^ (r >> 2)) * 16 + (cc & 1) * 8);
                if (out < M) *(float4 *)(x32 + (int64_t)out * K + 64 * ct + 4 * cc) = float4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
            }
        }
        barrier();  // the rows' scales
    }
    // Epilogue (as wave_epilogue): the lane holds C[m0 + 16 i + l15][n0 + 16 wave + 4 kq + 0..3]; the waves stage
    // their quarters of the 64 columns, then each stores a quarter of the block.
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int row = m0 + 16 * i + l15, col = 16 * wave + 4 * kq;
        uint8_t *const at = tr + (16 * i + l15) * kPitch;
        if (F32) {
            *(float4 *)(at + col * 4) = float4{acc[i][0], acc[i][1], acc[i][2], acc[i][3]};
        } else {
            float rs = OWN ? scale[16 * i + l15] : 1.f;
            if (ss_fast) {
                const float4 u = raw_ss[i][0], v = raw_ss[i][1];
                const float ss = nin.n_part == 8 ? ((u.x + u.y) + (u.z + u.w)) + ((v.x + v.y) + (v.z + v.w))
                                                 : ((u.x + u.y) + u.z) + u.w;
                rs = 1.f / sqrtf(ss * nin.inv_d + nin.eps);
            } else if (scaled) {
                rs = row_scale(nin, min(row, M - 1));
            }
            __attribute__((aligned(8))) __bf16 v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = acc[i][e] * rs;
                v[e] = (__bf16)(EPI == EPI_GELU_BF16 ? gelu_erf(x) : EPI == EPI_RELU_BF16 ? fmaxf(x, 0.f) : x);
            }
            if (to_cache && row - user.t0 >= user.l_valid) v[0] = v[1] = v[2] = v[3] = (__bf16)0.f;
            *(uint2 *)(at + col * 2) = *(const uint2 *)v;
        }
    }
    __syncthreads();
    if constexpr (F32) {
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const int r = 16 * i + (tid >> 4), cc = l15, out = m0 + r, col = n0 + cc * 4;
            float4 o = *(const float4 *)(tr + r * kPitch + cc * 16);
            const float4 rd = rsd[i];
            o.x += rd.x; o.y += rd.y; o.z += rd.z; o.w += rd.w;
            if (out < M) {
                *(float4 *)((float *)Cout + (int64_t)out * ldc + col) = o;
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
        store_block_to_cache<kPitch>(tr, qc, user, m0, n0, M, Cout, ldc, lane, wave, wave + 1);
    } else if (wave < 2 * RB) {
        if (EPI == EPI_GELU_BF16 && (tiled & kTiledC)) {
            // piece `wave` = (16-row group wave / 2, k-tile wave % 2) of the block
            const int rr = 16 * (wave >> 1) + (lane >> 2), c = (lane & 3) ^ (lane >> 4);
            if (m0 + rr < M)
                *(uint4 *)((uint8_t *)Cout + ((int64_t)((m0 >> 4) + (wave >> 1)) * (N / 32) + (n0 >> 5) + (wave & 1)) * 1024 +
                           lane * 16) = *(const uint4 *)(tr + rr * kPitch + ((wave & 1) * 4 + c) * 16);
        } else {
            const int r = tid >> 3, cc = tid & 7;
            if (m0 + r < M)
                *(uint4 *)((__bf16 *)Cout + (int64_t)(m0 + r) * ldc + n0 + cc * 8) = *(const uint4 *)(tr + r * kPitch + cc * 16);
        }
    }
}

template <int EPI, int IN = kSummed>
hipError_t launch_small(const GemmArgs &g, hipStream_t s, float *x32 = nullptr)
{
    const int n_ct = g.N / 64;
    // 16 rows a workgroup as long as that makes at most one per CU, two where K is short and no residual row waits for its sums (a direct cache write
    // has blocks of 32).  Us a call, four layers, the line at 128 / 256 workgroups of 32 rows: d_model 512, K = 512, score of 192 rows 102.0 / 98.5, 256
    // 104.0 / 100.7, 320 109.5 / 107.4; d_model 256, score of 400 rows 86.2 / 84.0, 640 92.6 / 88.6; with the residual projections score of 1600 rows 111.1 / 113.9;
    // with K = 2048 (at 192) score of 640 rows 128.0 / 132.8, encode of 600 100.1 / 103.6.  At 64: score of 128 rows 92.5 / 101.4, 400 119.5 / 123.
    const bool half = !g.qc.layer_base && (int64_t)n_ct * ((g.M + 31) / 32) <= (EPI != EPI_RESID_F32 && g.K <= 512 ? 256 : 128);
    const int rows = half ? 16 : 32, n_rt = (g.M + rows - 1) / rows;
    const int by_cols = g.M < g.N && n_ct % 8 == 0;
    const unsigned grid = by_cols ? (unsigned)n_ct * n_rt : (unsigned)((n_rt + 7) / 8 * 8) * n_ct;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(NW * 64), 0, s, (const __bf16 *)g.A, g.lda, (const __bf16 *)g.W, g.M, g.N, g.K,
                           g.C, g.ldc, g.resid, g.ldr, g.nin, g.nout, g.tiled, g.qc, by_cols, x32);
        return hipGetLastError();
    };
    auto of = [&](auto rb) {
        constexpr int RB = decltype(rb)::value;
        if (g.K % 512 == 0) return go(gemm_small_kernel<EPI, RB, 8, 2, IN>);
        if constexpr (IN != kSummed) {
            return go(gemm_small_kernel<EPI, RB, 8, 1, IN>);
        } else {
            if (g.K % 256 == 0) return go(gemm_small_kernel<EPI, RB, 8, 1, kSummed>);
            return go(gemm_small_kernel<EPI, RB, 4, 1, kSummed>);
        }
    };
    return half ? of(std::integral_constant<int, 1>{}) : of(std::integral_constant<int, 2>{});
}

}  // namespace

bool gemm_small_takes(int epi, int M, int N, int K)
{
    // Few rows: until the tiles' (gemm_bf16.hip) reuse of their operands wins: from one workgroup of 32 rows
    // per CU on for QKV, from two for the residual projections, from 2.5 for the up-projection, whose tiled store is a workgroup's own.  Us per call, four layers,
    // d_model 512.  QKV, the line at 256 / 512 / 640 workgroups: score of 560 rows 124.8 / 127.1, 640 127 / 128, 800 128 / - / 134, 1000 131 / - / 131 (768: 136).  Up, at 256
    // / 512 / 640: score of 320 rows 113.5 / 109.5, 400 119.5 / 115.3, 560 - / 127.1 / 124.5, 640 - / 128.1 / 127.4 (768 / 1024: request of 1000 behaviours 223
    // / 228 instead of 217).  Residual, at 384 / 512 / 640 or more: score of 1600 rows 204 / 182, 2000 203 / 185, 2400 223.3 / - / 222, 3200 251 / - / 262, encode of
    // 2048 rows 152.5 / 138; d_model 256, score of 3200 160.7 / 147.6, 4096 158.8 / 154.
    return K % 128 == 0 && (int64_t)(N / 64) * ((M + 31) / 32) <= (epi == EPI_RESID_F32 ? 512 : epi == EPI_GELU_BF16 ? 640 : 256);
}

bool gemm_small_sums(int M, int N, int K)
{
    // A launch less is worth a first projection of up to three workgroups per CU.  Us a call of four layers, the line at 256 / 768 workgroups: score of 336 rows of
    // 512 113.8 / 111.4, 680 126.7 / 124.8, 1000 130.6 / 128.7, of 256 680 92.9 / 90.4, 1600 111.4 / 109.9; encode of 512 rows 90.5 / 87.1, 1000 102.3 / 100.6 (one
    // layer 11.1 / 8.0), of 256 2048 87.4 / 85.9; fusion of 64 candidates x 4 of 512 46.5 / 43.6, 250 53.7 / 53.1, 1000 x 2 of 256 39.6 / 38.5; from there to 1024 even (score of 1200 rows of 512 167.4 / 167.4).
    return (K == 256 || K == 512) && !gemm_resident_takes(M, K, false) && !gemm_resident_takes(M, K, true) && (int64_t)(N / 64) * ((M + 31) / 32) <= 768;
}

hipError_t gemm_small_given(RowsIn in, const void *x, float *x32, const void *w_packed, int M, int N, int K, void *C, int64_t ldc, const RowNormIn &in_norm,
                            const QkvToCache &to_cache, hipStream_t s)
{
    if (M < 1 || N % 64 != 0 || N < K || (K != 256 && K != 512)) return hipErrorInvalidValue;
    const GemmArgs g{x, K, w_packed, M, N, K, C, ldc, nullptr, 0, in_norm, RowNormOut{}, 0, to_cache};
    return in == kRowsF32 ? launch_small<EPI_STORE_BF16, kGivenF32>(g, s) : launch_small<EPI_STORE_BF16, kGivenBf16>(g, s, x32);
}

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
