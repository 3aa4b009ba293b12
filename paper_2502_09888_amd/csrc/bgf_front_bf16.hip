// The front of the fusion layer (Eq. (4) of Climber, arXiv 2502.09888): its fused QKV projection and the attention over the N_b
// rows of a candidate, one launch from the fp32 block outputs to the bf16 attention outputs.  As launches of their own
// (gemm_resident_bf16.hip, bgf_attention_kernel) queries, keys and values of all rows go to memory and come back for N_b x N_b
// logits a head, twice the bytes of the rows themselves.
//
// A workgroup has two blocks of 32 rows (whole candidates, as many as fit: 32 rows for N_b of 2, 4 or 8, 30 of 3 or 5, 28 of 7, 24 of 6)
// in LDS as gemm_resident_bf16.hip has, and a wave one head (d_model 512: two workgroups share a block's rows): its queries, keys and values are three units of
// qkv_units.h whose accumulators become chunks of 8 features of one row per lane, so that a logit is a few products per lane
// and one exchange between the half-waves, and another row of the candidate is another lane: by DPP where a candidate has 2, 4 or 8
// lanes (6 and 7 rows: 8 lanes), else through the LDS crossbar.  Rounded to bf16 in between, and summed in the order of
// bgf_attention_kernel: same bits.
// 8192 candidates x 4 of 512: 76 us where the two launches take 82 + 23; without the loads of its rows 69, without the attention 68, without
// either 60: the products, whose weights take 27 of the vector cache's time (0.8 MB a workgroup).
#include "bgf.h"
#include "launch.h"
#include "qkv_units.h"

namespace climber {
namespace {

using namespace gemm;

constexpr int RB = 2, NW = 4, R = 4;

template <int K>
constexpr int front_lds_bytes() { return 32 * RB * (K * 2 + 4); }

__device__ __forceinline__ float low(uint32_t x) { return __uint_as_float(x << 16); }
__device__ __forceinline__ float high(uint32_t x) { return __uint_as_float(x & 0xffff0000u); }

__device__ __forceinline__ void spread(const u32x4 (&x)[4], float (&f)[4][8])
{
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int d = 0; d < 4; ++d) f[n][2 * d] = low(x[n][d]), f[n][2 * d + 1] = high(x[n][d]);
}

// Lanes of a candidate: N_b neighbours, or eight of which N_b count.
template <int NB>
constexpr int lanes_of() { return NB == 6 || NB == 7 ? 8 : NB; }
template <int NB>
constexpr bool by_dpp() { return lanes_of<NB>() == 2 || lanes_of<NB>() == 4 || lanes_of<NB>() == 8; }

// (by_dpp) x with the values of rows 4 G .. 4 G + 3 of the lane's candidate in the lane's four neighbours
template <int S, int G>
__device__ __forceinline__ void quad_of(const u32x4 (&x)[4], u32x4 (&y)[4])
{
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int d = 0; d < 4; ++d)
            y[n][d] = S != 8 ? x[n][d]
                      : G == 0 ? (uint32_t)__builtin_amdgcn_update_dpp((int)x[n][d], (int)x[n][d], 0x114, 0xf, 0xa, false)   // row_shr:4 into the odd fours
                               : (uint32_t)__builtin_amdgcn_update_dpp((int)x[n][d], (int)x[n][d], 0x104, 0xf, 0x5, false);  // row_shl:4 into the even ones
}

// sum += a[d] b[d] over d in their order, b of row J of the lane's candidate.  In assembly because the compiler makes a move and a multiply-add
// of it; the waits are what a lane-crossing read of a register just written takes, here and of the sum.  (Early clobber: the sums are written while rows are still to be read, and
// may not share a register with one of the same value.)
#define CLIMBER_DPP " quad_perm:[%[p0],%[p1],%[p2],%[p3]] row_mask:0xf bank_mask:0xf\n\t"
template <int S, int J>
__device__ __forceinline__ float dot_of_row(const float (&a)[8], const float (&b)[8])
{
    constexpr int p0 = S == 2 ? J : J % 4, p2 = S == 2 ? J + 2 : J % 4;
    float sum = 0.f;
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %1, %9" CLIMBER_DPP "v_fmac_f32_dpp %0, %2, %10" CLIMBER_DPP "v_fmac_f32_dpp %0, %3, %11" CLIMBER_DPP
        "v_fmac_f32_dpp %0, %4, %12" CLIMBER_DPP "v_fmac_f32_dpp %0, %5, %13" CLIMBER_DPP "v_fmac_f32_dpp %0, %6, %14" CLIMBER_DPP
        "v_fmac_f32_dpp %0, %7, %15" CLIMBER_DPP "v_fmac_f32_dpp %0, %8, %16" CLIMBER_DPP "s_nop 1"
        : "+&v"(sum)
        : "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]), "v"(b[4]), "v"(b[5]), "v"(b[6]), "v"(b[7]), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]),
          "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7]), [p0] "n"(p0), [p1] "n"(p0), [p2] "n"(p2), [p3] "n"(p2));
    return sum;
}
// out[d] += p b[d], likewise
template <int S, int J>
__device__ __forceinline__ void add_of_row(float p, const float (&b)[8], float (&out)[8])
{
    constexpr int p0 = S == 2 ? J : J % 4, p2 = S == 2 ? J + 2 : J % 4;
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %8, %16" CLIMBER_DPP "v_fmac_f32_dpp %1, %9, %16" CLIMBER_DPP "v_fmac_f32_dpp %2, %10, %16" CLIMBER_DPP
        "v_fmac_f32_dpp %3, %11, %16" CLIMBER_DPP "v_fmac_f32_dpp %4, %12, %16" CLIMBER_DPP "v_fmac_f32_dpp %5, %13, %16" CLIMBER_DPP
        "v_fmac_f32_dpp %6, %14, %16" CLIMBER_DPP "v_fmac_f32_dpp %7, %15, %16" CLIMBER_DPP
        : "+&v"(out[0]), "+&v"(out[1]), "+&v"(out[2]), "+&v"(out[3]), "+&v"(out[4]), "+&v"(out[5]), "+&v"(out[6]), "+&v"(out[7])
        : "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]), "v"(b[4]), "v"(b[5]), "v"(b[6]), "v"(b[7]), "v"(p), [p0] "n"(p0), [p1] "n"(p0), [p2] "n"(p2),
          [p3] "n"(p2));
}
#undef CLIMBER_DPP

template <int K, int NB>
__global__ __launch_bounds__(NW * 64, 2) void bgf_front_kernel(const float *e, const __bf16 *Wp, __bf16 *o, const int32_t *scen, const float *tau_scen,
                                                               int n_scen, int m, float scale_log2e, float inv_d, float eps)
{
    constexpr int S = lanes_of<NB>(), CB = 32 / S, U = CB * NB, H = K / 64;  // candidates and rows of a block, heads
    static_assert(H % NW == 0, "a head for each wave");
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    float *const scale = (float *)(lds + 32 * RB * K * 2);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hf = lane >> 5;
    const int turn = (int)blockIdx.x >> 3, part = turn % (H / NW);  // (parts of a tile on one XCD)
    const int c0 = (turn / (H / NW) * 8 + ((int)blockIdx.x & 7)) * (RB * CB);  // the tile's first candidate
    if (c0 >= m) return;
    const int n_rows = min(m - c0, RB * CB) * NB;  // of the tile; lane l of block i has row i U + l / S N_b + l % S, where there is one
    auto slot_row = [&](int r) __attribute__((always_inline)) { return min(min(r / S, CB - 1) * NB + min(r % S, NB - 1), U - 1); };
    const int64_t row0 = (int64_t)c0 * NB;

    const __amdgpu_buffer_rsrc_t w = __builtin_amdgcn_make_buffer_rsrc((void *)Wp, 0, 3 * K * K * 2, 0x00020000);
    u32x4 ring[2 * R];
    const int h = NW * part + wave;
    {   // rows into LDS, rounded; their sums of squares: as gemm_resident_bf16.hip
        constexpr int P = K / 256, kTurn = 32 * RB / NW;
        const int r0 = wave * kTurn;
        float4 raw[kTurn][P];
#pragma unroll
        for (int k = 0; k < kTurn; ++k) {
            const int r = r0 + k, row = min(r / 32 * U + slot_row(r % 32), n_rows - 1);
#pragma unroll
            for (int q = 0; q < P; ++q) raw[k][q] = *((const float4 *)e + (row0 + row) * (K / 4) + 64 * q + lane);
        }
        float sum[kTurn];
#pragma unroll
        for (int k = 0; k < kTurn; ++k) {
            const int r = r0 + k;
            sum[k] = 0.f;
#pragma unroll
            for (int q = 0; q < P; ++q) {
                const float4 f = raw[k][q];
                bf16x4 v;
                v[0] = (__bf16)f.x, v[1] = (__bf16)f.y, v[2] = (__bf16)f.z, v[3] = (__bf16)f.w;
                sum[k] += sumsq4(f.x, f.y, f.z, f.w);
                const int c = 32 * q + lane / 2;
                *(bf16x4 *)(lds + r * (K * 2) + ((c & ~15) | ((c & 15) ^ (r & 15))) * 16 + 8 * (lane & 1)) = v;
            }
        }
#pragma unroll
        for (int x = 32; x > 0; x >>= 1)
#pragma unroll
            for (int k = 0; k < kTurn; ++k) sum[k] += __shfl_xor(sum[k], x, 64);
#pragma unroll
        for (int k = 0; k < kTurn; ++k)
            if (lane == k) scale[r0 + k] = 1.f / sqrtf(sum[k] * inv_d + eps);
    }
#pragma unroll
    for (int f = 0; f < 2 * R; ++f) ring[f] = unit_frag<K>(w, 0, h, f, lane);
    const int mine = min(l32 / S, CB - 1);  // the lane's candidate of a block
    float cs[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) cs[i] = scale_log2e / tau_scen[min(max(scen[min(c0 + i * CB + mine, m - 1)], 0), n_scen - 1)];
    __syncthreads();

    const uint32_t a_base = LdsRows<K>::base(l32, hf);
    f32x16 acc[RB][2];
    u32x4 q[RB][4], k[RB][4], v[RB][4];
    auto unit = [&](int u, auto more_tag, u32x4 (&x)[RB][4]) __attribute__((always_inline)) {
        unit_product<K, RB, R, false, decltype(more_tag)::value>(acc, lds, w, 0, ring, a_base, u, H + u, lane);
#pragma unroll
        for (int i = 0; i < RB; ++i) row_chunks(acc[i], scale[32 * i + l32], false, x[i]);
    };
    unit(h, std::true_type{}, q);
    unit(H + h, std::true_type{}, k);
    unit(2 * H + h, std::false_type{}, v);
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        float t[NB], mx = -INFINITY;
        auto logit = [&](auto j_tag, const float (&dot)[4]) __attribute__((always_inline)) {
            constexpr int j = decltype(j_tag)::value;
            float s[4];
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(dot[n]), __float_as_uint(dot[n]), false, false);
                s[n] = __uint_as_float(both[0]) + __uint_as_float(both[1]);
            }
            t[j] = ((s[0] + s[1]) + (s[2] + s[3])) * cs[i];  // log2 units
            mx = fmaxf(mx, t[j]);
        };
        float sum = 0.f, out[4][8] = {};
        if constexpr (by_dpp<NB>()) {
            float a[4][8], b[4][8];
            u32x4 x[4];
            spread(q[i], a);
            static_for<(NB + 3) / 4>([&](auto g_tag) __attribute__((always_inline)) {
                constexpr int G = decltype(g_tag)::value;
                quad_of<S, G>(k[i], x);
                spread(x, b);
                static_for<(NB - 4 * G < 4 ? NB - 4 * G : 4)>([&](auto j_tag) __attribute__((always_inline)) {
                    constexpr int j = 4 * G + decltype(j_tag)::value;
                    float dot[4];
#pragma unroll
                    for (int n = 0; n < 4; ++n) dot[n] = dot_of_row<S, j>(a[n], b[n]);
                    logit(std::integral_constant<int, j>{}, dot);
                });
            });
            static_for<(NB + 3) / 4>([&](auto g_tag) __attribute__((always_inline)) {
                constexpr int G = decltype(g_tag)::value;
                quad_of<S, G>(v[i], x);
                spread(x, b);
                static_for<(NB - 4 * G < 4 ? NB - 4 * G : 4)>([&](auto j_tag) __attribute__((always_inline)) {
                    constexpr int j = 4 * G + decltype(j_tag)::value;
                    const float p = exp2f(t[j] - mx);
                    sum += p;
#pragma unroll
                    for (int n = 0; n < 4; ++n) add_of_row<S, j>(p, b[n], out[n]);
                });
            });
        } else {
            const int at = (hf * 32 + mine * S) * 4;
            static_for<NB>([&](auto j_tag) __attribute__((always_inline)) {
                constexpr int j = decltype(j_tag)::value;
                float dot[4] = {};
#pragma unroll
                for (int n = 0; n < 4; ++n)
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        const uint32_t b = (uint32_t)__builtin_amdgcn_ds_bpermute(at + 4 * j, (int)k[i][n][d]);
                        dot[n] = fmaf(high(q[i][n][d]), high(b), fmaf(low(q[i][n][d]), low(b), dot[n]));
                    }
                logit(j_tag, dot);
                __builtin_amdgcn_sched_barrier(0);  // (or the registers do not hold what is taken ahead)
            });
            static_for<NB>([&](auto j_tag) __attribute__((always_inline)) {
                constexpr int j = decltype(j_tag)::value;
                const float p = exp2f(t[j] - mx);
                sum += p;
#pragma unroll
                for (int n = 0; n < 4; ++n)
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        const uint32_t b = (uint32_t)__builtin_amdgcn_ds_bpermute(at + 4 * j, (int)v[i][n][d]);
                        out[n][2 * d] = fmaf(p, low(b), out[n][2 * d]);
                        out[n][2 * d + 1] = fmaf(p, high(b), out[n][2 * d + 1]);
                    }
                __builtin_amdgcn_sched_barrier(0);
            });
        }
        const float inv = 1.f / sum;
        u32x4 x[4];
#pragma unroll
        for (int n = 0; n < 4; ++n)
#pragma unroll
            for (int d = 0; d < 4; ++d) x[n][d] = pack2(out[n][2 * d] * inv, out[n][2 * d + 1] * inv);
        whole_rows(x);
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            const int l = 8 * n + (lane & 7), row = i * U + l / S * NB + l % S;
            if (l / S < CB && l % S < NB && row < n_rows) *(u32x4 *)(o + (row0 + row) * K + h * 64 + row_chunk(lane) * 8) = x[n];
        }
    }
}

template <int K, int NB>
hipError_t launch(const float *e, const void *wqkv, void *o, const int32_t *scen, const float *tau_scen, int n_scen, int64_t m, float qk_scale,
                  float inv_d, float eps, hipStream_t s)
{
    constexpr auto kernel = bgf_front_kernel<K, NB>;
    const hipError_t err = raise_lds_limit<kernel>(front_lds_bytes<K>());
    if (err != hipSuccess) return err;
    const int per = RB * (32 / lanes_of<NB>()), tiles = (int)((m + per - 1) / per), parts = K / 64 / NW;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((tiles + 7) / 8 * 8 * parts)), dim3(NW * 64), front_lds_bytes<K>(), s, e, (const __bf16 *)wqkv,
                       (__bf16 *)o, scen, tau_scen, n_scen, (int)m, qk_scale * 1.4426950408889634f, inv_d, eps);
    return hipGetLastError();
}

}  // namespace

// Us a call, one launch / projection and attention apart (with a launch for the rows' sums before them up to 8192 rows), N_b x d_model, d_gate 256 or 128:
// 4 x 512 250 candidates 65.8 / 60.2, 500 78.1 / 76.1, 1000 89.6 / 92.3, 2000 105 / 116, 8192 301 / 338; 4 x 256 1000 59.8 / 59.9, 8192 94.5 / 119; 2 x 512 2000
// 84.8 / 87.5, 4100 106 / 114; 8 x 512 400 101 / 105, 5000 393 / 429; 8 x 256 12000 273 / 337; 7 x 512 600 109 / 114; 6 x 256 1000 64.0 / 70.2.  Through the LDS
// crossbar: 3 x 512 1000 83.1 / 83.0, 1400 93.5 / 96.6, 9000 260 / 285; 3 x 256 1400 59.8 / 58.7, 12000 126 / 146; 5 x 512 800 102 / 99, 1000 105.6 / 104.5, 2000
// 132 / 134, 6000 298 / 311.  More than eight rows a candidate: one wave's registers do not hold them.
bool bgf_front_takes(int64_t m, int nb, int d)
{
    return nb >= 2 && nb <= 8 && (d == 256 || d == 512) && m * nb >= (nb == 3 || nb == 5 ? 6144 : 4000);
}

hipError_t launch_bgf_front(const float *e, const void *wqkv, void *o, const int32_t *scen, const float *tau_scen, int n_scen, int64_t m, int nb,
                            int d, float qk_scale, float inv_d, float eps, hipStream_t s)
{
    if (m <= 0) return hipSuccess;
    auto as = [&](auto nb_tag) {
        constexpr int NB = decltype(nb_tag)::value;
        if (d == 512) return launch<512, NB>(e, wqkv, o, scen, tau_scen, n_scen, m, qk_scale, inv_d, eps, s);
        if (d == 256) return launch<256, NB>(e, wqkv, o, scen, tau_scen, n_scen, m, qk_scale, inv_d, eps, s);
        return hipErrorInvalidValue;
    };
    switch (nb) {
    case 2: return as(std::integral_constant<int, 2>{});
    case 3: return as(std::integral_constant<int, 3>{});
    case 4: return as(std::integral_constant<int, 4>{});
    case 5: return as(std::integral_constant<int, 5>{});
    case 6: return as(std::integral_constant<int, 6>{});
    case 7: return as(std::integral_constant<int, 7>{});
    case 8: return as(std::integral_constant<int, 8>{});
    default: return hipErrorInvalidValue;
    }
}

}  // namespace climber
