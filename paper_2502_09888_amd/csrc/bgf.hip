// Bit-wise gating fusion of Climber (arXiv 2502.09888, Sec. 3.1.4, Eq. (4)): what stands
// around the projections of the fusion layer.
//   fusion attention: G = ATL(E): every one of a candidate's N_b block outputs attends to all N_b of
//     them, no relative attention bias, temperature from the candidate's scenario only;
//   gate + head: Y = G (.) sigmoid(f_gate(G)), score = <w_head, vec(Y)> + b;
//     with f_gate's projections in one launch (bgf_gate_kernel) or behind two launches of gemm_bf16.
// N_b is a handful (the number of extraction strategies), so the attention is N_b x N_b logits per
// (candidate, head), held in registers; d_head = 64.
#include "bgf.h"
#include "lanes.h"
#include "qkv_units.h"

namespace climber {
namespace {

constexpr int kMaxBlocks = 16;

using namespace gemm;

// sum over the 8 lanes 8s .. 8s+7, in each of them
__device__ __forceinline__ float sum8(float x)
{
    auto dpp = [](float v, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, false));
    };
    x += dpp(x, std::integral_constant<int, 0xB1>{});   // quad_perm [1,0,3,2]
    x += dpp(x, std::integral_constant<int, 0x4E>{});   // quad_perm [2,3,0,1]
    x += dpp(x, std::integral_constant<int, 0x141>{});  // row_half_mirror: the other quad of the eight
    return x;
}

// qkv: bf16 [m * NB][3 * d] (queries | keys | values, head h at column h * 64); o: bf16 [m * NB][d].
// One wavefront per (candidate, group of 8 heads): lane = (head 8g + lane / 8, features 8 (lane % 8) ..
// + 7), so that every row of a head is loaded and stored as whole 128-byte lines, 16 bytes per lane;
// a logit is 8 products per lane and a sum over the 8 lanes of the head.
template <int NB>
__global__ __launch_bounds__(256) void bgf_attention_kernel(const __bf16 *qkv, __bf16 *o, const int32_t *scen,
                                                            const float *tau_scen, int n_scen, int64_t m, int H,
                                                            float scale_log2e)
{
    const int lane = threadIdx.x & 63, c8 = lane & 7;
    const int groups = (H + 7) >> 3;
    const int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);  // (candidate, group of heads)
    if (item >= m * groups) return;
    const int64_t c = item / groups;
    const int h = (int)(item % groups) * 8 + (lane >> 3), d = H * 64;
    if (h >= H) return;  // whole groups of 8 lanes leave; the sums below stay inside such a group
    const int sc = min(max(scen[c], 0), n_scen - 1);
    const float cs = scale_log2e / tau_scen[sc];
    const __bf16 *base = qkv + c * NB * 3 * (int64_t)d + h * 64 + c8 * 8;
    bf16x8 kj[NB], vj[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        kj[j] = *(const bf16x8 *)(base + (int64_t)j * 3 * d + d);
        vj[j] = *(const bf16x8 *)(base + (int64_t)j * 3 * d + 2 * d);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const bf16x8 qi = *(const bf16x8 *)(base + (int64_t)i * 3 * d);
        float t[NB], mx = -INFINITY;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            float dot = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) dot = fmaf((float)qi[e], (float)kj[j][e], dot);
            t[j] = sum8(dot) * cs;  // log2 units
            mx = fmaxf(mx, t[j]);
        }
        float sum = 0.f, acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const float pj = exp2f(t[j] - mx);
            sum += pj;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] = fmaf(pj, (float)vj[j][e], acc[e]);
        }
        const float inv = 1.f / sum;
        bf16x8 ov;
#pragma unroll
        for (int e = 0; e < 8; ++e) ov[e] = (__bf16)(acc[e] * inv);
        *(bf16x8 *)(o + (c * NB + i) * (int64_t)d + h * 64 + c8 * 8) = ov;
    }
}

// four values of Y = G (.) sigmoid(pre), and their part of the head's sum
__device__ __forceinline__ float4 gated(const float4 &g, const bf16x4 &pre)
{
    float4 y;
    y.x = g.x * __builtin_amdgcn_rcpf(1.f + __expf(-(float)pre[0]));
    y.y = g.y * __builtin_amdgcn_rcpf(1.f + __expf(-(float)pre[1]));
    y.z = g.z * __builtin_amdgcn_rcpf(1.f + __expf(-(float)pre[2]));
    y.w = g.w * __builtin_amdgcn_rcpf(1.f + __expf(-(float)pre[3]));
    return y;
}
__device__ __forceinline__ float head_sum(const float4 &y, const float4 &w, float sum)
{
    return fmaf(y.x, w.x, fmaf(y.y, w.y, fmaf(y.z, w.z, fmaf(y.w, w.w, sum))));
}

// g: fp32 [m][nd] (the fusion layer's output), pre: bf16 [m][nd] (f_gate(G) before the sigmoid); y (nullable): fp32 [m][nd];
// score: [m].  One wavefront per candidate.
__global__ __launch_bounds__(256) void bgf_gate_head_kernel(const float *g, const __bf16 *pre, const float *w_head,
                                                            float b_head, float *y, float *score, int64_t m, int nd)
{
    const int lane = threadIdx.x & 63;
    const int64_t c = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (c >= m) return;
    float acc = 0.f;
    // four consecutive values per lane and step (nd is a multiple of 64): 16-byte loads and stores
    for (int e = lane * 4; e < nd; e += 256) {
        const float4 gv = *(const float4 *)(g + c * nd + e);
        const float4 wv = *(const float4 *)(w_head + e);
        const bf16x4 pv = *(const bf16x4 *)(pre + c * nd + e);
        const float4 yv = gated(gv, pv);
        if (y) *(float4 *)(y + c * nd + e) = yv;
        acc = head_sum(yv, wv, acc);
    }
    acc = wave_sum64(acc);
    if (lane == 0) score[c] = acc + b_head;
}

// Both projections of the gate, the gate and the head in one launch for 32 candidates a workgroup.  Down: a wave per 32 columns of the
// hidden, the rows by way of registers into a double buffer of 256 columns, weights from L2 into registers.  Up: 256 columns a
// step, a wave per 32 of them; their bf16 values meet G in LDS, where a wave takes whole rows as bgf_gate_head_kernel does: the same
// bits as by the three launches.  8192 candidates x 4 blocks of 512, d_gate 256: 66 us instead of 25 + 19 + 30, of which the bytes of G and
// Y take 33 and the weights' way from L2 (2 MB a workgroup) about as long (waves issue or wait to issue half of their time, matrix
// cores busy 10 %); fragments further ahead (16 instead of 8) and G two steps ahead change nothing.  Registers for two workgroups
// per CU, us the call with / without: 8500 candidates 432 / 437, 9500 438 / 444, 12000 x 4 of 256 202 / 205; up to 8192, a workgroup per CU, the
// three spilled registers cost 1 % (4200 254.5 / 251.6).
template <int DG>
__global__ __launch_bounds__(512, 4) void bgf_gate_kernel(const __bf16 *gb, const float *g, const __bf16 *w_down, const __bf16 *w_up,
                                                          const float *w_head, float b_head, float *y, float *score, int m, int nd)
{
    constexpr int NW = 8, R = 8, kRows = 32, kCols = 256, kStep = kCols / 16, S2 = DG / 16, kOwn = kRows / NW;
    constexpr int kBuf = kRows * kCols * 2, kPre = kCols * 2 + 16;
    constexpr int kSwap = 2 * kBuf > 2 * kRows * kPre ? 2 * kBuf : 2 * kRows * kPre;
    static_assert(kStep % R == 0 && S2 % R == 0 && DG / 32 <= NW, "");
    __shared__ __attribute__((aligned(16))) uint8_t lds[kSwap + kRows * DG * 2];
    uint8_t *const hid = lds + kSwap;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5, r15 = lane & 15;
    const int64_t m0 = (int64_t)blockIdx.x * kRows;
    const int n_steps = nd / kCols;
    auto frag = [&](const __amdgpu_buffer_rsrc_t &w, int at) __attribute__((always_inline)) {
        return __builtin_amdgcn_raw_buffer_load_b128(w, lane * 16, at * 1024, 0);
    };
    const __amdgpu_buffer_rsrc_t wd = __builtin_amdgcn_make_buffer_rsrc((void *)w_down, 0, nd * DG * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t wu = __builtin_amdgcn_make_buffer_rsrc((void *)w_up, 0, nd * DG * 2, 0x00020000);
    auto barrier = []() __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // ---- hidden = ReLU(G W_down) ----
    u32x4 ring[R];
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    {
        const int blk = min(wave, DG / 32 - 1), S = nd / 16;  // (waves beyond the last block copy only)
        u32x4 rows[2];
        auto fetch = [&](int t) __attribute__((always_inline)) {  // rows 4 wave .. + 3 of the step, two at a time
#pragma unroll
            for (int i = 0; i < 2; ++i)
                rows[i] = *(const u32x4 *)(gb + min(m0 + 4 * wave + 2 * i + hf, (int64_t)m - 1) * nd + t * kCols + l32 * 8);
        };
        auto put = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int r = 4 * wave + 2 * i + hf;
                *(u32x4 *)(lds + buf * kBuf + r * LdsRows<kCols>::kPitch + ((l32 & ~15) | (r15 ^ (r & 15))) * 16) = rows[i];
            }
        };
        fetch(0);
#pragma unroll
        for (int e = 0; e < R; ++e) ring[e] = frag(wd, blk * S + e);
        put(0);
        fetch(min(1, n_steps - 1));
        barrier();
        const uint32_t base = LdsRows<kCols>::base(l32, hf);
#pragma unroll 1
        for (int t = 0; t < n_steps; ++t) {
            const uint8_t *a = lds + (t & 1) * kBuf;
            static_for<kStep>([&](auto s_tag) __attribute__((always_inline)) {
                constexpr int s = decltype(s_tag)::value;
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ring[s % R]), LdsRows<kCols>::frag(a, base, s, 0), acc, 0, 0, 0);
                ring[s % R] = frag(wd, blk * S + min(t * kStep + s + R, S - 1));
                __builtin_amdgcn_sched_barrier(0);
            });
            if (t + 1 < n_steps) put((t + 1) & 1);
            fetch(min(t + 2, n_steps - 1));
            barrier();
        }
        if (wave < DG / 32) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int c = 4 * wave + q;
                bf16x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = (__bf16)fmaxf(acc[4 * q + e], 0.f);
                *(bf16x4 *)(hid + l32 * LdsRows<DG>::kPitch + ((c & ~15) | ((c & 15) ^ r15)) * 16 + 8 * hf) = v;
            }
        }
    }

    // ---- Y = G sigmoid(hidden W_up), score = <w_head, Y> + b_head ----
#pragma unroll
    for (int e = 0; e < R; ++e) ring[e] = frag(wu, wave * S2 + e);
    float4 gv[kOwn], wv;
    auto fetch = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < kOwn; ++k)
            gv[k] = *(const float4 *)(g + min(m0 + kOwn * wave + k, (int64_t)m - 1) * nd + t * kCols + lane * 4);
        wv = *(const float4 *)(w_head + t * kCols + lane * 4);
    };
    fetch(0);
    float sum[kOwn] = {};
    barrier();
    const uint32_t base = LdsRows<DG>::base(l32, hf);
#pragma unroll 1
    for (int t = 0; t < n_steps; ++t) {
        f32x16 up;
#pragma unroll
        for (int r = 0; r < 16; ++r) up[r] = 0.f;
        const int blk = NW * t + wave, next = min(blk + NW, nd / 32 - 1);
        static_for<S2>([&](auto s_tag) __attribute__((always_inline)) {
            constexpr int s = decltype(s_tag)::value;
            up = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ring[s % R]), LdsRows<DG>::frag(hid, base, s, 0), up, 0, 0, 0);
            ring[s % R] = frag(wu, s + R < S2 ? blk * S2 + s + R : next * S2 + s + R - S2);
            __builtin_amdgcn_sched_barrier(0);
        });
        uint8_t *pre = lds + (t & 1) * (kRows * kPre);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            bf16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (__bf16)up[4 * q + e];
            *(bf16x4 *)(pre + l32 * kPre + (32 * wave + 8 * q + 4 * hf) * 2) = v;
        }
        barrier();
#pragma unroll
        for (int k = 0; k < kOwn; ++k) {
            const bf16x4 pv = *(const bf16x4 *)(pre + (kOwn * wave + k) * kPre + lane * 8);
            const float4 yv = gated(gv[k], pv);
            sum[k] = head_sum(yv, wv, sum[k]);
            const int64_t row = m0 + kOwn * wave + k;
            if (y && row < m) *(float4 *)(y + row * nd + t * kCols + lane * 4) = yv;
        }
        fetch(min(t + 1, n_steps - 1));
    }
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
        const float total = wave_sum64(sum[k]);
        const int64_t row = m0 + kOwn * wave + k;
        if (lane == 0 && row < m) score[row] = total + b_head;
    }
}

}  // namespace

// A workgroup streams both weights for its 32 candidates, whoever else does, so few of them are better served by the projections for few rows
// (gemm_small_bf16.hip), further on with a wide G, whose weights the macro tiles read less often.  The lines lie where the two sides meet, which is
// earlier with Y than without it.  Us a call, one launch / three, G as blocks x d_model, with Y; in brackets without.
// d_gate 256: 1 x 512 1500 58.2 / 58.6, 3 x 256 2100 63.8 / 65.0; 2 x 512 2200 90.2 / 90.1, 2690 90.8 / 91.2 [2272 88.0 / 87.4, 2677 88.4 / 88.1], 4 x 256
// 2690 66.5 / 66.6 [2549 64.6 / 64.1], 5 x 256 2200 76.9 / 72.6, 2690 78.2 / 75.0 [2598 76.3 / 71.9], 3 x 512 2305 102.0 / 100.6, 2433 103.9 / 104.2, 2690
// 115.1 / 116.9 [2562 110.0 / 107.3], 6 x 256 2305 79.0 / 77.7, 2561 80.1 / 79.6, 2690 81.0 / 83.1, 7 x 256 2177 84.5 / 82.2, 2433 97.8 / 99.3, 2690 98.6 /
// 101.6 [2686 96.6 / 95.8]; 4 x 512 2305 126.3 / 124.6, 2433 127.1 / 128.6, 3391 145.6 / 148.1 [2448 124.4 / 120.8, 3239 136.9 / 136.4, 3500 146.8 / 145.2,
// 4200 224.8 / 229.0], 8 x 256 2500 106.1 / 104.2, 2817 108.6 / 110.9, 3333 113.3 / 117.2 [2743 104.1 / 101.8, 3221 108.6 / 107.7, 3400 111.1 / 111.6]; wider
// ones meet more than once, by the turns of the macro
// tiles: 6 x 512 3400 249.9 / 251.2 [247.7 / 245.2], 5800 387.1 / 402.7 [369.7 / 377.5], 12 x 256 3900 209.7 / 216.0 [203.3 / 204.1], 5000 284.1 / 278.0
// [267.5 / 258.5], 8 x 512 4300 386.5 / 398.0 [372.7 / 372.2], 5000 430 / 427, 6000 480 / 484; 12 x 512 3900 574 / 549, 6000 829 / 826, 16 x 512 5000
// 1038 / 1007, 6000 1204 / 1198.
// d_gate 128: 1 x 256 1500 34.9 / 37.4, 2 x 512 1500 80.5 / 80.3; 3 x 512 2000 107.9 / 105.9, 2600 112.7 / 112.6, 4 x 512 2000 111.0 / 106.7, 2800 127.3
// / 127.1, 3400 141.2 / 141.7, 6 x 512 2000 144.0 / 137.3, 2800 231.3 / 231.2; 7 x 512 1579 139.7 / 135.1, 2177 174.6 / 176.2, 2690 231.4 / 236.0, 3100
// 251.6 / 249.9 [2012 149.2 / 144.6, 2931 231.4 / 228.6]; 15 x 256 2177 211.2 / 205.9, 3190 277.4 / 276.1, 8 x 512 1607 151.1 / 144.9, 2500 242.2 / 242.1,
// 3190 274.2 / 263.2, 3400 264.8 / 270.0 [2469 238.9 / 231.1, 2947 240.1 / 236.4], 16 x 256 2177 263.3 / 252.8, 3190 333.5 / 325.7, 3300 320.1 / 323.2; 10 x
// 512 4000 470 / 457, 5000 602 / 616, 16 x 512 4000 789 / 760, 5000 968 / 998.
bool bgf_gate_takes(int64_t m, int nd, int dg, bool with_y)
{
    if (nd % 256 != 0) return false;
    if (dg == 128) return m >= (nd > 4096 ? 5000 : nd > 3584 || (nd > 3072 && !with_y) ? 3200 : nd > 3072 ? 2100 : nd > 1024 ? 2800 : 1500);
    return dg == 256 && m >= (nd > 2048 ? 6000 : nd <= 768 ? 2049 : with_y ? 2400 : nd > 1792 ? 3400 : 2700);
}

hipError_t launch_bgf_gate(const void *gb, const float *g, const void *w_down, const void *w_up, const float *w_head, float b_head, float *y,
                           float *score, int64_t m, int nd, int dg, hipStream_t s)
{
    if (m <= 0) return hipSuccess;
    const dim3 grid((unsigned)((m + 31) / 32)), block(512);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, 0, s, (const __bf16 *)gb, g, (const __bf16 *)w_down, (const __bf16 *)w_up, w_head, b_head, y,
                           score, (int)m, nd);
        return hipGetLastError();
    };
    if (dg == 128) return go(bgf_gate_kernel<128>);
    if (dg == 256) return go(bgf_gate_kernel<256>);
    return hipErrorInvalidValue;
}

hipError_t launch_bgf_attention(const void *qkv, void *o, const int32_t *scen, const float *tau_scen, int n_scen,
                                int64_t m, int nb, int H, float qk_scale, hipStream_t s)
{
    if (m <= 0) return hipSuccess;
    if (nb < 1 || nb > kMaxBlocks) return hipErrorInvalidValue;
    const int64_t items = m * ((H + 7) / 8);
    const dim3 grid((unsigned)((items + 3) / 4)), block(256);
    const float sl = qk_scale * 1.4426950408889634f;
    auto go = [&](auto nb_tag) {
        constexpr int NB = decltype(nb_tag)::value;
        hipLaunchKernelGGL(bgf_attention_kernel<NB>, grid, block, 0, s, (const __bf16 *)qkv, (__bf16 *)o, scen, tau_scen,
                           n_scen, m, H, sl);
    };
    switch (nb) {
#define CLIMBER_BGF_CASE(N) case N: go(std::integral_constant<int, N>{}); break;
        CLIMBER_BGF_CASE(1) CLIMBER_BGF_CASE(2) CLIMBER_BGF_CASE(3) CLIMBER_BGF_CASE(4) CLIMBER_BGF_CASE(5)
        CLIMBER_BGF_CASE(6) CLIMBER_BGF_CASE(7) CLIMBER_BGF_CASE(8) CLIMBER_BGF_CASE(9) CLIMBER_BGF_CASE(10)
        CLIMBER_BGF_CASE(11) CLIMBER_BGF_CASE(12) CLIMBER_BGF_CASE(13) CLIMBER_BGF_CASE(14) CLIMBER_BGF_CASE(15)
        CLIMBER_BGF_CASE(16)
#undef CLIMBER_BGF_CASE
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_bgf_gate_head(const float *g, const void *pre, const float *w_head, float b_head, float *y,
                                float *score, int64_t m, int nd, hipStream_t s)
{
    if (m <= 0) return hipSuccess;
    hipLaunchKernelGGL(bgf_gate_head_kernel, dim3((unsigned)((m + 3) / 4)), dim3(256), 0, s, g, (const __bf16 *)pre,
                       w_head, b_head, y, score, m, nd);
    return hipGetLastError();
}

int bgf_max_blocks() { return kMaxBlocks; }

}  // namespace climber
