// What follows the attention of a layer, up to the hidden of its feed-forward, for few rows of 256 columns (f_FFN of Eq. (3), Climber,
// arXiv 2502.09888):
//     h = x + o Wo;   hidden = GELU(RMSNorm(h; g2) W1)
// in one launch.  A request's launches are latency: 3.5 us each with nothing to do, then the weights' way through the vector cache of the
// CU that a tile is on.  Here a workgroup makes the whole h of 32 rows for itself and 128 columns of the hidden from it: the output
// projection is made d_ffn / 128 times over, which costs a workgroup 128 KiB of weights, 1 us, less than a launch of its own with its start, its
// end and the rows between.  (At d_model 512 it is 512 KiB, which come from beyond L2 as soon as a few layers share it: 2.7 us a layer slower
// than the two launches, 10 with all of a wave's W1 requested ahead.)  A wave has 64 columns of h and 32 of the hidden, its weights
// straight from L2 in registers, 16 fragments ahead across the two products.
// Products, row sums and their order are those of the separate launches (gemm_small_bf16.hip, gemm_bf16.hip): same bits.
#include "gemm_common.h"
#include "qkv_units.h"

namespace climber {
namespace {

using namespace gemm;

typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef const __attribute__((address_space(1))) uint8_t glb_u8;

// every wave's LDS accesses so far are done (loads stay in flight)
__device__ __forceinline__ void meet()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

constexpr int D = 256, NW = D / 64, kHidden = 32 * NW;

__global__ __launch_bounds__(NW * 64) void layer_head_kernel(const HeadArgs p)
{
    constexpr int S = D / 16, R = 16;
    static_assert(S % R == 0, "");
    __shared__ __attribute__((aligned(16))) uint8_t X[32 * D * 2];
    __shared__ __attribute__((aligned(16))) uint8_t corners[NW][32 * 80];
    __shared__ float ss[32 * (D / 64)];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hf = lane >> 5, r15 = lane & 15;
    // parts of a tile go round the XCDs, so that each of them has an eighth of W1 in its L2 (and all of Wo)
    const int part = (int)blockIdx.x % p.n_parts, m0 = (int)blockIdx.x / p.n_parts * 32, M = p.M, col0 = 64 * wave;

    {   // rows of o
        constexpr int kLanes = D * 2 / 16, kPer = 64 / kLanes;  // lanes per row, rows per copy of 1 KiB
#pragma unroll
        for (int c = 0; c < 32 / kPer / NW; ++c) {
            const int r0 = (wave * (32 / kPer / NW) + c) * kPer, r = r0 + lane / kLanes, slot = lane % kLanes, ch = (slot & ~15) | ((slot & 15) ^ (r & 15));
            __builtin_amdgcn_global_load_lds((glb_u8 *)((const uint8_t *)p.o + (int64_t)min(m0 + r, M - 1) * (D * 2) + ch * 16), (lds_u8 *)X + r0 * (D * 2), 16, 0, 0);
        }
    }
    const int64_t at = (int64_t)min(m0 + l32, M - 1) * D + col0 + 4 * hf;  // the lane's accumulators: [row m0 + l32][col0 + 32 j + 8 g + 4 hf + 0..3]
    f32x16 x[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) load_block(x[j], p.x + at + 32 * j);
    __builtin_amdgcn_sched_barrier(0);
    const __amdgpu_buffer_rsrc_t w = __builtin_amdgcn_make_buffer_rsrc((void *)p.wo, 0, p.w_bytes, 0x00020000);
    auto wo = [&](int e) __attribute__((always_inline)) {  // fragment of column block e % 2, k-step e / 2
        return __builtin_amdgcn_raw_buffer_load_b128(w, lane * 16, ((2 * wave + e % 2) * S + e / 2) * 1024, 0);
    };
    auto w1 = [&](int e) __attribute__((always_inline)) {
        return __builtin_amdgcn_raw_buffer_load_b128(w, lane * 16, p.w1 + ((part * NW + wave) * S + e) * 1024, 0);
    };
    u32x4 ring[R];
#pragma unroll
    for (int e = 0; e < R; ++e) ring[e] = wo(e);
    f32x16 acc[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
    __builtin_amdgcn_sched_barrier(0);
    static_assert(R == 16, "");
    __builtin_amdgcn_s_waitcnt(0x4f70);  // vmcnt(16): the rows are there, the weights stay in flight (and the compiler knows)
    meet();

    // ---- h = x + o Wo ----
    const uint32_t base = LdsRows<D>::base(l32, hf);
    bf16x8 fa[2] = {LdsRows<D>::frag(X, base, 0, 0), LdsRows<D>::frag(X, base, 1, 0)};
    auto steps = [&](int s0, auto last_tag) __attribute__((always_inline)) {
        constexpr bool LAST = decltype(last_tag)::value;
        static_for<R / 2>([&](auto t_tag) __attribute__((always_inline)) {
            constexpr int t = decltype(t_tag)::value;
            const bf16x8 a = fa[t & 1];
            if (!LAST || t + 2 < R / 2) fa[t & 1] = LdsRows<D>::frag(X, base, s0 + t + 2, 0);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ring[2 * t + j]), a, acc[j], 0, 0, 0);
                ring[2 * t + j] = LAST ? w1(2 * t + j) : wo(2 * s0 + R + 2 * t + j);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    steps(0, std::false_type{});
    static_assert(S == R, "two turns of the ring");
    steps(S - R / 2, std::true_type{});
    float half8[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        float pr[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
#pragma unroll
            for (int e = 4 * g; e < 4 * g + 4; ++e) acc[j][e] += x[j][e];
            const float q4 = sumsq4(acc[j][4 * g], acc[j][4 * g + 1], acc[j][4 * g + 2], acc[j][4 * g + 3]);
            pr[g] = q4 + __shfl_xor(q4, 32, 64);
        }
        half8[j] = (pr[0] + pr[1]) + (pr[2] + pr[3]);
    }
    if (hf == 0) ss[l32 * (D / 64) + wave] = half8[0] + half8[1];
    if (part == 0 && m0 + l32 < M) {
#pragma unroll
        for (int j = 0; j < 2; ++j) store_block(p.h + at + 32 * j, acc[j]);
    }
    meet();  // o has been read; the sums are there
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int c = col0 / 8 + 4 * j + g;
            bf16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (__bf16)acc[j][4 * g + e];
            *(bf16x4 *)(X + l32 * (D * 2) + (((c & ~15) | ((c & 15) ^ r15)) * 16) + 8 * hf) = v;
        }
    const float rs = row_scale(RowNormIn{ss, D / 64, p.inv_d, p.eps}, l32);
    meet();  // h is there

    // ---- hidden = GELU(r * (h W1)) ----
    f32x16 hid;
#pragma unroll
    for (int r = 0; r < 16; ++r) hid[r] = 0.f;
    fa[0] = LdsRows<D>::frag(X, base, 0, 0), fa[1] = LdsRows<D>::frag(X, base, 1, 0);
    static_for<S>([&](auto s_tag) __attribute__((always_inline)) {
        constexpr int s = decltype(s_tag)::value;
        const bf16x8 a = fa[s & 1];
        if constexpr (s + 2 < S) fa[s & 1] = LdsRows<D>::frag(X, base, s + 2, 0);
        hid = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ring[s % R]), a, hid, 0, 0, 0);
        if constexpr (s + R < S) ring[s % R] = w1(s + R);
        __builtin_amdgcn_sched_barrier(0);
    });
    // out, as the 1 KiB pieces (16 rows, 32 columns) that the down-projection copies (gemm.h)
    uint8_t *const tr = corners[wave];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (__bf16)gelu_erf(hid[4 * g + e] * rs);
        *(bf16x4 *)(tr + l32 * 80 + (8 * g + 4 * hf) * 2) = v;
    }
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int r = 16 * it + (lane >> 2), c = (lane & 3) ^ ((lane >> 4) & 3);
        if (m0 + r < M)
            *(uint4 *)((uint8_t *)p.u + ((int64_t)((m0 >> 4) + it) * (p.F / 32) + (part * kHidden) / 32 + wave) * 1024 + lane * 16) = *(const uint4 *)(tr + r * 80 + c * 16);
    }
}

}  // namespace

// At most a workgroup per CU.  Us a call, four layers, one launch / two.  d_ffn 128: score of 20 rows 65.8 / 77.2, 1064 81.5 / 86.1, 2904 111.1 / 121.9,
// request of 100 behaviours and candidates 132 / 140, packed forward of 656 candidates 123.5 / 131.2; 256: score of 64 70.6 / 77.7, 904 82.5 / 81.6, 1112
// 86.7 / 89.8, 1600 92.9 / 95.2, 2384 113.4 / 119.7, 3000 119.2 / 126.3, 4064 124.9 / 130.0, encode of 2048 73.1 / 73.5, forward of 3000 candidates 162.7 /
// 165.6; 512: score of 120 73.8 / 76.8, 1600 97.8 / 100.3, 2048 102.9 / 102.3, encode of 1024 65.2 / 64.3, 2048 78.5 / 77.1, forward of 1600
// 160.1 / 162.0; 640: score of 144 77.6 / 77.8, 1600 100.9 / 104.6, encode of 384 63.2 / 62.7; 768: score of 48 74.1 / 77.0, encode of 1024 69.6 / 70.8; 1024: score of
// 20 71.6 / 77.2, 144 77.3 / 78.1, 952 94.5 / 96.0, 1200 (304 workgroups) 115.3 / 103.4; 2048: score of 104 81.7 / 83.2, 408 87.9 / 94.1.
bool layer_head_takes(int M, int d, int F) { return d == D && F % kHidden == 0 && F > 0 && (M + 31) / 32 * (int64_t)(F / kHidden) <= 256; }

hipError_t layer_head_bf16(const HeadArgs &a, hipStream_t s)
{
    if (a.M < 1 || a.D != D || a.F < 1 || a.F % kHidden != 0) return hipErrorInvalidValue;
    HeadArgs p = a;
    p.n_parts = a.F / kHidden;
    hipLaunchKernelGGL(layer_head_kernel, dim3((unsigned)((a.M + 31) / 32 * p.n_parts)), dim3(NW * 64), 0, s, p);
    return hipGetLastError();
}

}  // namespace climber
