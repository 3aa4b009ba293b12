// The fused QKV projection (f_QKV of Eq. (3), Climber, arXiv 2502.09888) of many rows: 64 of them, whole, in the LDS of a workgroup
// (two per CU), and weights from L2 straight into registers (qkv_units.h).  The macro tiles of gemm_bf16.hip move 0.75 KiB out of LDS
// and 0.4 into it per MFMA, and copy every row as often as there are tiles in its line; here it is 0.5 KiB of rows out of
// LDS and 0.5 of weights, no barrier in the loop, and no LDS on the way out.  32768 rows in a stack: d_model 512 62 us (71), d_model 256 22 (30).
// fp32 rows (the fusion module's) are rounded, squared and summed on the way into LDS: 82 us where a launch for their bf16 copy and
// sums and this one took 94.  (The same for a stack's bf16 rows: 77, against 11 for their sums alone, which bring the rows near,
// and 63.)
// Without its stores it takes 48, without the loads of its rows 54, the products alone 38: HBM and the clock under the products.
#include "launch.h"
#include "qkv_units.h"

namespace climber {
namespace {

using namespace gemm;

typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef const __attribute__((address_space(1))) uint8_t glb_u8;

constexpr int RB = 2, ROWS = 32 * RB, NW = 4, R = 4;

template <int K>
constexpr int resident_lds_bytes() { return ROWS * (K * 2 + 4); }

template <int K, RowsIn IN>
__global__ __launch_bounds__(NW * 64, 2) void gemm_resident_kernel(const void *A, const __bf16 *Wp, int M, const RowNormIn nin,
                                                                   const QkvOut out, const int splits)
{
    constexpr int n_units = 3 * K / 64;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    float *const scale = (float *)(lds + ROWS * K * 2);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int turn = (int)blockIdx.x >> 3, m0 = (turn / splits * 8 + ((int)blockIdx.x & 7)) * ROWS, part = turn % splits;
    if (m0 >= M) return;
    const bool cached = m0 < out.n_cached;
    const int first = cached ? out.qc.which0 * (K / 64) : 0;
    const int end = first + (n_units - first) * (part + 1) / splits, u = first + (n_units - first) * part / splits + wave;

    const __amdgpu_buffer_rsrc_t w = __builtin_amdgcn_make_buffer_rsrc((void *)Wp, 0, 3 * K * K * 2, 0x00020000);
    u32x4 ring[2 * R];
    auto first_frags = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 2 * R; ++e) ring[e] = unit_frag<K>(w, 0, min(u, n_units - 1), e, lane);
    };
    if constexpr (IN == kRowsSummed) {
        constexpr int kLanes = K * 2 / 16, kPer = 64 / kLanes;  // lanes per row, rows per 1 KiB copy
#pragma unroll
        for (int c = 0; c < ROWS / kPer / NW; ++c) {
            const int r0 = (wave * (ROWS / kPer / NW) + c) * kPer, r = r0 + lane / kLanes, slot = lane % kLanes;
            const int ch = (slot & ~15) | ((slot & 15) ^ (r & 15));
            __builtin_amdgcn_global_load_lds((glb_u8 *)((const uint8_t *)A + (int64_t)min(m0 + r, M - 1) * (K * 2) + ch * 16),
                                             (lds_u8 *)lds + r0 * (K * 2), 16, 0, 0);
        }
        first_frags();
        if (tid < ROWS) scale[tid] = row_scale(nin, min(m0 + tid, M - 1));
    } else {
        // fp32 rows by way of registers, all rows of the wave at once: a row's columns 256 p + 4 lane .. + 3, squared and summed as in rowwise.hip
        constexpr int P = K / 256, kTurn = ROWS / NW;
        {
            const int r0 = wave * kTurn;
            float4 raw[kTurn][P];
#pragma unroll
            for (int k = 0; k < kTurn; ++k)
#pragma unroll
                for (int q = 0; q < P; ++q) raw[k][q] = *((const float4 *)A + (int64_t)min(m0 + r0 + k, M - 1) * (K / 4) + 64 * q + lane);
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
            for (int o = 32; o > 0; o >>= 1)
#pragma unroll
                for (int k = 0; k < kTurn; ++k) sum[k] += __shfl_xor(sum[k], o, 64);
#pragma unroll
            for (int k = 0; k < kTurn; ++k)
                if (lane == k) scale[r0 + k] = 1.f / sqrtf(sum[k] * nin.inv_d + nin.eps);
        }
        first_frags();
    }
    CacheUser user[1] = {CacheUser{0, 64, 0}};
    if (cached) user[0] = cache_user(out.qc, m0);
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    __syncthreads();
    if (cached) qkv_units<K, RB, R, true>(lds, scale, w, 0, ring, u, NW, end, out, user, m0, M, lane);
    else qkv_units<K, RB, R, false>(lds, scale, w, 0, ring, u, NW, end, out, user, m0, M, lane);
}

template <int K, RowsIn IN>
hipError_t launch(const void *A, const void *W, int M, const RowNormIn &nin, const QkvOut &out, hipStream_t s)
{
    constexpr auto kernel = gemm_resident_kernel<K, IN>;
    const hipError_t e = raise_lds_limit<kernel>(resident_lds_bytes<K>());
    if (e != hipSuccess) return e;
    // The units of a tile over three workgroups (two without queries): each wave has one (K = 256) or two.  Two for all, six: encode of 17 users 676,
    // 641 against 655, of 32 829, 825 against 827; d_model 256, 32 users 286, 293 against 286; one layer's keys and values 56 in two, 62 in three; fp32
    // rows 82 in one or two, 91 in three.
    const int splits = IN == kRowsF32 || (out.n_cached && out.qc.which0) ? 2 : 3, tiles = (M + ROWS - 1) / ROWS;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((tiles + 7) / 8 * 8 * splits)), dim3(NW * 64), resident_lds_bytes<K>(), s, A,
                       (const __bf16 *)W, M, nin, out, splits);
    return hipGetLastError();
}

}  // namespace

// Us per call here / by macro tiles, d_model 512: encode (four layers, projections of all of them) of 10 users x 1024 376 / 389, 13 420 / 432, 24
// 721 / 720, 32 852 / 865, 33 1035 / 1049; scoring of 8481 rows 531 / 523, 16448 913 / 893, 30840 1185 / 1204 (rows, no fragments, to
// write: left to the macro tiles); below 8192 rows there are too few tiles.  d_model 256: encode of 9 users x 1024 151 / 160, 64 581 / 612, scoring of 11565
// rows 250 / 255, 32896 539 / 564.
bool gemm_resident_takes(int M, int K, bool cached) { return M > 8192 && (K == 256 || (K == 512 && cached)); }

bool gemm_resident_sums(int M, int K) { return M > 8192 && (K == 256 || K == 512); }

hipError_t gemm_resident_bf16(RowsIn in, const void *A, const void *w_packed, int M, int K, const RowNormIn &nin, const QkvOut &out,
                              hipStream_t s)
{
    if (M <= 0) return hipSuccess;
    auto as = [&](auto in_tag) {
        constexpr RowsIn IN = decltype(in_tag)::value;
        if (K == 512) return launch<512, IN>(A, w_packed, M, nin, out, s);
        if (K == 256) return launch<256, IN>(A, w_packed, M, nin, out, s);
        return hipErrorInvalidValue;
    };
    switch (in) {
    case kRowsSummed: return as(std::integral_constant<RowsIn, kRowsSummed>{});
    case kRowsF32: return as(std::integral_constant<RowsIn, kRowsF32>{});
    }
    return hipErrorInvalidValue;
}

}  // namespace climber
