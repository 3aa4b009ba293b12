// bf16 MFMA GEMM for the projections of the layer stack (f_QKV and f_FFN of Eq. (3), Climber,
// arXiv 2502.09888): C[M][N] = A[M][K] * W[K][N] with fp32 accumulation and a fused epilogue
// (plain bf16 store, residual add into the fp32 stream, erf-GELU).
//
// W is first repacked (pack_weights) into B-operand fragments of v_mfma_f32_32x32x16_bf16:
//   chunk (nb, ks, lane), 16 B: W[16ks + 8(lane/32) + 0..7][32nb + lane%32]
// so that a k-tile of a 32-column block is contiguous and is copied HBM -> LDS linearly.
// A is row-major (its tile is copied row by row, 64 B per row and k-tile, with the 16-byte chunks
// of a row XOR-swizzled by (row / 4) % 4 through the choice of the global address each lane loads:
// 16 consecutive rows of one k chunk then cover all 64 banks) or in the tiled layout of gemm.h,
// where one copy is 1 KiB contiguous.
// Both copies are direct global_load_lds (no register staging) into a ring of 3, 4 or 6 k-tiles of 32,
// one to four tiles in flight behind the one that is waited for, one bare s_barrier per k-tile; the copies of a k-tile are dealt out
// between the MFMAs of the tile two ahead of it, not queued in front of them.
// Workgroup = 4 waves as 2 x 2; a wave owns WM x WN blocks of 32 x 32:
//   4 x 2 (macro tile 256 x 128): 128 accumulator registers, two workgroups per CU (the projections
//         here have K = 512 or 2048: short k-loops, and they sit near the HBM/MFMA ridge);
//   2 x 2 (macro tile 128 x 128): for problems too small to fill the chip with larger tiles.
// Workgroups that share A rows are launched onto the same XCD (see the kernel).
#include "gemm_common.h"
#include "lanes.h"
#include "launch.h"

#include <algorithm>
#include <cstdlib>
#include <type_traits>
#include <utility>

namespace climber {
namespace {

using namespace gemm;

typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef const __attribute__((address_space(1))) uint8_t glb_u8;

constexpr int BK = 32;      // k-tile

// blockIdx.y = job.  A lane packs 16 rows of two columns, i.e. four 16-byte chunks of a fragment (nb, ks): 64 lanes read whole
// lines of a row with one load, all 16 loads are in flight at once, and 16 lanes write the whole fragment.  Bound by memory.
// (A lane per chunk, eight 2-byte loads of half a line each: 25 MB of four layers 18.2 us that way, 13.7 this way; the fusion
// module 13.9 in two launches, 7.2 in one.)  Weights and gains are 16-byte aligned.
__global__ __launch_bounds__(256) void pack_weights_kernel(const PackJobs jobs)
{
    const int j = blockIdx.y, K = jobs.K[j], N = jobs.N[j];
    const uint32_t pairs = (uint32_t)N / 2, n_items = (uint32_t)K / 16 * pairs;
    const __bf16 *w = (const __bf16 *)jobs.w[j], *gain = (const __bf16 *)jobs.gain[j];
    for (uint32_t item = blockIdx.x * 256 + threadIdx.x; item < n_items; item += gridDim.x * 256) {
        const uint32_t ks = item / pairs, n = item % pairs * 2;
        uint32_t x[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) x[e] = *(const uint32_t *)(w + (int64_t)(16 * ks + e) * N + n);
        __bf16 v[2][16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            v[0][e] = __builtin_bit_cast(__bf16, (uint16_t)x[e]);
            v[1][e] = __builtin_bit_cast(__bf16, (uint16_t)(x[e] >> 16));
        }
        if (gain) {
            const bf16x8 g[2] = {*(const bf16x8 *)(gain + 16 * ks), *(const bf16x8 *)(gain + 16 * ks + 8)};
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                v[0][e] = (__bf16)((float)v[0][e] * (float)g[e / 8][e % 8]);
                v[1][e] = (__bf16)((float)v[1][e] * (float)g[e / 8][e % 8]);
            }
        }
        bf16x8 *out = (bf16x8 *)jobs.packed[j] + ((int64_t)(n / 32) * (K / 16) + ks) * 64 + n % 32;
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                bf16x8 y;
#pragma unroll
                for (int e = 0; e < 8; ++e) y[e] = v[c][8 * half + e];
                out[32 * half + c] = y;
            }
    }
}

template <int N>
__device__ __forceinline__ void wait_vm()
{
    static_assert(N < 64, "");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// WM, WN: 32 x 32 blocks per wave along M and N.  Macro tile (2*WM*32) x (2*WN*32) x 32.
template <int EPI, int WM, int WN, int kStages>
__global__ __launch_bounds__(256, 2) void gemm_bf16_kernel(
    const __bf16 *A, int64_t lda, const __bf16 *Wp, int M, int N, int K, void *C, int64_t ldc,
    const float *resid, int64_t ldr, const RowNormIn nin, const RowNormOut nout, const int tiled,
    const QkvToCache qc)
{
    constexpr int BM = 64 * WM, BN = 64 * WN;
    constexpr int kABytes = BM * BK * 2, kBBytes = BN * BK * 2, kStageBytes = kABytes + kBBytes;
    constexpr int NA = kABytes / 1024 / 4, NB = kBBytes / 1024 / 4;  // 1 KiB copies per wave and tile
    constexpr int NPRE = NA + NB;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    // the wave number as a scalar: LDS destinations of the copies (M0) are then scalar arithmetic
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    const int wm = wave >> 1, wn = wave & 1;
    // Tile of this workgroup.  Workgroups are dealt to the 8 XCDs round-robin in launch order and
    // every XCD has an L2 of its own; the n_col workgroups that share a block of A rows are therefore
    // given launch indices that are equal modulo 8 (one XCD, adjacent in time), so that the rows
    // come from HBM once instead of once per XCD.
    const int n_col = N / BN, n_tiles = n_col * ((M + BM - 1) / BM);
    int tile = blockIdx.x;
    if (n_tiles % 8 == 0) tile = (tile & 7) * (n_tiles >> 3) + (tile >> 3);
    const int m0 = (tile / n_col) * BM, n0 = (tile % n_col) * BN;
    const int n_kt = K / BK;

    // copy plan.  A: copy j of this wave covers rows 16*(wave*NA + j) .. +15, lane -> (row, slot),
    // global chunk = slot ^ ((row >> 2) & 3).  W: copy j covers fragment (nbl, ksl) of the tile.
    const __bf16 *a_src[NA];
    const bool a_tiled = tiled & kTiledA;
    const int a_step = a_tiled ? 512 : BK;   // elements from one k-tile of a copy to the next
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        const int r = 16 * (wave * NA + j) + (lane >> 2), slot = lane & 3;
        if (a_tiled)   // the 1 KiB piece is stored as it lands in LDS, swizzle included
            a_src[j] = A + (int64_t)min((m0 >> 4) + wave * NA + j, (M - 1) >> 4) * (K / BK) * 512 + lane * 8;
        else
            a_src[j] = A + (int64_t)min(m0 + r, M - 1) * lda + ((slot ^ ((r >> 2) & 3)) * 8);
    }
    const uint8_t *w_src[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int f = wave * NB + j, nbl = f >> 1, ksl = f & 1;
        w_src[j] = (const uint8_t *)Wp +
                   (((int64_t)(n0 / 32 + nbl) * (K / 16) + ksl) * 64 + lane) * 16;
    }
    // copy c (0 .. NPRE-1) of k-tile kt into the ring stage at byte offset `stage`: NA pieces of the
    // A tile, then NB pieces of the W tile
    auto issue_one = [&](int kt, int stage, auto c_tag) __attribute__((always_inline)) {
        constexpr int c = decltype(c_tag)::value;
        lds_u8 *base = (lds_u8 *)lds + stage;
        if constexpr (c < NA)
            __builtin_amdgcn_global_load_lds((glb_u8 *)(a_src[c] + kt * a_step), base + (wave * NA + c) * 1024, 16, 0, 0);
        else
            __builtin_amdgcn_global_load_lds((glb_u8 *)(w_src[c - NA] + (int64_t)kt * 2048),
                                             base + kABytes + (wave * NB + (c - NA)) * 1024, 16, 0, 0);
    };
    auto issue = [&](int kt) __attribute__((always_inline)) {
        static_for<NPRE>([&](auto c) __attribute__((always_inline)) { issue_one(kt, (kt % kStages) * kStageBytes, c); });
    };

    // the first tiles start their way in before anything else is set up (accumulators, row
    // statistics, cache geometry: a microsecond or two that the copies' latency covers)
    for (int kt = 0; kt < kStages - 1 && kt < n_kt; ++kt) issue(kt);

    f32x16 acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // Input rows that were not normalised: r = 1/sqrt(mean(x^2) + eps) of row 32i + l32 scales the
    // whole output row (a lane's accumulators of block row i all belong to that one row).  The
    // partial sums of squares are requested here, ahead of the k-loop, and first touched in the
    // epilogue, so nothing waits for them (8 partial sums per row, d_model = 512, is the fast path).
    constexpr bool SCALED = EPI != EPI_RESID_F32;
    float4 raw_ss[SCALED ? WM : 1][2];
    const bool ss8 = SCALED && nin.ss && nin.n_part == 8;
    if (ss8) {
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            const int row = min(m0 + 32 * (WM * wm + i) + l32, M - 1);
            raw_ss[i][0] = *(const float4 *)(nin.ss + (int64_t)row * 8);
            raw_ss[i][1] = *(const float4 *)(nin.ss + (int64_t)row * 8 + 4);
        }
    }

    // Direct cache write: the user of block row i of this wave (requested here, first used in the epilogue)
    CacheUser user[WM];
#pragma unroll
    for (int i = 0; i < WM; ++i) {
        user[i] = CacheUser{0, 64, 0};
        if (EPI == EPI_STORE_BF16 && qc.layer_base)
            user[i] = cache_user(qc, __builtin_amdgcn_readfirstlane(min(m0 + 32 * (WM * wm + i), M - 32)));
    }

    // One k-tile: wait for it, read both halves' fragments, then the MFMAs with the copies of tile
    // kt + kStages - 1 (if PREFETCH) dealt out between them, one copy after every kStep-th MFMA, so
    // that a wave never queues its copies back to back in front of its own MFMAs.
    constexpr int kMfma = 2 * WM * WN, kStep = kMfma / NPRE >= 1 ? kMfma / NPRE : 1;
    // The ring stages of tile kt and of the tile to prefetch come in as byte offsets carried by the
    // loop (derived from kt % kStages in here, every fragment address cost vector additions on the
    // path from the barrier to the first MFMA instead of being an immediate).
    auto k_tile = [&](int kt, int st_cur, int st_fill, auto ahead_tag, auto prefetch_tag) __attribute__((always_inline)) {
        constexpr bool PREFETCH = decltype(prefetch_tag)::value;
        wait_vm<decltype(ahead_tag)::value * NPRE>();  // tiles that may stay in flight
        __builtin_amdgcn_s_barrier();
        const uint8_t *sa = lds + st_cur;
        const uint8_t *sw = sa + kABytes;
        bf16x8 af[2][WM], bfr[2][WN];
        auto read_frags = [&](auto ks_tag) __attribute__((always_inline)) {
            constexpr int ks = decltype(ks_tag)::value;
#pragma unroll
            for (int i = 0; i < WM; ++i) {
                const int row = 32 * (WM * wm + i) + l32;
                af[ks][i] = *(const bf16x8 *)(sa + row * 64 + (((2 * ks + hf) ^ ((row >> 2) & 3)) * 16));
            }
#pragma unroll
            for (int j = 0; j < WN; ++j)
                bfr[ks][j] = *(const bf16x8 *)(sw + (((WN * wn + j) * 2 + ks) * 64 + lane) * 16);
        };
        // the second half's fragments are requested behind the first MFMA, not ahead of it: the four
        // waves leave the barrier together and queue their reads at the one LDS port
        read_frags(std::integral_constant<int, 0>{});
        __builtin_amdgcn_sched_barrier(0);
        static_for<kMfma>([&](auto m_tag) __attribute__((always_inline)) {
            constexpr int Ms = decltype(m_tag)::value;
            constexpr int ks = Ms / (WM * WN), i = (Ms % (WM * WN)) / WN, j = Ms % WN;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[ks][j], af[ks][i], acc[i][j], 0, 0, 0);
            if constexpr (Ms == 0) {
                read_frags(std::integral_constant<int, 1>{});
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (PREFETCH && Ms % kStep == kStep - 1 && Ms / kStep < NPRE) {
                issue_one(kt + kStages - 1, st_fill, std::integral_constant<int, Ms / kStep>{});
                __builtin_amdgcn_sched_barrier(0);
            }
        });
    };
    {
        constexpr int kRing = kStages * kStageBytes;
        int kt = 0, st_cur = 0, st_fill = kRing - kStageBytes;   // stage of tile kt, stage of tile kt - 1
        auto advance = [&]() __attribute__((always_inline)) {
            st_fill = st_cur;
            st_cur = st_cur + kStageBytes == kRing ? 0 : st_cur + kStageBytes;
        };
        for (; kt + kStages - 1 < n_kt; ++kt, advance()) k_tile(kt, st_cur, st_fill, std::integral_constant<int, kStages - 2>{}, std::true_type{});
        static_for<kStages - 1>([&](auto i_tag) __attribute__((always_inline)) {
            constexpr int left = kStages - 2 - decltype(i_tag)::value;
            if (n_kt - kt != left + 1) return;
            k_tile(kt, st_cur, st_fill, std::integral_constant<int, left>{}, std::false_type{});
            ++kt, advance();
        });
    }

    __syncthreads();  // every wave is done reading the last k-tile
    float rs[WM];
#pragma unroll
    for (int i = 0; i < WM; ++i) rs[i] = 1.f;
    if (SCALED && nin.ss) {
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            float ss = 0.f;
            if (ss8) {
                const float4 u = raw_ss[i][0], v = raw_ss[i][1];
                ss = ((u.x + u.y) + (u.z + u.w)) + ((v.x + v.y) + (v.z + v.w));
            } else {
                const int row = min(m0 + 32 * (WM * wm + i) + l32, M - 1);
                for (int q = 0; q < nin.n_part; ++q) ss += nin.ss[(int64_t)row * nin.n_part + q];
            }
            rs[i] = 1.f / sqrtf(ss * nin.inv_d + nin.eps);
        }
    }

    wave_epilogue<EPI, WM, WN>(acc, rs, user, lds + wave * 32 * epilogue_pitch<EPI, WN>(), m0 + 32 * WM * wm, n0 + WN * 32 * wn,
                               lane, M, N, C, ldc, resid, ldr, nout, tiled, qc);
}

template <int EPI, int WM, int WN, int kStages>
hipError_t launch(const GemmArgs &g, hipStream_t s)
{
    constexpr int BM = 64 * WM, BN = 64 * WN;
    constexpr size_t lds_bytes = (size_t)kStages * (BM + BN) * BK * 2;
    const hipError_t e = raise_lds_limit<gemm_bf16_kernel<EPI, WM, WN, kStages>>(lds_bytes);
    if (e != hipSuccess) return e;
    const dim3 grid((g.N / BN) * ((g.M + BM - 1) / BM)), block(256);
    hipLaunchKernelGGL((gemm_bf16_kernel<EPI, WM, WN, kStages>), grid, block, lds_bytes, s, (const __bf16 *)g.A, g.lda,
                       (const __bf16 *)g.W, g.M, g.N, g.K, g.C, g.ldc, g.resid, g.ldr, g.nin, g.nout, g.tiled, g.qc);
    return hipGetLastError();
}

template <int EPI>
hipError_t dispatch(const GemmArgs &g, hipStream_t s)
{
    if (gemm_small_takes(EPI, g.M, g.N, g.K)) return gemm_small_bf16(EPI, g, s);
    // macro tile 256 x 128 when that still gives every CU two workgroups, else 128 x 128
    const int64_t big_tiles = (int64_t)(g.N / 128) * ((g.M + 255) / 256);
    if (big_tiles >= 512) return launch<EPI, 4, 2, 3>(g, s);
    // 64 x 128 where 128 x 128 would leave CUs without a tile.  us per call with / without: one
    // request (1000 behaviours, 200 candidates, four layers) 271 / 285, 4 x 1500 behaviours with 300 candidates each 570 / 583,
    // encode of 8 x 1024 308 / 336, score of 4352 rows 421 / 436; with all CUs taken (score of 8192 rows) 565 / 558
    if ((int64_t)(g.N / 128) * ((g.M + 127) / 128) < 256) {
        // One workgroup per CU or two, whose k-tiles come from beyond L2 behind a launch that read a cache: a longer ring where the walk is long, which
        // a short one (K of 256 or 512) does not gain back at its start.  Us, four layers, d_model 512, ring of 4 / 6 / 8 / 12 k-tiles for the
        // down-projection: score of 1600 rows 277 / 267 / 268 / 270, 2400 312 / 301 / 302 / 305, 4096 373 / 367 / 368 / 368, encode of 4000 209 / 208 / 209 / 210; for
        // all projections score of 1000 197 / 197 / 199 / 204.
        if (g.K >= 1024) return launch<EPI, 1, 2, 6>(g, s);
        return launch<EPI, 1, 2, 4>(g, s);
    }
    return launch<EPI, 2, 2, 4>(g, s);
}

}  // namespace

hipError_t pack_weights(const PackJobs &jobs, hipStream_t s)
{
    if (jobs.n <= 0) return hipSuccess;
    if (jobs.n > kMaxPackJobs) return hipErrorInvalidValue;
    int64_t most = 0;
    for (int j = 0; j < jobs.n; ++j)
        most = std::max<int64_t>(most, (int64_t)(jobs.N[j] / 2) * (jobs.K[j] / 16));
    const unsigned gx = (unsigned)std::min<int64_t>((most + 255) / 256, 1024);
    hipLaunchKernelGGL(pack_weights_kernel, dim3(gx, (unsigned)jobs.n), dim3(256), 0, s, jobs);
    return hipGetLastError();
}

hipError_t gemm_bf16(int epi, const void *A, int64_t lda, const void *w_packed, int M, int N, int K,
                     void *C, int64_t ldc, const float *resid, int64_t ldr, const RowNormIn &nin,
                     const RowNormOut &nout, int tiled, hipStream_t s, const QkvToCache *to_cache)
{
    if (M <= 0) return hipSuccess;
    QkvToCache qc{};
    if (to_cache) {
        qc = *to_cache;
        if (epi != EPI_STORE_BF16 || !qc.layer_base || qc.d % 64 != 0 || qc.H * 64 != qc.d || qc.l_pad % 64 != 0 ||
            qc.l_pad < 0 || qc.l_valid < 0 || qc.l_valid > qc.l_pad || N != (3 - qc.which0) * qc.d ||
            M != qc.rows || M % 64 != 0 || (qc.l_pad > 0 && M % qc.l_pad != 0) ||
            (qc.l_pad == 0 && (!qc.seg || !qc.tok_off || !qc.hist_len)))
            return hipErrorInvalidValue;
    }
    if (N % 128 != 0 || K % 64 != 0) return hipErrorInvalidValue;
    if ((tiled & ~(kTiledA | kTiledC)) || ((tiled & kTiledC) && epi != EPI_GELU_BF16)) return hipErrorInvalidValue;
    const GemmArgs g{A, lda, w_packed, M, N, K, C, ldc, resid, ldr, nin, nout, tiled, qc};
    switch (epi) {
    case EPI_STORE_BF16: return dispatch<EPI_STORE_BF16>(g, s);
    case EPI_GELU_BF16: return dispatch<EPI_GELU_BF16>(g, s);
    case EPI_RESID_F32: return dispatch<EPI_RESID_F32>(g, s);
    case EPI_RELU_BF16: return dispatch<EPI_RELU_BF16>(g, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace climber
