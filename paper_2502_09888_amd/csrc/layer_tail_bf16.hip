// What follows the attention of a layer, in one kernel (f_FFN of Eq. (3), Climber, arXiv 2502.09888):
//     h = x + o Wo;   y = h + GELU(RMSNorm(h; g2) W1) W2
// for row counts that fill the chip.  As three launches, h (fp32 and bf16), its row sums and the feed-forward
// hidden (d_ffn columns) go out to memory and come back: at d_model 512, d_ffn 2048 a row moves 20 KiB, of which 6
// are the row's own input and output, and the launches wait for those bytes about as long as for their products.
// Here a workgroup owns 32*RB rows and all their columns: the bf16 copy of h and one chunk of the hidden live in LDS,
// h itself in registers or (64 rows of 512 columns, four waves) in the rows of y until y replaces it, and only weights -- packed
// fragments, L2-resident -- stream in, straight into registers.
//
// NW waves side by side over the columns: a wave owns D / NW columns of h / y and 32 columns of every chunk of the
// hidden.  Per chunk: the next chunk's hidden from the bf16 rows, then y += hidden W2 with the next chunk's GELU
// dealt out between the matrix instructions (neither waits for the other's pipe).  The weight fragments of all
// products form one stream of loads, R in flight per wave across phase changes and barriers; rows of LDS operands are
// XOR-swizzled so that the fragment reads are conflict-free.
// 64 rows (RB = 2): bound by the matrix cores at the clock that they leave and, nearly as much, by the weights' way
// through the vector cache (4.7 MB per workgroup at 64 bytes per clock).  32768 rows in a stack: d_model 512, eight waves,
// 193 us, against 230 as three launches; d_model 256, four waves and two workgroups per CU, 63 against 87.  Of the 193, 11
// pay for the residuals' exact place (h as the start value of the second sum: 3 to 11 times the rounding error) and 12
// for the GELU's relative error in the tail (see gelu_stage).  Four waves with h by way of memory (64 MB out and back,
// by all workgroups at once) take about 20 us more.  32 rows (RB = 1) where 64 would leave CUs without work: bound by
// the weights' way through the vector cache (the same bytes for half the products); 8192 rows 62 us between the other
// launches of a stack, 76 without the weights requested ahead (PRE below).  (Taller tiles would need less of the caches, but 128 rows do not fit the registers; separate waves
// for the two products gave the same times.)
// The rows that leave are the next layer's input: with QKV the workgroup goes on to that layer's fused QKV projection (qkv_units.h),
// its rows' bf16 copy in LDS once more.  They and their row sums do not go out and come back (66 MB a layer at 32768 rows of 512), and
// what the launch between two attentions starts and ends with goes away; y itself is left out where nobody reads it.  Encode of
// 32 users x 1024, four layers: 847 -> 808 us with the projection of the first layer's rows by gemm_resident_bf16.hip, packed forward
// 1010 -> 927; 0.9 PFLOP/s over the launch.
// X16: the residual rows are the bf16 rows that a call was given, so that no fp32 copy of them is made (that launch 18.7 us at 32768 rows, the
// sums alone 11; encode 823 -> 811, one layer of 32896 candidates and more 1 %).
// Products, row sums and their order are those of the separate launches (gemm_bf16.hip, gemm_small_bf16.hip): same
// bits.
#include "gemm_common.h"
#include "lanes.h"
#include "launch.h"
#include "qkv_units.h"

#include <utility>

namespace climber {
namespace {

using namespace gemm;

typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef const __attribute__((address_space(1))) uint8_t glb_u8;

// A fragment of the weights: 16 bytes per lane at a wave-uniform offset.  (Through the buffer builtin: the compiler
// counts the loads in flight itself, and an address takes one vector register throughout.)
__device__ __forceinline__ void load_frag(u32x4 &f, uint32_t lane_off, __amdgpu_buffer_rsrc_t w, int at)
{
    f = __builtin_amdgcn_raw_buffer_load_b128(w, (int)lane_off, at, 0);
}
// every wave's LDS accesses so far are done (the weights' loads stay in flight)
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// rows of h, a chunk of the hidden (at the end: 32 rows of y, fp32); with a projection behind it: sums of squares and scales of y
template <int D, int RB, int NW>
constexpr int tail_lds_bytes()
{
    constexpr int operands = 32 * RB * (D + 32 * NW) * 2, rows = 32 * D * 4;
    return operands > rows ? operands : rows;
}
template <int D, int RB>
constexpr int tail_scale_bytes() { return 32 * RB * (D / 64 + 1) * 4; }

template <int N>
using At = std::integral_constant<int, N>;

// The next fragments of the stream of weights: fragment e at base + (e % NJ) * a + (e / NJ) * b.
struct Next { int base, a, b; };

// PRE = 1: one more wave, which requests the weights for the L2 of its XCD ahead of their use.  A workgroup of its own has to
// itself a CU, and the 32 of an XCD walk over the same weights at the same time: what is not in L2 (kernels' boundaries
// and four layers with the cache between them see to that) costs all of them a trip to memory every 8 or 16 fragments.
// So every workgroup requests its share of them, one 8 KiB piece per load (a lane per 128-byte line; four bytes of each land
// in a corner of LDS that nobody reads), a chunk of the hidden ahead.  By one of the other waves those loads would delay
// its own, which return in order.  Us, four layers scored, 8192 rows: 484 with a 268 MB cache between (539 without), 379
// with a short one (389); by the computing waves at their start 493 and 393.  With it eight fragments in flight do what
// 16 did, and the registers hold a third wave per SIMD.  64-row tiles do not gain (and have no registers for it).
template <int D, int RB, int NW, int R, int PRE, bool QKV, bool X16>
__global__ __launch_bounds__((NW + PRE) * 64, 2 + PRE) void layer_tail_kernel(const TailArgs p)
{
    static_assert(!X16 || RB * (D / NW / 32) <= 4, "the residual's blocks are all requested ahead");
    static_assert(!QKV || D / NW == 64, "");
    constexpr int ROWS = 32 * RB, CW = D / NW, NJ = CW / 32;   // rows of the tile; columns and column blocks of a wave
    constexpr int kChunk = 32 * NW;                            // hidden columns of a chunk
    constexpr int S = D / 16, T = kChunk / 16;                 // k-steps of the products over h and over a chunk
    constexpr int kXPitch = D * 2, kHPitch = kChunk * 2;       // bytes per row of the two LDS operands
    static_assert(NJ == 2 || NJ == 4, "a wave owns whole 64-column slices of the row sums");
    static_assert(32 % (T * NJ) == 0, "a share of the GELU for every matrix instruction");
    static_assert(S % R == 0 && T * NJ % R == 0 && R % (2 * NJ) == 0, "ring slots are compile-time constants");
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    uint8_t *const X = lds, *const H = lds + ROWS * kXPitch;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5, r15 = lane & 15;
    const int m0 = blockIdx.x * ROWS, M = p.M, F = p.F, col0 = CW * wave, n_chunks = F / kChunk;

    // LDS operands: 16-byte chunk c of row r at slot c ^ (r % 16) of its group of 16
    const uint32_t x_base = (uint32_t)(l32 * kXPitch + ((hf ^ r15) << 4)), h_base = (uint32_t)(l32 * kHPitch + ((hf ^ r15) << 4));
    auto frag = [](const uint8_t *op, uint32_t base, int pitch, int step, int i) __attribute__((always_inline)) {
        return *(const bf16x8 *)(op + ((base ^ ((step & 7) << 5)) + (step >> 3) * 256 + i * 32 * pitch));
    };
    auto write_a = [&](uint8_t *op, int pitch, int i, int col, bf16x4 v) __attribute__((always_inline)) {  // columns col + 4 hf ..
        const int c = col / 8;
        *(bf16x4 *)(op + (32 * i + l32) * pitch + (((c & ~15) | ((c & 15) ^ r15)) * 16) + 8 * hf) = v;
    };

    if (PRE && wave == NW) {  // pieces in the order of use: Wo, W1 of chunk 0; per chunk W1 of the next, W2 of this one
        constexpr int PO = D * D * 2 / 8192, P1 = NW * S / 8, P2 = (D / 32) * (T / 8);
        static_assert(S % 8 == 0 && T % 8 == 0, "whole pieces");
        const int n_layer = PO + n_chunks * (P1 + P2), sharers = ((int)gridDim.x + 7) / 8;
        const int q_skip = QKV && m0 < p.next.n_cached ? p.next.qc.which0 * PO : 0, n_pieces = n_layer + (QKV ? 3 * PO - q_skip : 0);  // (the next layer's queries: nobody's)
        int k = blockIdx.x / 8;  // (workgroups go round the eight XCDs)
        auto request = [&](int end) __attribute__((always_inline)) {
            for (; k < min(end, n_pieces); k += sharers) {
                int at = k * 8192, r = k - PO - P1;
                if (QKV && k >= n_layer) {
                    at = p.wq + (k - n_layer + q_skip) * 8192;
                } else if (r >= 0) {
                    const int ch = r / (P1 + P2);
                    r %= P1 + P2;
                    const int c = r - (ch + 1 < n_chunks ? P1 : 0);
                    at = c < 0 ? p.w1 + (ch + 1) * (NW * S * 1024) + r * 8192
                               : p.w2 + (c / (T / 8)) * ((F / 16) * 1024) + ch * T * 1024 + (c % (T / 8)) * 8192;
                } else if (k >= PO) {
                    at = p.w1 + (k - PO) * 8192;
                }
                __builtin_amdgcn_global_load_lds((glb_u8 *)((const uint8_t *)p.wo + at + lane * 128),
                                                 (lds_u8 *)lds + tail_lds_bytes<D, RB, NW>() + (QKV ? tail_scale_bytes<D, RB>() : 0), 4, 0, 0);
            }
        };
        int ahead = PO + P1 + (P1 + P2);
        request(ahead);
        for (int i = 0; i < 4; ++i) __builtin_amdgcn_s_barrier();  // the barriers below, one for one
        for (int ch = 0; ch + 1 < n_chunks; ++ch) {
            request(ahead += P1 + P2);
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_s_barrier();
        }
        request(n_pieces);
        for (int i = 0; i < (QKV ? 3 : 1); ++i) __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): nothing may land in LDS that is no longer the workgroup's
        return;
    }

    // the attention output rows -> X, whole rows
    {
        constexpr int kLanes = kXPitch / 16, kPer = 64 / kLanes;  // lanes per row, rows per 1 KiB copy
#pragma unroll
        for (int c = 0; c < ROWS / kPer / NW; ++c) {
            const int r0 = (wave * (ROWS / kPer / NW) + c) * kPer, r = r0 + lane / kLanes, slot = lane % kLanes;
            const int ch = (slot & ~15) | ((slot & 15) ^ (r & 15));
            __builtin_amdgcn_global_load_lds((glb_u8 *)((const uint8_t *)p.o + (int64_t)min(m0 + r, M - 1) * kXPitch + ch * 16),
                                             (lds_u8 *)X + r0 * kXPitch, 16, 0, 0);
        }
    }
    f32x16 acc[RB][NJ];  // the lane's accumulators are [row 32i + l32][col0 + 32j + 8g + 4hf + 0..3]
    auto clear_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    };
    clear_acc();
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0), here and not in the loops below
    // Both residuals join a finished sum (see wave_epilogue), so h exists beside the accumulators of the second one: in
    // registers where they suffice, else in the rows of y, from which a lane reads back what it wrote itself.
    constexpr int NB = RB * NJ;
    constexpr bool kKeep = NB <= 4;
    constexpr int kAhead = kKeep ? NB : 1;  // blocks of residual rows requested ahead of the end of a product
    f32x16 side[kAhead];
    // (offsets made where they are used: held across the products they would cost registers the loops have not got)
    struct Rows { int64_t at[RB]; };
    auto rows = [&]() __attribute__((always_inline)) {
        int l = lane;
        asm volatile("" : "+v"(l));
        Rows r;
#pragma unroll
        for (int i = 0; i < RB; ++i) r.at[i] = (int64_t)min(m0 + 32 * i + (l & 31), M - 1) * D + col0 + 4 * (l >> 5);
        return r;
    };
    auto request_rows = [&](const float *from) __attribute__((always_inline)) {
        const Rows at = rows();
#pragma unroll
        for (int b = 0; b < kAhead; ++b) load_block(side[b], from + at.at[b / NJ] + 32 * (b % NJ));
    };
    auto request_rows16 = [&]() __attribute__((always_inline)) {  // as they are: two values in a register
        const bool second = m0 >= p.x16_split;
        const __bf16 *from = second ? (const __bf16 *)p.x16_b - (int64_t)p.x16_split * D : (const __bf16 *)p.x16;
        const Rows at = rows();
#pragma unroll
        for (int b = 0; b < kAhead; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float2 q = *(const float2 *)(from + at.at[b / NJ] + 32 * (b % NJ) + 8 * g);
                side[b][2 * g] = q.x, side[b][2 * g + 1] = q.y;
            }
    };
    auto add_rows16 = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const uint32_t two = __float_as_uint(side[b % kAhead][r / 2]);
                acc[b / NJ][b % NJ][r] += __uint_as_float(two << 16);
                acc[b / NJ][b % NJ][r + 1] += __uint_as_float(two & 0xffff0000u);
            }
    };
    auto add_rows = [&](const float *from) __attribute__((always_inline)) {  // acc += rows, block by block
        const Rows at = rows();
        static_for<NB>([&](auto b_tag) __attribute__((always_inline)) {
            constexpr int b = decltype(b_tag)::value;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[b / NJ][b % NJ][r] += side[b % kAhead][r];
            if constexpr (b + kAhead < NB) load_block(side[b % kAhead], from + at.at[(b + kAhead) / NJ] + 32 * ((b + kAhead) % NJ));
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    auto keep_rows = [&]() __attribute__((always_inline)) {
        const Rows at = rows();
        static_for<NB>([&](auto b_tag) __attribute__((always_inline)) {
            constexpr int b = decltype(b_tag)::value;
            if constexpr (kKeep) side[b] = acc[b / NJ][b % NJ];
            else if (m0 + 32 * (b / NJ) + l32 < M) store_block(p.y + at.at[b / NJ] + 32 * (b % NJ), acc[b / NJ][b % NJ]);
        });
        __builtin_amdgcn_sched_barrier(0);
    };

    // the stream of weight fragments, 1 KiB each: Wo; W1 of chunk 0; then, per chunk, W1 of the next and W2 of this one
    const uint32_t w_lane = lane * 16;
    const __amdgpu_buffer_rsrc_t w = __builtin_amdgcn_make_buffer_rsrc((void *)p.wo, 0, p.w_bytes, 0x00020000);
    const int wo = (col0 / 32) * S * 1024, w1 = p.w1 + wave * S * 1024, w2_col = (F / 16) * 1024, w2 = p.w2 + (col0 / 32) * w2_col;
    constexpr int w1_chunk = NW * S * 1024;
    auto next_up = [&](int ch) __attribute__((always_inline)) { return Next{w1 + ch * w1_chunk, 1024, NJ * 1024}; };
    auto next_down = [&](int ch) __attribute__((always_inline)) { return Next{w2 + ch * T * 1024, w2_col, 1024}; };
    u32x4 ring[R];
    auto load_next = [&](auto slot_tag, const Next &n, int e) __attribute__((always_inline)) {
        load_frag(ring[decltype(slot_tag)::value], w_lane, w, n.base + (e % NJ) * n.a + (e / NJ) * n.b);
    };
    {
        const Next n{wo, S * 1024, 1024};
        static_for<R>([&](auto e) __attribute__((always_inline)) { load_next(e, n, decltype(e)::value); });
    }
    lds_barrier();  // o is there

    // One k-step of a product into acc: operand rows fa, NJ fragments from ring slot q on.  Behind every MFMA goes
    // `between(index)`; operand rows of the next step (`refill(i)`) and fragments (`reload(j)`) as their registers fall free.
    bf16x8 fa[2][RB];
    auto mfma_step = [&](auto q_tag, auto &&refill, auto &&reload, auto &&between) __attribute__((always_inline)) {
        constexpr int q = decltype(q_tag)::value;
        __builtin_amdgcn_sched_barrier(0);
        static_for<RB * NJ>([&](auto m_tag) __attribute__((always_inline)) {
            constexpr int m = decltype(m_tag)::value, i = m / NJ, j = m % NJ;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ring[q + j]), fa[0][i], acc[i][j], 0, 0, 0);
            if constexpr (j == NJ - 1) refill(i);
            if constexpr (i == RB - 1) reload(std::integral_constant<int, j>{});
            between(m_tag);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    auto nothing = [](auto) __attribute__((always_inline)) {};

    // ---- h = x + o Wo ----
#pragma unroll
    for (int i = 0; i < RB; ++i) fa[0][i] = frag(X, x_base, kXPitch, 0, i);
    auto o_steps = [&](int s0, auto last_tag) __attribute__((always_inline)) {
        constexpr bool LAST = decltype(last_tag)::value;
        static_for<8>([&](auto u_tag) __attribute__((always_inline)) {
            constexpr int u = decltype(u_tag)::value, q = (u * NJ) % R, un = u + R / NJ;
            mfma_step(std::integral_constant<int, q>{},
                      [&](int i) __attribute__((always_inline)) { if (!LAST || u < 7) fa[0][i] = frag(X, x_base, kXPitch, s0 + u + 1, i); },
                      [&](auto j_tag) __attribute__((always_inline)) {
                          constexpr int j = decltype(j_tag)::value;
                          load_frag(ring[q + j], w_lane, w, LAST && un >= 8 ? w1 + ((un - 8) * NJ + j) * 1024 : wo + j * (S * 1024) + (s0 + un) * 1024);
                      },
                      nothing);
        });
    };
#pragma unroll 1
    for (int s0 = 0; s0 + 8 < S; s0 += 8) o_steps(s0, std::false_type{});
    if constexpr (X16) request_rows16();
    else request_rows(p.x);
    o_steps(S - 8, std::true_type{});
    if constexpr (X16) add_rows16();  // h
    else add_rows(p.x);
    keep_rows();
    // sums of squares of the rows' 64-column slices, as the separate launches form them
    auto slice_sums = [&](auto &&put) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int sl = 0; sl < NJ / 2; ++sl) {
                float half8[2];
#pragma unroll
                for (int jj = 0; jj < 2; ++jj) {
                    float pr[4];
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const f32x16 &a = acc[i][2 * sl + jj];
                        const float q4 = sumsq4(a[4 * g], a[4 * g + 1], a[4 * g + 2], a[4 * g + 3]);
                        pr[g] = q4 + __shfl_xor(q4, 32, 64);
                    }
                    half8[jj] = (pr[0] + pr[1]) + (pr[2] + pr[3]);
                }
                put(i, sl, half8[0] + half8[1]);
            }
    };
    float *ss = (float *)H;  // [ROWS][D / 64], until the hidden moves in
    slice_sums([&](int i, int sl, float v) __attribute__((always_inline)) {
        if (hf == 0) ss[(32 * i + l32) * (D / 64) + wave * (NJ / 2) + sl] = v;
    });
    lds_barrier();  // o has been read; the sums are there
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                bf16x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = (__bf16)acc[i][j][4 * g + e];
                write_a(X, kXPitch, i, col0 + 32 * j + 8 * g, v);
            }
    clear_acc();
    float rs[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) rs[i] = row_scale(RowNormIn{ss, D / 64, p.inv_d, p.eps}, 32 * i + l32);
    lds_barrier();  // h is there; the sums have been read

    // ---- y = h + GELU(r * (h W1)) W2, a chunk of the hidden at a time ----
    f32x16 hid[RB];
    bf16x4 hb[RB][4];
    // hid = h W1 of a chunk
    auto up = [&](int w1c, const Next &n) __attribute__((always_inline)) {
        uint32_t x_at = x_base;
        asm("" : "+v"(x_at));  // (the k-steps' addresses are made anew for every chunk, not kept in registers throughout)
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) hid[i][r] = 0.f;
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int i = 0; i < RB; ++i) fa[s][i] = frag(X, x_at, kXPitch, s, i);
        auto steps = [&](int s0, auto last_tag) __attribute__((always_inline)) {
            constexpr bool LAST = decltype(last_tag)::value;
            static_for<R>([&](auto u_tag) __attribute__((always_inline)) {
                constexpr int u = decltype(u_tag)::value;
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < RB; ++i) {
                    hid[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ring[u]), fa[u & 1][i], hid[i], 0, 0, 0);
                    if (!LAST || u < R - 2) fa[u & 1][i] = frag(X, x_at, kXPitch, s0 + u + 2, i);
                    if (i == RB - 1) {
                        if constexpr (LAST) load_next(u_tag, n, u);
                        else load_frag(ring[u], w_lane, w, w1c + (s0 + u + R) * 1024);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
        };
#pragma unroll 1
        for (int s0 = 0; s0 + R < S; s0 += R) steps(s0, std::false_type{});
        steps(S - R, std::true_type{});
    };
    // values 4g .. 4g + 3 of hid[i] through the scale and the GELU, in eight pieces of about 40 clocks
    float gx[4], gt[4], gp[4];
    auto gelu_piece = [&](auto piece_tag, auto group_tag) __attribute__((always_inline)) {
        constexpr int piece = decltype(piece_tag)::value, i = decltype(group_tag)::value / 4, g = decltype(group_tag)::value % 4;
        auto each = [&](auto from, auto to, int e0, int e1) __attribute__((always_inline)) {  // stages [from, to) of values [e0, e1)
            constexpr int s0 = decltype(from)::value;
            static_for<decltype(to)::value - s0>([&](auto s) __attribute__((always_inline)) {
#pragma unroll
                for (int e = e0; e < e1; ++e) gelu_stage<s0 + decltype(s)::value>(gx[e], gt[e], gp[e]);
            });
        };
        if constexpr (piece == 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e) gx[e] = hid[i][4 * g + e] * rs[i];
            each(At<0>{}, At<1>{}, 0, 4);
        } else if constexpr (piece == 1) {
            each(At<1>{}, At<2>{}, 0, 3);   // a reciprocal or an exponential takes as long as four other instructions
        } else if constexpr (piece == 2) {
            each(At<1>{}, At<2>{}, 3, 4);
            each(At<2>{}, At<4>{}, 0, 4);
        } else if constexpr (piece == 3) {
            each(At<4>{}, At<6>{}, 0, 4);
            each(At<6>{}, At<7>{}, 0, 2);
        } else if constexpr (piece == 4) {
            each(At<6>{}, At<7>{}, 2, 4);
            each(At<7>{}, At<8>{}, 0, 4);
        } else if constexpr (piece == 5) {
            each(At<8>{}, At<9>{}, 0, 2);
            each(At<9>{}, At<10>{}, 0, 2);
        } else if constexpr (piece == 6) {
            each(At<8>{}, At<9>{}, 2, 4);
            each(At<9>{}, At<10>{}, 2, 4);
        } else {
            each(At<10>{}, At<11>{}, 0, 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) hb[i][g][e] = (__bf16)gx[e];
        }
    };
    auto write_hidden = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int g = 0; g < 4; ++g) write_a(H, kHPitch, i, 32 * wave + 8 * g, hb[i][g]);
    };
    // y += hidden W2 of chunk ch; between the products, the GELU of the chunk in hid
    auto down = [&](int ch, const Next &n, auto gelu_tag) __attribute__((always_inline)) {
        constexpr bool GELU = decltype(gelu_tag)::value;
        const Next own = next_down(ch);
        uint32_t h_at = h_base;
        asm("" : "+v"(h_at));
#pragma unroll
        for (int i = 0; i < RB; ++i) fa[0][i] = frag(H, h_at, kHPitch, 0, i);
        static_for<T>([&](auto t_tag) __attribute__((always_inline)) {
            constexpr int t = decltype(t_tag)::value, q = (t * NJ) % R, tn = t + R / NJ;
            mfma_step(std::integral_constant<int, q>{},
                      [&](int i) __attribute__((always_inline)) { if (t + 1 < T) fa[0][i] = frag(H, h_at, kHPitch, t + 1, i); },
                      [&](auto j_tag) __attribute__((always_inline)) {
                          constexpr int j = decltype(j_tag)::value;
                          load_next(std::integral_constant<int, q + j>{}, tn < T ? own : n, (tn < T ? tn : tn - T) * NJ + j);
                      },
                      [&](auto m_tag) __attribute__((always_inline)) {
                          if constexpr (GELU) {
                              constexpr int per = 32 / (T * NJ), at = (t * RB * NJ + decltype(m_tag)::value) * per;
                              static_for<per>([&](auto k) __attribute__((always_inline)) {
                                  constexpr int pc = at + decltype(k)::value;
                                  gelu_piece(std::integral_constant<int, pc % 8>{}, std::integral_constant<int, pc / 8>{});
                              });
                          }
                      });
        });
    };

    up(w1, n_chunks > 1 ? next_up(1) : next_down(0));
    static_for<RB * 32>([&](auto k) __attribute__((always_inline)) {
        gelu_piece(std::integral_constant<int, decltype(k)::value % 8>{}, std::integral_constant<int, decltype(k)::value / 8>{});
    });
    write_hidden();
    lds_barrier();
#pragma unroll 1
    for (int ch = 0; ch + 1 < n_chunks; ++ch) {
        up(w1 + (ch + 1) * w1_chunk, next_down(ch));
        down(ch, ch + 2 < n_chunks ? next_up(ch + 2) : next_down(ch + 1), std::true_type{});
        lds_barrier();  // chunk ch has been read
        write_hidden();
        lds_barrier();  // chunk ch + 1 is there
    }
    if constexpr (!kKeep) request_rows(p.y);
    const bool cached = QKV && m0 < p.next.n_cached;
    const int u0 = (cached ? p.next.qc.which0 * (D / 64) : 0) + wave;  // the wave's first unit of the projection
    down(n_chunks - 1, QKV ? Next{p.wq + 2 * u0 * (S * 1024), S * 1024, 1024} : next_down(n_chunks - 1), std::false_type{});  // (without it, what it loads ahead is not used)
    add_rows(p.y);  // y

    // ---- y out: rows through LDS, whole lines ----
    float *const y_ss = (float *)(lds + tail_lds_bytes<D, RB, NW>()), *const y_scale = y_ss + ROWS * (D / 64);
    if constexpr (QKV) {
        slice_sums([&](int i, int sl, float v) __attribute__((always_inline)) {
            if (hf == 0) y_ss[(32 * i + l32) * (D / 64) + wave * (NJ / 2) + sl] = v;
        });
    } else if (p.ss) {
        slice_sums([&](int i, int sl, float v) __attribute__((always_inline)) {
            const int row = m0 + 32 * i + l32;
            if (hf == 0 && row < M) p.ss[(int64_t)row * (D / 64) + wave * (NJ / 2) + sl] = v;
        });
    }
    lds_barrier();
    constexpr int kRowB = CW * 4, kPieces = kRowB / 16;  // fp32 bytes and 16-byte pieces of a wave's part of a row
    uint8_t *tr = lds + wave * (32 * kRowB);
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        if (QKV && m0 < p.y_first) break;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *(float4 *)(tr + l32 * kRowB + (((8 * j + 2 * g + hf) ^ r15) * 16)) =
                    float4{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
#pragma unroll
        for (int it = 0; it < 32 * kPieces / 64; ++it) {
            const int id = it * 64 + lane, r = id / kPieces, c = id % kPieces, row = m0 + 32 * i + r, col = col0 + 4 * c;
            const float4 v = *(const float4 *)(tr + r * kRowB + ((c ^ (r & 15)) * 16));
            if (row < M) {
                *(float4 *)(p.y + (int64_t)row * D + col) = v;
                if (!QKV && p.yb) {
                    bf16x4 b;
                    b[0] = (__bf16)v.x, b[1] = (__bf16)v.y, b[2] = (__bf16)v.z, b[3] = (__bf16)v.w;
                    *(bf16x4 *)((__bf16 *)p.yb + (int64_t)row * D + col) = b;
                }
            }
        }
    }
    if constexpr (QKV) {
        lds_barrier();  // (everybody's corner of LDS is free; the sums are there)
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    bf16x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = (__bf16)acc[i][j][4 * g + e];
                    write_a(X, kXPitch, i, col0 + 32 * j + 8 * g, v);
                }
        if (tid < ROWS) y_scale[tid] = row_scale(RowNormIn{y_ss, D / 64, p.inv_d, p.eps}, tid);
        CacheUser user[(RB + 1) / 2];
#pragma unroll
        for (int b = 0; b < (RB + 1) / 2; ++b) user[b] = cached ? cache_user(p.next.qc, min(m0 + 64 * b, p.next.n_cached - 32)) : CacheUser{0, 64, 0};
        lds_barrier();  // y is there
        if (cached) qkv_units<D, RB, R / 2, true>(X, y_scale, w, p.wq, ring, u0, NW, 3 * D / 64, p.next, user, m0, M, lane);
        else qkv_units<D, RB, R / 2, false>(X, y_scale, w, p.wq, ring, u0, NW, 3 * D / 64, p.next, user, m0, M, lane);
    }
}

template <int D, int RB, int NW, int R, int PRE, bool QKV = false, bool X16 = false>
hipError_t launch_tail(const TailArgs &a, hipStream_t s)
{
    if constexpr (!X16 && D / NW == 64)
        if (a.x16) return launch_tail<D, RB, NW, R, PRE, QKV, true>(a, s);
    constexpr size_t lds = tail_lds_bytes<D, RB, NW>() + PRE * 256 + (QKV ? tail_scale_bytes<D, RB>() : 0);
    constexpr auto kernel = layer_tail_kernel<D, RB, NW, R, PRE, QKV, X16>;
    const hipError_t e = raise_lds_limit<kernel>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((a.M + 32 * RB - 1) / (32 * RB))), dim3((NW + PRE) * 64), lds, s, a);
    return hipGetLastError();
}

}  // namespace

// A launch takes the time of one workgroup until every CU has one; the separate launches grow with the rows.  Weights that
// four layers and the cache between them have pushed out of L2 count here, so whole calls decide (four layers, with /
// without, us).  d_model 512, d_ffn 2048: score of 4096 rows 353 / 333, 4352 431 / 444, 8192 549 / 559, 16384 795 / 964,
// encode of 4096 222 / 209, 5120 235 / 257 (without weights requested ahead; with them score of 4096 rows 298 / 282 and 362 / 361
// with a short and a long history, 3072 280 / 255 and 321 / 304); d_ffn 1408 (four waves): score of 8704 rows 642 / 603, 12288 729 / 735,
// 24576 1129 / 1237; d_model 256: score of 4096 rows 192 / 188, 4608 194 / 204, 32768 521 / 713.  Other widths have no kernel: the
// stacks that this is configured and measured with have 256 or 512 columns.
bool layer_tail_takes(int M, int D, int F)
{
    return F % 128 == 0 && F > 0 && ((D == 512 && M > (F % 256 == 0 ? 4096 : 12288)) || (D == 256 && M > 4096));
}

// With the next layer's projection in the same launch its input rows, their row sums and that launch's start and end are saved; without,
// it is dealt out over all CUs whatever the tail's last turn (a tile of 64 rows per CU) leaves idle.  d_model 512:
// - Keys and values only (encode, before the last layer), where y is left out as well: always.  Us, encode of two layers with / without, users x
//   1024 (16 tiles each): 9 users 109 / 118, 12 122 / 136, 17 220 / 235, 24 245 / 259, 33 364 / 381, 49 501 / 519, 64 569 / 601.
// - Whole layers of an encode: from two turns on, and as many CUs as those pay for may stay idle, 32 for each but the first.  Us, four layers, all
//   tails / the last one only: 10 users (160 tiles, 96 idle) 355 / 351, 14 (32 idle) 424 / 415, 16 (none) 448 / 444; 17 (272 tiles, 240 idle) 670 / 636, 24 (128)
//   696 / 683, 28 (64) 755 / 752, 30 (32) 783 / 787, 32 (none) 822 / 825; 33 (528 tiles, 240) 1037 / 1011, 38 (160) 1057 / 1045, 40 (128) 1069 / 1066, 44 (64)
//   1132 / 1140, 48 (none) 1201 / 1216; 49 (784 tiles, 240) 1409 / 1399, 56 (128) 1452 / 1456, 64 (none) 1601 / 1619.
// - Packed forward: the candidates' rows besides, which are a launch of their own otherwise: 190 more.  Us, four layers, all / none: 129 tiles 354 / 371,
//   252 511 / 552; 264 (248 idle) 764 / 742, 287 (225) 808 / 797, 297 (215) 725 / 733, 355 (157) 767 / 771, 422 842 / 879, 492 947 / 1013; 516 (252) 1092 /
//   1100, 542 1150 / 1162, 659 1227 / 1265; 774 (250) 1558 / 1567.  271 tiles (241 idle), six layers, 1191 / 1151.
// - Candidates alone, against the 128 x 128 tiles: 9766 rows 554 / 530, 16448 944 / 896, 24672 1020 / 1015, 30840 1173 / 1204: not.
// - Tiles of 32 rows (up to 8192 of them), with / without: with a history always, us, four layers, encode of 4500 rows 237 / 242, 6000 252 / 263, 7168
//   263 / 274, 8192 280 / 296, packed forward of 5200 352 / 364, 7200 386 / 410 (encode of 5120 to 8192 rows with d_ffn 256 to 4096: 0.93 to 0.97).
//   Candidates alone from where the 128 x 128 tiles of their own launch begin a third turn: d_ffn 2048, 16 users x 1024, 5120 rows 359.7 / 357.6, 5376
//   363.6 / 362.2, 5440 364.7 / 377.4, 6400 379.5 / 387.6, 7680 401.0 / 409.7, 7792 403.0 / 417.5, 8192 411.2 / 421.0; the same line with 64 x 256 (5376
//   312.4 / 308.6, 5440 315.4 / 321.7, 8192 352.9 / 357.1), 8 x 3000 (8192 521 / 533), and with d_ffn 256 (5376 233.1 / 228.5, 5440 235.1 / 245.0, 7400
//   253.2 / 257.5, 8192 260.8 / 265.3), 512, 1024 and 4096 (8192 586.8 / 595.7).
// d_model 256 (tiles two per CU): encode of 5 users 127 / 132, 9 141 / 151, 17 218 / 236, 32 280 / 316, 64 530 / 581, scoring of 4500 rows 195 / 193, 8481
// 206 / 213, 32896 517 / 539: always.
bool layer_tail_projects(int M, int D, int F, int n_cached, bool ends)
{
    if (!layer_tail_takes(M, D, F)) return false;
    if (D == 256) return true;
    if (F % 256 != 0) return false;
    if (M <= 8192) return n_cached > 0 || M > 5376;
    if (n_cached == 0) return false;
    const int tiles = (M + 63) / 64, turns = (tiles + 255) / 256, idle = turns * 256 - tiles;
    return n_cached < M ? idle <= 32 * (turns - 1) + 190 : ends || (turns > 1 && idle <= 32 * (turns - 1));
}

bool layer_tail_reads_bf16(int M, int D, int F) { return layer_tail_takes(M, D, F) && (D == 256 || F % 256 == 0); }

hipError_t layer_tail_bf16(const TailArgs &a, hipStream_t s)
{
    if (a.M < 1 || a.F < 128 || a.F % 128 != 0) return hipErrorInvalidValue;
    if (a.x16 && (!layer_tail_reads_bf16(a.M, a.D, a.F) || a.x16_split % 64 != 0)) return hipErrorInvalidValue;
    if (a.wq) {
        if (!layer_tail_takes(a.M, a.D, a.F) || (a.D == 512 && a.F % 256 != 0) || a.next.n_cached % 64 != 0 || a.y_first % 64 != 0) return hipErrorInvalidValue;
        if (a.D == 256) return launch_tail<256, 2, 4, 8, 0, true>(a, s);
        return a.M <= 8192 ? launch_tail<512, 1, 8, 8, 1, true>(a, s) : launch_tail<512, 2, 8, 8, 0, true>(a, s);
    }
    // d_model 512: eight waves need chunks of 256; no more than a 32-row tile per CU: those (fewer rows in line behind one
    // another).  Four waves hold twice the columns each, and h has to wait in memory.  Us, stack calls of four layers, eight
    // / four waves: encode of 32768 rows 853 / 907, score of 8704 594 / 727, of 16384 772 / 919.
    if (a.D == 512 && a.F % 256 == 0) return a.M <= 8192 ? launch_tail<512, 1, 8, 8, 1>(a, s) : launch_tail<512, 2, 8, 8, 0>(a, s);
    if (a.D == 512) return launch_tail<512, 2, 4, 8, 0>(a, s);
    if (a.D == 256) return launch_tail<256, 2, 4, 8, 0>(a, s);
    return hipErrorInvalidValue;
}

}  // namespace climber
