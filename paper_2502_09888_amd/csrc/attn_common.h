// Device-side building blocks shared by the bf16 MFMA attention kernels (attn_bf16.hip,
// hist_fused_bf16.hip): operand fragment types, the per-wave softmax state and the block-level
// steps S^T = K Q^T, softmax (FAST: no reference; SAFE: running maximum) and O^T += V^T P^T of
// Eq. (3) of Climber (arXiv 2502.09888) in the transposed formulation described in attn_bf16.hip.
#pragma once
#include "internal.h"

namespace climber {
namespace attn {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef const __attribute__((address_space(1))) uint8_t glb_u8;

constexpr float kSafeSlack = 8.0f;           // SAFE: exp2-domain slack before the row maximum moves
// FAST is accepted iff kDenomLo < denominator < kDenomHi for every row.  The window bounds the
// largest logit of a row (in log2 units it is at most log2 of the denominator), and with it the
// error that rounding q * c to bf16 puts on the dominant probabilities; rows beyond it are redone
// by the SAFE pass, which scales in fp32.
constexpr float kDenomHi = 1048576.f;        // 2^20
constexpr float kDenomLo = 1.f / 1048576.f;  // 2^-20
// The exact-scale form of the FAST pass (queries unrounded, p = exp2(s * c) with c in fp32) has no
// error that grows with the logits; its window only keeps the exponentials inside the fp32 / bf16
// exponent range.
constexpr float kDenomHiExact = 1.0e30f;
constexpr float kDenomLoExact = 1.0e-30f;
// largest root mean square of the first block's exponents s * c (log2 units) for which a wave
// folds c into its bf16 queries (the benchmark's logits have 2.9 at the smallest temperature), and
// the fewest keys a row must see for it: the folded form's error per logit averages out over
// many comparable keys, not over a few
constexpr float kPilotSpread = 4.25f;
constexpr int kFoldMinKeys = 256;
constexpr float kSafeNoRef = -1.0e30f;       // SAFE: "no reference yet", below any finite logit
// LDS floats for one head's rows of the bias tables: what two workgroups per CU leave beside the rings (80 KiB each).  Beyond it
// they are looked up in global memory, behind the tiles in flight.  Us that way / from LDS, 32 rows of 129 + 12 or 129 + 20 entries: history
// of 64 x 1024 in subsequences of 256 261 / 185, causal of 20 x 2000 171 / 121, scoring 512 of 64 136 / 109, 128 of 32 27.5 / 28.8.
constexpr int kBiasLdsFloats = 6656;

// What the attention kernels are given.
struct KParams {
    const uint8_t *layer_base;
    const int32_t *hist_len, *tok_off, *order, *cand_off;
    const __bf16 *q, *k_self, *v_self;
    const int32_t *scen, *beh;
    const float *tau;
    __bf16 *o;
    int64_t ld_q, ld_kv, ld_o;
    int B, H, n_scen, n_beh, sub_len, n_qtiles;
    int uni_len, uni_pad;  // >= 0: every user has this valid / padded history length
    int uni_cand;          // >= 0: every user has this many candidates (SUMI)
    int pilot_pairs;       // attn_wave_bf16.hip, attn_split_bf16.hip: the choice of the softmax form is made for 64 queries
    float scale_log2e, inv_qk_scale;
    BiasArgs bias;  // relative attention bias (attn_bias_bf16.hip)
    int bias_H;
};

static inline KParams make_params(const AttnArgs &a, int n_qtiles)
{
    KParams p;
    p.layer_base = a.cache.layer_base;
    p.hist_len = a.cache.hist_len;
    p.tok_off = a.cache.tok_off;
    p.order = a.cache.order;
    p.cand_off = a.cand_off;
    p.q = (const __bf16 *)a.q;
    p.k_self = (const __bf16 *)a.k_self;
    p.v_self = (const __bf16 *)a.v_self;
    p.scen = a.scen;
    p.beh = a.beh;
    p.tau = a.tau;
    p.o = (__bf16 *)a.o;
    p.ld_q = a.ld_q;
    p.ld_kv = a.ld_kv;
    p.ld_o = a.ld_o;
    p.B = a.cache.B;
    p.H = a.H;
    p.n_scen = a.n_scen;
    p.n_beh = a.n_beh;
    p.sub_len = a.sub_len;
    p.n_qtiles = n_qtiles;
    p.scale_log2e = a.qk_scale * 1.4426950408889634f;
    p.inv_qk_scale = 1.f / a.qk_scale;
    p.bias = a.bias;
    p.bias_H = a.H;
    p.uni_len = a.uni_len;
    p.uni_pad = a.uni_pad;
    p.uni_cand = a.uni_cand;
    p.pilot_pairs = 0;
    return p;
}

// Per-wave softmax state for QB blocks of 32 queries.
template <int QB>
struct QState {
    bf16x8 qf[QB][4];  // B operands of S^T: FAST q' = bf16(q*c), SAFE q; [query][16s + 8hf + 0..7]
    float c[QB];      // qk_scale * log2(e) / tau_row                       (SAFE)
    float m_ref[QB];  // running reference maximum, raw logit units         (SAFE)
    float l[QB];      // this half-wave's share of the softmax denominator
    f32x16 O[2][QB];  // O^T[d block][query block]
};

struct KFrags { bf16x8 a[4]; };  // K A-operands of a 32-key block (4 k-steps of 16 dims)
struct VFrags { bf16x8 a[2][2]; };  // V^T A-operands [16-key group][32-dim block]

// A pointer the caller knows to be wave-uniform, as a value in scalar registers.
static __device__ __forceinline__ const uint8_t *uniform_ptr(const uint8_t *p)
{
    const uint64_t a = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    return (const uint8_t *)(((uint64_t)hi << 32) | lo);
}

static __device__ __forceinline__ float xhalf(float x) { return __shfl_xor(x, 32, 64); }

// Exchange between the two half-waves: returns max(x, x of the lane 32 away).
static __device__ __forceinline__ float xhalf_max(float x)
{
    const unsigned u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

static __device__ __forceinline__ KFrags load_k(const uint8_t *blk, int lane)
{
    KFrags f;
#pragma unroll
    for (int s = 0; s < 4; ++s) f.a[s] = *(const bf16x8 *)(blk + (s * 64 + lane) * 16);
    return f;
}

static __device__ __forceinline__ VFrags load_v(const uint8_t *blk, int lane)
{
    VFrags f;
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int db = 0; db < 2; ++db)
            f.a[g][db] = *(const bf16x8 *)(blk + 4096 + ((g * 2 + db) * 64 + lane) * 16);
    return f;
}

// S^T[qb] = K_blk q_qb^T for both query blocks
template <int QB>
static __device__ __forceinline__ void qk_block(const QState<QB> &st, const KFrags &k, f32x16 (&S)[QB])
{
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int r = 0; r < 16; ++r) S[qb][r] = 0.f;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
            S[qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k.a[s], st.qf[qb][s], S[qb], 0, 0, 0);
}

// O^T[db][qb] += V^T_{g,db} P^T
template <int QB>
static __device__ __forceinline__ void pv_block(QState<QB> &st, const VFrags &v, const bf16x8 (&P)[QB][2])
{
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
                st.O[db][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v.a[g][db], P[qb][g], st.O[db][qb], 0, 0, 0);
}

// keys with index >= k_hi are excluded (last blocks of a range only)
template <int QB>
static __device__ __forceinline__ void mask_block(f32x16 (&S)[QB], int hf, int blk_lo, int k_hi)
{
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int kidx = blk_lo + 8 * (r >> 2) + 4 * hf + (r & 3);
        if (kidx >= k_hi) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) S[qb][r] = -INFINITY;
        }
    }
}

// causal history attention: the lane's query of block qb sees keys with index < lim[qb] only
template <int QB>
static __device__ __forceinline__ void mask_causal(f32x16 (&S)[QB], int hf, int blk_lo, const int (&lim)[QB])
{
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int kidx = blk_lo + 8 * (r >> 2) + 4 * hf + (r & 3);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
            if (kidx >= lim[qb]) S[qb][r] = -INFINITY;
    }
}

// p = exp2(S*scale - sub) rounded to bf16 in B-operand order (P[g] holds the keys of 16-key
// group g); returns the row's share of the denominator.
//   AFFINE = false (scale folded into the query, logits of ordinary size): the sum of the values
//     before rounding.  Round-to-nearest is unbiased, so with many comparable terms the denominator
//     and the bf16 numerators agree to well below the bf16 rounding of a single term, and the sum
//     costs one addition per value.
//     Plain v_add_f32 on purpose: the v_dot2 family issues into the matrix pipe and would take MFMA
//     slots there, whereas adds overlap with the MFMAs of the other wave on the SIMD.
//   AFFINE = true (fp32 scale: large logits, causal rows, bias, the history pass that is bound by
//     memory, the running-maximum pass): the sum of the ROUNDED values.  These rows can be sharply
//     peaked; a single dominant probability rounded to bf16 in the numerator and not in the
//     denominator would put its rounding, a relative 2^-9, straight into the output.
template <bool AFFINE>
static __device__ __forceinline__ float exp_pack(const f32x16 &S, float scale, float sub, bf16x8 (&P)[2])
{
    float sum = 0.f;
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const float p0 = __builtin_amdgcn_exp2f(AFFINE ? fmaf(S[8 * g + e], scale, -sub) : S[8 * g + e]);
            const float p1 = __builtin_amdgcn_exp2f(AFFINE ? fmaf(S[8 * g + e + 1], scale, -sub) : S[8 * g + e + 1]);
            P[g][e] = (__bf16)p0;
            P[g][e + 1] = (__bf16)p1;
            if constexpr (AFFINE) {
                // sum += P[e] * 1 + P[e + 1] * 1 on the rounded pair, one instruction (it issues into the
                // matrix pipe, which these forms leave room in).  Through the builtin, not inline assembly:
                // the compiler knows the wait states the instruction needs before its result is read.
                typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
                const bf16x2_t pr = {P[g][e], P[g][e + 1]}, ones = {(__bf16)1.f, (__bf16)1.f};
                sum = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, sum, false);
            } else {
                sum += p0 + p1;
            }
        }
    return sum;
}

// FAST softmax of one block: p = exp2(t)
template <int QB>
static __device__ __forceinline__ void softmax_fast(QState<QB> &st, const f32x16 (&S)[QB], bf16x8 (&P)[QB][2])
{
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) st.l[qb] += exp_pack<false>(S[qb], 1.f, 0.f, P[qb]);
}

// SAFE softmax of one block: running maximum in raw logit units, p = exp2((s - m) * c)
template <int QB>
static __device__ __forceinline__ void softmax_safe(QState<QB> &st, const f32x16 (&S)[QB], bf16x8 (&P)[QB][2])
{
    float mx[QB];
    bool need[QB];
    bool any = false;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        float v = fmaxf(S[qb][0], S[qb][1]);
#pragma unroll
        for (int r = 2; r < 16; r += 2) v = fmaxf(fmaxf(v, S[qb][r]), S[qb][r + 1]);
        mx[qb] = xhalf_max(v);  // same in both half-waves
        need[qb] = (mx[qb] - st.m_ref[qb]) * st.c[qb] > kSafeSlack;
        any |= need[qb];
    }
    if (__builtin_amdgcn_ballot_w64(any) != 0) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float alpha =
                need[qb] ? __builtin_amdgcn_exp2f((st.m_ref[qb] - mx[qb]) * st.c[qb]) : 1.f;
            st.m_ref[qb] = need[qb] ? mx[qb] : st.m_ref[qb];
            st.l[qb] *= alpha;
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) st.O[db][qb][r] *= alpha;
        }
    }
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
        st.l[qb] += exp_pack<true>(S[qb], st.c[qb], st.m_ref[qb] * st.c[qb], P[qb]);
}

// ---- keys and values as rows (history pass that writes the cache itself) --------------------------
// A tile of 64 keys in LDS: 64 key rows of 128 bytes and 64 value rows, 16-byte chunk c of row r at slot c ^ (r / 2) % 8.  Key
// fragments are row pieces; value fragments come out of the rows by LDS transpose reads (addresses as derived in
// hist_fused_bf16.hip).  256 threads.
struct RawTiles {
    const uint8_t *k, *v;  // first row of the range, the head's columns
    int64_t row_bytes;
    uint32_t row_at, k_at[4], v_at;
};

static __device__ __forceinline__ RawTiles raw_tiles(const KParams &p, int64_t row, int h, int tid)
{
    const int lane = tid & 63, l32 = lane & 31, hf = lane >> 5, r = tid >> 3;
    RawTiles t;
    t.k = uniform_ptr((const uint8_t *)(p.k_self + row * p.ld_kv + h * kDHead));
    t.v = uniform_ptr((const uint8_t *)(p.v_self + row * p.ld_kv + h * kDHead));
    t.row_bytes = p.ld_kv * 2;
    t.row_at = (uint32_t)r * (uint32_t)p.ld_kv * 2u + (uint32_t)((tid & 7) ^ ((r >> 1) & 7)) * 16u;
#pragma unroll
    for (int s = 0; s < 4; ++s) t.k_at[s] = (uint32_t)(l32 * 128 + (((2 * s + hf) ^ ((l32 >> 1) & 7)) * 16));
    const int G = lane >> 4, i16 = lane & 15, x = 2 * (G & 1) + ((i16 >> 1) & 1), y = 2 * (G >> 1) + (i16 >> 3);
    t.v_at = (uint32_t)((4 * (G >> 1) + (i16 >> 2)) * 128 + (x ^ y) * 16 + 8 * (i16 & 1));
    return t;
}

// rows 64 n .. 64 n + 63 of the range (they exist: padded lengths are multiples of 64); to_k, to_v: the wave's first KiB of the key
// and of the value rows
static __device__ __forceinline__ void raw_issue(const RawTiles &t, int n, lds_u8 *to_k, lds_u8 *to_v)
{
    const int64_t at = (int64_t)n * 64 * t.row_bytes, half = 32 * t.row_bytes;
    __builtin_amdgcn_global_load_lds((glb_u8 *)(t.k + at) + t.row_at, to_k, 16, 0, 0);
    __builtin_amdgcn_global_load_lds((glb_u8 *)(t.k + at + half) + t.row_at, to_k + 4096, 16, 0, 0);
    __builtin_amdgcn_global_load_lds((glb_u8 *)(t.v + at) + t.row_at, to_v, 16, 0, 0);
    __builtin_amdgcn_global_load_lds((glb_u8 *)(t.v + at + half) + t.row_at, to_v + 4096, 16, 0, 0);
}

// (keys, values: a tile's rows of either kind)
static __device__ __forceinline__ KFrags raw_k(const RawTiles &t, const uint8_t *keys, int blk)
{
    KFrags f;
#pragma unroll
    for (int s = 0; s < 4; ++s) f.a[s] = *(const bf16x8 *)(keys + t.k_at[s] + blk * 4096);
    return f;
}

// (One block of inline assembly with its wait: for the builtin, with copies in flight, the compiler waits until all of
// them have landed.  In a loop it belongs behind the MFMAs of the next logits, which run meanwhile.)
static __device__ __forceinline__ VFrags raw_v(const RawTiles &t, const uint8_t *values, int blk)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    s16x4 x[8];
    asm volatile("ds_read_b64_tr_b16 %0, %8 offset:0\n\tds_read_b64_tr_b16 %1, %8 offset:1088\n\t"
                 "ds_read_b64_tr_b16 %2, %8 offset:64\n\tds_read_b64_tr_b16 %3, %8 offset:1024\n\t"
                 "ds_read_b64_tr_b16 %4, %8 offset:2048\n\tds_read_b64_tr_b16 %5, %8 offset:3136\n\t"
                 "ds_read_b64_tr_b16 %6, %8 offset:2112\n\tds_read_b64_tr_b16 %7, %8 offset:3072\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5]), "=&v"(x[6]), "=&v"(x[7])
                 : "v"((uint32_t)(uintptr_t)(lds_u8 *)values + t.v_at + (uint32_t)blk * 4096u)
                 : "memory");
    VFrags f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        f.a[i >> 1][i & 1] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(x[2 * i], x[2 * i + 1], 0, 1, 2, 3, 4, 5, 6, 7));
    return f;
}

// the value rows of a tile from row `first` on, which may hold anything: zeros, before they meet probabilities of 0
static __device__ __forceinline__ void raw_clear(uint8_t *values, int first, int tid)
{
    for (int i = tid; i < (64 - first) * 8; i += 256) *(uint4 *)(values + first * 128 + i * 16) = uint4{0, 0, 0, 0};
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
}

// The cache block of 32 rows that lie in LDS (chunk c of row r at slot c ^ r % 8; no copy in flight), of which `n` count: key
// and value fragments as laid out in internal.h, zeros in the slots beyond.
static __device__ __forceinline__ void own_block_k(uint8_t *block, const uint8_t *rows, int n, int lane)
{
    const int r = lane & 31, hf = lane >> 5;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        u32x4 x = *(const u32x4 *)(rows + r * 128 + (((2 * s + hf) ^ (r & 7)) * 16));
        if (r >= n) x = u32x4{0, 0, 0, 0};
        *(u32x4 *)(block + (s * 64 + lane) * 16) = x;
    }
}
static __device__ __forceinline__ void own_block_v(uint8_t *block, const uint8_t *rows, int n, int lane)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    const int G = lane >> 4, i16 = lane & 15, hf = lane >> 5;
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int db = 0; db < 2; ++db) {
            bf16x8 x;
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const int r = 16 * g + 8 * hh + 4 * (G >> 1) + (i16 >> 2), c = 4 * db + 2 * (G & 1) + ((i16 >> 1) & 1);
                const bf16x4 part = __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(
                                                                   (lds_u8 *)const_cast<uint8_t *>(rows) + r * 128 + ((c ^ (r & 7)) * 16) + 8 * (i16 & 1))));
#pragma unroll
                for (int e = 0; e < 4; ++e) x[4 * hh + e] = 16 * g + 8 * hh + 4 * hf + e < n ? part[e] : (__bf16)0.f;
            }
            *(u32x4 *)(block + 4096 + ((g * 2 + db) * 64 + lane) * 16) = __builtin_bit_cast(u32x4, x);
        }
}

}  // namespace attn
}  // namespace climber
