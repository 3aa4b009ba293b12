// bf16 MFMA attention for launches of few queries (gfx950): the SUMI candidate pass and the block-diagonal
// history pass of Climber (arXiv 2502.09888, Eq. (3), Sec. 3.1.2, Sec. 3.2) where the 128- and 256-query tiles
// of attn_bf16.hip make too few workgroups: 200 candidates of eight users are 64 workgroups there, one per head,
// and the launch takes as long as one of them walks over the history.  (Fewer still share a tile's keys out among waves,
// attn_split_bf16.hip.)  Us there / here, 8 heads: those 200 against 1000 20.0 / 14.3, of 12 users against 4000 59.6 / 36.6, 256 of 16 against
// 1024 21.9 / 18.9; history pass of one user's 4096 in one subsequence 52.5 / 45.8.
//
// One wave = one workgroup = 32 queries of one (user, head).  The cache holds keys and values as MFMA operand
// fragments, so the wave loads them from global memory (L2; the waves of a head run on one XCD) straight into
// registers, two blocks of 32 keys ahead: no LDS, no barrier, no other wave to wait for.  Bound by the wave's
// own chain per block: 8 MFMAs, 16 exponentials and the conversions between them (about 0.2 us per 32 keys).
//
// The steps and their order are those of attn_bf16.hip's FAST pass -- logits, exponentials, sums and products of
// a block in the same order, the candidate's own key and value joining at the same place -- and so are the
// bits, within one form of the softmax.  Forms (folded, exact scale, SAFE) as described there.  Whether to fold is decided
// for the same queries as there: the wave's 32, or the 64 that a wave of the 256-query tiles holds (a second product
// against the first block of keys, 0.1 us); a SAFE pass is the wave's alone, where the tiled kernel repeats a
// whole tile.
#include "attn_common.h"

#include <type_traits>

namespace climber {
namespace {

using namespace attn;

constexpr int kRing = 2;  // blocks of 32 keys (and as many of 32 values) in flight or in use

// (Two waves per SIMD in the bounds, although a launch has at most one: with all the registers to itself the candidate pass
// uses no scratch memory and takes 15.3 us instead of 14.3 for 200 candidates of 8 users, the history pass of 4096 rows 48.4 instead of 45.8.)
template <bool SUMI, bool CAUSAL>
__global__ __launch_bounds__(64, 2) void attn_wave_kernel(const KParams p)
{
    constexpr int kRowPitch = 144;  // 128 B of a row + 16 B pad
    __shared__ __attribute__((aligned(16))) uint8_t tr[32 * kRowPitch];
    const int lane = threadIdx.x, l32 = lane & 31, hf = lane >> 5;

    // workgroup -> (user, head, query tile); tiles of a head on one XCD (see attn_bf16.hip)
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int qt = j % p.n_qtiles, bh = (j / p.n_qtiles) * 8 + xcd;
    if (bh >= p.B * p.H) return;
    const int h = bh % p.H;
    int b = bh / p.H, Lb, t0, Lpad;
    if (p.uni_len >= 0) {
        Lb = p.uni_len;
        Lpad = p.uni_pad;
        t0 = b * Lpad;
    } else {
        b = p.order[b];
        Lb = p.hist_len[b];
        t0 = p.tok_off[b];
        Lpad = p.tok_off[b + 1] - t0;
    }
    const int q0 = qt * 32;
    int64_t row0;
    int nq, k_lo, k_hi, nq_mate = 0;  // (nq_mate: queries of the 32 that share this wave's pilot)
    if (SUMI) {
        int c0, Mb;
        if (p.uni_cand >= 0) {
            Mb = p.uni_cand;
            c0 = b * Mb;
        } else {
            c0 = p.cand_off[b];
            Mb = p.cand_off[b + 1] - c0;
        }
        if (q0 >= Mb) return;
        row0 = (int64_t)c0 + q0;
        nq = min(32, Mb - q0);
        if (p.pilot_pairs) nq_mate = min(32, Mb - (q0 ^ 32));
        k_lo = 0;
        k_hi = Lb;
    } else {
        if (q0 >= Lpad) return;
        row0 = (int64_t)t0 + q0;
        nq = max(0, min(32, Lb - q0));
        if (nq == 0) {  // padding rows only: defined output, zeros (padded lengths are multiples of 64)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *(uint4 *)(p.o + (row0 + 8 * i + (lane >> 3)) * p.ld_o + h * kDHead + (lane & 7) * 8) = uint4{0, 0, 0, 0};
            return;
        }
        k_lo = p.sub_len > 0 ? (q0 / p.sub_len) * p.sub_len : 0;
        k_hi = p.sub_len > 0 ? min(k_lo + p.sub_len, Lb) : Lb;
        if (CAUSAL) k_hi = min(k_hi, q0 + 32);  // no query of this tile sees a later key
    }
    const int n_blk = (k_hi - k_lo + kBlockKeys - 1) / kBlockKeys;
    const uint8_t *kv = p.layer_base + ((size_t)t0 * p.H + (size_t)h * Lpad) * (kDHead * 4) +
                        (size_t)(k_lo / kBlockKeys) * kBlockBytes;
    const int64_t row = row0 + min(l32, nq - 1);

    QState<1> st;
    KFrags kf[kRing];
    VFrags vf[kRing];
    auto load_block_k = [&](int blk, KFrags &f) __attribute__((always_inline)) { f = load_k(kv + (size_t)min(blk, n_blk - 1) * kBlockBytes, lane); };
    auto load_block_v = [&](int blk, VFrags &f) __attribute__((always_inline)) { f = load_v(kv + (size_t)min(blk, n_blk - 1) * kBlockBytes, lane); };
    const __bf16 *q_row = p.q + row * p.ld_q + h * kDHead + 8 * hf;
    auto load_q = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 4; ++s) st.qf[0][s] = *(const bf16x8 *)(q_row + 16 * s);
    };
    // masks of a block that is not wholly visible: the end of the range, and the diagonal of the causal pass
    // (queries q0 .. q0 + 31 and a range that ends with them)
    auto mask_tail = [&](f32x16 (&S)[1], int blk) __attribute__((always_inline)) {
        const int blk_lo = k_lo + blk * kBlockKeys;
        const int lim[1] = {CAUSAL ? min(q0 + l32 + 1, k_hi) : k_hi};
        mask_causal(S, hf, blk_lo, lim);
    };
    // the candidate's own key and value rows
    auto own_dot = [&]() __attribute__((always_inline)) {  // <q, k_own>, in the units of the query as it stands
        const __bf16 *kp = p.k_self + row * p.ld_kv + h * kDHead + 8 * hf;
        bf16x8 kk[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) kk[s] = *(const bf16x8 *)(kp + 16 * s);
        float dot = 0.f;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            u32x4 qv = __builtin_bit_cast(u32x4, st.qf[0][s]);  // (the empty asm: or its unpacked halves stay live)
            asm volatile("" : "+v"(qv));
            const bf16x8 qq = __builtin_bit_cast(bf16x8, qv);
#pragma unroll
            for (int e = 0; e < 8; ++e) dot += (float)qq[e] * (float)kk[s][e];
        }
        return dot + xhalf(dot);
    };
    // (the value row waits in the wave's corner of LDS, idle until the output, rather than in 16 registers)
    auto fetch_own_v = [&]() __attribute__((always_inline)) {
        const __bf16 *vp = p.v_self + row * p.ld_kv + h * kDHead + 4 * hf;
#pragma unroll
        for (int i = 0; i < 8; ++i) *(uint2 *)(tr + (i * 64 + lane) * 8) = *(const uint2 *)(vp + 8 * i);
    };
    auto own_v = [&](float w) __attribute__((always_inline)) {  // O += w * v_own
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const bf16x4 vv = *(const bf16x4 *)(tr + (i * 64 + lane) * 8);
#pragma unroll
            for (int e = 0; e < 4; ++e) st.O[i >> 2][0][4 * (i & 3) + e] = fmaf(w, (float)vv[e], st.O[i >> 2][0][4 * (i & 3) + e]);
        }
    };
    auto store_rows = [&](float lt) __attribute__((always_inline)) {
        const float inv = 1.f / lt;
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                bf16x4 ov;
#pragma unroll
                for (int e = 0; e < 4; ++e) ov[e] = (__bf16)(st.O[db][0][4 * g + e] * inv);
                *(bf16x4 *)(tr + l32 * kRowPitch + (32 * db + 8 * g + 4 * hf) * 2) = ov;
            }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 8 * i + (lane >> 3), cc = lane & 7;
            const uint4 val = *(const uint4 *)(tr + r * kRowPitch + cc * 16);
            __bf16 *op = p.o + (row0 + r) * p.ld_o + h * kDHead + cc * 8;
            if (r < nq) *(uint4 *)op = val;
            else if (!SUMI && q0 + r < Lpad) *(uint4 *)op = uint4{0, 0, 0, 0};
        }
    };

    load_q();
    QState<1> mate;
    int mate_scen = 0, mate_beh = 0;
    if (SUMI && nq_mate > 0) {
        const int64_t r = row0 + ((q0 ^ 32) - q0) + min(l32, nq_mate - 1);
#pragma unroll
        for (int s = 0; s < 4; ++s) mate.qf[0][s] = *(const bf16x8 *)(p.q + r * p.ld_q + h * kDHead + 8 * hf + 16 * s);
        mate_scen = p.scen[r], mate_beh = p.beh[r];
    }
    if (n_blk > 0) {
#pragma unroll
        for (int i = 0; i < kRing; ++i) {
            load_block_k(i, kf[i]);
        }
    }
    const int sc = min(max(p.scen[row], 0), p.n_scen - 1), bhv = min(max(p.beh[row], 0), p.n_beh - 1);
    st.c[0] = p.scale_log2e / p.tau[sc * p.n_beh + bhv];
    st.l[0] = 0.f;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) st.O[db][0][r] = 0.f;

    // FAST pass
    bool fold = false;
    float w_own = 0.f;
    auto own_weight = [&]() __attribute__((always_inline)) {
        if (SUMI) w_own = __builtin_amdgcn_exp2f(own_dot() * (fold ? 1.f : st.c[0]));
    };
    f32x16 S0[1], S1[1];
    bf16x8 P0[1][2], P1[1][2] = {};  // (no block before the first: zeros)
    if (n_blk > 0) {
        load_block_v(0, vf[0]);
        vf[1] = VFrags{};
        qk_block(st, kf[0], S0);
        f32x16 S_mate[1];
        if (SUMI && nq_mate > 0) qk_block(mate, kf[0], S_mate);
        load_block_k(kRing, kf[0]);
        // fold the row scale into a bf16 query?  (the pilot of attn_bf16.hip)
        {
            float ss = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) ss = fmaf(S0[0][r], S0[0][r], ss);
            ss += xhalf(ss);
            bool big = k_hi - k_lo < kFoldMinKeys || !(ss * st.c[0] * st.c[0] < kBlockKeys * kPilotSpread * kPilotSpread);
            if (SUMI && nq_mate > 0) {  // the tiled kernel's waves have 64 queries here and fold for all of them or none
                ss = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r) ss = fmaf(S_mate[0][r], S_mate[0][r], ss);
                ss += xhalf(ss);
                const float c = p.scale_log2e / p.tau[min(max(mate_scen, 0), p.n_scen - 1) * p.n_beh + min(max(mate_beh, 0), p.n_beh - 1)];
                big |= !(ss * c * c < kBlockKeys * kPilotSpread * kPilotSpread);
            }
            fold = SUMI && __builtin_amdgcn_ballot_w64(big) == 0;
            if (fold) {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const bf16x8 qq = st.qf[0][s];
#pragma unroll
                    for (int e = 0; e < 8; ++e) st.qf[0][s][e] = (__bf16)((float)qq[e] * st.c[0]);
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) S0[0][r] *= st.c[0];
            }
        }
        auto run = [&](auto fold_tag) __attribute__((always_inline)) {
            constexpr bool FOLD = decltype(fold_tag)::value;
            // Step `blk` (slot U of the group): the logits of block blk + 1, the exponentials of block blk (whose logits
            // are in Sc) and the value product of block blk - 1 (whose probabilities are in Pp) -- three chains that
            // do not depend on each other.  TAIL: the last group; keys past the end of the range (the whole block,
            // where it lies beyond) get the logit -inf, i.e. add zeros, and nothing is requested that is not used.
            auto step = [&](int blk, f32x16 (&Sc)[1], f32x16 (&Sn)[1], bf16x8 (&Pc)[1][2], const bf16x8 (&Pp)[1][2], auto u_tag,
                            auto tail_tag) __attribute__((always_inline)) {
                constexpr int U = decltype(u_tag)::value;
                constexpr bool TAIL = decltype(tail_tag)::value;
                if constexpr (!TAIL || U < 3) qk_block(st, kf[(U + 1) % kRing], Sn);
                if constexpr (!TAIL || U == 0) load_block_k(blk + 1 + kRing, kf[(U + 1) % kRing]);
                if constexpr (TAIL) mask_tail(Sc, blk);
                if constexpr (FOLD) softmax_fast(st, Sc, Pc);
                else st.l[0] += exp_pack<true>(Sc[0], st.c[0], 0.f, Pc[0]);
                pv_block(st, vf[(U + 1) % kRing], Pp);
                if constexpr (!TAIL || U < 3) load_block_v(blk + 1, vf[(U + 1) % kRing]);
                // the wave issues in order: a product, then exponentials while it runs
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x2, FOLD ? 3 : 4, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            const std::integral_constant<int, 0> u0;
            const std::integral_constant<int, 1> u1;
            const std::integral_constant<int, 2> u2;
            const std::integral_constant<int, 3> u3;
            const std::true_type tail;
            const std::false_type whole;
            int blk = 0;
            auto groups = [&](int end, auto own_tag) __attribute__((always_inline)) {  // whole groups of four, a further block exists
                for (; blk + 4 < end; blk += 4) {
                    step(blk, S0, S1, P0, P1, u0, whole);
                    step(blk + 1, S1, S0, P1, P0, u1, whole);
                    step(blk + 2, S0, S1, P0, P1, u2, whole);
                    if constexpr (decltype(own_tag)::value) st.l[0] += blk == 0 && hf == 0 ? w_own : 0.f;
                    step(blk + 3, S1, S0, P1, P0, u3, whole);
                }
            };
            if (SUMI) {
                own_weight();
                fetch_own_v();
                groups(min(n_blk, 9), std::true_type{});
                if (n_blk > 8) own_v(w_own);  // behind the products of blocks 0 .. 6
            }
            groups(n_blk, std::false_type{});
            step(blk, S0, S1, P0, P1, u0, tail);  // one to four blocks are left
            step(blk + 1, S1, S0, P1, P0, u1, tail);
            if (blk + 2 < n_blk) {
                step(blk + 2, S0, S1, P0, P1, u2, tail);
                step(blk + 3, S1, S0, P1, P0, u3, tail);
            }
            // (of an odd number the last one is missing: zeros times the values of the one before, which an infinite one among
            // them would make NaN)
            if ((n_blk & 1) == 0) pv_block(st, vf[1], P1);
        };
        if (fold) run(std::true_type{});
        else run(std::false_type{});
    }
    if (SUMI) {
        if (n_blk == 0) {
            own_weight();
            fetch_own_v();
        }
        if (n_blk <= 8) own_v(w_own);
        if (n_blk <= 4) st.l[0] += hf == 0 ? w_own : 0.f;
    }
    float lt = st.l[0] + xhalf(st.l[0]);
    const bool bad = fold ? !(lt > kDenomLo && lt < kDenomHi) : !(lt > kDenomLoExact && lt < kDenomHiExact);
    if (__builtin_amdgcn_ballot_w64(bad) != 0) {
        // SAFE pass (rare): queries as given, running maximum; the own key / value is the first member
        int again = l32;
        asm volatile("" : "+v"(again));  // keeps the compiler from holding the first pass's rows in registers
        const int64_t r2 = row0 + min(again, nq - 1);
        const __bf16 *qp = p.q + r2 * p.ld_q + h * kDHead + 8 * hf;
#pragma unroll
        for (int s = 0; s < 4; ++s) st.qf[0][s] = *(const bf16x8 *)(qp + 16 * s);
        st.m_ref[0] = SUMI ? own_dot() : kSafeNoRef;
        st.l[0] = SUMI && hf == 0 ? 1.f : 0.f;
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) st.O[db][0][r] = 0.f;
        if (SUMI) own_v(1.f);
        for (int blk = 0; blk < n_blk; ++blk) {
            load_block_k(blk, kf[0]);
            load_block_v(blk, vf[0]);
            qk_block(st, kf[0], S0);
            if (blk == n_blk - 1) mask_tail(S0, blk);
            softmax_safe(st, S0, P0);
            pv_block(st, vf[0], P0);
        }
        lt = st.l[0] + xhalf(st.l[0]);
    }
    store_rows(lt);
}

}  // namespace

hipError_t launch_attn_wave_bf16(const AttnArgs &a, bool sumi, hipStream_t s)
{
    const int n_qtiles = (a.max_rows_per_user + 31) / 32;
    const int64_t grid = (int64_t)8 * n_qtiles * ((a.cache.B * a.H + 7) / 8);
    if (grid <= 0 || grid > 0x7fffffff) return hipErrorInvalidValue;
    KParams p = make_params(a, n_qtiles);
    p.pilot_pairs = sumi && a.max_rows_per_user > 128;
    const dim3 g((unsigned)grid), t(64);
    if (sumi) hipLaunchKernelGGL((attn_wave_kernel<true, false>), g, t, 0, s, p);
    else if (a.causal) hipLaunchKernelGGL((attn_wave_kernel<false, true>), g, t, 0, s, p);
    else hipLaunchKernelGGL((attn_wave_kernel<false, false>), g, t, 0, s, p);
    return hipGetLastError();
}

}  // namespace climber
