// bf16 MFMA attention for launches of so few queries that a wave per 32 of them (attn_wave_bf16.hip) leaves most SIMDs without
// one (gfx950): the SUMI candidate pass and the history pass of Climber (arXiv 2502.09888, Eq. (3), Sec. 3.1.2, Sec. 3.2) of
// one to a few users.  Such a launch takes as long as one wave walks over its keys.
//
// One workgroup = 32 queries of one (user, head), NP + 2 waves.  The blocks of 32 keys are shared out among NP of them, a round of NP
// blocks at a time: logits, exponentials, probabilities as the operand of the value product into LDS, and each lane's sum of
// them.  The last two waves add up: the value products, 32 dimensions each, and the sums, block after block in the order of the
// keys.  So every addition is made in the order in which the other kernels make it, and the bits are theirs: no merging of partial
// outputs, and one form of the softmax for all keys.  A round's probabilities are added up while the next round's are made.
//
// Bound by its beginning (about 5 us for a launch: first touches of rows, keys and code) and then by a round's chain, exponentials,
// LDS, meeting, value products that wait for each other: 0.10 us per 32 keys, 0.21 where one wave does all of it.  NP:
// 200 candidates of one user against 1000, 8 heads, 8.7 us with 2, 9.2 with 3, 8.4 with 4, 8.6 with 6, against 4000 (values one
// round ahead) 20.6, 22.1, 18.2, 17.5.  Keys four rounds ahead instead of two, or a round's probabilities read under the products of the round before: no faster.
//
// The pilot (which decides whether to fold, attn_bf16.hip), the own key and value and the SAFE pass as in attn_wave_bf16.hip.
#include "attn_common.h"

#include <type_traits>

namespace climber {
namespace {

using namespace attn;

constexpr int NP = 4;  // waves that make probabilities
constexpr int kHalfPitch = 80;  // 32 dimensions of an output row and 16 B, in LDS

struct Slot {  // a block's probabilities (B operands of the value product) and each lane's sum of them
    bf16x8 p[2][64];
    float sum[64];
};

// VR: rounds that the values are requested ahead.
template <bool SUMI, bool CAUSAL, int VR>
__global__ __launch_bounds__((NP + 2) * 64, 2) void attn_split_kernel(const KParams p)
{
    __shared__ __attribute__((aligned(16))) uint8_t tr[2 * 32 * kHalfPitch];
    __shared__ Slot slots[2][NP];
    __shared__ int no_fold[2];
    const int lane = threadIdx.x & 63, l32 = lane & 31, hf = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

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
    int nq, k_lo, k_hi, nq_mate = 0;  // (nq_mate: queries of the 32 that share this tile's pilot)
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
            if (wave < 4) *(uint4 *)(p.o + (row0 + 8 * wave + (lane >> 3)) * p.ld_o + h * kDHead + (lane & 7) * 8) = uint4{0, 0, 0, 0};
            return;
        }
        k_lo = p.sub_len > 0 ? (q0 / p.sub_len) * p.sub_len : 0;
        k_hi = p.sub_len > 0 ? min(k_lo + p.sub_len, Lb) : Lb;
        if (CAUSAL) k_hi = min(k_hi, q0 + 32);  // no query of this tile sees a later key
    }
    const int n_blk = (k_hi - k_lo + kBlockKeys - 1) / kBlockKeys, n_rounds = (n_blk + NP - 1) / NP;
    const uint8_t *kv = p.layer_base + ((size_t)t0 * p.H + (size_t)h * Lpad) * (kDHead * 4) +
                        (size_t)(k_lo / kBlockKeys) * kBlockBytes;
    const int64_t row = row0 + min(l32, nq - 1);

    QState<1> st, mate;
    auto load_q = [&](QState<1> &to, int64_t r) __attribute__((always_inline)) {
        const __bf16 *q_row = p.q + r * p.ld_q + h * kDHead + 8 * hf;
#pragma unroll
        for (int s = 0; s < 4; ++s) to.qf[0][s] = *(const bf16x8 *)(q_row + 16 * s);
    };
    auto load_block_k = [&](int blk, KFrags &f) __attribute__((always_inline)) { f = load_k(kv + (size_t)min(blk, n_blk - 1) * kBlockBytes, lane); };
    // the end of the range, and the diagonal of the causal pass (queries q0 .. q0 + 31 and a range that ends with them)
    auto mask_tail = [&](f32x16 (&S)[1], int blk) __attribute__((always_inline)) {
        const int lim[1] = {CAUSAL ? min(q0 + l32 + 1, k_hi) : k_hi};
        mask_causal(S, hf, k_lo + blk * kBlockKeys, lim);
    };
    // barrier for what lies in LDS
    auto meet = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // What is waited for first, all of it requested before any of it is used.  The temperatures: the table's entries, a lane each, where
    // a wave holds them all, rather than a second trip to memory behind the row's indices.
    const int64_t mate_row = SUMI && nq_mate > 0 ? row0 + ((q0 ^ 32) - q0) + min(l32, nq_mate - 1) : row;  // (no mate: itself)
    const int n_tau = p.n_scen * p.n_beh;
    const float tau = p.tau[min(lane, n_tau - 1)];
    const int scen = p.scen[row], beh = p.beh[row], mate_scen = SUMI ? p.scen[mate_row] : 0, mate_beh = SUMI ? p.beh[mate_row] : 0;
    KFrags pilot_k, kf[2];
    load_q(st, row);
    if (SUMI && wave == 1) load_q(mate, mate_row);
    bf16x8 k_own[4] = {};
    bf16x4 v_own[4] = {};
    const int db = wave - NP;  // the last two waves' 32 dimensions
    if (n_blk > 0) {
        if (SUMI && wave == 1) load_block_k(0, pilot_k);
        if (wave < NP) {
            load_block_k(wave, kf[0]);
            load_block_k(NP + wave, kf[1]);
        }
    }
    auto load_own_k = [&]() __attribute__((always_inline)) {
        const __bf16 *kp = p.k_self + row * p.ld_kv + h * kDHead + 8 * hf;
#pragma unroll
        for (int s = 0; s < 4; ++s) k_own[s] = *(const bf16x8 *)(kp + 16 * s);
    };
    if (SUMI && wave >= NP) {
        load_own_k();
        const __bf16 *vp = p.v_self + row * p.ld_kv + h * kDHead + 4 * hf + 32 * db;
#pragma unroll
        for (int i = 0; i < 4; ++i) v_own[i] = *(const bf16x4 *)(vp + 8 * i);
    }
    auto own_dot = [&]() __attribute__((always_inline)) {  // <q, k_own>, in the units of the query as it stands
        float dot = 0.f;
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int e = 0; e < 8; ++e) dot += (float)st.qf[0][s][e] * (float)k_own[s][e];
        return dot + xhalf(dot);
    };
    auto row_scale = [&](int sc, int bh_) __attribute__((always_inline)) {
        const int at = min(max(sc, 0), p.n_scen - 1) * p.n_beh + min(max(bh_, 0), p.n_beh - 1);
        return p.scale_log2e / (n_tau <= 64 ? __shfl(tau, at, 64) : p.tau[at]);
    };
    st.c[0] = row_scale(scen, beh);

    // FAST pass
    f32x16 S0[1], S1[1];
    bool fold = false;
    if (SUMI && n_blk > 0) {
        // Fold the row scale into a bf16 query?  The first block's logits are looked at by wave 0, which has them to make, and those of
        // the other 32 queries by wave 1.
        if (wave < 2) {
            if (wave == 0) qk_block(st, kf[0], S0);
            else qk_block(mate, pilot_k, S0);
            const float c = wave == 0 ? st.c[0] : row_scale(mate_scen, mate_beh);
            float ss = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) ss = fmaf(S0[0][r], S0[0][r], ss);
            ss += xhalf(ss);
            const bool wide = !(ss * c * c < kBlockKeys * kPilotSpread * kPilotSpread);
            no_fold[wave] = __builtin_amdgcn_ballot_w64(wide) != 0;
        }
        meet();
        fold = k_hi - k_lo >= kFoldMinKeys && !(no_fold[0] | no_fold[1]);
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

    if (wave < NP) {
        // Block r * NP + wave of round r; the logits of the next round's run while its exponentials do.  (The last rounds
        // request blocks again that are not used.)
        auto produce = [&](int r, f32x16 (&Sc)[1], f32x16 (&Sn)[1], KFrags &k, auto fold_tag) __attribute__((always_inline)) {
            constexpr bool FOLD = decltype(fold_tag)::value;
            const int blk = r * NP + wave;
            qk_block(st, k, Sn);
            load_block_k(blk + 3 * NP, k);
            if (blk >= n_blk - 1) mask_tail(Sc, blk);
            Slot &to = slots[r & 1][wave];
            bf16x8 P[2];
            to.sum[lane] = exp_pack<!FOLD>(Sc[0], FOLD ? 1.f : st.c[0], 0.f, P);
            to.p[0][lane] = P[0];
            to.p[1][lane] = P[1];
            meet();
        };
        auto all = [&](auto fold_tag) __attribute__((always_inline)) {
            for (int r = 0; r < n_rounds; r += 2) {
                produce(r, S0, S1, kf[1], fold_tag);
                if (r + 1 < n_rounds) produce(r + 1, S1, S0, kf[0], fold_tag);
            }
        };
        if (n_blk > 0) {
            if (!SUMI || wave > 0) qk_block(st, kf[0], S0);
            load_block_k(2 * NP + wave, kf[0]);
        }
        if (fold) all(std::true_type{});
        else all(std::false_type{});
        meet();
        return;
    }

    f32x16 &O = st.O[0][0];
#pragma unroll
    for (int r = 0; r < 16; ++r) O[r] = st.O[1][0][r] = 0.f;
    st.l[0] = 0.f;
    bf16x8 v[VR][NP][2];
    auto load_block_v = [&](int blk, bf16x8 (&f)[2]) __attribute__((always_inline)) {
        const uint8_t *from = kv + (size_t)min(blk, n_blk - 1) * kBlockBytes + 4096 + (db * 64 + lane) * 16;
        f[0] = *(const bf16x8 *)from;
        f[1] = *(const bf16x8 *)(from + 2048);
    };
    if (n_blk > 0) {
#pragma unroll
        for (int i = 0; i < VR * NP; ++i) load_block_v(i, v[i / NP][i % NP]);
    }
    float w_own = 0.f;
    if (SUMI) w_own = __builtin_amdgcn_exp2f(own_dot() * (fold ? 1.f : st.c[0]));
    auto own_v = [&](float w) __attribute__((always_inline)) {  // O += w * v_own
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) O[4 * i + e] = fmaf(w, (float)v_own[i][e], O[4 * i + e]);
    };
    // (one loop body, not a lambda called for each u: that one's schedule takes 17 registers more, and 0.4 us of the shortest launches)
    for (int r0 = 0; r0 < n_rounds; r0 += VR)
#pragma unroll
    for (int u = 0; u < VR; ++u) {
        const int r = r0 + u;
        if (u > 0 && r >= n_rounds) break;
        meet();
        bf16x8 P[NP][2];
        float sum[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) {  // (what is not a block's: not used)
            const Slot &from = slots[r & 1][i];
            P[i][0] = from.p[0][lane];
            P[i][1] = from.p[1][lane];
            sum[i] = from.sum[lane];
        }
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            if (SUMI) {  // the own key and value join where they do in the other kernels
                if (i == 3 % NP && r == 3 / NP && n_blk > 4) st.l[0] += hf == 0 ? w_own : 0.f;
                if (i == 7 % NP && r == 7 / NP && n_blk > 8) own_v(w_own);
            }
            if (r * NP + i < n_blk) {
                st.l[0] += sum[i];
                O = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[u][i][0], P[i][0], O, 0, 0, 0);
                O = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[u][i][1], P[i][1], O, 0, 0, 0);
            }
        }
#pragma unroll
        for (int i = 0; i < NP; ++i) load_block_v((r + VR) * NP + i, v[u][i]);  // (not under the condition: the waits would lose count)
    }
    if (SUMI) {
        if (n_blk <= 8) own_v(w_own);
        if (n_blk <= 4) st.l[0] += hf == 0 ? w_own : 0.f;
    }
    float lt = st.l[0] + xhalf(st.l[0]);
    const bool bad = fold ? !(lt > kDenomLo && lt < kDenomHi) : !(lt > kDenomLoExact && lt < kDenomHiExact);
    if (__builtin_amdgcn_ballot_w64(bad) != 0) {
        // SAFE pass (rare): queries as given, running maximum; the own key / value is the first member.  Both waves make all
        // the logits, and the products of their own 32 dimensions.
        int again = l32;
        asm volatile("" : "+v"(again));  // keeps the compiler from holding the first pass's rows in registers
        load_q(st, row0 + min(again, nq - 1));
        if (SUMI) load_own_k();
        st.m_ref[0] = SUMI ? own_dot() : kSafeNoRef;
        st.l[0] = SUMI && hf == 0 ? 1.f : 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) O[r] = 0.f;
        if (SUMI) own_v(1.f);
        for (int blk = 0; blk < n_blk; ++blk) {
            bf16x8 P[1][2];
            load_block_k(blk, pilot_k);
            load_block_v(blk, v[0][0]);
            qk_block(st, pilot_k, S0);
            if (blk == n_blk - 1) mask_tail(S0, blk);
            softmax_safe(st, S0, P);
            O = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[0][0][0], P[0][0], O, 0, 0, 0);
            O = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[0][0][1], P[0][1], O, 0, 0, 0);
        }
        lt = st.l[0] + xhalf(st.l[0]);
    }
    // No wave of the workgroup reads the tile's rows any more: a history tile's output may lie on its key and value rows.  (Candidates'
    // outputs lie apart from their inputs: with pilot_pairs the neighbouring workgroup reads these query rows, in no order.)
    meet();
    uint8_t *half = tr + db * 32 * kHalfPitch;
    const float inv = 1.f / lt;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        bf16x4 ov;
#pragma unroll
        for (int e = 0; e < 4; ++e) ov[e] = (__bf16)(O[4 * g + e] * inv);
        *(bf16x4 *)(half + l32 * kHalfPitch + (8 * g + 4 * hf) * 2) = ov;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = 16 * i + (lane >> 2), cc = lane & 3;
        const uint4 val = *(const uint4 *)(half + r * kHalfPitch + cc * 16);
        __bf16 *op = p.o + (row0 + r) * p.ld_o + h * kDHead + 32 * db + cc * 8;
        if (r < nq) *(uint4 *)op = val;
        else if (!SUMI && q0 + r < Lpad) *(uint4 *)op = uint4{0, 0, 0, 0};
    }
}

}  // namespace

hipError_t launch_attn_split_bf16(const AttnArgs &a, bool sumi, hipStream_t s)
{
    const int n_qtiles = (a.max_rows_per_user + 31) / 32;
    const int64_t grid = (int64_t)8 * n_qtiles * ((a.cache.B * a.H + 7) / 8);
    if (grid <= 0 || grid > 0x7fffffff) return hipErrorInvalidValue;
    KParams p = make_params(a, n_qtiles);
    p.pilot_pairs = sumi && a.max_rows_per_user > 128;
    const dim3 g((unsigned)grid), t((NP + 2) * 64);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, g, t, 0, s, p); };
    // Values a round further ahead where the walk is long, and what is requested in vain at its end little of it.  Us the call, one round ahead / two: 200
    // candidates against 4000 behaviours 18.5 / 18.0, two users x 64 20.9 / 18.6, eight x 20 against 1000 to 4000 18.7 / 16.7, three x 32 against 2500 14.5 /
    // 13.4, 200 against 2500 13.2 / 13.1, 2000 11.5 / 11.5, 1500 9.9 / 10.0, five users against 355 to 1421 8.6 / 8.8, 4 x 64 against 256 5.6 / 6.0.  A history
    // tile's subsequence is short, and without them even.
    if (sumi && a.max_hist_len > 2048) go(attn_split_kernel<true, false, 2>);
    else if (sumi) go(attn_split_kernel<true, false, 1>);
    else if (a.causal) go(attn_split_kernel<false, true, 1>);
    else go(attn_split_kernel<false, false, 1>);
    return hipGetLastError();
}

}  // namespace climber
