// bf16 MFMA flash attention for gfx950 (CDNA4): the SUMI candidate pass and the block-diagonal
// history pass of Climber (arXiv 2502.09888): Eq. (3) attention with a per-query-row temperature,
// the "single user, multiple items" mask of Sec. 3.2 and the per-subsequence attention of
// Sec. 3.1.2.
//
// Shape of the computation (one workgroup = one (user, head, tile of NW*64 query rows)):
//   - the transposed problem is computed: S^T = K Q^T and O^T = V^T P^T with
//     v_mfma_f32_32x32x16_bf16.  In the accumulator layout of that instruction a lane owns ONE
//     query column (lane % 32), so the softmax statistics of a query are per-lane scalars and the
//     probabilities leave the S^T accumulator already in the B-operand layout the P V product
//     needs (the cache stores V with the matching key permutation).
//   - history K/V tiles of 64 keys are copied HBM -> LDS directly (global_load_lds, no register
//     staging; the cache is stored as MFMA fragments so the copy is linear) into a ring of 3
//     buffers (the tile being computed, the next one, and the one being refilled) and are reused
//     by every wave, i.e. by the whole query tile.  Query rows and the candidates' own key / value
//     rows arrive the same way in a landing buffer behind the ring, one slice per wave.
//   - FAST pass.  Softmax does not depend on the reference subtracted from the logits as long as
//     numerator and denominator share it, and fp32 / bf16 carry 8 exponent bits, so for logits of
//     ordinary size NO reference is needed at all: p = exp2(t) with t the logit in log2 units, one
//     v_exp_f32, half a v_cvt_pk_bf16_f32 and one v_add_f32 (denominator) per logit -- no row
//     maximum, no subtraction, no rescale of O.  Two forms, chosen per wave from the first block's
//     logits: "folded", q' = bf16(q * c) with c = qk_scale*log2(e)/tau_row, so that t = <q',k>
//     comes straight out of the MFMA (rounding q*c costs every logit a relative 2^-9: kept only
//     while a row's denominator stays in [kDenomLo, kDenomHi]); and "exact scale", q as given and
//     t = <q,k> * c in fp32 (one more multiplication per logit; the denominator only has to stay
//     inside the exponent range, [kDenomLoExact, kDenomHiExact]; the denominator is summed from the
//     probabilities as rounded to bf16, so that a one-hot row does not carry the rounding of its
//     dominant term into the output).  Only the candidate pass folds; history rows always take the
//     exact form.  The loop is software pipelined
//     over 32-key blocks: the S^T MFMAs of block i+1 are issued before the exponentials of block
//     i, so matrix and vector pipes overlap inside one wave.
//   - SAFE pass.  If any row's denominator leaves its window (or is not finite) the workgroup
//     redoes its work with the classical online softmax: unscaled q, fp32 scale
//     p = exp2(s*c - m*c), running row maximum (moved when exceeded by 2^8, O and l rescaled).
//     This covers logits of any size.  The choice of form is per wave and the redo per workgroup,
//     so a row's rounding depends on whether a neighbour of its tile has large logits: results
//     are bitwise independent of the other rows only within one form.
//   - SUMI: the candidate's own key / value join the softmax as one more member (FAST: between
//     two tiles, from the landing buffer; SAFE: as the initial state): the "+ itself" term of the
//     mask.
#include "attn_common.h"

#include <algorithm>
#include <type_traits>

namespace climber {
namespace {

using namespace attn;

constexpr int kTileKeys = 64;                // keys per LDS tile = 2 cache blocks
constexpr int kTileBytes = 2 * kBlockBytes;  // 16 KiB
constexpr int kStages = 3;                   // LDS ring of K/V tiles

// wait until at most `tiles_in_flight` later tiles (NPRE loads each) are still outstanding
template <int NPRE>
__device__ __forceinline__ void wait_tiles(int tiles_in_flight)
{
    static_assert(NPRE == 2 || NPRE == 4 || NPRE == 8, "vmcnt immediates below");
    if (tiles_in_flight >= 2) {
        if (NPRE == 8) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
        if (NPRE == 4) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        if (NPRE == 2) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
    } else if (tiles_in_flight == 1) {
        if (NPRE == 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        if (NPRE == 4) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
        if (NPRE == 2) asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
    } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
}

// RAW (history pass): the keys and values are rows, as the projection wrote them, and this launch writes them into the cache
// as well.  Key and value tiles travel into the ring as rows (RawTiles, attn_common.h).  Every
// wave writes the cache blocks of its own rows, which come by the landing buffer while it attends, as a candidate's own rows
// do: nothing of it is in the loop.
template <int NW, int QB, bool SUMI, bool CAUSAL = false, bool RAW = false>
__global__ __launch_bounds__(NW * 64, 2) void attn_bf16_kernel(const KParams p)
{
    static_assert(!(SUMI && CAUSAL), "the causal flag concerns the history pass");
    static_assert(!(SUMI && RAW) && (!RAW || NW == 4), "rows: the history pass, two slabs of 32 rows");
    constexpr bool OWN = SUMI || RAW;  // the tile's own key and value rows come by the landing buffer
    static_assert(kStages == 3, "tile t+1 is read while tile t is computed and one more is in flight; "
                                "every wait in the FAST loop drains all copies");
    constexpr int NT = NW * 64;
    constexpr int WQ = 32 * QB;  // query rows per wave
    constexpr int TQ = NW * WQ;  // query rows per workgroup
    constexpr int NPRE = kTileBytes / 16 / NT;
    __shared__ __attribute__((aligned(16))) uint8_t lds[kStages * kTileBytes + TQ * 128];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // scalar
    int l32 = lane & 31;
    const int hf = lane >> 5;

    // workgroup -> (user, head, query tile).  Consecutive workgroup ids are dealt round-robin to
    // the 8 XCDs; tiles of the same (user, head) get ids congruent mod 8 so that they run on one
    // XCD and share its L2 copy of that head's K/V.
    const int wg = blockIdx.x;
    const int xcd = wg & 7, j = wg >> 3;
    const int qt = j % p.n_qtiles;
    const int bh = (j / p.n_qtiles) * 8 + xcd;
    if (bh >= p.B * p.H) return;
    // Uniform batches (the host knows): user geometry comes from kernel arguments, which saves
    // two dependent trips to memory at the start of every workgroup.
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

    const int q0 = qt * TQ;
    int64_t row0;
    int nq, k_lo, k_hi;
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
        nq = min(TQ, Mb - q0);
        k_lo = 0;
        k_hi = Lb;
    } else {
        if (q0 >= Lpad) return;
        row0 = (int64_t)t0 + q0;
        nq = max(0, min(TQ, Lb - q0));
        if (nq == 0) {  // a tile of padding rows only: defined output, zeros (and zeros in the cache)
            if (RAW) {
                uint8_t *dst = const_cast<uint8_t *>(p.layer_base) + ((size_t)t0 * p.H + (size_t)h * Lpad) * (kDHead * 4) +
                               (size_t)(q0 / kBlockKeys) * kBlockBytes;
                for (int i = tid; i < min(TQ, Lpad - q0) * (kDHead * 4 / 16); i += NT) ((uint4 *)dst)[i] = uint4{0, 0, 0, 0};
            }
            for (int idx = tid; idx < TQ * (kDHead / 8); idx += NT) {
                const int r = idx / (kDHead / 8), cc = idx % (kDHead / 8);
                if (q0 + r < Lpad)
                    *(uint4 *)(p.o + (row0 + r) * p.ld_o + h * kDHead + cc * 8) = uint4{0, 0, 0, 0};
            }
            return;
        }
        k_lo = p.sub_len > 0 ? (q0 / p.sub_len) * p.sub_len : 0;
        k_hi = p.sub_len > 0 ? min(k_lo + p.sub_len, Lb) : Lb;
        if (CAUSAL) k_hi = min(k_hi, q0 + TQ);  // no query of this tile sees a later key
    }
    // Causal history pass: token i sees the keys j <= i of its subsequence.  A block of 32 keys is
    // masked per lane (the lane's queries are q0 + wave*WQ + 32 qb + lane%32) when it reaches up to
    // or beyond the wave's first query; blocks wholly beyond a wave's queries contribute zeros.
    int lim[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) lim[qb] = q0 + wave * WQ + qb * 32 + l32 + 1;
    const int q_wave_lo = q0 + wave * WQ;
    auto causal = [&](f32x16 (&S)[QB], int blk_lo) __attribute__((always_inline)) {
        if (CAUSAL && blk_lo + kBlockKeys > q_wave_lo) mask_causal(S, hf, blk_lo, lim);
    };
    const int n_tiles = (k_hi - k_lo + kTileKeys - 1) / kTileKeys;
    const uint8_t *kv = p.layer_base + ((size_t)t0 * p.H + (size_t)h * Lpad) * (kDHead * 4) +
                        (size_t)(k_lo / kBlockKeys) * kBlockBytes;

    // K/V tiles go HBM -> LDS directly (no register staging): every wave copies NPRE slabs of
    // 1 KiB (64 lanes x 16 B) per tile; the LDS image equals the HBM image.
    // tile t into the ring stage at byte offset `stage` (= (t % kStages) * kTileBytes)
    RawTiles raw;
    if constexpr (RAW) raw = raw_tiles(p, (int64_t)t0 + k_lo, h, tid);
    auto issue_tile_at = [&](int t, int stage) __attribute__((always_inline)) {
        if constexpr (RAW) return raw_issue(raw, t, (lds_u8 *)lds + stage + wave * 1024, (lds_u8 *)lds + stage + 8192 + wave * 1024);
        glb_u8 *src = (glb_u8 *)(kv + (size_t)t * kTileBytes + (size_t)tid * 16);
        lds_u8 *dst = (lds_u8 *)lds + stage + wave * 1024;
#pragma unroll
        for (int i = 0; i < NPRE; ++i)
            __builtin_amdgcn_global_load_lds(src + i * NT * 16, dst + i * NT * 16, 16, 0, 0);
    };
    auto issue_tile = [&](int t) __attribute__((always_inline)) { issue_tile_at(t, (t % kStages) * kTileBytes); };
    // fragments of block blk of the tile in the ring stage at byte offset `so`
    auto tile_k = [&](int so, int blk) __attribute__((always_inline)) {
        if constexpr (RAW) return raw_k(raw, lds + so, blk);
        else return load_k(lds + so + blk * kBlockBytes, lane);
    };
    auto tile_v = [&](int so, int blk) __attribute__((always_inline)) {
        if constexpr (RAW) return raw_v(raw, lds + so + 8192, blk);
        else return load_v(lds + so + blk * kBlockBytes, lane);
    };
    auto clear_tail = [&](int so, int tile_lo) __attribute__((always_inline)) {
        if constexpr (RAW)
            if (tile_lo + kTileKeys > k_hi) raw_clear(lds + so + 8192, k_hi - tile_lo, tid);
    };
    QState<QB> st;
    // FAST start: the raw query rows stay in st.qf and the row scale in st.c until the first block's
    // logits have shown which form of the pass the wave takes; empty state (the candidate's own
    // key/value joins later, from the landing buffer).
    auto init_fast = [&](const float (&c)[QB]) __attribute__((always_inline)) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            st.c[qb] = c[qb];
            st.l[qb] = 0.f;
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) st.O[db][qb][r] = 0.f;
        }
    };
    // SAFE start (rare): everything is fetched again, straight from global memory, so that nothing
    // of it has to stay in registers across the FAST pass (the empty asm keeps the compiler from
    // reusing the FAST pass's row addresses).  q unscaled; the own key/value is the first member
    // of the softmax and its logit the first reference.
    auto init_safe = [&]() __attribute__((always_inline)) {
        int l32s = l32, hfs = hf;
        asm volatile("" : "+v"(l32s), "+v"(hfs));
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const int64_t row = row0 + min(wave * WQ + qb * 32 + l32s, nq - 1);
            const int sc = min(max(p.scen[row], 0), p.n_scen - 1);
            const int bhv = min(max(p.beh[row], 0), p.n_beh - 1);
            st.c[qb] = p.scale_log2e / p.tau[sc * p.n_beh + bhv];
            const __bf16 *qp = p.q + row * p.ld_q + h * kDHead + 8 * hfs;
            float dot = 0.f;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                st.qf[qb][s] = *(const bf16x8 *)(qp + 16 * s);
                if (SUMI) {
                    const bf16x8 kk = *(const bf16x8 *)(p.k_self + row * p.ld_kv + h * kDHead + 8 * hfs + 16 * s);
#pragma unroll
                    for (int e = 0; e < 8; ++e) dot += (float)st.qf[qb][s][e] * (float)kk[e];
                }
            }
            // SUMI: the own logit (both halves add the same two numbers).  History pass: no member
            // of the row is known yet; a reference far below any logit makes the first block's
            // maximum the reference (0 would leave rows whose logits are all very negative with an
            // empty sum).  Every row sees a key of its first block, so the reference is finite
            // before the first exponential.
            st.m_ref[qb] = SUMI ? dot + xhalf(dot) : kSafeNoRef;
            st.l[qb] = (SUMI && hfs == 0) ? 1.f : 0.f;
            if (SUMI) {
                const __bf16 *vp = p.v_self + row * p.ld_kv + h * kDHead + 4 * hfs;
#pragma unroll
                for (int db = 0; db < 2; ++db)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const bf16x4 vv = *(const bf16x4 *)(vp + 32 * db + 8 * g);
#pragma unroll
                        for (int e = 0; e < 4; ++e) st.O[db][qb][4 * g + e] = (float)vv[e];
                    }
            } else {
#pragma unroll
                for (int db = 0; db < 2; ++db)
#pragma unroll
                    for (int r = 0; r < 16; ++r) st.O[db][qb][r] = 0.f;
            }
        }
    };
    auto prologue = [&]() __attribute__((always_inline)) {
        // tiles 0 .. kStages-2 in flight (SAFE pass)
        for (int t = 0; t < kStages - 1 && t < n_tiles; ++t) issue_tile(t);
    };

    // ---- FAST pass, software pipelined over 32-key blocks -----------------------------------
    // Start-up order = what the first MFMA needs first: tile 0, the query rows, then the tiles
    // that are only needed a little later (loads return in order).
    // ... and the row ids and the temperature table, whose values are needed together with the
    // query rows.  Both are staged in the last ring buffer (first refilled during tile 0, i.e.
    // after the lookups), so the per-row lookup is not a second dependent trip to memory.  They too arrive by
    // global_load_lds: before it uses a value that it loads into a register while such copies are in flight, or stores to LDS,
    // the compiler waits until every copy has landed, tile 1 included (32 users x 128 candidates against 512
    // behaviours 11.5 us that way, 11.0 this way).
    constexpr int kIdsBytes = 512;  // per wave: 64 scenario ids, 64 behaviour ids
    constexpr int kTauLds = (kTileBytes - NW * kIdsBytes) / 4;
    static_assert(kTauLds % NT == 0, "the last copy of the table stays clear of the end of the buffer");
    uint8_t *ids_lds = lds + (kStages - 1) * kTileBytes + wave * kIdsBytes;
    float *tau_lds = (float *)(lds + (kStages - 1) * kTileBytes + NW * kIdsBytes);
    const int n_tau = p.n_scen * p.n_beh;
    const bool tau_in_lds = n_tau <= kTauLds;
    // Query rows land in the landing buffer behind the ring: whole 128-byte rows, copied
    // HBM -> LDS by the wave that owns them (8 lanes per row, so every request is a full line),
    // 16-byte chunks XOR-swizzled by the row number so that the fragment reads below are
    // conflict-free.  A wave only ever touches its own slice of that buffer.
    uint8_t *rows_lds = lds + kStages * kTileBytes + wave * (WQ * 128);
    auto issue_rows = [&](const __bf16 *base, int64_t ld) __attribute__((always_inline)) {
        // wave-uniform base (the tile's first row) in scalar registers + a 32-bit offset per lane (at most
        // TQ - 1 rows): half the address registers of 64-bit lane addresses
        const uint8_t *sb = uniform_ptr((const uint8_t *)(base + row0 * ld + h * kDHead));
#pragma unroll
        for (int i = 0; i < WQ / 8; ++i) {
            const int pos = i * 64 + lane, r = pos >> 3, c = (pos & 7) ^ (r & 7);
            const uint32_t off = ((uint32_t)min(wave * WQ + r, nq - 1) * (uint32_t)ld + (uint32_t)c * 8u) * 2u;
            __builtin_amdgcn_global_load_lds((glb_u8 *)sb + off, (lds_u8 *)rows_lds + i * 1024, 16, 0, 0);
        }
    };
    auto load_q_lds = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int r = qb * 32 + l32, c = (2 * s + hf) ^ (r & 7);
                st.qf[qb][s] = *(const bf16x8 *)(rows_lds + r * 128 + c * 16);
            }
    };
    // FAST, SUMI: the candidate's own key/value.  Their rows travel through the same landing
    // buffer while the history loop runs (keys first, values once the keys are consumed), so no
    // wave ever waits for them: weight w = exp2(<q', k_own>), l += w (behind the third block of 32 keys; behind the last
    // one against at most 128 keys), then O += w * v_own (behind the seventh; behind the last against at most 256).
    float w_own[QB];
    bool fold = false;  // the wave runs the pass with the scale folded into a bf16 query (decided below)
    // RAW: the cache blocks of the wave's rows, zeros where a slot has no row
    auto own_block = [&](int qb) __attribute__((always_inline)) {
        return const_cast<uint8_t *>(p.layer_base) + ((size_t)t0 * p.H + (size_t)h * Lpad) * (kDHead * 4) +
               (size_t)((q0 + wave * WQ) / kBlockKeys + qb) * kBlockBytes;
    };
    auto own_k = [&]() __attribute__((always_inline)) {
        if constexpr (RAW) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
                if (q0 + wave * WQ + qb * 32 < Lpad) own_block_k(own_block(qb), rows_lds + qb * 4096, nq - wave * WQ - qb * 32, lane);
            return;
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const int r = qb * 32 + l32;
            float dot = 0.f;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const bf16x8 kk = *(const bf16x8 *)(rows_lds + r * 128 + (((2 * s + hf) ^ (r & 7)) * 16));
                // read q' back out of the packed operand registers (the empty asm hides where
                // they came from: otherwise the unpacked halves stay live across the whole loop)
                u32x4 qv = __builtin_bit_cast(u32x4, st.qf[qb][s]);
                asm volatile("" : "+v"(qv));
                const bf16x8 qq = __builtin_bit_cast(bf16x8, qv);
#pragma unroll
                for (int e = 0; e < 8; ++e) dot += (float)qq[e] * (float)kk[e];
            }
            w_own[qb] = __builtin_amdgcn_exp2f((dot + xhalf(dot)) * (fold ? 1.f : st.c[qb]));
            st.l[qb] += hf == 0 ? w_own[qb] : 0.f;
        }
    };
    auto own_v = [&]() __attribute__((always_inline)) {
        if constexpr (RAW) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
                if (q0 + wave * WQ + qb * 32 < Lpad) own_block_v(own_block(qb), rows_lds + qb * 4096, nq - wave * WQ - qb * 32, lane);
            return;
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const int r = qb * 32 + l32;
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const bf16x4 vv =
                        *(const bf16x4 *)(rows_lds + r * 128 + (((4 * db + g) ^ (r & 7)) * 16) + 8 * hf);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        st.O[db][qb][4 * g + e] = fmaf(w_own[qb], (float)vv[e], st.O[db][qb][4 * g + e]);
                }
        }
    };
    if (n_tiles > 0) issue_tile(0);
    {
        const int64_t row = row0 + min(wave * WQ + lane % WQ, nq - 1);
        __builtin_amdgcn_global_load_lds((glb_u8 *)(p.scen + row), (lds_u8 *)ids_lds, 4, 0, 0);
        __builtin_amdgcn_global_load_lds((glb_u8 *)(p.beh + row), (lds_u8 *)ids_lds + 256, 4, 0, 0);
        if (tau_in_lds)
            for (int i = 0; i < n_tau; i += NT)
                __builtin_amdgcn_global_load_lds((glb_u8 *)(p.tau + min(i + tid, n_tau - 1)), (lds_u8 *)(tau_lds + i + wave * 64), 4, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    issue_rows(p.q, p.ld_q);
    if (n_tiles > 1) issue_tile(1);
    __builtin_amdgcn_sched_barrier(0);
    // tile 0 and the query rows of this wave have landed (only tile 1 may still be in flight);
    // tau_lds is visible to the workgroup after the bare barrier (a fence would also wait for
    // tile 1)
    if (n_tiles > 1)
        wait_tiles<NPRE>(1);
    else
        wait_tiles<NPRE>(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    {
        float c[QB];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const int *ids = (const int *)ids_lds + qb * 32 + l32;
            const int sc = min(max(ids[0], 0), p.n_scen - 1), bhv = min(max(ids[64], 0), p.n_beh - 1), at = sc * p.n_beh + bhv;
            if (tau_in_lds) {
                c[qb] = tau_lds[at];
            } else {
                c[qb] = p.tau[at];
                asm volatile("" : "+v"(c[qb]));  // (waited for here, not where the two ways meet)
            }
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) c[qb] = p.scale_log2e / c[qb];
        load_q_lds();
        init_fast(c);
    }
    if (n_tiles > 0) {
        f32x16 S0[QB], S1[QB];
        bf16x8 P[QB][2];
        // every wave has looked up its temperatures in the table staged in the last ring stage,
        // which the first refill (tile 2) overwrites
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        {
            const KFrags k0 = tile_k(0, 0);
            qk_block(st, k0, S0);
            // Which form of the FAST pass?  Folding the row scale c = qk_scale*log2(e)/tau into the bf16
            // query saves a multiplication per logit but rounds q*c to 8 bits, an error of 2^-9 of every
            // logit: harmless while the exponents stay small.  The first block's exponents s*c tell:
            // their root mean square estimates the spread of the row's exponents, and with it the size of
            // the denominator (log2 of it ~ log2(keys) + 0.35 spread^2 for bell-shaped logits).  Below
            // kPilotSpread for every row of the wave -> fold; otherwise the queries stay exact and every
            // logit is multiplied by c in fp32.  A wrong guess is caught by the window on the denominators.
            // (Waves decide on their own: both forms read the same tiles and pass the same barriers.)
            bool big = k_hi - k_lo < kFoldMinKeys;  // (a short history: too few keys to average the folded form's error over)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                float ss = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r) ss = fmaf(S0[qb][r], S0[qb][r], ss);
                ss += xhalf(ss);  // the 32 keys of the block
                big |= !(ss * st.c[qb] * st.c[qb] < kBlockKeys * kPilotSpread * kPilotSpread);
            }
            // Only the candidate pass folds, and only against a history of some length: its rows then have
            // many comparable keys to average the per-logit error over.  History rows
            // see one subsequence (a few keys only under the causal flag) and can be sharply peaked, where
            // the folded form's error shows in the output: they always take the exact form.
            fold = SUMI && __builtin_amdgcn_ballot_w64(big) == 0;
            if (fold) {
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
                    for (int sx = 0; sx < 4; ++sx) {
                        const bf16x8 qq = st.qf[qb][sx];
#pragma unroll
                        for (int e = 0; e < 8; ++e) st.qf[qb][sx][e] = (__bf16)((float)qq[e] * st.c[qb]);
                    }
#pragma unroll
                    for (int r = 0; r < 16; ++r) S0[qb][r] *= st.c[qb];  // the first block's logits, formed already
                }
            }
            causal(S0, k_lo);
        }
        auto run = [&](auto fold_tag) __attribute__((always_inline)) {
        constexpr bool FOLD = decltype(fold_tag)::value;
        // p = exp2(t): t straight from the MFMA (FOLD), or s * c in fp32
        auto soft = [&](const f32x16 (&S)[QB]) __attribute__((always_inline)) {
            if constexpr (FOLD) {
                softmax_fast(st, S, P);
            } else {
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) st.l[qb] += exp_pack<true>(S[qb], st.c[qb], 0.f, P[qb]);
            }
        };
        // One step = every tile but the last: 64 unmasked keys.  EV numbers the tile that becomes
        // readable in the middle of the step when something rides along with its refill or is
        // due afterwards (the own rows of a candidate tile); 0 = plain step.  The steps with
        // events are peeled off the loop: inside it they would make the compiler shuffle the
        // accumulators around the branches.
        // The ring stages of tiles t, t + 1 and t + 2 come in as byte offsets that the loop carries
        // along: derived from t % kStages inside the loop, every fragment address took two vector
        // additions and its own address register instead of an immediate.
        auto tile_step = [&](int t, int so_cur, int so_nxt, int so_fill, auto ev_tag) __attribute__((always_inline)) {
            constexpr int EV = decltype(ev_tag)::value;
            {   // block 0 of tile t: its logits are in S0; start block 1's logits
                const KFrags k1 = tile_k(so_cur, 1);
                VFrags v0;
                if (!RAW) v0 = tile_v(so_cur, 0);
                __builtin_amdgcn_sched_barrier(0);
                qk_block(st, k1, S1);
                if (RAW) v0 = tile_v(so_cur, 0);
                causal(S1, k_lo + t * kTileKeys + kBlockKeys);
                soft(S0);
                pv_block(st, v0, P);
            }
            // tile t+1 becomes readable (kStages == 3: no later tile is in flight, the wait
            // drains every copy, own rows included); the own rows ride along with the refill
            wait_tiles<NPRE>(0);
            __builtin_amdgcn_s_barrier();
            // the landing slice is overwritten: this wave's earlier reads of it must have returned
            if (OWN && (EV == 1 || EV == 3)) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (OWN && EV == 1) issue_rows(p.k_self, p.ld_kv);
            if (OWN && EV == 3) issue_rows(p.v_self, p.ld_kv);
            if (t + 2 < n_tiles) issue_tile_at(t + 2, so_fill);
            if (OWN && EV == 2) own_k();
            if (OWN && EV == 4) own_v();
            {   // block 1 of tile t; start block 0 of tile t+1
                const KFrags k0 = tile_k(so_nxt, 0);
                VFrags v1;
                if (!RAW) v1 = tile_v(so_cur, 1);
                __builtin_amdgcn_sched_barrier(0);
                qk_block(st, k0, S0);
                if (RAW) v1 = tile_v(so_cur, 1);
                causal(S0, k_lo + (t + 1) * kTileKeys);
                soft(S1);
                pv_block(st, v1, P);
            }
        };
        static_assert(kStages == 3, "stage offsets below are written out for a ring of three");
        constexpr int T1 = kTileBytes, T2 = 2 * kTileBytes;
        if (n_tiles > 1) {
            tile_step(0, 0, T1, T2, std::integral_constant<int, 1>{});
            if (n_tiles > 2) {
                tile_step(1, T1, T2, 0, std::integral_constant<int, 2>{});
                if (n_tiles > 3) {
                    tile_step(2, T2, 0, T1, std::integral_constant<int, 3>{});
                    if (n_tiles > 4) {
                        tile_step(3, 0, T1, T2, std::integral_constant<int, 4>{});
                        int so_cur = T1, so_nxt = T2, so_fill = 0;
                        for (int t = 4; t + 1 < n_tiles; ++t) {
                            tile_step(t, so_cur, so_nxt, so_fill, std::integral_constant<int, 0>{});
                            const int so = so_cur;
                            so_cur = so_nxt, so_nxt = so_fill, so_fill = so;
                        }
                    }
                }
            }
        }
        {   // last tile: 1..64 keys, S0 holds its first block
            const int t = n_tiles - 1;
            const int so_cur = (t % kStages) * kTileBytes;
            const int tile_lo = k_lo + t * kTileKeys;
            clear_tail(so_cur, tile_lo);
            const bool two = tile_lo + kBlockKeys < k_hi;
            if (two) {
                const KFrags k1 = tile_k(so_cur, 1);
                qk_block(st, k1, S1);
                causal(S1, tile_lo + kBlockKeys);
            }
            if (tile_lo + kBlockKeys > k_hi) mask_block(S0, hf, tile_lo, k_hi);
            {
                const VFrags v0 = tile_v(so_cur, 0);
                soft(S0);
                pv_block(st, v0, P);
            }
            if (two) {
                if (tile_lo + kTileKeys > k_hi) mask_block(S1, hf, tile_lo + kBlockKeys, k_hi);
                const VFrags v1 = tile_v(so_cur, 1);
                soft(S1);
                pv_block(st, v1, P);
            }
        }
        };
        if (__builtin_expect(fold, 1))
            run(std::true_type{});
        else
            run(std::false_type{});
    }

    // lane % 32 again, opaquely: otherwise the compiler carries the old copy across the loop, in
    // scratch memory (where the 256-query scoring kernel already keeps 12 registers)
    asm volatile("v_and_b32 %0, 31, %1" : "=v"(l32) : "v"(tid));
    if (OWN) {  // whatever part of the own-row schedule a short history left undone
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (n_tiles < 2) issue_rows(p.k_self, p.ld_kv);
        if (n_tiles < 3) {
            wait_tiles<NPRE>(0);
            own_k();
        }
        if (n_tiles < 4) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            issue_rows(p.v_self, p.ld_kv);
        }
        if (n_tiles < 5) {
            wait_tiles<NPRE>(0);
            own_v();
        }
    }

    // ---- SAFE pass (rare): whole workgroup redoes its rows with a running maximum -----------
    float lt[QB];
    bool bad = false;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        lt[qb] = st.l[qb] + xhalf(st.l[qb]);
        bad |= fold ? !(lt[qb] > kDenomLo && lt[qb] < kDenomHi) : !(lt[qb] > kDenomLoExact && lt[qb] < kDenomHiExact);
    }
    // Workgroup-wide OR of `bad` through the (idle) landing buffer: one flag per wave in its own
    // slice, one barrier; the barrier also orders the reuse of the LDS ring below.
    // (Redoing 32 queries at a time is faster, but leaves the rest of the tile in the folded form: 2.3e-3 -> 2.8e-3 off the
    // results in 64 bits.  With the keys split over the waves, a causal row may see none in some wave's share.)
    int *flag_lds = (int *)(lds + kStages * kTileBytes);
    // (the ballot is taken by the whole wave: inside the branch it would see lane 0 only)
    const int wave_bad = __builtin_amdgcn_ballot_w64(bad) != 0;
    if (lane == 0) flag_lds[wave * (WQ * 32)] = wave_bad;
    __syncthreads();
    int any_bad = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) any_bad |= flag_lds[w * (WQ * 32)];
    if (any_bad) {
        prologue();
        init_safe();
        for (int t = 0; t < n_tiles; ++t) {
            wait_tiles<NPRE>(min(t + kStages - 1, n_tiles) - (t + 1));
            __builtin_amdgcn_s_barrier();
            if (t + kStages - 1 < n_tiles) issue_tile(t + kStages - 1);
            const int so_cur = (t % kStages) * kTileBytes;
            const int tile_lo = k_lo + t * kTileKeys;
            clear_tail(so_cur, tile_lo);
#pragma unroll
            for (int blk = 0; blk < 2; ++blk) {
                const int blk_lo = tile_lo + blk * kBlockKeys;
                if (blk_lo < k_hi) {
                    f32x16 S[QB];
                    bf16x8 P[QB][2];
                    const KFrags kf = tile_k(so_cur, blk);
                    qk_block(st, kf, S);
                    if (blk_lo + kBlockKeys > k_hi) mask_block(S, hf, blk_lo, k_hi);
                    causal(S, blk_lo);
                    softmax_safe(st, S, P);
                    const VFrags vf = tile_v(so_cur, blk);
                    pv_block(st, vf, P);
                }
            }
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) lt[qb] = st.l[qb] + xhalf(st.l[qb]);
    }

    // ---- normalise and store ----------------------------------------------------------------
    // A lane holds O^T[32db + 8g + 4hf + 0..3][query]: 8-byte pieces of 32 different rows.  Each
    // wave turns its 32 x 64 block around in its own corner of the (now idle) LDS ring so that
    // the global stores are whole 128-byte rows, 16 bytes per lane.
    if (any_bad) __syncthreads();  // SAFE pass: every wave is done reading K/V tiles
    constexpr int kRowPitch = 144;  // 128 B of a row + 16 B pad, keeps 16-byte alignment
    uint8_t *tr = lds + wave * (32 * kRowPitch);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const float inv = 1.f / lt[qb];
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                bf16x4 ov;
#pragma unroll
                for (int e = 0; e < 4; ++e) ov[e] = (__bf16)(st.O[db][qb][4 * g + e] * inv);
                *(bf16x4 *)(tr + l32 * kRowPitch + (32 * db + 8 * g + 4 * hf) * 2) = ov;
            }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int id = i * 64 + lane, r = id >> 3, cc = id & 7;
            const int wq = wave * WQ + qb * 32 + r;
            uint4 val = *(const uint4 *)(tr + r * kRowPitch + cc * 16);
            __bf16 *op = p.o + (row0 + wq) * p.ld_o + h * kDHead + cc * 8;
            if (wq < nq) {
                __builtin_nontemporal_store(__builtin_bit_cast(u32x4, val), (u32x4 *)op);
            } else if (!SUMI && q0 + wq < Lpad) {
                *(uint4 *)op = uint4{0, 0, 0, 0};
            }
        }
    }
}

template <int NW, int QB, bool SUMI, bool CAUSAL = false, bool RAW = false>
hipError_t launch(const AttnArgs &a, hipStream_t s)
{
    constexpr int TQ = NW * 32 * QB;
    const int n_qtiles = (a.max_rows_per_user + TQ - 1) / TQ;
    const int groups = (a.cache.B * a.H + 7) / 8;
    const int64_t grid = (int64_t)8 * n_qtiles * groups;
    if (grid <= 0 || grid > 0x7fffffff) return hipErrorInvalidValue;
    const KParams p = make_params(a, n_qtiles);
    hipLaunchKernelGGL((attn_bf16_kernel<NW, QB, SUMI, CAUSAL, RAW>), dim3((unsigned)grid), dim3(NW * 64), 0, s, p);
    return hipGetLastError();
}

// Query-tile shape: 4 waves x QB blocks of 32 queries per workgroup.  QB = 2 (256 queries) re-reads
// a head's K/V from L2 half as often and reuses every LDS fragment for two MFMAs; QB = 1 (128
// queries) keeps two waves per SIMD busy when a head has few queries.  Scoring takes 128 only for users of up to 128
// candidates: where a row leaves the softmax's window all rows of its tile are redone with unrounded queries, so
// smaller tiles would hold more rows in the folded form.  (They pad less and deal the work out in smaller pieces; us, 256 / 128
// queries, 8 heads: 64 x 257 75.7 / 68.3, 40 x 300 against 600 40.5 / 33.0, 64 x 512 76.0 / 83.3.)
// The history pass: a query tile lies inside one subsequence (sub_len is 0 or a multiple of 128); 256 queries where that allows them,
// they are well filled, and there are many of them or just enough for the 512 workgroups that the chip holds at a time: with a few
// more a nearly empty second turn costs more than the tiles' economy gives, and under the causal flag half-empty tiles balance
// badly.  Us, 256 / 128 queries, rows and caches that no earlier call left in the last-level cache, 8 heads:
//   from the cache, writer's launch included: 12 users x 1000 in subsequences of 512 (384 workgroups of 256) 33.0 / 31.6, 16 (512) 38.4 / 39.9,
//     18 (576) 46.4 / 45.3, 32 (1024) 67.1 / 71.5; in one subsequence 16 52.8 / 57.3, 18 68.7 / 65.7; causal, 512 each, 16 38.7 / 38.5, 18
//     48.5 / 44.6, 32 69.1 / 69.7; of 256 to 1024 behaviours 16 (512 launched) 6 % for 256, 18 (576) 8 % for 128; poorly filled: 32 x 600 50.2 / 47.4, 36 x 300 34.7 / 31.0
//   from rows: 12 x 1000 in 512 29.8 / 28.5, 16 32.0 / 35.9, 18 42.9 / 42.5, 32 60.0 / 65.3; causal 16 33.0 / 36.9 (but 16 of 256 to 1024
//     8 % the other way), 18 45.8 / 43.8; 32 x 600 46.5 / 42.7, 36 x 300 30.6 / 27.4
bool hist_wide_tiles(const AttnArgs &a)
{
    if (a.sub_len % 256 != 0) return false;
    const int64_t r1 = hist_tile_rows(a, 128), r2 = hist_tile_rows(a, 256), tiles = r2 / 256 * a.H;
    const int64_t launched = (int64_t)a.cache.B * a.H * ((a.max_rows_per_user + 255) / 256);  // those beyond a user's end, too
    return 6 * r1 > 5 * r2 && (tiles > 640 || (!a.causal && tiles > 384 && launched <= 512));
}

// Launches of few queries go to attn_wave_bf16.hip: at most one wave of 32 per SIMD (1024), fewer where the tiles are well
// filled or the walk is too short to hide a launch's ends.  Us per call there / here, 8 heads.
//   candidates, more than 128 or up to 64 a user: 200 of 8 against 1000 (448 waves) 14.3 / 20.0, 256 of 16 (1024)
//     against 1024 17.8 / 20.9, against 256 9.0 / 9.0, against 128 9.0 / 8.0; 64 of 64 (1024) against 512 14.8 / 15.8,
//     against 128 9.2 / 7.6; 10 of 66 (528) against 193, the history pass with it, 40.7 / 44.9; 256 of 32 (2048) 31 / 27
//   65 to 128 (128-query tiles, full ones): 128 of 8 (256) against 1024 11.5 / 12.8, of 16 (512) 13.4 / 14.0, against 512
//     9.5 / 9.3, 96 of 32, 4 heads (384) against 512 9.4 / 9.0, 128 of 32 (1024) against 1024 18.0 / 16.5
//   history pass: one user's 4096 (1024) 48 / 73, 16 of 256 13.7 / 14.7, 8 of 1024 (2048) 24.5 / 22.5; subsequences of 384
//     (128-query tiles) of 2 x 1024 (512) 11.3 / 11.3, of 4 x 1024 (1024) 15.1 / 14.3
bool few_queries(const AttnArgs &a, bool sumi)
{
    const int64_t waves = (int64_t)a.cache.B * a.H * ((a.max_rows_per_user + 31) / 32);
    if (!sumi) return waves <= (a.sub_len % 256 == 0 || a.sub_len == 128 ? 1024 : 512);
    if (a.max_rows_per_user > 64 && a.max_rows_per_user <= 128) return waves <= (a.max_hist_len > 640 ? 512 : 256);
    return waves <= (a.max_hist_len >= 256 || a.max_rows_per_user <= 32 ? 1024 : 512);
}

// Launches of at most a workgroup per CU of an XCD (the tiles of a head are on one) share a tile's keys out among waves
// (attn_split_bf16.hip) but for the shortest walks.  Us there / with a wave per 32 queries, 8 heads: candidates of one user against 1000,
// 10 to 256 of them 7.8 to 8.4 / 11.3 to 11.9, against 4000 18.2 / 31.4, against 256 5.9 / 6.8, against 64 5.8 / 5.8; the most workgroups (256):
// 128 of 8 against 1024 9.6 / 12.8, 10 of 32 against 1000 13.1 / 14.5; one more per CU: 256 of 8 against 512 (512) 12.3 / 9.6, 128
// of 10 against 1000 (320) 17.3 / 13.3; two heads of one user's 4000 in one subsequence (125 on each of two XCDs) 72 / 45.
bool split_keys(const AttnArgs &a, bool sumi)
{
    const int64_t per_xcd = ((int64_t)a.cache.B * a.H + 7) / 8 * ((a.max_rows_per_user + 31) / 32);
    const int walk = !sumi && a.sub_len > 0 ? std::min(a.sub_len, a.max_hist_len) : a.max_hist_len;
    return per_xcd <= 32 && walk >= 128;
}
}  // namespace

// From rows, one launch, or the cache writer and a launch that reads the cache: two launches only where a wave per 32 queries
// (attn_wave_bf16.hip) has a long walk to make, which tiles make more slowly, or where the walk is shared out among waves (split_keys).  Us from
// rows / as two, 8 heads: 4 users x 1024 behaviours in one subsequence 16.8 / 22.3, in two 11.2 / 16.9, one user's 2000 in one 28.1 / 23.9, 4096 in
// one 53.5 / 47.9; shared out: one user's 1000 in one 16.5 / 11.4, causal 16.7 / 10.8, in two 10.6 / 10.1, 2 x 500 in one 10.4 / 9.5, one user's
// 300 8.0 / 8.7, 1000 in four 7.7 / 8.5; where two would be the tiled kernel: 16 x up to 4096 in subsequences of 512 77.8 / 93.1, 64 x 1024 in one 167.6 / 187.9, causal 64 x 1000 in two 113 / 124.
bool attn_hist_rows_bf16_takes(const AttnArgs &a)
{
    if (a.bias.pos_table) return attn_hist_rows_bias_bf16_takes(a);
    const int walk = a.sub_len > 0 ? std::min(a.sub_len, a.max_hist_len) : a.max_hist_len;
    if (split_keys(a, false)) return walk <= 384;
    return walk <= 1024 || !few_queries(a, false);
}

hipError_t launch_attn_hist_rows_bf16(const AttnArgs &a, hipStream_t s)
{
    if (a.bias.pos_table) return launch_attn_hist_rows_bias_bf16(a, s);
    const bool wide = hist_wide_tiles(a);
    if (a.causal) return wide ? launch<4, 2, false, true, true>(a, s) : launch<4, 1, false, true, true>(a, s);
    return wide ? launch<4, 2, false, false, true>(a, s) : launch<4, 1, false, false, true>(a, s);
}

hipError_t launch_attn_sumi_bf16(const AttnArgs &a, hipStream_t s)
{
    if (a.bias.pos_table) return launch_attn_bias_bf16(a, true, s);
    if (split_keys(a, true)) return launch_attn_split_bf16(a, true, s);
    if (few_queries(a, true)) return launch_attn_wave_bf16(a, true, s);
    return a.max_rows_per_user > 128 ? launch<4, 2, true>(a, s) : launch<4, 1, true>(a, s);
}

hipError_t launch_attn_hist_bf16(const AttnArgs &a, hipStream_t s)
{
    if (a.bias.pos_table) return launch_attn_bias_bf16(a, false, s);
    if (split_keys(a, false)) return launch_attn_split_bf16(a, false, s);
    if (few_queries(a, false)) return launch_attn_wave_bf16(a, false, s);
    const bool wide = hist_wide_tiles(a);
    if (a.causal) return wide ? launch<4, 2, false, true>(a, s) : launch<4, 1, false, true>(a, s);
    return wide ? launch<4, 2, false>(a, s) : launch<4, 1, false>(a, s);
}

}  // namespace climber
