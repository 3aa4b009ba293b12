// bf16 MFMA attention with the relative attention bias of Eq. (3) of Climber (arXiv 2502.09888) for gfx950:
// R = Q K^T + f_b, divided by the temperature afterwards; candidate pass (SUMI mask of Sec. 3.2) and history
// pass (subsequences of Sec. 3.1.2, also causal).  Formulation, cache layout, LDS ring and softmax as in
// attn_bf16.hip; always the exact-scale form of the softmax (the logits are larger by the bias).
//
// The bias of a (query, key) pair is two table entries chosen by a clipped position distance and a log2 bucket of
// the time distance: about a dozen instructions and two LDS gathers per logit, four times the softmax itself.  But
// buckets are coarse: against a block of 32 keys that lies a clip distance and an octave of time away, all of a
// wave's 32 queries x 32 keys fall into one position and one time bucket.  So every wave classifies the blocks
// first (extremes of the keys' positions and times against the extremes of its queries'), and a
// uniform block costs one pair of gathers per query, its bias joining as the addend of the fused
// multiply-add that scales the logit.  The other blocks -- those around the query's own place and the ones an
// octave boundary falls into -- look up every logit and apply it with the same operations, so that a row's bits do
// not depend on which way its wave took.
#include "attn_common.h"
#include "launch.h"

#include <algorithm>
#include <type_traits>

namespace climber {
namespace {

using namespace attn;

constexpr int kTileKeys = 64, kTileBytes = 2 * kBlockBytes, kStages = 3, NW = 4;

// Tiles of 64 keys in LDS: a ring of three stages of keys, values, positions and time stamps, or (SPLIT) two rings: the keys themselves,
// two stages, as all of a tile have been read when the next one's first block is started; and what is read later, three.  The
// latter takes 8 KiB less, which makes room for a third workgroup per CU, and where there is none it gains nothing: us with one / two, QB = 2, 512
// candidates of 32 users against 4000 162 / 171; QB = 1, tables of 129 + 20 entries, 300 of 64 users 101.5 / 102.6, 128 of 96 69.5 / 68.1, history of
// 64 x 1024 in one, from the cache, 291.0 / 292.6, of 30 x 1000 in four 98.3 / 98.3.  From rows it is always two.
template <bool SPLIT>
struct Ring {
    static constexpr int kKeyStage = SPLIT ? kTileBytes / 2 : 0;                                  // stages of keys begin at 0
    static constexpr int kRest = 2 * kKeyStage, kCoords = SPLIT ? kTileBytes / 2 : kTileBytes;  // those of the rest; coordinates in them
    static constexpr int kStage = kCoords + kTileKeys * 8, kBytes = kRest + kStages * kStage;
};

template <bool RAW, int PER_CU>
constexpr bool two_rings = RAW || PER_CU == 3;

// minimum over the 32 lanes of a half-wave, as a scalar (both halves hold the same 32 values)
template <class F>
__device__ __forceinline__ int half_wave_reduce(int x, F &&f)
{
    auto dpp = [](int v, auto ctrl) { return __builtin_amdgcn_update_dpp(0, v, decltype(ctrl)::value, 0xf, 0xf, false); };
    x = f(x, dpp(x, std::integral_constant<int, 0xB1>{}));   // quad_perm [1,0,3,2]
    x = f(x, dpp(x, std::integral_constant<int, 0x4E>{}));   // quad_perm [2,3,0,1]
    x = f(x, dpp(x, std::integral_constant<int, 0x141>{}));  // row_half_mirror
    x = f(x, dpp(x, std::integral_constant<int, 0x140>{}));  // row_mirror
    return f(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16));
}

// LDS: rings, tables of the head, one flag per wave; at the end, over the first two, a wave's corner for 32 rows of outputs, and of keys
// and values on their way to the cache.
template <bool RAW>
constexpr int kCorner = RAW ? 12288 : 4096;
template <bool SPLIT, bool RAW>
__host__ __device__ constexpr int bias_flags_at(int entries)
{
    const int used = Ring<SPLIT>::kBytes + entries * 4, corners = NW * kCorner<RAW>;
    return used > corners ? used : corners;
}

// IN_LDS: the head's rows of the tables are copied into LDS (else looked up in global memory).
// RAW (history pass): keys and values are rows, and this launch writes them into the cache as well (RawTiles, attn_common.h);
// every wave the blocks of its own rows, which it fetches once more behind its last tile.
// PER_CU: workgroups per CU, which the registers have to leave room for (168 a lane for three).
template <int QB, bool SUMI, bool CAUSAL, bool IN_LDS, bool RAW, int PER_CU>
__global__ __launch_bounds__(NW * 64, PER_CU) void attn_bias_kernel(const KParams p)
{
    static_assert(!(SUMI && CAUSAL), "the causal flag concerns the history pass");
    static_assert(!RAW || (!SUMI && QB == 1), "rows: the history pass");
    constexpr int NT = NW * 64, WQ = 32 * QB, TQ = NW * WQ, NPRE = kTileBytes / 16 / NT;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    constexpr bool SPLIT = two_rings<RAW, PER_CU>;
    using LdsRing = Ring<SPLIT>;
    float *bias_lds = (float *)(lds + LdsRing::kBytes);  // the head's table rows: [n_tau][n_pos], [n_tau][n_time]
    // (behind everything: a wave's corner is in use while others may still read the flags)
    int *flag_lds = (int *)(lds + bias_flags_at<SPLIT, RAW>(IN_LDS ? p.n_scen * p.n_beh * (p.bias.n_pos + p.bias.n_time) : 0));

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;

    // workgroup -> (user, head, query tile), the tiles of a head on one XCD; geometry as in attn_bf16.hip
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
                if (q0 + r < Lpad) *(uint4 *)(p.o + (row0 + r) * p.ld_o + h * kDHead + cc * 8) = uint4{0, 0, 0, 0};
            }
            return;
        }
        k_lo = p.sub_len > 0 ? (q0 / p.sub_len) * p.sub_len : 0;
        k_hi = p.sub_len > 0 ? min(k_lo + p.sub_len, Lb) : Lb;
        if (CAUSAL) k_hi = min(k_hi, q0 + TQ);
    }
    const int n_tiles = (k_hi - k_lo + kTileKeys - 1) / kTileKeys;
    const uint8_t *kv = p.layer_base + ((size_t)t0 * p.H + (size_t)h * Lpad) * (kDHead * 4) +
                        (size_t)(k_lo / kBlockKeys) * kBlockBytes;
    RawTiles raw;
    if constexpr (RAW) raw = raw_tiles(p, (int64_t)t0 + k_lo, h, tid);
    // tile t: its keys to stage t % 2 of theirs (SPLIT; `keys`: byte offset), the rest to the stage of the ring at byte offset `stage`
    auto issue_tile = [&](int t, int keys, int stage) __attribute__((always_inline)) {
        lds_u8 *to = (lds_u8 *)lds + LdsRing::kRest + stage, *to_k = (lds_u8 *)lds + keys + wave * 1024, *to_v = to + wave * 1024;
        if constexpr (RAW) {
            raw_issue(raw, t, to_k, to_v);
        } else {  // a block of the cache is 4 KiB of keys and 4 KiB of values
            glb_u8 *src = (glb_u8 *)(kv + (size_t)t * kTileBytes + (size_t)tid * 16);
            static_assert(NPRE == 4 && NT * 16 == kBlockBytes / 2, "");
            __builtin_amdgcn_global_load_lds(src, SPLIT ? to_k : to_v, 16, 0, 0);
            __builtin_amdgcn_global_load_lds(src + 4096, SPLIT ? to_v : to_v + 4096, 16, 0, 0);
            __builtin_amdgcn_global_load_lds(src + 8192, SPLIT ? to_k + 4096 : to_v + 8192, 16, 0, 0);
            __builtin_amdgcn_global_load_lds(src + 12288, SPLIT ? to_v + 4096 : to_v + 12288, 16, 0, 0);
        }
        if (wave < 2)  // wave 0: positions, wave 1: time stamps of the tile's keys, 4 bytes per lane
            __builtin_amdgcn_global_load_lds((glb_u8 *)((wave ? p.bias.key_ts : p.bias.key_pos) + t0 + k_lo + t * kTileKeys + lane),
                                             to + LdsRing::kCoords + wave * (kTileKeys * 4), 4, 0, 0);
    };
    auto tile_k = [&](int keys, int stage, int blk) __attribute__((always_inline)) {
        if constexpr (RAW) return raw_k(raw, lds + keys, blk);
        else return load_k(SPLIT ? lds + keys + blk * (kBlockBytes / 2) : lds + stage + blk * kBlockBytes, lane);
    };
    auto tile_v = [&](const uint8_t *stage, int blk) __attribute__((always_inline)) {
        if constexpr (RAW) return raw_v(raw, stage, blk);
        else return load_v(SPLIT ? stage + blk * (kBlockBytes / 2) - kBlockBytes / 2 : stage + blk * kBlockBytes, lane);
    };
    auto clear_tail = [&](uint8_t *stage, int t) __attribute__((always_inline)) {
        if constexpr (RAW)
            if (k_lo + (t + 1) * kTileKeys > k_hi) raw_clear(stage, k_hi - k_lo - t * kTileKeys, tid);
    };
    auto wait_copies = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
    if (n_tiles > 0) issue_tile(0, 0, 0);

    // the lane's queries: rows, scales, bias coordinates
    QState<QB> st;
    int b_pos[QB], tau_idx[QB];
    uint32_t b_ts[QB];          // time stamp, sign bit flipped
    // (recomputed where it is needed: held across the loop, the rows would cost registers the loop has not got)
    auto row_of = [&](int qb) __attribute__((always_inline)) {
        int l = l32;
        asm volatile("" : "+v"(l));
        return row0 + min(wave * WQ + qb * 32 + l, nq - 1);
    };
    const int n_groups = p.n_scen * p.n_beh, n_pos = p.bias.n_pos, n_time = p.bias.n_time, half = (n_pos - 1) >> 1;
    // (requests of everything the start needs go out before the first of them is waited for)
    int scen[QB], beh[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int64_t row = row_of(qb);
        scen[qb] = p.scen[row];
        beh[qb] = p.beh[row];
        b_pos[qb] = p.bias.q_pos[row];
        b_ts[qb] = bias_time_key(p.bias.q_ts[row]);
    }
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const __bf16 *qp = p.q + row_of(qb) * p.ld_q + h * kDHead + 8 * hf;
#pragma unroll
        for (int s = 0; s < 4; ++s) st.qf[qb][s] = *(const bf16x8 *)(qp + 16 * s);
    }
    if constexpr (IN_LDS) {  // eight table rows per wave and turn, a lane per entry; time rows reversed (see entry)
        constexpr int kTurn = 8;
        const bool short_rows = n_pos <= 64 && n_time <= 64;
        for (int g0 = wave * kTurn; g0 < n_groups; g0 += NW * kTurn) {
            if (short_rows) {
                float pr[kTurn], tr[kTurn];
#pragma unroll
                for (int k = 0; k < kTurn; ++k) {
                    const int row = min(g0 + k, n_groups - 1) * p.bias_H + h;
                    pr[k] = p.bias.pos_table[row * n_pos + min(lane, n_pos - 1)];
                    tr[k] = p.bias.time_table[row * n_time + min(lane, n_time - 1)];
                }
#pragma unroll
                for (int k = 0; k < kTurn; ++k) {
                    const int g = min(g0 + k, n_groups - 1);
                    bias_lds[g * n_pos + min(lane, n_pos - 1)] = pr[k];
                    bias_lds[n_groups * n_pos + g * n_time + n_time - 1 - min(lane, n_time - 1)] = tr[k];
                }
            } else {
                for (int g = g0; g < min(g0 + kTurn, n_groups); ++g) {
                    for (int i = lane; i < n_pos; i += 64) bias_lds[g * n_pos + i] = p.bias.pos_table[(g * p.bias_H + h) * n_pos + i];
                    for (int i = lane; i < n_time; i += 64)
                        bias_lds[n_groups * n_pos + g * n_time + n_time - 1 - i] = p.bias.time_table[(g * p.bias_H + h) * n_time + i];
                }
            }
        }
    }
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        tau_idx[qb] = min(max(scen[qb], 0), p.n_scen - 1) * p.n_beh + min(max(beh[qb], 0), p.n_beh - 1);
        st.c[qb] = p.scale_log2e / p.tau[tau_idx[qb]];
        st.l[qb] = 0.f;
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) st.O[db][qb][r] = 0.f;
    }
    if (n_tiles > 1) issue_tile(1, LdsRing::kKeyStage, LdsRing::kStage);

    // Classes of 64 blocks: do a wave's 32 queries of a query block share one position and one time bucket with all
    // keys of the block, and which.  Distances are monotonic in both ends, so the buckets of the extreme pairs decide.
    // Eight lanes per block, four keys each.
    // A class holds the clipped distance above eight bits of time bucket: blocks with a distance that does not fit there
    // (tables of more than 2^23 entries a row) are looked up per logit.
    constexpr int kMixed = 0x7fffffff, kClassPos = 1 << 22;
    int qp_min[QB], qp_max[QB];
    uint32_t qt_min[QB], qt_max[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        qp_min[qb] = half_wave_reduce(b_pos[qb], [](int x, int y) { return min(x, y); });
        qp_max[qb] = half_wave_reduce(b_pos[qb], [](int x, int y) { return max(x, y); });
        qt_min[qb] = half_wave_reduce((int)b_ts[qb], [](int x, int y) { return (int)min((uint32_t)x, (uint32_t)y); });
        qt_max[qb] = half_wave_reduce((int)b_ts[qb], [](int x, int y) { return (int)max((uint32_t)x, (uint32_t)y); });
    }
    // The classes of the wave's blocks, a lane per block, and what the last uniform class came to: neighbouring blocks mostly
    // share it (everything clipped), and then a block costs no trip to LDS.  Scoring 512 of 64 users against 1024 97.9 -> 95.2 us,
    // 128 of 32 28.1 -> 26.8, causal history pass of 20 x 2000 in subsequences of 512 191 -> 169.
    int classes[QB] = {}, last_class[QB];
    float last_add[QB] = {};
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) last_class[qb] = kMixed;
    // position distance clipped to the table; leading zeros of a time distance, from those of the last bucket (the
    // hardware's count of 0 is all ones, which the unsigned clamp takes to 31: bucket 0)
    int half_v = half, z_min_v = max(32 - n_time, 0);
    asm volatile("" : "+v"(half_v), "+v"(z_min_v));  // in vector registers: one scalar operand per instruction is the limit
    auto clip = [&](int d) __attribute__((always_inline)) {
        int x;
        asm("v_med3_i32 %0, %1, %2, %3" : "=v"(x) : "v"(d), "v"(-half_v), "v"(half_v));
        return x;
    };
    auto clip_zeros = [&](uint32_t d) __attribute__((always_inline)) {
        uint32_t z;
        asm("v_ffbh_u32 %0, %1" : "=v"(z) : "v"(d));
        asm("v_med3_u32 %0, %1, %2, 31" : "=v"(z) : "v"(z), "v"(z_min_v));
        return (int)z;
    };
    auto zeros = [&](uint32_t a, uint32_t b) __attribute__((always_inline)) {
        uint32_t d;
        asm("v_sad_u32 %0, %1, %2, 0" : "=v"(d) : "v"(a), "v"(b));  // |a - b|
        return clip_zeros(d);
    };
    auto classes_from = [&](int blk0) __attribute__((always_inline)) {
        auto dpp = [](int v, auto ctrl) { return __builtin_amdgcn_update_dpp(0, v, decltype(ctrl)::value, 0xf, 0xf, false); };
        auto over8 = [&](int x, auto &&f) {  // over the eight lanes of a block
            x = f(x, dpp(x, std::integral_constant<int, 0xB1>{}));
            x = f(x, dpp(x, std::integral_constant<int, 0x4E>{}));
            return f(x, dpp(x, std::integral_constant<int, 0x141>{}));
        };
        constexpr int kTurn = 4;  // 32 blocks per turn
#pragma unroll 1
        for (int g0 = 0; g0 < 8 && k_lo + (blk0 + 8 * g0) * kBlockKeys < k_hi; g0 += kTurn) {
            int4 kp[kTurn], kt[kTurn];
#pragma unroll
            for (int k = 0; k < kTurn; ++k) {
                // (past the range: its last four keys again)
                const int key = min(k_lo + (blk0 + 8 * (g0 + k)) * kBlockKeys + 4 * lane, (k_hi - 1) & ~3);
                kp[k] = *(const int4 *)(p.bias.key_pos + (int64_t)t0 + key);
                kt[k] = *(const int4 *)(p.bias.key_ts + (int64_t)t0 + key);
            }
#pragma unroll
            for (int k = 0; k < kTurn; ++k) {
                const int key = min(k_lo + (blk0 + 8 * (g0 + k)) * kBlockKeys + 4 * lane, (k_hi - 1) & ~3);
                const int pe[4] = {kp[k].x, kp[k].y, kp[k].z, kp[k].w}, te[4] = {kt[k].x, kt[k].y, kt[k].z, kt[k].w};
                int p_min = pe[0], p_max = pe[0], t_min = te[0], t_max = te[0];
#pragma unroll
                for (int e = 1; e < 4; ++e) {
                    const bool in = key + e < k_hi;
                    const int pp = in ? pe[e] : pe[0], tt = in ? te[e] : te[0];
                    p_min = min(p_min, pp), p_max = max(p_max, pp), t_min = min(t_min, tt), t_max = max(t_max, tt);
                }
                auto lesser = [](int x, int y) { return min(x, y); };
                auto greater = [](int x, int y) { return max(x, y); };
                p_min = over8(p_min, lesser), p_max = over8(p_max, greater);
                const uint32_t kt_min = bias_time_key(over8(t_min, lesser)), kt_max = bias_time_key(over8(t_max, greater));
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    const int ip = clip(__builtin_elementwise_sub_sat(qp_min[qb], p_max)), ip2 = clip(__builtin_elementwise_sub_sat(qp_max[qb], p_min));
                    uint32_t d_min = 0, d_max;
                    if (qt_min[qb] >= kt_max) d_min = qt_min[qb] - kt_max, d_max = qt_max[qb] - kt_min;
                    else if (kt_min >= qt_max[qb]) d_min = kt_min - qt_max[qb], d_max = kt_max - qt_min[qb];
                    else d_max = max(qt_max[qb] - kt_min, kt_max - qt_min[qb]);
                    const int it = clip_zeros(d_min);
                    const int cls = ip == ip2 && abs(ip) < kClassPos && it == clip_zeros(d_max) ? (ip << 8) + it : kMixed;
                    const int mine = __builtin_amdgcn_ds_bpermute(32 * (lane & 7), cls);  // (the eight lanes of a block hold it)
                    if (lane >> 3 == g0 + k) classes[qb] = mine;
                }
            }
        }
    };
    if (n_tiles > 0) classes_from(0);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();  // tile 0 and the tables are in LDS

    // Bias of the lane's query for a clipped position distance and the leading zeros (32 - n_time .. 31) of a time
    // distance, in the units of the exponent.  The time rows are kept reversed in LDS: indexed by the leading zeros.
    uint32_t p_row[QB], t_row[QB];  // LDS byte addresses of entry 0 of either
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        p_row[qb] = (uint32_t)(tau_idx[qb] * n_pos + half) * 4u;
        t_row[qb] = (uint32_t)(n_groups * n_pos + tau_idx[qb] * n_time + n_time - 32) * 4u;
    }
    auto entry = [&](int qb, int dp, int z) __attribute__((always_inline)) {
        float x;
        if constexpr (IN_LDS) {
            x = *(const float *)((const uint8_t *)bias_lds + (p_row[qb] + 4 * dp)) + *(const float *)((const uint8_t *)bias_lds + (t_row[qb] + 4 * z));
        } else {
            const int g = tau_idx[qb] * p.bias_H + h;
            x = p.bias.pos_table[g * n_pos + half + dp] + p.bias.time_table[g * n_time + 31 - z];
        }
        return st.c[qb] * p.inv_qk_scale * x;
    };
    // S of a block that is not uniform: t = S * c + bias, looked up per logit (coords: the block's positions in LDS)
    auto lookup_block = [&](int qb, f32x16 (&S)[QB], const uint8_t *coords) __attribute__((always_inline)) {
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
            const int4 kp = *(const int4 *)(coords + 32 * g4 + 16 * hf), kt = *(const int4 *)(coords + kTileKeys * 4 + 32 * g4 + 16 * hf);
            const int kpe[4] = {kp.x, kp.y, kp.z, kp.w}, kte[4] = {kt.x, kt.y, kt.z, kt.w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                S[qb][4 * g4 + e] = fmaf(S[qb][4 * g4 + e], st.c[qb],
                                         entry(qb, clip(__builtin_elementwise_sub_sat(b_pos[qb], kpe[e])), zeros(b_ts[qb], bias_time_key(kte[e]))));
        }
    };
    // Raw products S of block `blk` of the range -> what the exponentials take: t = S * scale + add, the exponent in
    // log2 units with the bias in it.
    auto bias_block = [&](int qb, f32x16 (&S)[QB], int blk, const uint8_t *stage, float &scale, float &add) __attribute__((always_inline)) {
        const int cls = __builtin_amdgcn_readlane(classes[qb], blk & 63);
        if (cls != kMixed) {
            if (cls != last_class[qb]) last_class[qb] = cls, last_add[qb] = entry(qb, cls >> 8, cls & 255);
            scale = st.c[qb];
            add = last_add[qb];
        } else {
            lookup_block(qb, S, stage + LdsRing::kCoords + (blk & 1) * (kBlockKeys * 4));
            scale = 1.f;
            add = 0.f;
        }
    };
    const int whole_hi = CAUSAL ? min(q0 + wave * WQ, k_hi) : k_hi;  // keys below it are visible to every query of the wave
    // A block with keys that not every query sees: the bias is applied here, then those keys are taken out.  (The other
    // way round a table entry that only they select, be it infinite or NaN, would reach the rows.)
    auto mask = [&](int qb, f32x16 (&S)[QB], int blk, float &scale, float &add) __attribute__((always_inline)) {
        const int lo = k_lo + blk * kBlockKeys;
        if (lo + kBlockKeys > whole_hi) {
            const int lim[1] = {CAUSAL ? min(q0 + wave * WQ + qb * 32 + l32 + 1, k_hi) : k_hi};
            f32x16 T[1];
#pragma unroll
            for (int r = 0; r < 16; ++r) T[0][r] = fmaf(S[qb][r], scale, add);
            scale = 1.f, add = 0.f;
            mask_causal(T, hf, lo, lim);
            S[qb] = T[0];
        }
    };

    // FAST pass (exact-scale form), software pipelined over 32-key blocks as in attn_bf16.hip
    if (n_tiles > 0) {
        f32x16 S0[QB], S1[QB];
        bf16x8 P[QB][2];
        // (without the causal flag only the last tile has keys that are not visible)
        auto soft = [&](f32x16 (&S)[QB], int blk, const uint8_t *stage, auto last_tag) __attribute__((always_inline)) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                float scale, add;
                bias_block(qb, S, blk, stage, scale, add);
                if constexpr (CAUSAL || decltype(last_tag)::value) mask(qb, S, blk, scale, add);
                st.l[qb] += exp_pack<true>(S[qb], scale, -add, P[qb]);
            }
        };
        qk_block(st, tile_k(0, 0, 0), S0);
        int ko_cur = 0, so_cur = 0, so_nxt = LdsRing::kStage, so_fill = 2 * LdsRing::kStage;
        for (int t = 0; t + 1 < n_tiles; ++t) {
            const uint8_t *cur = lds + LdsRing::kRest + so_cur;
            if (t > 0 && (t & 31) == 0) classes_from(2 * t);
            {   // block 0 of tile t: its logits are in S0; start block 1's
                const KFrags k1 = tile_k(ko_cur, so_cur, 1);
                VFrags v0;
                if (!RAW) v0 = tile_v(cur, 0);
                __builtin_amdgcn_sched_barrier(0);
                qk_block(st, k1, S1);
                if (RAW) v0 = tile_v(cur, 0);
                soft(S0, 2 * t, cur, std::false_type{});
                pv_block(st, v0, P);
            }
            // Tile t + 1 has landed; nobody reads tile t - 1 any more, nor the keys of tile t, whose reads have returned before the copies
            // behind the barrier overwrite them: raw_v has waited for all of a wave's reads, load_v leaves it to the compiler, whose waits may
            // as well stand behind the barrier.
            if constexpr (RAW) wait_copies();
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            if (t + 2 < n_tiles) issue_tile(t + 2, ko_cur, so_fill);
            ko_cur ^= LdsRing::kKeyStage;
            {   // block 1 of tile t; start block 0 of tile t + 1
                const KFrags k0 = tile_k(ko_cur, so_nxt, 0);
                VFrags v1;
                if (!RAW) v1 = tile_v(cur, 1);
                __builtin_amdgcn_sched_barrier(0);
                qk_block(st, k0, S0);
                if (RAW) v1 = tile_v(cur, 1);
                soft(S1, 2 * t + 1, cur, std::false_type{});
                pv_block(st, v1, P);
            }
            const int so = so_cur;
            so_cur = so_nxt, so_nxt = so_fill, so_fill = so;
        }
        {   // last tile: 1..64 keys
            const int blk = 2 * (n_tiles - 1);
            uint8_t *cur = lds + LdsRing::kRest + so_cur;
            clear_tail(cur, n_tiles - 1);
            if (blk > 0 && (blk & 63) == 0) classes_from(blk);
            const bool two = k_lo + (blk + 1) * kBlockKeys < k_hi;
            if (two) qk_block(st, tile_k(ko_cur, so_cur, 1), S1);
            const VFrags v0 = tile_v(cur, 0);
            soft(S0, blk, cur, std::true_type{});
            pv_block(st, v0, P);
            if (two) {
                const VFrags v1 = tile_v(cur, 1);
                soft(S1, blk + 1, cur, std::true_type{});
                pv_block(st, v1, P);
            }
        }
    }
    // SUMI: the candidate's own key (its exponent, log2 units) and value
    float w_own[QB];
    if (SUMI) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const __bf16 *kp = p.k_self + row_of(qb) * p.ld_kv + h * kDHead + 8 * hf;
            float dot = 0.f;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const bf16x8 kk = *(const bf16x8 *)(kp + 16 * s);
#pragma unroll
                for (int e = 0; e < 8; ++e) dot += (float)st.qf[qb][s][e] * (float)kk[e];
            }
            // zero distance in position and time
            w_own[qb] = fmaf(dot + xhalf(dot), st.c[qb], entry(qb, 0, 31));
        }
    }
    auto own_v = [&](int qb, float w) __attribute__((always_inline)) {  // O += w * v_own
        const __bf16 *vp = p.v_self + row_of(qb) * p.ld_kv + h * kDHead + 4 * hf;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const bf16x4 vv = *(const bf16x4 *)(vp + 8 * i);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                st.O[i >> 2][qb][4 * (i & 3) + e] = fmaf(w, (float)vv[e], st.O[i >> 2][qb][4 * (i & 3) + e]);
        }
    };
    float lt[QB];
    bool bad = false;
    if (SUMI) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float w = __builtin_amdgcn_exp2f(w_own[qb]);
            st.l[qb] += hf == 0 ? w : 0.f;
            own_v(qb, w);
        }
    }
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        lt[qb] = st.l[qb] + xhalf(st.l[qb]);
        bad |= !(lt[qb] > kDenomLoExact && lt[qb] < kDenomHiExact);
    }
    // SAFE pass (rare): the whole workgroup redoes its rows with a running maximum, in log2 units
    const int wave_bad = __builtin_amdgcn_ballot_w64(bad) != 0;
    if (lane == 0) flag_lds[wave] = wave_bad;
    __syncthreads();  // (and every wave is done with the ring)
    int any_bad = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) any_bad |= flag_lds[w];
    if (any_bad) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            st.m_ref[qb] = SUMI ? w_own[qb] : kSafeNoRef;
            st.l[qb] = (SUMI && hf == 0) ? 1.f : 0.f;
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) st.O[db][qb][r] = 0.f;
        }
        if (SUMI) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) own_v(qb, 1.f);
        }
        for (int t = 0; t < n_tiles; ++t) {
            __syncthreads();
            issue_tile(t, 0, 0);
            wait_copies();
            __syncthreads();
            clear_tail(lds + LdsRing::kRest, t);
            for (int k = 0; k < 2; ++k) {
                const int blk = 2 * t + k;
                if (k_lo + blk * kBlockKeys >= k_hi) break;
                if ((blk & 63) == 0) classes_from(blk);
                f32x16 S[QB];
                bf16x8 P[QB][2];
                qk_block(st, tile_k(0, 0, k), S);
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    float scale, add;
                    bias_block(qb, S, blk, lds + LdsRing::kRest, scale, add);
                    mask(qb, S, blk, scale, add);
#pragma unroll
                    for (int r = 0; r < 16; ++r) S[qb][r] = fmaf(S[qb][r], scale, add);
                }
                float c_keep[QB];
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) c_keep[qb] = st.c[qb], st.c[qb] = 1.f;  // (t is scaled already)
                softmax_safe(st, S, P);
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) st.c[qb] = c_keep[qb];
                pv_block(st, tile_v(lds + LdsRing::kRest, k), P);
            }
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) lt[qb] = st.l[qb] + xhalf(st.l[qb]);
        __syncthreads();
    }

    // normalise and store: each wave turns its 32 x 64 blocks around in its corner of the idle ring (chunk c of row r at
    // slot c ^ r % 8); behind it in the corner, RAW: its own key and value rows, on their way into the cache
    uint8_t *tr = lds + wave * kCorner<RAW>;
    if constexpr (RAW) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int pos = i * 64 + lane, r = pos >> 3, c = (pos & 7) ^ (r & 7);
            const int64_t at = (row0 + min(wave * WQ + r, nq - 1)) * p.ld_kv + h * kDHead + c * 8;
            __builtin_amdgcn_global_load_lds((glb_u8 *)(p.k_self + at), (lds_u8 *)tr + 4096 + i * 1024, 16, 0, 0);
            __builtin_amdgcn_global_load_lds((glb_u8 *)(p.v_self + at), (lds_u8 *)tr + 8192 + i * 1024, 16, 0, 0);
        }
    }
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
                *(bf16x4 *)(tr + l32 * 128 + (((4 * db + g) ^ (l32 & 7)) * 16) + 8 * hf) = ov;
            }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int id = i * 64 + lane, r = id >> 3, cc = id & 7;
            const int wq = wave * WQ + qb * 32 + r;
            const u32x4 val = *(const u32x4 *)(tr + r * 128 + ((cc ^ (r & 7)) * 16));
            __bf16 *op = p.o + (row0 + wq) * p.ld_o + h * kDHead + cc * 8;
            if (wq < nq) __builtin_nontemporal_store(val, (u32x4 *)op);
            else if (!SUMI && q0 + wq < Lpad) *(uint4 *)op = uint4{0, 0, 0, 0};
        }
    }
    if constexpr (RAW) {
        wait_copies();
        if (q0 + wave * WQ < Lpad) {
            uint8_t *block = const_cast<uint8_t *>(p.layer_base) + ((size_t)t0 * p.H + (size_t)h * Lpad) * (kDHead * 4) +
                             (size_t)((q0 + wave * WQ) / kBlockKeys) * kBlockBytes;
            own_block_k(block, tr + 4096, nq - wave * WQ, lane);
            own_block_v(block, tr + 8192, nq - wave * WQ, lane);
        }
    }
}

// one head's rows of the tables
int64_t bias_entries(const AttnArgs &a)
{
    return (int64_t)a.n_scen * a.n_beh * ((int64_t)a.bias.n_pos + a.bias.n_time);
}

template <bool SPLIT, bool RAW>
size_t bias_lds_bytes(const AttnArgs &a)
{
    const int64_t entries = bias_entries(a);
    return (size_t)bias_flags_at<SPLIT, RAW>(entries <= kBiasLdsFloats ? (int)entries : 0) + NW * 4;
}

// (LDS is given out by 1280 bytes)
template <bool RAW>
bool three_per_cu(const AttnArgs &a)
{
    constexpr size_t kLds = 160 * 1024, kUnit = 1280;
    return (bias_lds_bytes<true, RAW>(a) + kUnit - 1) / kUnit * kUnit * 3 <= kLds;
}

template <int QB>
int64_t bias_workgroups(const AttnArgs &a)
{
    constexpr int TQ = NW * 32 * QB;
    return (int64_t)8 * ((a.max_rows_per_user + TQ - 1) / TQ) * (((int64_t)a.cache.B * a.H + 7) / 8);
}

// three: the instance whose registers are held to what three workgroups per CU leave (QB = 1; their LDS: three_per_cu)
template <int QB, bool SUMI, bool CAUSAL, bool RAW = false>
hipError_t launch_bias(const AttnArgs &a, bool three, hipStream_t s)
{
    constexpr int TQ = NW * 32 * QB;
    const int64_t grid = bias_workgroups<QB>(a);
    if (grid <= 0 || grid > 0x7fffffff) return hipErrorInvalidValue;
    const KParams p = make_params(a, (a.max_rows_per_user + TQ - 1) / TQ);
    const bool in_lds = bias_entries(a) <= kBiasLdsFloats;
    auto go = [&](auto in_lds_tag, auto per_cu) {
        constexpr int PER_CU = decltype(per_cu)::value;
        constexpr auto kernel = attn_bias_kernel<QB, SUMI, CAUSAL, decltype(in_lds_tag)::value, RAW, PER_CU>;
        const hipError_t e = raise_lds_limit<kernel>(bias_flags_at<two_rings<RAW, PER_CU>, RAW>(kBiasLdsFloats) + NW * 4);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(NW * 64), (bias_lds_bytes<two_rings<RAW, PER_CU>, RAW>(a)), s, p);
        return hipGetLastError();
    };
    using Two = std::integral_constant<int, 2>;
    using Three = std::integral_constant<int, 3>;
    if constexpr (QB == 1) {
        if (in_lds) return three ? go(std::true_type{}, Three{}) : go(std::true_type{}, Two{});
        if constexpr (SUMI || (CAUSAL && !RAW))
            if (three) return go(std::false_type{}, Three{});
        return go(std::false_type{}, Two{});
    } else {
        return in_lds ? go(std::true_type{}, Two{}) : go(std::false_type{}, Two{});
    }
}

}  // namespace

hipError_t launch_attn_bias_bf16(const AttnArgs &a, bool sumi, hipStream_t s)
{
    // Candidates: 256-query tiles once 128-query tiles make more than two workgroups per CU.  Us, 256 / 128, 8 heads,
    // histories of 1024: 200 candidates of one user (16 workgroups of 128) 35 / 22, 512 of 16 (512) 36 / 31, of 24 (768)
    // 49 / 46, of 32 (1024) 53 / 58, 128 of 64 (512) 49 / 33; histories of 215, 692 of 5 users, 2 heads (60) 15.7 / 10.5, of
    // 16, 8 heads (768) 21.9 / 24.9.  Same bits.
    // Where three workgroups of 128 fit a CU (the tables), the busiest CU's share of queries decides: 512 of 24 users 49.9 / 40.9, 256 of 40 49.4 /
    // 39.5, 300 of 64 104 / 79, 1000 of 20 against 4000 234 / 205; equal shares: 512 of 32 54.3 / 55.2, 200 of 64 54.4 / 58.5, 1024 of 16 51.6 / 52.7,
    // 512 of 64 111 / 111, with 17 + 8 entries 101 / 105; tables beyond LDS (257 + 20): 512 of 24 84.9 / 62.1, 300 of 64 168.6 / 115.5, up to 200 of 100
    // that differ 137.9 / 131.7 (142.8 where registers leave room for two).  Where two do: poorly filled tiles only (512 of 64, 129 + 20
    // entries, 118 / 137).
    // A third workgroup where there are more than two per CU: with two / three, 128 of 72 users 52.5 / 43.6, of 64 (512) 37.3 / 37.0, of 48 30.9 / 31.3, up
    // to 300 of 32 that differ (about 500 with work) 28.8 / 35.6 (three on some CUs, one on others), beyond LDS 45.4 / 50.2.
    if (sumi) {
        const int64_t B = a.cache.B, H = a.H;
        const bool few = B * H * ((a.max_rows_per_user + 127) / 128) <= 512, fit = three_per_cu<false>(a);
        auto rows = [&](int tile) {  // (of users that differ, about half a tile each is padding)
            return a.uni_cand >= 0 ? B * ((a.uni_cand + tile - 1) / tile * tile) : a.total_q_rows + B * (tile / 2);
        };
        const int64_t narrow = H * rows(128) / 128, wide = H * rows(256) / 256;
        const bool better = fit ? (narrow + 255) / 256 < (wide + 255) / 256 * 2 : 6 * narrow <= 10 * wide;
        return few || a.max_rows_per_user <= 128 || better ? launch_bias<1, true, false>(a, fit && narrow > 512, s)
                                                           : launch_bias<2, true, false>(a, false, s);
    }
    // History from the cache: three where they fit; tables beyond LDS: under the causal flag, whose tiles' walks differ.  Us with two / three, 100 x
    // 100 in one (800 workgroups) 35.5 / 33.3; tables beyond LDS, causal, 64 x 1024 in one 402 / 370, 16 x 1000 in two 97 / 93, 8 x 1000 in four
    // 48.8 / 49.1; not causal, 64 x 1024 in one 512 / 465, but 16 x 1000 (1024 workgroups) 137 / 144.
    const bool three = three_per_cu<false>(a);
    return a.causal ? launch_bias<1, false, true>(a, three, s) : launch_bias<1, false, false>(a, three, s);
}

// From rows with the tables in LDS.  With look-ups in global memory the cache writer and a launch that reads the cache are the faster
// way but for causal passes and short walks: 32 rows of 257 + 20 entries, us from rows / as two, causal: subsequences of 256, one
// user's 1000 24.2 / 23.0, 24.7 / 26.2; 4 x 300 24.5 / 23.4, 24.8 / 26.4; 30 x 1000 131 / 128, 132 / 124; 8 x 2000 70.1 / 70.6, 70.7 / 81.2;
// 64 x 1024 260 / 254, 259 / 245; histories of 60 x 200 32.2 / 36.9, 31.6 / 34.7, 100 x 100 23.4 / 26.2, 23.7 / 26.9.
bool attn_hist_rows_bias_bf16_takes(const AttnArgs &a)
{
    const int walk = a.sub_len > 0 ? std::min(a.sub_len, a.max_hist_len) : a.max_hist_len;
    return a.causal || walk < 256 || bias_entries(a) <= kBiasLdsFloats;
}

hipError_t launch_attn_hist_rows_bias_bf16(const AttnArgs &a, hipStream_t s)
{
    // A third workgroup per CU where the tables leave it room in LDS and there are that
    // many.  From rows it costs the compiler the order it likes best: us with two / three, subsequences of 256, one row of 33 + 20 entries,
    // full and causal: 64 users x 1024 142 / 125, 146 / 126; 30 x 1000 74.3 / 67.4, 74.6 / 68.3; 8 x 2000 (1024 workgroups) 41.9 / 41.5, 42.3 /
    // 41.6; 100 x 100 (800) 32.9 / 34.9, 33.6 / 36.4; 4 x 300 14.2 / 14.2, 14.4 / 15.2; 32 rows of 33 + 12, 64 x 1024 137 / 120, 139 / 119.
    const bool three = three_per_cu<true>(a) && bias_workgroups<1>(a) >= 1024;
    return a.causal ? launch_bias<1, false, true, true>(a, three, s) : launch_bias<1, false, false, true>(a, three, s);
}

}  // namespace climber
