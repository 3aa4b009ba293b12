// fp32 attention on the matrix cores (gfx950): both masks of Climber (arXiv 2502.09888, Sec. 3.1.2, Sec. 3.2) with the
// per-row temperature of Eq. (3), for d_head 32, 64 and 128 without a relative bias.
//
// A workgroup owns 16 query rows of one (user, head) and splits their keys over its four waves, 16 keys a turn
// (wave w takes blocks w, w + 4, ...), because these launches are small: what counts is the length of one wave's chain of
// loads, products and exponentials, and a row's keys are the only work there is to share out.  Every wave carries a
// running maximum; the four partial results meet in LDS.  As in the bf16 kernels the transposed problem is
// computed, S^T = K Q^T and O^T = V^T P^T, here with v_mfma_f32_16x16x4_f32 (fp32 operands and sums): the lane holds four
// logits of one query, which are at once the operand of the second product.
//   lane = (g = lane / 16, i = lane % 16);  16-key block:
//   first product, step 4t + e:   K[key i][16t + 4g + e], Q[query i][16t + 4g + e]   -> S[key 4g + r][query i]
//   second product, step r:       V[key 4g + r][d], d = VD (i) + ..., P[key 4g + r][query i] -> O[d of row 4g + r][query i]
// so that keys, values and queries are read as 16-byte pieces of whole row segments.  No fp32 value is rounded on the way.
// The history pass reads its keys and values from the rows it is given and writes the cache rows of its own 16 rows:
// one launch instead of a cache writer and an attention that has to wait for it.
// One user, 64 behaviours, 8 candidates, 2 heads of 32: history pass 4.8 us (cache writer and a wave per row 14.0), candidates
// 4.0 (10.3): launch latency and one trip to memory.
#include "internal.h"

#include <algorithm>

namespace climber {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kRows = kTileRowsF32, kKeys = 16, kWaves = 4;
constexpr float kLog2e = 1.4426950408889634f;

// the four lanes that hold logits of one query
__device__ __forceinline__ float quad_max(float v)
{
    v = fmaxf(v, __shfl_xor(v, 16, 64));
    return fmaxf(v, __shfl_xor(v, 32, 64));
}
__device__ __forceinline__ float quad_sum(float v)
{
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
}

struct TileArgs {
    AttnArgs a;
    float *cache_k, *cache_v;  // this layer's keys and values, [rows][H][d_head]
    int n_tiles;               // tiles per (user, head) of the grid
    int sub, tiles_per_sub;    // history: rows and tiles of a subsequence
    int from_rows;             // history: keys and values come from a.k_self / a.v_self and go into the cache here
};

template <int DH, bool SUMI, bool CAUSAL>
__global__ __launch_bounds__(kWaves * 64) void attn_tile_f32_kernel(const TileArgs p)
{
    static_assert(!(SUMI && CAUSAL), "the causal flag concerns the history pass");
    constexpr int NB = DH / 16, VW = NB < 4 ? NB : 4;  // 16-wide blocks of d; consecutive d of a lane
    typedef float vec __attribute__((ext_vector_type(VW)));
    constexpr int NV = NB / VW;                        // pieces of VW floats per lane and row
    __shared__ __attribute__((aligned(16))) float part[kWaves][4][NV][64][VW];
    __shared__ float part_m[kWaves][kRows], part_l[kWaves][kRows];

    const AttnArgs &a = p.a;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, i = lane & 15;
    const int tile = blockIdx.x % p.n_tiles, bh = blockIdx.x / p.n_tiles, h = bh % a.H, b = bh / a.H;
    // (uniform batches: geometry from the arguments, a trip to memory less)
    const bool uni = a.uni_pad >= 0;
    const int t0 = uni ? b * a.uni_pad : a.cache.tok_off[b], Lb = uni ? a.uni_len : a.cache.hist_len[b];
    int64_t base;              // the user's first query row
    int q0, q_end, lo, hi;     // rows [q0, q_end) of the user see keys [lo, hi)
    if (SUMI) {
        base = max(a.uni_cand >= 0 ? b * a.uni_cand : a.cand_off[b], 0);
        q0 = tile * kRows;
        q_end = (int)(min(a.uni_cand >= 0 ? base + a.uni_cand : (int64_t)a.cand_off[b + 1], a.total_q_rows) - base);
        lo = 0, hi = Lb;
    } else {
        const int Lpad = uni ? a.uni_pad : a.cache.tok_off[b + 1] - t0;
        base = t0;
        lo = tile / p.tiles_per_sub * p.sub;
        q0 = lo + tile % p.tiles_per_sub * kRows, q_end = min(Lpad, lo + p.sub);
        hi = min(lo + p.sub, Lb);
    }
    // the temperature table in a register (entry lane), if it has no more than 64 entries
    const int n_tau = a.n_scen * a.n_beh;
    const float tau_reg = a.tau[min(lane, n_tau - 1)];
    const bool from_rows = !SUMI && p.from_rows;
    const int64_t ld_key = from_rows ? a.ld_kv : (int64_t)a.H * DH;
    const float *kb = from_rows ? (const float *)a.k_self : p.cache_k, *vb = from_rows ? (const float *)a.v_self : p.cache_v;
    kb += (int64_t)t0 * ld_key + h * DH;
    vb += (int64_t)t0 * ld_key + h * DH;

    // (candidates: the grid covers the longest user the caller announced; a longer one takes several turns)
    for (; q0 < q_end; q0 += p.n_tiles * kRows) {
        const int n_rows = min(kRows, q_end - q0);                       // rows that exist
        const int nq = SUMI ? n_rows : max(0, min(n_rows, Lb - q0));     // rows that count
        float *const o = (float *)a.o + (base + q0) * a.ld_o + h * DH;
        if (!SUMI && nq < n_rows)  // padding rows: zeros
            for (int x = tid; x < (n_rows - nq) * DH; x += kWaves * 64) o[(int64_t)(nq + x / DH) * a.ld_o + x % DH] = 0.f;
        // cache rows of this tile (zeros past the valid length): fetched here, stored behind the products
        constexpr int kPieces = DH / 4, kPer = (kRows * kPieces + kWaves * 64 - 1) / (kWaves * 64);
        f32x4 ck[kPer], cv[kPer];
        auto fetch_cache_rows = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < kPer; ++x) {
                const int r = (x * kWaves * 64 + tid) / kPieces, cc = tid % kPieces * 4;
                const int64_t src = (int64_t)(q0 + min(r, max(nq, 1) - 1)) * ld_key + cc;
                ck[x] = *(const f32x4 *)(kb + src);
                cv[x] = *(const f32x4 *)(vb + src);
            }
        };
        auto store_cache_rows = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < kPer; ++x) {
                const int r = (x * kWaves * 64 + tid) / kPieces, cc = tid % kPieces * 4;
                if (r >= n_rows) continue;
                const int64_t dst = ((int64_t)(t0 + q0 + r) * a.H + h) * DH + cc;
                const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                *(f32x4 *)(p.cache_k + dst) = r < nq ? ck[x] : zero;
                *(f32x4 *)(p.cache_v + dst) = r < nq ? cv[x] : zero;
            }
        };
        if (nq == 0) {  // (candidates: never)
            if (from_rows) {
                fetch_cache_rows();
                store_cache_rows();
            }
            return;
        }

        const int k_end = CAUSAL ? min(hi, q0 + kRows) : hi, n = k_end - lo, n_blk = (n + kKeys - 1) / kKeys;
        f32x4 kf[NB];
        vec vf[4][NV];
        auto load_k = [&](int blk) __attribute__((always_inline)) {
            const float *src = kb + (int64_t)(lo + min(blk * kKeys + i, n - 1)) * ld_key + 4 * g;
#pragma unroll
            for (int t = 0; t < NB; ++t) kf[t] = *(const f32x4 *)(src + 16 * t);
        };
        auto load_v = [&](int blk) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float *src = vb + (int64_t)(lo + min(blk * kKeys + 4 * g + r, n - 1)) * ld_key + VW * i;
#pragma unroll
                for (int v = 0; v < NV; ++v) vf[r][v] = *(const vec *)(src + 16 * VW * v);
            }
        };
        const int64_t row = base + q0 + min(i, nq - 1);
        const int sc = min(max(a.scen[row], 0), a.n_scen - 1), bv = min(max(a.beh[row], 0), a.n_beh - 1);
        f32x4 q[NB];
#pragma unroll
        for (int t = 0; t < NB; ++t) q[t] = *(const f32x4 *)((const float *)a.q + row * a.ld_q + h * DH + 16 * t + 4 * g);
        if (wave < n_blk) {
            load_k(wave);
            load_v(wave);
        }
        if (from_rows) fetch_cache_rows();
        const float tau = n_tau <= 64 ? __shfl(tau_reg, sc * a.n_beh + bv, 64) : a.tau[sc * a.n_beh + bv];
        const float c = a.qk_scale * kLog2e / tau;  // logits in log2 units

        float m = -INFINITY, l = 0.f;  // running maximum of the query; this lane's share of the denominator
        f32x4 O[NB];                   // [VW v + e][r]: d = 16 VW v + VW (4g + r) + e
#pragma unroll
        for (int x = 0; x < NB; ++x) O[x] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (SUMI && wave == 0) {  // the candidate's own key and value: the first member of its softmax
            const float *ks = (const float *)a.k_self + row * a.ld_kv + h * DH, *vs = (const float *)a.v_self + row * a.ld_kv + h * DH;
            float dot = 0.f;
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                const f32x4 kk = *(const f32x4 *)(ks + 16 * t + 4 * g);
#pragma unroll
                for (int e = 0; e < 4; ++e) dot = fmaf(q[t][e], kk[e], dot);
            }
            m = quad_sum(dot) * c;
            l = g == 0 ? 1.f : 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const vec own = *(const vec *)(vs + 16 * VW * v + VW * (4 * g + r));
#pragma unroll
                    for (int e = 0; e < VW; ++e) O[VW * v + e][r] = own[e];
                }
        }
        const int lim = CAUSAL ? min(n, q0 + i + 1 - lo) : n;  // keys [0, lim) of the range are the query's
        for (int blk = wave; blk < n_blk; blk += kWaves) {
            const bool more = blk + kWaves < n_blk;
            f32x4 S = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < NB; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) S = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[t][e], q[t][e], S, 0, 0, 0);
            if (more) load_k(blk + kWaves);
            const bool edge = (blk + 1) * kKeys > (CAUSAL ? q0 - lo : n);  // not every key is every query's
            float mx = m;
            bool out[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int key = blk * kKeys + 4 * g + r;
                out[r] = edge && key >= lim;
                mx = fmaxf(mx, out[r] ? -INFINITY : S[r] * c);
                if (edge && key >= n)
#pragma unroll
                    for (int v = 0; v < NV; ++v) vf[r][v] = (vec)(0.f);
            }
            mx = quad_max(mx);
            const float ref = mx == -INFINITY ? 0.f : mx;  // (no key seen yet: all terms are exp2(-inf) = 0)
            const float alpha = __builtin_amdgcn_exp2f(m - ref);
            m = mx;
            float P[4];
            l *= alpha;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                P[r] = __builtin_amdgcn_exp2f(out[r] ? -INFINITY : fmaf(S[r], c, -ref));
                l += P[r];
            }
#pragma unroll
            for (int x = 0; x < NB; ++x) O[x] *= alpha;
            bool apart = false;
            if (CAUSAL && edge) {
                // a value that is not finite must not reach the queries that do not see its key (0 * inf): then the block
                // goes key by key, and only the queries that see the key take the sum
                bool odd = false;
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int x = 0; x < NB; ++x) odd |= !(fabsf(vf[r][x / VW][x % VW]) < INFINITY);
                apart = __builtin_amdgcn_ballot_w64(odd) != 0;
            }
            if (!apart) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int x = 0; x < NB; ++x) O[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][x / VW][x % VW], P[r], O[x], 0, 0, 0);
            } else {
                for (int key = 0; key < min(kKeys, n - blk * kKeys); ++key)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if ((key & 3) != r) continue;
                        const bool mine = g == key >> 2, sees = blk * kKeys + key < lim;
#pragma unroll
                        for (int x = 0; x < NB; ++x) {
                            const f32x4 with = __builtin_amdgcn_mfma_f32_16x16x4f32(mine ? vf[r][x / VW][x % VW] : 0.f, mine ? P[r] : 0.f, O[x], 0, 0, 0);
                            O[x] = sees ? with : O[x];
                        }
                    }
            }
            if (more) load_v(blk + kWaves);
        }

        if (from_rows) store_cache_rows();

        // ---- the waves' shares together ----
        l = quad_sum(l);
        if (g == 0) part_m[wave][i] = m, part_l[wave][i] = l;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                vec x;
#pragma unroll
                for (int e = 0; e < VW; ++e) x[e] = O[VW * v + e][r];
                *(vec *)part[wave][r][v][lane] = x;
            }
        __syncthreads();
        float mm = part_m[0][i];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) mm = fmaxf(mm, part_m[w][i]);
        const float ref = mm == -INFINITY ? 0.f : mm;
        float f[kWaves], sum = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            f[w] = __builtin_amdgcn_exp2f(part_m[w][i] - ref);
            sum = fmaf(f[w], part_l[w][i], sum);
        }
        // wave r finishes the values of accumulator register r
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            vec x = (vec)(0.f);
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const vec y = *(const vec *)part[w][wave][v][lane];
#pragma unroll
                for (int e = 0; e < VW; ++e) x[e] = fmaf(f[w], y[e], x[e]);
            }
#pragma unroll
            for (int e = 0; e < VW; ++e) x[e] /= sum;
            if (i < nq) *(vec *)(o + (int64_t)i * a.ld_o + 16 * VW * v + VW * (4 * g + wave)) = x;
        }
        if (!SUMI) return;
        __syncthreads();
    }
}

template <int DH>
hipError_t launch_tile(const TileArgs &p, bool sumi, unsigned grid, hipStream_t s)
{
    const dim3 t(kWaves * 64);
    if (sumi) hipLaunchKernelGGL((attn_tile_f32_kernel<DH, true, false>), dim3(grid), t, 0, s, p);
    else if (p.a.causal) hipLaunchKernelGGL((attn_tile_f32_kernel<DH, false, true>), dim3(grid), t, 0, s, p);
    else hipLaunchKernelGGL((attn_tile_f32_kernel<DH, false, false>), dim3(grid), t, 0, s, p);
    return hipGetLastError();
}

}  // namespace

// Grid: every head of every user gets the tiles of the longest one.  Where lengths differ much most of them are empty.
struct TileGrid { int sub, tiles_per_sub; int64_t heads, tiles; };
static TileGrid tile_grid(const AttnArgs &a, bool sumi)
{
    TileGrid g;
    g.sub = !sumi && a.sub_len > 0 ? std::min(a.sub_len, a.max_rows_per_user) : a.max_rows_per_user;
    g.tiles_per_sub = (g.sub + kRows - 1) / kRows;
    g.heads = (int64_t)a.cache.B * a.H;
    g.tiles = (int64_t)((a.max_rows_per_user + g.sub - 1) / g.sub) * g.tiles_per_sub;
    return g;
}

// Whole 16-byte pieces of rows; other widths and the relative bias take the kernel of attn_f32.hip, a wave per row.  So do
// launches that it is the faster way for, by what either costs in ns (d_head 64; the ratio is alike for 32 and 128):
//   a wave per row   2.3 a row and 0.2 a key it sees; 4000 for the cache writer that the history pass then needs
//   tiles            1.2 (history) or 4.5 (candidates) a workgroup, empty or not, and for a tile with rows 3.3 (history)
//                    and 0.07 a key
// Us, there / here, 8 heads: 4096 rows in subsequences of 1 76 / 108, of 2 80 / 58; one candidate for each of 4096
// users with histories of 4 78 / 141, of 64 1680 / 250; 16000 histories of 2 and one of 1024, subsequences of 16, 471 /
// 10388; 1024 of 16 and one of 2048, whole, 7567 / 1687; 1 candidate each for 4096 users and 512 for one 1247 / 4392.
// A grid has less than 2^32 threads; beyond that the launch would leave rows out.
bool attn_tile_f32_takes(const AttnArgs &a, bool sumi)
{
    if ((a.d_head != 32 && a.d_head != 64 && a.d_head != 128) || a.bias.pos_table || a.ld_q % 4 != 0 || a.ld_kv % 4 != 0 || a.ld_o % 4 != 0)
        return false;
    const TileGrid g = tile_grid(a, sumi);
    const double grid = (double)g.heads * g.tiles, rows = (double)a.total_q_rows, users = a.cache.B;
    if (grid * (kWaves * 64) >= 4294967296.0) return false;
    if (grid <= 2048) return true;  // all of them at once: the length of one wave's chain counts
    if (!sumi) {
        const double keys = a.hist_pairs / rows;
        return 1.2 * grid + a.hist_tiles * a.H * (3.3 + 0.07 * keys) < 4000 + rows * a.H * (2.3 + 0.2 * keys);
    }
    // (who has how many candidates is not known here: the longest history the most, the rest alike)
    const double most = a.max_rows_per_user, keys = (most * a.max_hist_len + (rows - most) * (a.valid_rows / users)) / rows;
    return 4.5 * grid + std::min(rows, users + rows / kRows) * a.H * 0.07 * keys < rows * a.H * (2.3 + 0.2 * keys);
}

hipError_t launch_attn_tile_f32(const AttnArgs &a, bool sumi, int64_t cache_rows, bool write_cache, hipStream_t s)
{
    TileArgs p;
    p.a = a;
    p.cache_k = (float *)a.cache.layer_base;
    p.cache_v = p.cache_k + cache_rows * a.H * a.d_head;
    p.from_rows = write_cache;
    const TileGrid tg = tile_grid(a, sumi);
    p.sub = tg.sub;
    p.tiles_per_sub = tg.tiles_per_sub;
    p.n_tiles = (int)tg.tiles;
    if (tg.heads <= 0 || tg.heads * tg.tiles > 0xffffffffll / (kWaves * 64)) return hipErrorInvalidValue;
    const unsigned grid = (unsigned)(tg.heads * tg.tiles);
    switch (a.d_head) {
    case 32: return launch_tile<32>(p, sumi, grid, s);
    case 64: return launch_tile<64>(p, sumi, grid, s);
    case 128: return launch_tile<128>(p, sumi, grid, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace climber
