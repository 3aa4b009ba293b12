// GEMM and row-wise kernels of the layer stack (internal).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace climber {

enum { EPI_STORE_BF16 = 0, EPI_GELU_BF16 = 1, EPI_RESID_F32 = 2, EPI_RELU_BF16 = 3 };

// RMSNorm folded into the projections around it.  A projection whose input is RMSNorm(x; g) runs on
// the plain bf16 rows of x with the gain folded into the weight rows (pack job with `gain`) and
// multiplies every output row by r = 1/sqrt(mean(x^2) + eps) in its epilogue (`in_norm`).  The
// projection that produces x (EPI_RESID_F32) writes, besides the fp32 rows, their bf16 copy and
// the sums of squares of its 64-column slices (`out_norm`); d/64 partial sums per row.
struct RowNormIn {          // consumer side; ss == nullptr: no scaling
    const float *ss;        // [rows][n_part] partial sums of squares of the input rows
    int n_part;
    float inv_d, eps;
};
struct RowNormOut {         // producer side; ss == nullptr: fp32 rows only
    float *ss;              // [rows][N/64]
    void *xb;               // bf16 copy of the output rows, [rows][ldb]
    int64_t ldb;
};

// W [K][N] bf16 row-major -> MFMA B-operand fragments (same byte size).  K % 16 == 0, N % 32 == 0.
// Several weights in one launch (n <= kMaxPackJobs): job i packs w[i] [K[i]][N[i]] into packed[i].
constexpr int kMaxPackJobs = 16;
struct PackJobs {
    const void *w[kMaxPackJobs];
    const void *gain[kMaxPackJobs];  // bf16 [K] multiplied into the rows of w, or nullptr
    void *packed[kMaxPackJobs];
    int K[kMaxPackJobs], N[kMaxPackJobs];
    int n;
};
hipError_t pack_weights(const PackJobs &jobs, hipStream_t s);

// Tiled activation layout (bf16, X columns): the rows are cut into groups of 16 and the columns into
// k-tiles of 32; piece (g, t) = 1 KiB at ((g * X/32) + t) * 1024, holding for row r of the group and
// 16-byte slot s (at r*64 + s*16) the 8 columns 32t + 8(s ^ (r >> 2)) ..: exactly the bytes one
// global->LDS copy of the consuming projection lands, so that the copy reads 1 KiB contiguous and
// the k-tiles of a row group follow each other in memory.  Buffers hold a multiple of 16 rows.
// Used for the FFN hidden (X = d_ffn: with row-major rows a copy would touch 16 rows 4 KiB apart).
enum { kTiledA = 1, kTiledC = 2 };

// Fused QKV projection of the history rows of a batch (all `rows` padded rows of the cache):
// output columns [0, d) (queries) go to C as rows of d, columns [d, 2d) and [2d, 3d) (keys, values)
// straight into the layer's bf16 KV cache as MFMA operand fragments (the layout of internal.h;
// slots past a user's valid length as zeros), so that no key / value rows are written and read back.
// which0 = 1: the weight and N cover the key and value columns only (last layer: no attention).
// l_pad > 0: every user has this padded and l_valid valid rows; l_pad == 0: ragged batch, a block of
// 32 rows finds its user in seg (one entry per 64 rows) and the user's rows in tok_off / hist_len.
struct QkvToCache {         // layer_base == nullptr: plain store
    uint8_t *layer_base;    // cache payload of the layer
    int H, l_valid, l_pad;  // heads of 64; uniform batches: every user's valid and padded length
    int d, which0;
    const int32_t *seg, *tok_off, *hist_len;  // dev: [rows/64], [B+1], [B]
    int64_t rows;
};

// C = A W (+ epilogue).  A: bf16 [M][lda], or tiled (kTiledA; lda unused); w_packed from pack_weights;
// N % 128 == 0, K % 64 == 0.  EPI_STORE_BF16 / EPI_GELU_BF16 / EPI_RELU_BF16: C is bf16 [M][ldc] (EPI_GELU_BF16 with
// kTiledC: tiled, ldc unused).  EPI_RESID_F32: C is fp32, C = acc + resid.
hipError_t gemm_bf16(int epi, const void *A, int64_t lda, const void *w_packed, int M, int N, int K,
                     void *C, int64_t ldc, const float *resid, int64_t ldr, const RowNormIn &in_norm,
                     const RowNormOut &out_norm, int tiled, hipStream_t s, const QkvToCache *to_cache = nullptr);

// The arguments of one projection launch, as the kernels' host side passes them around.
struct GemmArgs {
    const void *A;
    int64_t lda;
    const void *W;
    int M, N, K;
    void *C;
    int64_t ldc;
    const float *resid;
    int64_t ldr;
    RowNormIn nin;
    RowNormOut nout;
    int tiled;
    QkvToCache qc;
};
// gemm_small_bf16.hip: few rows.  N % 64 == 0, K % 128 == 0.
bool gemm_small_takes(int epi, int M, int N, int K);  // instead of the macro tiles
hipError_t gemm_small_bf16(int epi, const GemmArgs &g, hipStream_t s);
// The fused QKV projection of few rows as a call has them (x: [M][K], fp32 with kRowsF32, else bf16) with what row_prep_f32 or row_prep_bf16 does for
// them: their sums of squares and, of bf16 rows, their fp32 copy [M][K] in x32 (in_norm: inv_d and eps).  N >= K.
bool gemm_small_sums(int M, int N, int K);
enum RowsIn { kRowsSummed, kRowsF32 };
hipError_t gemm_small_given(RowsIn in, const void *x, float *x32, const void *w_packed, int M, int N, int K, void *C, int64_t ldc, const RowNormIn &in_norm,
                            const QkvToCache &to_cache, hipStream_t s);

// Where the fused QKV projection of a call's rows goes: rows [0, n_cached), the history's, keys and values into the cache and
// queries to rows of q; the others as rows of `rows`, row n_cached first.  n_cached: none, or qc.rows.
struct QkvOut {
    QkvToCache qc;        // (qc.which0 = 1: no queries of the history)
    int n_cached;
    void *q, *rows;
    int64_t ld_q, ld_rows;
};

// gemm_resident_bf16.hip: the fused QKV projection of many rows.  A: [M][K], bf16 with their sums of squares in in_norm.ss, or fp32
// rows, whose sums it forms itself (row_prep_f32's bits; in_norm: inv_d and eps); N = 3 K.
bool gemm_resident_takes(int M, int K, bool cached);   // rows with their sums
bool gemm_resident_sums(int M, int K);                 // fp32 rows, instead of a launch for their sums before
hipError_t gemm_resident_bf16(RowsIn in, const void *A, const void *w_packed, int M, int K, const RowNormIn &in_norm, const QkvOut &out,
                              hipStream_t s);

// layer_tail_bf16.hip: y = h + GELU(RMSNorm(h) W1) W2 with h = x + o Wo, one launch.  Rows of D columns: o bf16,
// x / y fp32, yb (nullable) bf16; ss (nullable) [M][D / 64] sums of squares of y; wo [D][D], w1 [D][F] (gains
// multiplied in), w2 [F][D] packed.  y may be x, or lies apart from it; its rows may hold h for a while.
struct TailArgs {
    const void *o;
    const float *x;   // or, where layer_tail_reads_bf16, bf16 rows: x16, from row x16_split on x16_b
    const void *wo;   // the three packed weights are one block of memory: wo here,
    int w1, w2;       // w1 and w2 that many bytes further on,
    int w_bytes;      // all of them in so many bytes (< 2^31)
    float *y;
    void *yb;
    float *ss;
    int M, D, F;
    float inv_d, eps;
    // The next layer's QKV projection behind it, on the rows as they leave (where layer_tail_projects; yb and ss are then not written):
    int wq;           // its packed weights, so many bytes behind wo (within w_bytes); 0: no projection
    int y_first;      // y is wanted from this row on (a multiple of 64)
    QkvOut next;
    const void *x16, *x16_b;
    int x16_split;    // a multiple of 64
};
bool layer_tail_takes(int M, int D, int F);  // shapes it has a kernel for and is the faster way
// where that is the faster way; n_cached of the rows go to a cache, and if `ends` only their keys and values are wanted
bool layer_tail_projects(int M, int D, int F, int n_cached, bool ends);
bool layer_tail_reads_bf16(int M, int D, int F);
hipError_t layer_tail_bf16(const TailArgs &a, hipStream_t s);

// layer_head_bf16.hip: the tail's beginning for few rows, one launch: h = x + o Wo (fp32 rows, apart from x) and the hidden GELU(RMSNorm(h) W1),
// tiled (kTiledA of the down-projection).
struct HeadArgs {
    const void *o;
    const float *x;
    const void *wo;   // packed; w1 (gains multiplied in) so many bytes further on,
    int w1, w_bytes;  // both in so many bytes
    float *h;
    void *u;
    int M, D, F;
    float inv_d, eps;
    int n_parts;      // (layer_head_bf16's own)
};
bool layer_head_takes(int M, int D, int F);  // shapes it has a kernel for and is the faster way
hipError_t layer_head_bf16(const HeadArgs &a, hipStream_t s);

// What the first projection of a stack call needs of its input rows: the sum of squares of every
// row into ss[row][0] (ss[row][1 .. n_part-1] = 0) and
//   from bf16 rows x (the embeddings): the fp32 copy x32 (the residual stream; nullable);
//   from fp32 rows x: the bf16 copy xb.
hipError_t row_prep_bf16(const void *x, float *x32, float *ss, int n_part, int64_t rows, int d, hipStream_t s);
hipError_t row_prep_f32(const float *x, void *xb, float *ss, int n_part, int64_t rows, int d, hipStream_t s);

}  // namespace climber
