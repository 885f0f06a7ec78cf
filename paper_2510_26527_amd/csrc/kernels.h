// Internal launch interface between the C-ABI layer (api.hip) and the kernel files.
// Every launcher only enqueues work on `stream`; shapes were validated by the caller.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace psd {

// ---------------------------------------------------------------- acceptance (accept.hip)
struct AcceptArgs {
    const void *p, *q;            // logits, [rows][n_p_rows][V] / [rows][gamma][V]
    const int32_t *x;             // draft tokens [rows][gamma]
    const float *u;               // uniforms [rows][gamma+1]
    int rows, gamma, n_p_rows, V;
    int64_t p_stride, q_stride;   // elements between consecutive sequences
    int dtype;                    // PSD_F32 / PSD_BF16
    float temperature;
    int chunkA, n_chunksA;        // statistics pass: elements per block, blocks per logits row
    int chunkE, n_chunksE;        // draw pass chunking
    int groupE;                   // consecutive entries per thread of it
    float2 *stats;                // [rows][n_p_rows+gamma][n_chunksA] (max raw logit, sum exp)
    float *xlogit;                // [rows][gamma][2] the draft token's logit under p and under q
    double *part;                 // [rows][n_piecesE][6] fp64 sums of the draw position (accept.hip)
    uint32_t *counter;            // [rows] chunks of the draw position done so far
    int32_t *out_n, *out_tok, *flags;
    int pieceE, n_piecesE;        // draw pass: entries whose sums are kept together (a chunk or a quarter of one), how many per row
};
// vec: rows are 16-byte aligned and V is a multiple of the elements per 16-byte load
void accept_plan(int rows, int gamma, int n_p_rows, int V, int dtype, bool vec, AcceptArgs *a);
size_t accept_workspace_bytes(const AcceptArgs &a);
void accept_bind_workspace(AcceptArgs *a, void *ws, int32_t *out_flags);
void launch_accept(const AcceptArgs &a, bool vec_ok, hipStream_t stream);
// temperature 0: greedy verification (greedy.hip); reads p and x only, same workspace
void launch_accept_greedy(const AcceptArgs &a, bool vec_ok, hipStream_t stream);

// ---------------------------------------------------------------- GEMMs (gemm.hip)
// Up to this many rows (one 16-row MFMA tile) the bf16 projections stream the weights straight into MFMA
// operands (HBM-bound); above it the activation operand traffic of that scheme outgrows the weights and kernels that stage
// the activations in LDS win (measured on two LLaMA2-7B-shaped layers: 0.28 ms at 16 rows; at 32 rows 0.43 ms
// streaming against 0.38 ms tiled, at 64 rows 0.66 against 0.38).
constexpr int kStreamMaxRows = 16;
// Up to this many rows a pass' operand-order activations (common.h) are folded: both parts in one fragment.
constexpr int kOpFoldRows = 8;
// y[m][n] = sum_k x[m][k] * W[n][k]; W is up to three row-major [n_i][K] matrices whose
// outputs are concatenated along n (QKV, gate|up).
// r_m from per-tile sums of squares: rsqrt(sum_t sumsq[t * M + m] * inv_d + eps); sumsq NULL: 1
struct RowScale {
    const float *sumsq;
    int tiles;
    float inv_d, eps;
};
// How a packed copy groups its strips of 16 rows: `strips` of them a band, the strips of all matrices one behind the other, or, paired
// (gate|up), each matrix in whole bands.  Bands of four are the 64-row tiles of the unit kernel.
struct GemmBands {
    int strips;
    int paired;                   // bands of each matrix; 0: not paired
    uint32_t inverse;             // ceil(2^32 / strips)
    bool owned;                   // up to kStreamMaxRows rows the band kernel runs: one block a band, or a pair of them
};
constexpr GemmBands kUnitBands{4, 0, 1u << 30, false};
// What the kernels read first stands first: a block begins by waiting for the 64-byte lines of arguments that it needs, every launch
// brings them in anew (the implicit ones, the grid's size among them, lie behind this struct).  Tiled launches of 22 rows, us, with
// M, K, n, the tile count and the grid's size on four lines / on the first: 4608 x 3584 12.3 / 11.9, 3584 x 3584 11.0 / 10.5.
struct GemmArgs {
    int M, K, N, nseg;            // N = sum n[i]
    int n[3];
    int splitk;
    int tiled_tiles, blocks;      // M > kStreamMaxRows: tiles of the product, and the tiled kernel's grid; set by launch_gemm
    int pack_tiles;               // 64-row tiles of wpack
    int lens_n;                   // lengths that the kernel moves on (`lens`); set only for the last kernel (gemm_moves_lens)
    bool whole;                   // blocks take whole tiles: rows kernel, set by launch_gemm; unit kernel, a head's, set by the caller
                                  //   (gemm_stream_whole): `partial` are then the logits, the row scale is applied
    bool w4;                      // 4-bit weights, see below
    bool op_folded;               // x_op, xg_op: high part and remainder in one fragment (at most 8 rows)
    const uint16_t *x16;          // M > kStreamMaxRows and 4-bit projections: the activations rounded to fp16
    float *partial;               // [splitk][M][N] fp32: split s holds its share of the K sum
    const void *w[3];
    const void *wpack;            // optional repacked copy of all segments (bf16: M <= 128; 4-bit: M <= kStreamMaxRows): see gemm.hip
    int x_rows_per_group, x_group_stride, x_group_offset;      // row m is read from source row
                                  //   (m / x_rows_per_group) * x_group_stride + x_group_offset + m % x_rows_per_group
    int scale_rows;               // rows per tile slab of scale.sumsq
    uint16_t *swiglu16;           // M > kStreamMaxRows and 4-bit ones; segments are (gate, up): [M][n[0]] fp16 <- silu(gate) * up instead of `partial`
    const uint16_t *x_op;         // bf16, packed weights, M <= kStreamMaxRows: the activations in operand order (common.h)
    const float *x;               // fp32 activations, K contiguous: fp32 models, and bf16 ones without packed weights up to kStreamMaxRows rows
    float *reduced;               // if non-NULL: [M][N] <- sum over splits (logits), times the row scale if given
    // -- bf16, M <= kStreamMaxRows, packed weights only: RMSNorm folded into the projections around it -----------
    // rmsnorm(x) W^T = r_m * ((x * gain) W^T) with r_m = rsqrt(mean_k x[m][k]^2 + eps).  A projection with x_resid
    // set adds its output into the residual stream x_resid [M][N], writes
    // xg_op[m][n] = x_resid[m][n] * gain[n] (the operand of the next projection, in operand order; gain = the next norm's)
    // and sumsq_out[strip or tile][m] = sum of x_resid[m][n]^2 over the 16 (column kernel) or 64 (with tile_counter)
    // columns one block finishes; the consumer of the next projection's output multiplies by r_m (RowScale).
    float *x_resid;
    uint16_t *xg_op;              // NULL: nobody reads it
    uint16_t *xg16_out;           // optional: the same rounded to fp16, row-major (the operand of the 4-bit projections)
    const void *gain;             // [N] bf16
    float *sumsq_out;             // [N/16][M] (column kernel) or [N/64][M] (with tile_counter)
    unsigned *tile_counter;       // non-NULL: by tiles of 64 columns that several blocks share and the last to arrive finishes (4-bit, unit
                                  //   kernel): [N/64] arrival counters, zero before the launch and left at zero by it
    // -- 4-bit weights (W4A16, groups of 128 along K): wpack holds the 4-bit quad layout of
    // launch_gemm_pack_w4; the projection writes `splitk` partial slots (gemm_w4_slots)
    const void *w4_scale[3], *w4_zero[3];   // M > kStreamMaxRows: w[] are the codes [n][K/2], these the bf16 scales and uint8 zero points [n][K/128]
    RowScale scale;               // applied when writing `reduced`, a head in whole tiles (row = the source row of m), or by bands or 4-bit gate tiles
    int32_t *lens;                // lens_n of them move on by lens_add, up to lens_max
    int lens_add, lens_max;
    // (behind the rest: ahead of it they moved what the tiled kernel reads first, 2 us over the launches of a small model's two layers)
    uint16_t *swiglu_op;          // bf16, packed weights, M <= kStreamMaxRows; segments are (gate, up): silu(gate) * up, scaled, in operand order
    GemmBands bands;              // of wpack
};
struct GemmTiledPlan {
    int ta, cols;                 // block tile: 64 ta rows x cols columns
    int tiles, blocks;            // tiles of the product; blocks, each of which takes an equal range of all their K steps
    int slots;                    // partial slots per output
    int first, cols2, tiles2;     // first > 0: only the first `first` tiles side by side are of this kind; the columns left over go in a
                                  //   second launch, in tiles2 tiles of cols2 columns
};
bool gemm_tiles_whole(int M, int K, const int *n, int nseg, bool packed);     // up to 128 rows: no tile shared; once true for M rows, for more (to 64, to 128) too
GemmTiledPlan gemm_tiled_plan(int M, int K, const int *n, int nseg, bool gated, bool w4);
bool gemm_tiled_gates(int M, int K, const int *n, bool packed);                // whether the gate|up projection n = {f, f} applies SwiGLU itself
// 17 to 128 rows on unit-packed weights: whether the rows kernel takes the product, and how
struct RowsPlan {
    bool used, whole;             // whole: no tile is shared between blocks
    int waves, tiles, blocks, slots;      // wavefronts = 16-column strips of a tile
};
RowsPlan gemm_rows_plan(int M, int K, const int *n, int nseg, bool gated);
// packed: a unit-packed bf16 copy of the weights is there
int gemm_pick_splitk(int dtype, int M, int K, int N, const int *n, int nseg, bool packed, bool w4);
// repacked weights for the M <= kStreamMaxRows path
int gemm_pack_tiles(const int *n, int nseg);
GemmBands gemm_gate_bands(int f);
GemmBands gemm_qkv_bands(const int *n);
size_t gemm_pack_bytes(const int *n, int nseg, int K, GemmBands b);
bool gemm_w4_gates(int d_model, int d_ffn);              // ... and the gate|up projection applies SwiGLU itself, up to kStreamMaxRows rows
int gemm_w4_slots(int K, const int *n, int nseg, bool resid);  // partial slots of a 4-bit projection (resid: the arrival epilogue's grid)
bool gemm_down_by_units(int d_model, int d_ffn);          // packed: the down projection (4-bit: O too) runs with tile_counter, on unit-major weights
int gemm_resid_slots(int tiles, int K);                  // ... its partial slots
int gemm_packed_splits(int K, const int *n, int nseg);   // partial slots (the splitk to use) with packed weights
void launch_gemm_pack(const void *const *w, const int *n, int nseg, int K, void *dst, GemmBands b, hipStream_t stream);
void launch_gemm_pack_strips(const void *w, int n, int K, void *dst, hipStream_t stream);      // the layout of the column kernel
// 4-bit weight-only quantised projections: q [n][K/2] bytes (low nibble = even k), scale bf16 [n][K/128],
// zero u8 [n][K/128]; w = scale * (q - zero).  Each n[s] a multiple of 64.
size_t gemm_pack_w4_bytes(const int *n, int nseg, int K);
void launch_gemm_pack_w4(const void *const *q, const void *const *scale, const void *const *zero, const int *n,
                         int nseg, int K, void *dst, hipStream_t stream);
bool gemm_stream_whole(const int *n, int nseg);
bool gemm_moves_lens(int dtype, const GemmArgs &g);               // whether launch_gemm has a kernel that can
void launch_gemm(int dtype, const GemmArgs &g, hipStream_t stream);

// ---------------------------------------------------------------- attention (attention.hip)
struct AttnArgs {
    const float *q;               // [B][R][h_q][d_h] rotated queries, fp32
    const void *k;                // this layer's K cache [B][h_kv][max_len][d_h]
    const void *v;                // this layer's V cache [B][h_kv][d_h][max_len]
    const int32_t *lens;          // [B] valid positions BEFORE this forward
    float *out;                   // [B][R][h_q*d_h] fp32; NULL where only the next one is read
    uint16_t *out16;              // optional: the same rounded to fp16 (the operand of the tiled and the 4-bit O projection)
    uint16_t *out_op;             // optional: the same in operand order (common.h; the operand of the packed O projection)
    bool op_folded;
    int B, R, h_q, h_kv, d_h, max_len;
    int len_bound;                // host upper bound of lens[b] + R
    float *part_o;                // split scratch [B][h_q][R][splits][d_h]
    float *part_ml;               // [B][h_q][R][splits][2]
    int splits;
    // Fused operand build (bf16, at most 32 query rows per KV head and at most 32 new rows): q is not read;
    // the kernel takes q, k, v of the new rows from the QKV projection's split-K partial sums
    // qkv_partial [qkv_splits][B*R][(h_q + 2 h_kv) d_h], applies the row scale rs and the rotation by
    // rope_cs [B*R][d_h/2] = (cos, sin) of position lens[b] + r at frequency i, and appends k, v to the cache.
    const float *qkv_partial;     // NULL: q holds the rotated queries and the cache already holds the new rows
    int qkv_splits;
    RowScale rs;
    const float2 *rope_cs;
    // Token tree (fused build only): tree_anc[r] has bit j set when row j of the step is row r itself or one of its
    // ancestors; row r then sees the cache and exactly those rows.  NULL: rows see the rows before them.
    const uint32_t *tree_anc;
};
constexpr int kMaxGroupRows = 4096;        // query rows per KV head (group * R) of a forward pass
// The order of the LDS-staged kernel's blocks: heads_inner: chunk[i] is the i-th chunk of query rows, of all heads before the next one;
// else each head's chunks one behind the other.  Four chunks to a word, which a block reads with the scalar unit: a byte comes through the
// vector one, and with it every bound and address that follows would be held per lane (1 to 2 us a launch).
struct ChunkOrder {
    uint32_t heads_inner, chunk[kMaxGroupRows / 128 / 4];
    __host__ __device__ __forceinline__ int at(unsigned i) const { return (int)(chunk[i / 4] >> 8 * (i % 4) & 255u); }
};
ChunkOrder attn_chunk_order(int R, int group, int rows);
bool attn_longest_first(int B, int R, int h_kv, int d_h, int len_bound);
// the step's row (0 .. R - 1) whose position bounds what the query rows [c * rows, (c + 1) * rows) of a KV head see; query row i is row i % R
// of head i / R of the group (a chunk that reaches into the next head's rows: the last one)
__host__ __device__ inline int chunk_last_row(int c, int rows, int R, int group) {
    const int q0 = c * rows, q1 = (group * R < q0 + rows ? group * R : q0 + rows) - 1;
    return q0 / R == q1 / R ? q1 % R : R - 1;
}
// whether launch_attention builds its operands itself for this shape (then no rotation / append kernel runs before it)
bool attn_fuses_rope(int dtype, int R, int h_q, int h_kv, int d_h, bool tree);
int attn_max_splits(int dtype, int B, int R, int h_q, int h_kv, int d_h, int len_bound, bool tree);
int attn_pick_splits(int dtype, int B, int R, int h_q, int h_kv, int d_h, int len_bound, bool tree);
void launch_attention(int dtype, const AttnArgs &a, hipStream_t stream);

// ---------------------------------------------------------------- token trees (tree.hip)
constexpr int kTreeMaxNodes = 32;          // nodes of a tree forward pass (root included): one 32-key tile of new rows
constexpr int kTreeMaxAcceptNodes = 64;    // nodes of a tree acceptance call
struct TreeShape {
    uint32_t anc[kTreeMaxNodes];  // bit j of anc[r]: node j is node r or one of its ancestors
    int32_t depth[kTreeMaxNodes];
    int n;
};
struct TreeAcceptArgs {
    const void *p, *q;            // [rows][n_nodes][vocab] logits (strides in elements per sequence), q unused when greedy
    int64_t p_stride, q_stride;
    const int32_t *tokens;        // [rows][n_nodes], tokens[.][0] unused
    const float *uniforms;        // [rows][n_nodes + 1]
    float temperature;            // 0: greedy matching
    int32_t *out_path_len, *out_path, *out_token, *out_flags;   // [rows], [rows][n_nodes], [rows], [rows] or NULL
    int rows, n_nodes, vocab;
    int32_t parents[kTreeMaxAcceptNodes];
};
void launch_tree_accept(int dtype, const TreeAcceptArgs &a, hipStream_t stream);
void launch_kv_compact_tree(int dtype, void *k, void *v, int32_t *lens, const int32_t *base, const int32_t *path,
                            const int32_t *path_len, int path_stride, int n_nodes, int L, int B, int h_kv, int d_h,
                            int max_len, int cap, hipStream_t stream);

// ---------------------------------------------------------------- measured ceilings (ceilings.hip)
void launch_probe_read(const void *src, size_t bytes, void *sink, int blocks, hipStream_t stream);
void launch_probe_mfma(const void *seed, void *sink, int blocks, int iters, hipStream_t stream);

// ---------------------------------------------------------------- row-wise kernels (rowwise.hip)
// optional by-product of the embedding kernel: cs[m][i] = (cos, sin) of (the position of row m) * theta^(-2i/d_h)
struct RopeTable {
    float2 *cs;                   // [M][d_h/2], NULL: not wanted
    const int32_t *lens;
    int R, d_h;
    float theta;
};
struct ZeroFill {
    unsigned *words;              // n 32-bit words set to zero by the first kernel of a forward pass (NULL / 0: none)
    int n;
};
// xn in operand order (common.h), one behind the other: rows first .. per_group - 1 of each group of per_group rows, 16 at most
struct OpRows {
    uint16_t *op;                 // NULL: not wanted
    int per_group, first;
    bool folded;
};
// tree (or NULL): row r sits at position lens[b] + depth[r], and tree_anc receives the ancestor masks
// x = embed[token]; then xn = rmsnorm(x) * gain, or (sumsq_out non-NULL) xn = x * gain and sumsq_out[m] = sum_k x[m][k]^2;
// with `op` xn goes there too, and may be NULL
void launch_embed_norm(int dtype, const void *embed, const int32_t *tokens, float *x, const void *gain, float *xn,
                       float *sumsq_out, int M, int d, int vocab, float eps, RopeTable rt, uint16_t *xn16, OpRows op, ZeroFill zf,
                       const TreeShape *tree, uint32_t *tree_anc, hipStream_t stream);
// qkv = sum over splits of partial [S][M][(h_q+2h_kv) d_h] -> rotated q (fp32), rotated k and v appended
// to the cache (model dtype); cs_table: RopeTable::cs of these rows, NULL: the angles are evaluated again
void launch_reduce_rope_append(int dtype, const float *partial, int S, RowScale rs, float *q_out, void *k_cache,
                               void *v_cache, const int32_t *lens, int B, int R, int h_q, int h_kv, int d_h,
                               int max_len, float theta, const float2 *cs_table, hipStream_t stream);
// x += sum over splits of partial [S][M][d]; xn = rmsnorm(x) * gain (xn16, if given: the same rounded to fp16; xn may be NULL
// beside that or op)
void launch_reduce_residual_norm(int dtype, const float *partial, int S, float *x, const void *gain, float *xn,
                                 int M, int d, float eps, uint16_t *xn16, OpRows op, hipStream_t stream);
// h = silu(g) * u with [g | u] = sum over splits of partial [S][M][2f]: fp32, fp16 or both
void launch_reduce_swiglu(const float *partial, int S, RowScale rs, float *h, int M, int f, uint16_t *h16, hipStream_t stream);
void launch_advance_lens(int32_t *lens, int B, int delta, int max_len, hipStream_t stream);
void launch_truncate(int32_t *lens, const int32_t *base, const int32_t *keep, int offset, int cap, int B,
                     hipStream_t stream);
void launch_truncate_to(int32_t *lens, int new_len, int B, hipStream_t stream);

}  // namespace psd
