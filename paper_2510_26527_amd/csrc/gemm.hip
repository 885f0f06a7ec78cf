// Decoder projections y[m][n] = sum_k x[m][k] W[n][k] on gfx950.
//
// The kernels, chosen by model dtype and row count M (M = batch * n_new of a verify step):
//   gemm_f32_kernel          fp32 weights, plain ALU dot products, one wavefront per output
//                            column (the tiny fp32 chain; fp32 1e-4 parity, not speed).
//   gemm_bf16_skinny_kernel  M <= 16, weights as the caller stores them (row-major).  HBM-bound weight
//                            streaming: W rows go straight from global memory into MFMA A-operand registers
//                            with 16-byte loads (no LDS), the few activation rows are the B operand, K is
//                            split over the four wavefronts of a block and over blocks.
//   gemm_bf16_unit_kernel    M <= 16 (heads, narrow QKV) on weights repacked by gemm_pack_kernel: the same MFMA tiling, but every
//                            16 KB unit (64 rows x 128 k) is stored in exactly the order the lanes load it,
//                            units of a GEMM are contiguous, and the grid is persistent: each block streams
//                            an equal, contiguous range of units (stream-K), its four wavefronts on the four
//                            K quarters of every unit, and writes one partial per tile it touches.
//                            With RESID (the down projection of wide models and very long ones) the block that arrives
//                            last at a tile adds the tile's partials and runs the residual epilogue below.
//   gemm_bf16_band_kernel    M <= 16: QKV (wide ones) and gate|up, one block per band of 16-row strips over the whole K range, the row
//                            scale in its epilogue, gate|up with SwiGLU.
//   gemm_bf16_rows_kernel    17 to 128 rows on the same units and bands: the weights stream into MFMA operands as above, the
//                            activations (fp16) go through LDS; whole tiles where they fill the chip.
//   gemm_bf16_column_kernel  M <= 16, the projections that write the residual stream (O, most models' down): one
//                            block per 16 output columns over the whole K range; the residual add, the
//                            gain-scaled copy and the RMSNorm statistics happen in its epilogue.
//   gemm_w4_unit_kernel      M <= 16, 4-bit weight-only quantised projections (groups of 128 along K): the unit
//                            kernel's stream-K over quads of four K steps, the codes multiplied as exact fp16
//                            integers against fp16-rounded activations, scale and zero point applied per group in
//                            fp32; one partial slot per block and tile, or (O, down of wide models) the residual epilogue run by
//                            the block that arrives last.
//   gemm_w4_column_kernel, gemm_w4_gate_kernel   the same arithmetic with one owner per output: O and down by strips of 16 columns, gate|up
//                            by tiles of 64 with the row scale and SwiGLU in its epilogue (where they fill the chip).
//   gemm_f16_tiled_kernel    M > 16 otherwise.  (64, 128 or 256) x (128, 192, 256) x 64 LDS-staged tiles, 32x32x16 fp16 MFMA
//                            (weights convert to fp16 exactly, activations are rounded to fp16); the gate|up projection
//                            applies SwiGLU itself where its tiles alone fill the chip.
// Activations are fp32 in memory in every case (the rows and tiled kernels read an fp16 copy their producers leave beside
// them; between the packed M <= 16 kernels they travel as bf16 pairs hi + lo in operand order, common.h).  The M <= 16 bf16
// kernels feed each activation to the matrix cores as that pair (two MFMAs against the same weight operand): with plain
// bf16 activations the logits of the 7B-shaped random-init models are 3e-2 off the fp64 result, above the 2e-2 bar; the
// weights, which are what streams from HBM, stay bf16.
// Every kernel but the ones with an epilogue of their own (residual, SwiGLU, logits in whole tiles) writes its result as split-K partials [splitk][M][N]
// (splitk >= 1); the consumer (the fused row-wise kernels, the attention kernel's operand build, or
// gemm_splitk_reduce_kernel for the logits) adds them in split order, so results are bit-reproducible.
#include <type_traits>
#include "common.h"
#include "kernels.h"
#include "prof.h"
#include "../../include/psd.h"

namespace psd {
namespace {

// source row of activation row m: rows may be a strided subset (the last rows of each sequence)
__host__ __device__ __forceinline__ size_t x_row(const GemmArgs &g, int m) {
    return (size_t)(m / g.x_rows_per_group) * g.x_group_stride + g.x_group_offset + (m % g.x_rows_per_group);
}

// ------------------------------------------------------------------------------ fp32
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs g) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int n = blockIdx.x * 4 + wave;
    if (n >= g.N) return;
    int seg = 0, nl = n;
    while (seg < g.nseg - 1 && nl >= g.n[seg]) { nl -= g.n[seg]; ++seg; }
    const float *wrow = (const float *)g.w[seg] + (size_t)nl * g.K;
    const float *x = (const float *)g.x;
    for (int m0 = 0; m0 < g.M; m0 += 8) {
        float acc[8];
#pragma unroll
        for (int mm = 0; mm < 8; ++mm) acc[mm] = 0.f;
        for (int k = lane; k < g.K; k += 64) {
            const float w = wrow[k];
#pragma unroll
            for (int mm = 0; mm < 8; ++mm)
                if (m0 + mm < g.M) acc[mm] += w * x[x_row(g, m0 + mm) * g.K + k];
        }
#pragma unroll
        for (int mm = 0; mm < 8; ++mm) acc[mm] = wave_sum(acc[mm]);
        if (lane == 0) {
#pragma unroll
            for (int mm = 0; mm < 8; ++mm)
                if (m0 + mm < g.M) {
                    g.partial[(size_t)(m0 + mm) * g.N + n] = acc[mm];
                }
        }
    }
}

// ------------------------------------------------------------------------------ bf16 helpers
struct TileRef {
    int seg;       // which weight matrix
    int row0;      // first row of the tile inside that matrix
    int col0;      // first output column of that matrix in the concatenated output
};
__device__ __forceinline__ TileRef find_tile(const GemmArgs &g, int tile, int tile_rows) {
    TileRef t;
    t.seg = 0;
    t.col0 = 0;
    while (t.seg < g.nseg - 1) {
        const int nt = (g.n[t.seg] + tile_rows - 1) / tile_rows;
        if (tile < nt) break;
        tile -= nt;
        t.col0 += g.n[t.seg];
        ++t.seg;
    }
    t.row0 = tile * tile_rows;
    return t;
}

// 8 consecutive activations of one row (zeros for a row past M)
__device__ __forceinline__ f32x8 load_act8(const float *xrow, int k, bool valid) {
    return valid ? load_f32x8(xrow + k) : f32x8{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
}

__device__ __forceinline__ void store_out(const GemmArgs &g, int ks, int m, int col, float v) {
    g.partial[((size_t)ks * g.M + m) * g.N + col] = v;
}



// the kernel that writes the logits also moves the lengths on
__device__ __forceinline__ void advance_lens(const GemmArgs &g) {
    for (int b = threadIdx.x; b < g.lens_n; b += blockDim.x) g.lens[b] = min(g.lens[b] + g.lens_add, g.lens_max);
}

// reduced[m][:] = (sum over splits, in split order) * r_m; one row per blockIdx.y
__global__ __launch_bounds__(256) void gemm_splitk_reduce_kernel(GemmArgs g) {
    __shared__ float red[4];
    const int m = blockIdx.y;
    if (m == 0 && blockIdx.x == 0) advance_lens(g);
    float sc = 1.0f;
    if (g.scale.sumsq) {
        const size_t src = x_row(g, m);
        float v = 0.f;
        for (int t = threadIdx.x; t < g.scale.tiles; t += 256) v += g.scale.sumsq[(size_t)t * g.scale_rows + src];
        v = wave_sum(v);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
        __syncthreads();
        sc = 1.0f / sqrtf((((red[0] + red[1]) + red[2]) + red[3]) * g.scale.inv_d + g.scale.eps);
    }
    const int col = blockIdx.x * 256 + threadIdx.x;
    if (col >= g.N) return;
    const size_t idx = (size_t)m * g.N + col;
    float v = 0.f;
    for (int ks = 0; ks < g.splitk; ++ks) v += g.partial[(size_t)ks * g.M * g.N + idx];
    g.reduced[idx] = v * sc;
}

// ------------------------------------------------------------------------------ bf16 skinny
// Block = 4 wavefronts, one 64-row tile of W (4 strips of 16 rows per wavefront, all four
// wavefronts on the same rows, each on its own K range).  Per 128-wide K step a lane issues
// 16 independent 16-byte loads of W (4 strips x 4) and keeps the next step's loads in flight
// while the current one feeds the MFMAs.  The K index inside a step is permuted so that a
// lane's four loads of one row are 2 x 32 contiguous bytes and the four lane groups of a row
// cover 2 x 128 contiguous bytes; the activation operand uses the same permutation.
constexpr int kSkinnyRows = 64;
constexpr int kSkinnyStepK = 128;
constexpr int kStreamBlocks = 512;                 // persistent grid of the unit kernel: 2 blocks per CU

template <int MT>
__global__ __launch_bounds__(256) void gemm_bf16_skinny_kernel(GemmArgs g) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = lane & 15, gq = lane >> 4;
    const TileRef t = find_tile(g, blockIdx.x, kSkinnyRows);
    const int seg_rows = g.n[t.seg];
    const uint16_t *W = (const uint16_t *)g.w[t.seg];
    const float *X = (const float *)g.x;
    const int K = g.K;

    const int nsteps = K / kSkinnyStepK;
    const int S = g.splitk * 4, slot = blockIdx.y * 4 + wave;
    const int s0 = (int)((long)slot * nsteps / S), s1 = (int)((long)(slot + 1) * nsteps / S);

    const uint16_t *wp[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int r = min(t.row0 + s * 16 + i, seg_rows - 1);
        wp[s] = W + (size_t)r * K + gq * 16;
    }
    const float *xp[MT];
    bool xvalid[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int tok = mt * 16 + i;
        xvalid[mt] = tok < g.M;
        xp[mt] = X + x_row(g, min(tok, g.M - 1)) * K + gq * 16;
    }

    f32x4 acc[4][MT];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[s][mt] = f32x4{0.f, 0.f, 0.f, 0.f};

    bf16x8 a_cur[4][4], a_nxt[4][4];
    auto load_a = [&](bf16x8 (&dst)[4][4], int step) {
        const int kk = step * kSkinnyStepK;
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int q = 0; q < 4; ++q) dst[s][q] = *reinterpret_cast<const bf16x8 *>(wp[s] + kk + (q >> 1) * 64 + (q & 1) * 8);
    };
    if (s0 < s1) load_a(a_cur, s0);
    for (int step = s0; step < s1; ++step) {
        if (step + 1 < s1) load_a(a_nxt, step + 1);
        const int kk = step * kSkinnyStepK;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            bf16x8 bh[MT], bl[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int k = kk + (q >> 1) * 64 + (q & 1) * 8;
                const f32x8 xv = load_act8(xp[mt], k, xvalid[mt]);
                split_bf16(xv, &bh[mt], &bl[mt]);
            }
            // hi parts over all accumulators, then lo parts: no back-to-back MFMAs on one accumulator
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    acc[s][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_cur[s][q], bh[mt], acc[s][mt], 0, 0, 0);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    acc[s][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_cur[s][q], bl[mt], acc[s][mt], 0, 0, 0);
        }
        if (step + 1 < s1) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int q = 0; q < 4; ++q) a_cur[s][q] = a_nxt[s][q];
        }
    }

    // acc[s][mt][v] = y[token mt*16 + i][row0 + s*16 + 4*gq + v]: add the four wavefronts (K split)
    __shared__ float red[4][kSkinnyRows][17];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        if (mt) __syncthreads();
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[wave][s * 16 + 4 * gq + v][i] = acc[s][mt][v];
        __syncthreads();
        const int nn = threadIdx.x & 63;
        const int row = t.row0 + nn;
        if (row < seg_rows) {
            for (int mm = threadIdx.x >> 6; mm < 16; mm += 4) {
                const int tok = mt * 16 + mm;
                if (tok < g.M) {
                    const float v = ((red[0][nn][mm] + red[1][nn][mm]) + red[2][nn][mm]) + red[3][nn][mm];
                    store_out(g, blockIdx.y, tok, t.col0 + row, v);
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------ bf16 stream-K on packed weights (unit kernel)
// Packed layout of one GEMM (all its weight matrices, in segment order): tiles of 64 rows, each
// tile ns = K/128 units of 16 KB.  Unit = 16 slots of 1 KB, slot index q*4 + strip; slot (q, strip) holds, for
// lane l = (i = l & 15, gq = l >> 4), the 8 bf16 W[tile*64 + strip*16 + i][step*128 + (q>>1)*64 + gq*16 + (q&1)*8 ...]:
// the 4 KB of K quarter q are contiguous.  Rows past the end of a matrix are stored as zeros.
constexpr int kUnitBytes = kSkinnyRows * kSkinnyStepK * 2;
constexpr int kUnitVec = kUnitBytes / 16;          // 16-byte vectors per unit
constexpr int kBandBlocks = 256;
constexpr int kGateLeast = 1, kGateMost = 7, kQkvLeast = 3, kQkvMost = 6;      // strips a band (the widths that are built)

// GemmBands (kernels.h): a band of S strips is ns steps of 4 S KB, a step its four K quarters, a quarter the S strips' slots: what the
// unit above is for S = 4.
struct PackArgs {
    const uint16_t *w[3];
    int n[3], nseg, K;
    GemmBands bands;
    u32x4 *dst;
};
__host__ __device__ __forceinline__ int strips_of(int n) { return (n + kSkinnyRows - 1) / kSkinnyRows * 4; }
// where the strip of 16 rows that begins at `row` of matrix `seg` lies: its band and its place there
struct BandRef { int band, slot; };
__device__ __forceinline__ BandRef band_of(const GemmBands &b, const int *n, int seg, int row) {
    int strip = row / 16;
    for (int s = 0; s < seg && !b.paired; ++s) strip += strips_of(n[s]);
    const int band = b.strips == 1 ? strip : (int)__umulhi((uint32_t)strip, b.inverse);
    return {band + seg * b.paired, strip - band * b.strips};
}

__global__ __launch_bounds__(256) void gemm_pack_kernel(PackArgs p) {
    // one block per (band, K step), one thread per 16-byte vector of a 4 KB piece
    const int S = p.bands.strips, ns = p.K / kSkinnyStepK, band = (int)(blockIdx.x / (unsigned)ns), step = (int)(blockIdx.x % (unsigned)ns);
    const int half = p.bands.paired;
    u32x4 *dst = p.dst + (size_t)blockIdx.x * S * 256;
    for (int v = threadIdx.x; v < S * 256; v += 256) {
        const int piece = v >> 6, lane = v & 63, q = piece / S, slot = piece % S, i = lane & 15, gq = lane >> 4;
        int seg = 0, strip = band * S + slot;
        if (p.bands.paired && band >= half) { seg = 1; strip -= half * S; }
        for (; !p.bands.paired && seg < p.nseg - 1 && strip >= strips_of(p.n[seg]); ++seg) strip -= strips_of(p.n[seg]);
        const int row = strip * 16 + i, k = step * kSkinnyStepK + (q >> 1) * 64 + gq * 16 + (q & 1) * 8;
        u32x4 x = u32x4{0u, 0u, 0u, 0u};
        if (row < p.n[seg]) x = *reinterpret_cast<const u32x4 *>(p.w[seg] + (size_t)row * p.K + k);
        dst[v] = x;
    }
}

// first unit of block b when U units are dealt to P blocks in contiguous, near-equal ranges
__host__ __device__ __forceinline__ long range_begin(long b, long U, long P) { return b * U / P; }
// the block whose range holds unit u
__host__ __device__ __forceinline__ long range_owner(long u, long U, long P) { return ((u + 1) * P - 1) / U; }

// The residual epilogue of one 64-column output tile that several blocks contributed partial sums to.  The calling
// thread holds, for column `col` of the tile (the 64 lanes of its wavefront = the tile's 64 columns), this block's
// sums of rows row0, row0 + rstep, ...: it publishes them in partial slot `slot` with agent-scope stores, waits for
// them, and the block counts itself in on the tile's counter.  Whichever block arrives last adds the tile's
// n_contrib slots in slot order (so the sum does not depend on who that was), adds into the residual stream, writes
// the gain-scaled copy and the rows' sums of squares over the tile, and leaves the counter at zero for the next
// launch.  No block waits for another.  Every thread of the block must call it (it synchronises the block).
template <int NR>
__device__ __forceinline__ void resid_tile_finish(const GemmArgs &g, int tile, int slot, int n_contrib, const float (&mine)[NR],
                                                  int row0, int rstep, bool col_ok, size_t col, int *s_last) {
    bool last = true;
    if (n_contrib > 1) {                                        // the same for the whole block
        if (col_ok)
#pragma unroll
            for (int r = 0; r < NR; ++r)
                if (row0 + r * rstep < g.M)
                    __hip_atomic_store(&g.partial[((size_t)slot * g.M + row0 + r * rstep) * g.N + col], mine[r],
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0)
            *s_last = __hip_atomic_fetch_add(&g.tile_counter[tile], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                      (unsigned)(n_contrib - 1);
        __syncthreads();
        last = *s_last != 0;
    }
    if (!last) return;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int tok = row0 + r * rstep;
        float v = 0.f, sq = 0.f;
        if (tok < g.M && col_ok) {
            if (n_contrib > 1) {
                for (int sl = 0; sl < n_contrib; ++sl)
                    v += __hip_atomic_load(&g.partial[((size_t)sl * g.M + tok) * g.N + col], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
            } else {
                v = mine[r];
            }
            const size_t o = (size_t)tok * g.N + col;
            v += g.x_resid[o];
            g.x_resid[o] = v;
            const float xg = v * (g.gain ? bf16_bits_to_f32(((const uint16_t *)g.gain)[col]) : 1.0f);
            if (g.xg_op) op_store(g.xg_op, tok, (int)col, g.op_folded, xg);
            if (g.xg16_out) g.xg16_out[o] = f32_to_f16_bits(xg);
            sq = v * v;
        }
        sq = wave_sum(sq);                                      // the tile's 64 columns of row tok sit in this wavefront
        if ((threadIdx.x & 63) == 0 && tok < g.M && g.sumsq_out) g.sumsq_out[(size_t)tile * g.M + tok] = sq;
    }
    if (n_contrib > 1 && threadIdx.x == 0)
        __hip_atomic_store(&g.tile_counter[tile], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A block of a unit kernel is done with a tile (the tile's last unit, or the end of the block's range): red[q][row][token]
// holds the sums of its four wavefronts.  They are added in wavefront order and the block writes ONE partial, slot =
// its index among the blocks that share the tile (the block that finishes the tile zeroes the slots nobody writes),
// or, RESID, hands them to the arrival epilogue above.  The tile's units are [first, first + upt) of the U that P blocks share.
template <bool RESID, bool FOLD = false>
__device__ __forceinline__ void unit_tile_flush(const GemmArgs &g, const float (&red)[4][kSkinnyRows][17], int tile, long first,
                                                int upt, long U, long P, bool tile_end, int *s_last, const float *s_scale = nullptr) {
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const TileRef t = find_tile(g, tile, kSkinnyRows);
    const long first_owner = g.whole ? blockIdx.x : range_owner(first, U, P);
    const int slot = (int)(blockIdx.x - first_owner);
    const int row = t.row0 + lane;                                  // lane = row of the tile
    const bool row_ok = row < g.n[t.seg];
    const size_t col = (size_t)t.col0 + row;
    constexpr int NR = FOLD ? 2 : 4;
    auto sum = [&](int tok) {
        float v = ((red[0][lane][tok] + red[1][lane][tok]) + red[2][lane][tok]) + red[3][lane][tok];
        if constexpr (FOLD)                                // the products with the remainders stand eight columns further on
            v += ((red[0][lane][tok + 8] + red[1][lane][tok + 8]) + red[2][lane][tok + 8]) + red[3][lane][tok + 8];
        return v;
    };
    if constexpr (RESID) {
        const int n_contrib = (int)(range_owner(first + upt - 1, U, P) - first_owner) + 1;
        float mine[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) mine[r] = sum(q + 4 * r);
        resid_tile_finish<NR>(g, tile, slot, n_contrib, mine, q, 4, row_ok, col, s_last);
    } else if (row_ok) {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int tok = q + 4 * r;
            if (tok < g.M) {
                float v = sum(tok);
                if (s_scale && g.whole) v *= s_scale[tok];
                g.partial[((size_t)slot * g.M + tok) * g.N + col] = v;
                if (tile_end)
                    for (int jj = slot + 1; jj < g.splitk; ++jj) g.partial[((size_t)jj * g.M + tok) * g.N + col] = 0.f;
            }
        }
    }
}

// Block b streams the contiguous units [range_begin(b), range_begin(b + 1)); wavefront q multiplies the q-th 4 KB of
// every unit (K offsets (q>>1)*64 + (q&1)*8 + 16 gq of the unit's 128), so the four wavefronts of a block read 16 KB
// in one piece and the blocks of the grid adjacent ranges: the access pattern of a plain streaming read.  Weights
// and the matching 8 activations per lane travel through a ring of register stages filled by buffer loads that return zeros
// past the end of the block's range, so that every wavefront runs the same straight-line loop, and a stage's data is waited for
// with the other stages still in flight.  At the end of a
// tile (or of the range) the four K quarters are added through LDS in wavefront order and the block writes ONE partial: slot =
// its index among the blocks that share the tile; the block that finishes a tile zeroes the slots nobody writes.
//
// A head whose whole tiles keep the chip busy (gemm_stream_whole) is given out in whole tiles: the block then applies the rows' scale, works
// that out itself (its sums of squares requested ahead of the first weights), and writes the logits: no slot and no reduction
// (128256 x 4096, us with the reduction: 7 rows 166.6 -> 157.6, 14 rows 189.8 -> 171.9).
//
// RESID: every output element still gets one owner, found at run time.  A block publishes its partial with agent-scope stores, waits for
// them, and counts itself in on the tile's counter; whichever block arrives last adds the tile's slots in slot order (so the sum does
// not depend on who that was) and runs the column kernel's epilogue on the tile's 64 columns, sum of squares per row into
// sumsq_out[tile][m].  It leaves the counter at zero for the next launch.  No block waits for another.
//
// Activations: in operand order, two fragments or (folded) one a quarter.  Row-major, as fp32 split here, every lane's 16 bytes come
// out of another line, and at 16 rows they cost the vector memory path twice what the weights do.  Measured, QKV, gate|up and head of
// the 32-layer 7B shape averaged (us a launch; row-major and two stages in an order of the compiler's / this): 1 row 24.0 / 23.6, 8 rows
// 25.1 / 24.7, 9 rows 25.5 / 25.2, 16 rows 27.2 (two tiles at a time) / 26.4; plain reads of the same weights 22.1.  Two tiles at a time,
// which share a K step's activations, gain nothing in operand order (two layers and head, 16 rows 30.6 / 29.7), nor does a fourth stage.
template <bool FOLD, bool RESID>
__global__ __launch_bounds__(256) void gemm_bf16_unit_kernel(GemmArgs g) {
    constexpr int R = 3, XV = FOLD ? 1 : 2;                // units in flight per wavefront (its 4 KB of each)
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int i = lane & 15, gq = lane >> 4;
    const int K = g.K, ns = K / kSkinnyStepK;
    const long U = (long)g.pack_tiles * ns, P = gridDim.x;
    const int u0 = (int)(g.whole ? range_begin(blockIdx.x, g.pack_tiles, P) * ns : range_begin(blockIdx.x, U, P));
    const int u1 = (int)(g.whole ? range_begin(blockIdx.x + 1, g.pack_tiles, P) * ns : range_begin(blockIdx.x + 1, U, P));
    if (g.lens_n && blockIdx.x == 0) advance_lens(g);
    if (u0 >= u1) return;
    const int n_my = u1 - u0;
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        (char *)const_cast<void *>(g.wpack) + (size_t)u0 * kUnitBytes, 0, n_my * kUnitBytes, 0x00020000);
    // whole: sixteen lanes a row take its sums of squares, the first sixteen each now (past the end: zeros)
    __shared__ float s_scale[16];
    const int sm = threadIdx.x >> 4, sl = threadIdx.x & 15;
    const bool scaled = g.whole && g.scale.sumsq;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(g.scale.sumsq), 0,
                                                                        scaled ? g.scale.tiles * g.scale_rows * 4 : 0, 0x00020000);
    const unsigned soff = sm < g.M ? (unsigned)(sl * g.scale_rows + (int)x_row(g, sm)) * 4 : 0x80000000u;
    uint32_t ssq[16];
    if (scaled)
#pragma unroll
        for (int t = 0; t < 16; ++t) ssq[t] = __builtin_amdgcn_raw_buffer_load_b32(rs, soff + (unsigned)(t * 16 * g.scale_rows) * 4, 0, 0);
    // activations: a row past M points past the buffer and reads zeros
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(g.x_op), 0, K * (FOLD ? 32 : 64), 0x00020000);
    constexpr unsigned kStepX = kSkinnyStepK * (FOLD ? 32 : 64);             // bytes from one K step to the next
    const int xm = FOLD ? i & 7 : i;
    const unsigned xbase = xm < g.M ? (unsigned)(q * (FOLD ? 1024 : 2048) + (gq * 16 + (int)x_row(g, xm) + (FOLD ? i & 8 : 0)) * 16) : 0x80000000u;
    const unsigned lane_off = q * 4096u + lane * 16u;

    u32x4 A[R][4], X[R][XV];
    int step_issue = u0 % ns;
    auto issue = [&](int j, int n) {                       // n = index of the unit inside the block's range
        const unsigned xo = n < n_my ? xbase + (unsigned)step_issue * kStepX : 0x80000000u;
        X[j][0] = __builtin_amdgcn_raw_buffer_load_b128(rx, xo, 0, 0);
        if constexpr (!FOLD) X[j][1] = __builtin_amdgcn_raw_buffer_load_b128(rx, xo + 1024, 0, 0);
        const unsigned wo = (unsigned)n * kUnitBytes + lane_off;
#pragma unroll
        for (int s = 0; s < 4; ++s) A[j][s] = __builtin_amdgcn_raw_buffer_load_b128(rw, wo + s * 1024, 0, 2);   // 2: streaming
        step_issue = step_issue + 1 == ns ? 0 : step_issue + 1;
        // The loads stay in this order.  Left to itself the compiler requests the first units in another order than the loop
        // does, and as loads return in order, a wait for one stage is then a wait for all of them.
        __builtin_amdgcn_sched_barrier(0);
    };
    f32x4 acc[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int j) {
        const bf16x8 bh = __builtin_bit_cast(bf16x8, X[j][0]), bl = __builtin_bit_cast(bf16x8, X[j][XV - 1]);
        // hi parts over all accumulators, then lo parts: no back-to-back MFMAs on one accumulator
#pragma unroll
        for (int s = 0; s < 4; ++s)
            acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, A[j][s]), bh, acc[s], 0, 0, 0);
#pragma unroll
        for (int s = 0; s < 4 && !FOLD; ++s)
            acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, A[j][s]), bl, acc[s], 0, 0, 0);
    };
    __shared__ float red[4][kSkinnyRows][17];
    __shared__ int s_last;
    int step_use = u0 % ns, tile = u0 / ns;
    long first = (long)tile * ns;                          // first unit of the tile
#pragma unroll
    for (int j = 0; j < R; ++j) issue(j, j);
    if (scaled) {                                          // (read after the barrier of the first flush)
        float v = 0.f;
#pragma unroll
        for (int t = 0; t < 16; ++t) v += __uint_as_float(ssq[t]);
        for (int t = 256 + sl; t < g.scale.tiles; t += 16)
            v += __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, sm < g.M ? (unsigned)(t * g.scale_rows + (int)x_row(g, sm)) * 4 : 0x80000000u, 0, 0));
        v += __shfl_xor(v, 8, 64);
        v += __shfl_xor(v, 4, 64);
        v += __shfl_xor(v, 2, 64);
        v += __shfl_xor(v, 1, 64);
        if (sl == 0) s_scale[sm] = 1.0f / sqrtf(v * g.scale.inv_d + g.scale.eps);
    } else if (g.whole && threadIdx.x < 16) {
        s_scale[threadIdx.x] = 1.0f;
    }
    for (int base = 0; base < n_my; base += R) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int n = base + j;
            multiply(j);
            issue(j, n + R);
            const bool tile_end = step_use + 1 == ns;
            step_use = tile_end ? 0 : step_use + 1;
            if (n < n_my && (tile_end || n + 1 == n_my)) {                  // the same for all four wavefronts
                // acc[s][v] = y[token i][row s*16 + 4*gq + v of the tile] over this wavefront's K quarter
#pragma unroll
                for (int s = 0; s < 4; ++s) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) red[q][s * 16 + 4 * gq + v][i] = acc[s][v];
                    acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
                __syncthreads();
                unit_tile_flush<RESID, FOLD>(g, red, tile, first, ns, U, P, tile_end, &s_last, s_scale);
                __syncthreads();
            }
            if (tile_end) { ++tile; first += ns; }
        }
    }
}

// ------------------------------------------------------------------------------ bf16 band kernel (M <= 16: QKV, gate|up)
// One block per band of S strips over the whole K range (GATED: the gate band and the up band of the same columns), on weights packed
// in these bands (gemm_qkv_bands, gemm_gate_bands), so that a block streams one contiguous range (GATED: two).  Wavefront (q, half) takes
// K quarter q of the even or the odd steps, through a ring of two; the eight wavefronts' sums meet in LDS.  Every output has one owner:
// QKV scales its rows and writes one partial slot, gate|up scales, applies SwiGLU and writes the operand of the down projection, so neither needs
// partial slots of several blocks to be written and read, nor gate|up the launch that did.
// What bounds it: streaming the weights (180 MB of the 7B shape's gate|up in 31 us = 5.9 TB/s, its QKV of 101 MB in 18 at 15 rows) and the
// fixed cost of a launch.  Against the unit kernel with shared tiles, and the SwiGLU launch behind it, on one box: gate|up 32.5 + 4.9 -> 30.9 us
// and QKV 19.6 -> 18.3 at 15 rows; the 32-layer 7B step at 8 rows 3 340 -> 3 070, two layers of the 8B shape at 11 rows 409 -> 397.
// The blocks begin at different steps of their bands: bands lie a multiple of a large power of two apart, and in step all blocks would
// ask the same channels at once (7B step 3 100 -> 3 079 us; beginnings 1, 3, 4 or 5 steps apart are no better than 2).  One stage in
// flight: 3 135 us, three: 3 123.  Slots of a step ordered strip by strip, or the gate and up strips of a step side by side: no change here,
// the latter 1 % slower in the rows kernel.
template <bool FOLD, int S, bool GATED>
__global__ __launch_bounds__(512) void gemm_bf16_band_kernel(GemmArgs g) {
    constexpr int R = 2, XV = FOLD ? 1 : 2, NS = GATED ? 2 * S : S;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = wave & 3, half = wave >> 2;
    const int i = lane & 15, gq = lane >> 4;
    const int K = g.K, ns = K / kSkinnyStepK;
    // the rows' sums of squares, requested ahead of the first weights: 32 threads a row, the first eight strips or tiles each
    __shared__ float s_scale[16];
    const int sm = threadIdx.x >> 5, sl = threadIdx.x & 31;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(g.scale.sumsq), 0, g.scale.tiles * g.M * 4, 0x00020000);
    const uint32_t soff = sm < g.M ? (uint32_t)(sl * g.M + sm) * 4 : 0x80000000u;
    uint32_t ssq[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) ssq[t] = __builtin_amdgcn_raw_buffer_load_b32(rs, soff + (uint32_t)(t * 32 * g.M) * 4, 0, 0);
    constexpr uint32_t kPiece = S * 1024, kStepW = 4 * kPiece;               // a quarter of a step, a step
    auto band = [&](unsigned b) {
        return __builtin_amdgcn_make_buffer_rsrc((char *)const_cast<void *>(g.wpack) + (size_t)b * ns * kStepW, 0, ns * kStepW, 0x00020000);
    };
    const __amdgpu_buffer_rsrc_t rw = band(blockIdx.x), ru = band(GATED ? blockIdx.x + gridDim.x : blockIdx.x);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(g.x_op), 0, K * (FOLD ? 32 : 64), 0x00020000);
    constexpr uint32_t kStepX = kSkinnyStepK * (FOLD ? 32 : 64);
    const int xm = FOLD ? i & 7 : i;
    const uint32_t xbase = xm < g.M ? (uint32_t)(q * (FOLD ? 1024 : 2048) + lane * 16) : 0x80000000u;       // a row past M reads zeros
    const uint32_t wbase = q * kPiece + lane * 16;
    const int turn = (int)(2 * blockIdx.x % (unsigned)ns);

    u32x4 A[R][NS], X[R][XV];
    auto issue = [&](int j, int n) {                       // this wavefront's n-th step; past the last one, zeros
        const int at = 2 * n + half, step = at + turn < ns ? at + turn : at + turn - ns;
        const uint32_t xo = at < ns ? xbase + (uint32_t)step * kStepX : 0x80000000u, wo = at < ns ? wbase + (uint32_t)step * kStepW : 0x80000000u;
        X[j][0] = __builtin_amdgcn_raw_buffer_load_b128(rx, xo, 0, 0);
        if constexpr (!FOLD) X[j][1] = __builtin_amdgcn_raw_buffer_load_b128(rx, xo + 1024, 0, 0);
#pragma unroll
        for (int s = 0; s < NS; ++s) A[j][s] = __builtin_amdgcn_raw_buffer_load_b128(s < S ? rw : ru, wo + s % S * 1024, 0, 2);      // 2: streaming
        __builtin_amdgcn_sched_barrier(0);                 // (as in the unit kernel: the loads stay in this order)
    };
    f32x4 acc[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int j) {
#pragma unroll
        for (int v = 0; v < XV; ++v)
#pragma unroll
            for (int s = 0; s < NS; ++s)
                acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, A[j][s]), __builtin_bit_cast(bf16x8, X[j][v]), acc[s], 0, 0, 0);
    };
#pragma unroll
    for (int j = 0; j < R; ++j) issue(j, j);
    {
        float v = 0.f;
#pragma unroll
        for (int t = 0; t < 8; ++t) v += __uint_as_float(ssq[t]);
        for (int t = 256 + sl; t < g.scale.tiles; t += 32)
            v += __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, sm < g.M ? (uint32_t)(t * g.M + sm) * 4 : 0x80000000u, 0, 0));
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if (sl == 0) s_scale[sm] = 1.0f / sqrtf(v * g.scale.inv_d + g.scale.eps);
    }
    const int n_my = (ns + 1) / 2;
    for (int base = 0; base + R < n_my; base += R) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            multiply(j);
            issue(j, base + j + R);
        }
    }
#pragma unroll
    for (int j = 0; j < R; ++j) multiply(j);
    // acc[s][v] = y[token i][column 4*gq + v of strip s] over this wavefront's quarters: the odd steps' wavefronts hand theirs over first
    __shared__ float red[4][NS * 16][17];
    if (half)
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[q][s * 16 + 4 * gq + v][i] = acc[s][v];
    __syncthreads();
    if (!half)
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[q][s * 16 + 4 * gq + v][i] += acc[s][v];
    __syncthreads();
    constexpr int kCols = S * 16;
    for (int e = threadIdx.x; e < kCols * (FOLD ? 8 : 16); e += 512) {
        const int col = e % kCols, tok = e / kCols, c = blockIdx.x * kCols + col;
        auto sum = [&](int row) {
            float v = ((red[0][row][tok] + red[1][row][tok]) + red[2][row][tok]) + red[3][row][tok];
            if constexpr (FOLD)                            // the products with the remainders stand eight columns further on
                v += ((red[0][row][tok + 8] + red[1][row][tok + 8]) + red[2][row][tok + 8]) + red[3][row][tok + 8];
            return v;
        };
        if (tok >= g.M || c >= (GATED ? g.n[0] : g.N)) continue;
        if constexpr (GATED) {
            const float gt = sum(col) * s_scale[tok], up = sum(kCols + col) * s_scale[tok];
            op_store(g.swiglu_op, tok, c, FOLD, gt / (1.0f + expf(-gt)) * up);
        } else {
            g.partial[(size_t)tok * g.N + c] = sum(col) * s_scale[tok];
        }
    }
}

// ------------------------------------------------------------------------------ bf16 one-slot column kernel
// For the projections that write the residual stream (N = d_model): one block per 16 output columns over the whole K range,
// its sixteen wavefronts on equal ranges of the K quarters, added through LDS in wavefront order.
// Every output element has a single owner, so the block finishes the job itself: x_resid[m][n] += y[m][n],
// xg_op[m][n] = x_resid[m][n] * gain_next[n] (the operand of the next projection, RMSNorm gain folded in),
// and the sum of squares of the updated 16 columns per row goes to sumsq_out, from which the consumer of the
// next projection derives the RMSNorm scale.  No partial slots, no reduce kernel, no norm kernel.
// Weights are packed strip-major for this kernel (gemm_pack_strip_kernel): strip (16 rows) x K step is 4 KB
// = 4 slots of 1 KB in lane order, all K steps of a strip contiguous, so a block streams one contiguous
// range and a wavefront a contiguous part of it.
// What bounds it: the block reads all activations, at 16 rows twice as many bytes as weights, so how they are read decides.  They
// come in operand order, whole 1 KB pieces, D quarters at a time and ahead of these quarters' weights: the weights, which come
// from farther, are then not waited for twice.  Measured, O and down of the 32-layer 7B shape averaged (us a launch; O so on row-major
// activations and down on the unit kernel with the residual epilogue by the last block to arrive at a tile / this): 1 row
// 14.1 / 13.1, 8 rows 16.3 / 13.4, 9 rows 17.2 / 15.9, 16 rows 20.2 / 16.2; plain reads 10.7.  Weights and activations in turn
// 18.2 at 15 rows; a ring of quarters that is refilled one by one 19.7, most of it for its loads past the end, which cost
// like any other though they touch no memory.  How many quarters at a time hardly matters: 8, 10, 11, 12 or 13 folded and 6 to 9 not are
// within 0.3 us of each other at 1, 8, 9 and 16 rows of 1024 x 4096, 2048 x 5632, 3584 x 18944 and 4096 x 4096, 11008 and 14336; these
// leave no spills at 1024 threads (128 registers).
constexpr int kStripVec = 16 * kSkinnyStepK * 2 / 16;   // 16-byte vectors per (strip, step)

__global__ __launch_bounds__(256) void gemm_pack_strip_kernel(const uint16_t *W, int N, int K, u32x4 *dst) {
    const size_t vec = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int ns = K / kSkinnyStepK;
    const size_t strips = (size_t)((N + kSkinnyRows - 1) / kSkinnyRows) * 4;
    if (vec >= strips * ns * kStripVec) return;
    const size_t strip = vec / ((size_t)ns * kStripVec);
    const int rem = (int)(vec % ((size_t)ns * kStripVec));
    const int step = rem / kStripVec, q = (rem % kStripVec) >> 6, lane = rem & 63;
    const int i = lane & 15, gq = lane >> 4;
    const size_t row = strip * 16 + i;
    const int k = step * kSkinnyStepK + (q >> 1) * 64 + gq * 16 + (q & 1) * 8;
    u32x4 v = u32x4{0u, 0u, 0u, 0u};
    if (row < (size_t)N) v = *reinterpret_cast<const u32x4 *>(W + row * K + k);
    dst[vec] = v;
}

// 4-bit weights (W4A16, asymmetric, groups of 128 along K = one K step): w = scale * (q - zero).  Packed layout
// of one GEMM: tiles of 64 rows, each tile ceil(ns / 4) quads, a quad = four consecutive K steps of the tile
// (K steps past the end of K are stored with scale 0), a step = 4352 bytes: four 1 KB slots of codes, one per
// strip of 16 rows, in lane order (lane (n, gq) owns one 16-byte vector: dword kb holds its eight nibbles of row
// strip*16 + n, K offsets kb*32 + gq*8 ..+7 of the step, element e at bit 4*(e/2) + 16*(e&1), so that
// (dword >> 4p) & 0x000F000F is the element pair (2p, 2p+1)), then 256 bytes of scales and zero points: the word
// of (row n, strip s) at [n][s] holds the bf16 scale in its high half and the fp16 number 1024 + zero (bit
// pattern 0x6400 | zero) in its low half.  The kernel multiplies the nibbles as the exact fp16 integers
// 1024 + q (bit pattern 0x6400 | q) and takes scale * (sum (1024 + q) x - (1024 + zero) sum x) per group, so
// no weight is ever rounded.
constexpr int kW4StepBytes = 4096 + 256;
constexpr int kW4QuadBytes = 4 * kW4StepBytes;
__host__ __device__ __forceinline__ int w4_quads(int K) { return (K / kSkinnyStepK + 3) / 4; }

__global__ __launch_bounds__(64) void gemm_pack_w4_kernel(const uint8_t *Q, const uint16_t *scale, const uint8_t *zero,
                                                          int N, int K, uint8_t *dst) {
    // one block per stored K step: blockIdx.x = tile * (4 * quads) + step
    const int ns = K / kSkinnyStepK, ns4 = 4 * w4_quads(K);
    const size_t tile = blockIdx.x / ns4;
    const int step = blockIdx.x % ns4, lane = threadIdx.x, n = lane & 15, gq = lane >> 4;
    uint8_t *out = dst + (size_t)blockIdx.x * kW4StepBytes;
#pragma unroll
    for (int strip = 0; strip < 4; ++strip) {
        const size_t row = tile * kSkinnyRows + strip * 16 + n;
        u32x4 v = u32x4{0u, 0u, 0u, 0u};
        if (row < (size_t)N && step < ns) {
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                const int k = step * kSkinnyStepK + kb * 32 + gq * 8;
                const uint32_t raw = *reinterpret_cast<const uint32_t *>(Q + (row * K + k) / 2);   // byte b: k + 2b, k + 2b + 1
                uint32_t w = 0;
#pragma unroll
                for (int bb = 0; bb < 4; ++bb) {
                    w |= ((raw >> (8 * bb)) & 0xFu) << (4 * bb);                // element 2 bb
                    w |= ((raw >> (8 * bb + 4)) & 0xFu) << (16 + 4 * bb);       // element 2 bb + 1
                }
                v[kb] = w;
            }
        }
        reinterpret_cast<u32x4 *>(out + strip * 1024)[lane] = v;
    }
    {
        const int strip = lane >> 4;
        const size_t row = tile * kSkinnyRows + strip * 16 + n;
        uint32_t sz = 0x6400u;                                                   // rows and steps past the end: scale 0
        if (row < (size_t)N && step < ns)
            sz = ((uint32_t)scale[row * ns + step] << 16) | (0x6400u | zero[row * ns + step]);   // zero <= 15
        reinterpret_cast<uint32_t *>(out + 4096)[n * 4 + strip] = sz;
    }
}

template <bool FOLD>
__global__ __launch_bounds__(1024) void gemm_bf16_column_kernel(GemmArgs g) {
    constexpr int W = 16, D = FOLD ? 11 : 8, XV = FOLD ? 1 : 2;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i = lane & 15, gq = lane >> 4;
    const int nq = g.K / 32, q0 = wave * nq / W, q1 = (wave + 1) * nq / W;

    // the epilogue's operands, fetched before the main loop: thread t < 256 owns column n = t & 15 of row mm = t >> 4
    const int en = threadIdx.x & 15, tok = threadIdx.x >> 4;
    const int ecol = blockIdx.x * 16 + en;
    const bool mine = tok < g.M;                            // one of the first 256 threads; N is a multiple of 16
    // (buffer loads, for the others out of range: a load under a branch would be waited for where the branch ends)
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(g.x_resid, 0, g.M * g.N * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(g.gain), 0, g.N * 2, 0x00020000);
    const uint32_t e_res = __builtin_amdgcn_raw_buffer_load_b32(rr, mine ? (uint32_t)(tok * g.N + ecol) * 4 : 0x80000000u, 0, 0);
    const uint16_t e_gain = __builtin_amdgcn_raw_buffer_load_b16(rg, (uint32_t)ecol * 2, 0, 0);
    const u32x4 *wp = reinterpret_cast<const u32x4 *>(g.wpack) + (size_t)blockIdx.x * nq * 64 + lane;
    const u32x4 *xp = reinterpret_cast<const u32x4 *>(g.x_op) + lane;                 // rows past M hold anything: their columns are dropped
    f32x4 acc[2];
    acc[0] = acc[1] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 A[D], X[D][XV];
    auto load_x = [&](int j, int qn) {
#pragma unroll
        for (int v = 0; v < XV; ++v) X[j][v] = xp[(size_t)(qn * XV + v) * 64];
    };
    auto load_w = [&](int j, int qn) { A[j] = __builtin_nontemporal_load(wp + (size_t)qn * 64); };
    auto multiply = [&](int j) {
#pragma unroll
        for (int v = 0; v < XV; ++v)
            acc[FOLD ? j & 1 : v] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, A[j]), __builtin_bit_cast(bf16x8, X[j][v]),
                                                                            acc[FOLD ? j & 1 : v], 0, 0, 0);
    };
    int qn = q0;
    for (; qn + D <= q1; qn += D) {
#pragma unroll
        for (int j = 0; j < D; ++j) load_x(j, qn + j);
#pragma unroll
        for (int j = 0; j < D; ++j) load_w(j, qn + j);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < D; ++j) multiply(j);
    }
#pragma unroll
    for (int j = 0; j < D - 1; ++j)
        if (qn + j < q1) load_x(j, qn + j);
#pragma unroll
    for (int j = 0; j < D - 1; ++j)
        if (qn + j < q1) load_w(j, qn + j);
#pragma unroll
    for (int j = 0; j < D - 1; ++j)
        if (qn + j < q1) multiply(j);

    // acc[.][v] = y[token i][column 4*gq + v of the strip] over this wavefront's quarters (FOLD: the products with the
    // remainders stand eight tokens further on)
    __shared__ float red[W][16][17];
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][4 * gq + v][i] = acc[0][v] + acc[1][v];
    __syncthreads();
    if (threadIdx.x < 256) {
        float v = 0.f, sq = 0.f;
        if (tok < (FOLD ? 8 : 16)) {
#pragma unroll
            for (int w = 0; w < W; ++w) v += FOLD ? red[w][en][tok] + red[w][en][tok + 8] : red[w][en][tok];
        }
        if (mine) {
            v += __uint_as_float(e_res);
            g.x_resid[(size_t)tok * g.N + ecol] = v;
            if (g.xg_op) op_store(g.xg_op, tok, ecol, FOLD, v * bf16_bits_to_f32(e_gain));
            sq = v * v;
        }
        // the 16 columns of one row sit in 16 consecutive lanes
        sq += __shfl_xor(sq, 8, 64);
        sq += __shfl_xor(sq, 4, 64);
        sq += __shfl_xor(sq, 2, 64);
        sq += __shfl_xor(sq, 1, 64);
        if (en == 0 && tok < g.M && g.sumsq_out) g.sumsq_out[(size_t)blockIdx.x * g.M + tok] = sq;
    }
}

// ------------------------------------------------------------------------------ 4-bit weights, M <= 16
// The unit kernel's scheme on the 4-bit layout: the unit is a quad (four K steps of a 64-row tile, 17 KB), block b
// streams the contiguous quads [range_begin(b), range_begin(b + 1)), wavefront q multiplies step q of every quad
// (its 4352 contiguous bytes), the four wavefronts' sums meet in LDS at the end of a tile, one partial slot per
// block and tile or the arrival epilogue (O, down).  Codes, scales and activations travel through a ring of
// register stages filled by buffer loads that return zeros past the end of the block's range.
// The activations are the MFMA's row operand here and the weights its column operand, so that a lane holds four
// tokens of ONE weight row per strip and applies that row's scale and zero point as two scalars per group:
// u = sum (1024 + q) x on the matrix cores with the codes as exact fp16 integers, xs = sum x with an all-ones
// operand, then acc += scale * (u - (1024 + zero) * xs) in fp32.  The activations are read from the fp16 copy their
// producers leave beside the fp32 ones (11 significant bits, as for the tiled kernel; activations beyond +-65504
// would overflow): half the bytes every block re-reads from L2, which weigh as much as the 4-bit weights themselves.
constexpr int kW4Ring = 2;                         // quads in flight per wavefront (its K step of each)

// One K step (group) of NS strips: acc[s][v] += y[token 4 gq + v][row i of strip s]; codes, scale words and activations as the packing and
// the fp16 copy hold them (see above)
template <int NS>
__device__ __forceinline__ void w4_step(const u32x4 (&C)[NS], const uint32_t (&S)[NS], const u32x4 (&X)[4], f32x4 (&acc)[NS]) {
    const u32x4 ones4 = u32x4{0x3C003C00u, 0x3C003C00u, 0x3C003C00u, 0x3C003C00u};
    const f16x8 ones = __builtin_bit_cast(f16x8, ones4);
    f32x4 u[NS], xs = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NS; ++s) u[s] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
        const f16x8 xa = __builtin_bit_cast(f16x8, X[kb]);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const uint32_t w = C[s][kb];
            const u32x4 wi = u32x4{(w & 0x000F000Fu) | 0x64006400u, ((w >> 4) & 0x000F000Fu) | 0x64006400u,
                                   ((w >> 8) & 0x000F000Fu) | 0x64006400u, ((w >> 12) & 0x000F000Fu) | 0x64006400u};
            u[s] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa, __builtin_bit_cast(f16x8, wi), u[s], 0, 0, 0);
        }
        xs = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa, ones, xs, 0, 0, 0);       // sum of x over the group
    }
    // u[s][v] = sum over the group of x[token 4 gq + v] * (1024 + q[row s*16 + i]); xs[v] = sum of x[token 4 gq + v]
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const float sc = __uint_as_float(S[s] & 0xffff0000u);
        const float zf = (float)__builtin_bit_cast(_Float16, (uint16_t)(S[s] & 0xffffu));
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[s][v] += sc * (u[s][v] - zf * xs[v]);
    }
}

template <bool RESID>
__global__ __launch_bounds__(256) void gemm_w4_unit_kernel(GemmArgs g) {
    constexpr int R = kW4Ring;
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int i = lane & 15, gq = lane >> 4;
    const int K = g.K, ns = K / kSkinnyStepK, nq = w4_quads(K);
    const long U = (long)g.pack_tiles * nq, P = gridDim.x;
    const int u0 = (int)range_begin(blockIdx.x, U, P), u1 = (int)range_begin(blockIdx.x + 1, U, P);
    if (u0 >= u1) return;
    const int n_my = u1 - u0;
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        (char *)const_cast<void *>(g.wpack) + (size_t)u0 * kW4QuadBytes, 0, n_my * kW4QuadBytes, 0x00020000);
    // activations (the fp16 copy): offsets from the first row's source row; a row past M points past the buffer and
    // reads zeros.  Lane (token i, gq) multiplies K offsets kb*32 + gq*8 ..+7 of its step in MFMA kb.
    const size_t row_first = x_row(g, 0);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(g.x16) + row_first * K, 0, 0x7ffffff0, 0x00020000);
    const unsigned xbase = i < g.M ? (unsigned)((x_row(g, i) - row_first) * K * 2) + gq * 16u : 0x80000000u;

    u32x4 C[R][4], S[R], X[R][4];
    int quad_issue = u0 % nq;
    auto issue = [&](int j, int n) {                       // n = index of the quad inside the block's range
        const unsigned woff = (unsigned)n * kW4QuadBytes + q * kW4StepBytes;
#pragma unroll
        for (int s = 0; s < 4; ++s) C[j][s] = __builtin_amdgcn_raw_buffer_load_b128(rw, woff + s * 1024 + lane * 16u, 0, 2);   // 2: streaming
        S[j] = __builtin_amdgcn_raw_buffer_load_b128(rw, woff + 4096 + i * 16u, 0, 2);
        const int step = quad_issue * 4 + q;
        const unsigned xoff = n < n_my && step < ns ? xbase + (unsigned)step * (kSkinnyStepK * 2) : 0x80000000u;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) X[j][kb] = __builtin_amdgcn_raw_buffer_load_b128(rx, xoff + kb * 64, 0, 0);
        quad_issue = quad_issue + 1 == nq ? 0 : quad_issue + 1;
    };
    f32x4 acc[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
    __shared__ float red[4][kSkinnyRows][17];
    __shared__ int s_last;
#pragma unroll
    for (int j = 0; j < R; ++j) issue(j, j);
    int quad_use = u0 % nq, tile = u0 / nq;
    for (int base = 0; base < n_my; base += R) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int n = base + j;
            if (n >= n_my) break;                                           // the same for all four wavefronts
            const uint32_t sw[4] = {S[j][0], S[j][1], S[j][2], S[j][3]};
            w4_step<4>(C[j], sw, X[j], acc);
            issue(j, n + R);
            const bool tile_end = quad_use + 1 == nq;
            quad_use = tile_end ? 0 : quad_use + 1;
            if (tile_end || n + 1 == n_my) {
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int v = 0; v < 4; ++v) red[q][s * 16 + i][4 * gq + v] = acc[s][v];
                __syncthreads();
                unit_tile_flush<RESID>(g, red, tile, (long)tile * nq, nq, U, P, tile_end, &s_last);
                __syncthreads();
#pragma unroll
                for (int s = 0; s < 4; ++s) acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
            if (tile_end) ++tile;
        }
    }
}

// The 4-bit O and down projections: the column kernel's scheme (one block per 16 output columns, sixteen wavefronts on equal ranges of the K
// steps, one owner per output, its epilogue) on the quad layout, whose steps of a tile are contiguous: a block reads its strip's 1 KB of
// each and the strip's scale words out of the 256 bytes behind them.  What bounds it: the trip to memory and the activations, twice the
// codes' bytes at 7 rows; but a block ends with its own sums, where the unit kernel's end with an arrival (5 us of a launch of 11 or 15).  Two
// layers and a small head, the other projections alike (us, by units / this): 4096 x 14336 1 row 141 / 131, 7 rows 146 / 137, 16 rows
// 172 / 161; 2048 x 8192 7 rows 112 / 94; 1024 x 4096 7 rows 104 / 84.  Not for more than 256 strips, whose blocks come in two rounds, nor
// for a K seven times the width (gemm_down_by_units): 5120 x 13824 7 rows 175 / 190, 8192 x 28672 258 / 297, 4096 x 28672 178 / 178 and
// at 16 rows 209 / 220.
__global__ __launch_bounds__(1024) void gemm_w4_column_kernel(GemmArgs g) {
    constexpr int W = 16, D = 4;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i = lane & 15, gq = lane >> 4;
    const int K = g.K, ns = K / kSkinnyStepK, s0 = wave * ns / W, s1 = (wave + 1) * ns / W, strip = blockIdx.x & 3;
    const size_t tile_bytes = (size_t)w4_quads(K) * kW4QuadBytes;

    const int en = threadIdx.x & 15, tok = threadIdx.x >> 4;                 // (the epilogue's operands: as in the column kernel)
    const int ecol = blockIdx.x * 16 + en;
    const bool mine = tok < g.M;
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(g.x_resid, 0, g.M * g.N * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(g.gain), 0, g.N * 2, 0x00020000);
    const uint32_t e_res = __builtin_amdgcn_raw_buffer_load_b32(rr, mine ? (uint32_t)(tok * g.N + ecol) * 4 : 0x80000000u, 0, 0);
    const uint16_t e_gain = __builtin_amdgcn_raw_buffer_load_b16(rg, (uint32_t)ecol * 2, 0, 0);

    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        (char *)const_cast<void *>(g.wpack) + (blockIdx.x >> 2) * tile_bytes, 0, (int)tile_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(g.x16), 0, g.M * K * 2, 0x00020000);
    const uint32_t xbase = i < g.M ? (uint32_t)(i * K * 2) + gq * 16u : 0x80000000u;      // a row past M reads zeros
    const uint32_t cbase = strip * 1024u + lane * 16u, sbase = 4096u + i * 16u + strip * 4u;
    u32x4 C[D][1], X[D][4];
    uint32_t S[D][1];
    f32x4 acc[1];
    acc[0] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto load_x = [&](int j, int st) {
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) X[j][kb] = __builtin_amdgcn_raw_buffer_load_b128(rx, xbase + (uint32_t)st * (kSkinnyStepK * 2) + kb * 64, 0, 0);
    };
    auto load_w = [&](int j, int st) {
        C[j][0] = __builtin_amdgcn_raw_buffer_load_b128(rw, (uint32_t)st * kW4StepBytes + cbase, 0, 2);      // 2: streaming
        S[j][0] = __builtin_amdgcn_raw_buffer_load_b32(rw, (uint32_t)st * kW4StepBytes + sbase, 0, 0);
    };
    int st = s0;
    for (; st + D <= s1; st += D) {
#pragma unroll
        for (int j = 0; j < D; ++j) load_x(j, st + j);
#pragma unroll
        for (int j = 0; j < D; ++j) load_w(j, st + j);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < D; ++j) w4_step<1>(C[j], S[j], X[j], acc);
    }
#pragma unroll
    for (int j = 0; j < D - 1; ++j)
        if (st + j < s1) load_x(j, st + j);
#pragma unroll
    for (int j = 0; j < D - 1; ++j)
        if (st + j < s1) load_w(j, st + j);
#pragma unroll
    for (int j = 0; j < D - 1; ++j)
        if (st + j < s1) w4_step<1>(C[j], S[j], X[j], acc);

    __shared__ float red[W][16][17];
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][i][4 * gq + v] = acc[0][v];
    __syncthreads();
    if (threadIdx.x < 256) {
        float v = 0.f, sq = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) v += red[w][en][tok];
        if (mine) {
            const size_t o = (size_t)tok * g.N + ecol;
            v += __uint_as_float(e_res);
            g.x_resid[o] = v;
            const float xg = v * bf16_bits_to_f32(e_gain);
            if (g.xg_op) op_store(g.xg_op, tok, ecol, g.op_folded, xg);
            if (g.xg16_out) g.xg16_out[o] = f32_to_f16_bits(xg);
            sq = v * v;
        }
        sq += __shfl_xor(sq, 8, 64);
        sq += __shfl_xor(sq, 4, 64);
        sq += __shfl_xor(sq, 2, 64);
        sq += __shfl_xor(sq, 1, 64);
        if (en == 0 && tok < g.M && g.sumsq_out) g.sumsq_out[(size_t)blockIdx.x * g.M + tok] = sq;
    }
}

// The 4-bit gate|up projection with SwiGLU: one block per tile of 64 columns over the whole K range, four wavefronts on its gate rows and four
// on its up rows, each on one step of every quad; the block scales its rows, applies SwiGLU and writes the fp16 operand of the down projection:
// no partial slots and no launch to add them (two layers of the 8B shape and its head, 7 rows 303 -> 289 us; of 8192 x 28672 274 -> 258).
__global__ __launch_bounds__(512) void gemm_w4_gate_kernel(GemmArgs g) {
    constexpr int R = kW4Ring;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = wave & 3, up = wave >> 2;
    const int i = lane & 15, gq = lane >> 4;
    const int K = g.K, ns = K / kSkinnyStepK, nq = w4_quads(K), tiles = gridDim.x;
    // the rows' sums of squares, requested ahead of the first weights: 32 threads a row, up to eight strips or tiles each (O leaves a sum per
    // strip up to a width of 4096, per tile of 64 columns above: 256 at most)
    __shared__ float s_scale[16];
    const int sm = threadIdx.x >> 5, sl = threadIdx.x & 31;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(g.scale.sumsq), 0, g.scale.tiles * g.M * 4, 0x00020000);
    const uint32_t soff = sm < g.M ? (uint32_t)(sl * g.M + sm) * 4 : 0x80000000u;
    uint32_t ssq[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) ssq[t] = __builtin_amdgcn_raw_buffer_load_b32(rs, soff + (uint32_t)(t * 32 * g.M) * 4, 0, 0);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        (char *)const_cast<void *>(g.wpack) + (size_t)(blockIdx.x + up * tiles) * nq * kW4QuadBytes, 0, nq * kW4QuadBytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(g.x16), 0, g.M * K * 2, 0x00020000);
    const uint32_t xbase = i < g.M ? (uint32_t)(i * K * 2) + gq * 16u : 0x80000000u;
    u32x4 C[R][4], S[R], X[R][4];
    auto issue = [&](int j, int n) {                       // quad n; past the last one, zeros
        const uint32_t woff = (uint32_t)n * kW4QuadBytes + q * kW4StepBytes;
#pragma unroll
        for (int s = 0; s < 4; ++s) C[j][s] = __builtin_amdgcn_raw_buffer_load_b128(rw, woff + s * 1024 + lane * 16u, 0, 2);
        S[j] = __builtin_amdgcn_raw_buffer_load_b128(rw, woff + 4096 + i * 16u, 0, 2);
        const int step = n * 4 + q;
        const uint32_t xoff = step < ns ? xbase + (uint32_t)step * (kSkinnyStepK * 2) : 0x80000000u;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) X[j][kb] = __builtin_amdgcn_raw_buffer_load_b128(rx, xoff + kb * 64, 0, 0);
    };
    f32x4 acc[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int j) {
        const uint32_t sw[4] = {S[j][0], S[j][1], S[j][2], S[j][3]};
        w4_step<4>(C[j], sw, X[j], acc);
    };
#pragma unroll
    for (int j = 0; j < R; ++j) issue(j, j);
    {
        float v = 0.f;
#pragma unroll
        for (int t = 0; t < 8; ++t) v += __uint_as_float(ssq[t]);
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if (sl == 0) s_scale[sm] = 1.0f / sqrtf(v * g.scale.inv_d + g.scale.eps);
    }
    for (int base = 0; base + R < nq; base += R) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            multiply(j);
            issue(j, base + j + R);
        }
    }
#pragma unroll
    for (int j = 0; j < R; ++j) multiply(j);
    __shared__ float red[2][4][kSkinnyRows][17];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[up][q][s * 16 + i][4 * gq + v] = acc[s][v];
    __syncthreads();
    const int row = threadIdx.x & 63, c = blockIdx.x * kSkinnyRows + row;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int tok = (threadIdx.x >> 6) + 8 * t;
        if (tok >= g.M) break;
        const float gt = (((red[0][0][row][tok] + red[0][1][row][tok]) + red[0][2][row][tok]) + red[0][3][row][tok]) * s_scale[tok];
        const float uv = (((red[1][0][row][tok] + red[1][1][row][tok]) + red[1][2][row][tok]) + red[1][3][row][tok]) * s_scale[tok];
        g.swiglu16[(size_t)tok * g.n[0] + c] = f32_to_f16_bits(gt / (1.0f + expf(-gt)) * uv);
    }
}

// ------------------------------------------------------------------------------ bf16 rows kernel (17 to 128 rows, packed weights)
// Between the unit kernel and the tiled one: the weights go from the packed copy straight into MFMA operands, a strip of 16
// rows of W per wavefront and 128 k a step, R steps in flight, and become fp16 (exactly) in registers; the fp16 activations, MT
// tiles of 16 rows, are what a block's wavefronts share and go through LDS, one barrier a step.  They travel
// one step ahead of the weights, so that in the in-order return queue they never wait for them.  NW wavefronts = strips make a tile of
// 16 NW columns.  The grid is one block per CU; block b takes whole tiles (whole) or, where no tile width fills the chip with
// whole ones, an equal range of the product's steps.  gated: whole tiles of NW / 2 gate and as many up strips, whose products
// meet in LDS at the end.
// LDS: fragment (quarter q, tile mt) of a step is 64 lanes x 16 bytes; lane (i, g) lies at 16 g + (i ^ (4 q + g)): threads write
// whole rows, 16 bytes to each of 16 fragments, which without the xor were all in one bank (0.65 us a step).
// GATED is a build of its own: with both epilogues inlined at every ring stage the code of the loop is twice as long, which shows little, in
// launches of one round (a head of 32000 x 4096 at 45 rows 44.8 -> 44.5 us, two layers and head of the 7B shape 333 -> 330.5 on one box;
// boxes differ by more).
constexpr int kRowsBlocks = 256, kRowsMax = 128;

template <int NW, int MT, bool GATED>
__global__ __launch_bounds__(64 * NW) void gemm_bf16_rows_kernel(GemmArgs g) {
    constexpr int R = 4, NT = 64 * NW;
    constexpr int XV = MT * 16 * 16, XCH = (XV + NT - 1) / NT;        // 16-byte vectors of a step of X, per thread
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, gq = lane >> 4;
    const int K = g.K, ns = K / kSkinnyStepK;
    const long U = (long)g.tiled_tiles * ns, P = gridDim.x;
    const int u0 = __builtin_amdgcn_readfirstlane(g.whole ? (int)range_begin(blockIdx.x, g.tiled_tiles, P) * ns : (int)range_begin(blockIdx.x, U, P));
    const int u1 = __builtin_amdgcn_readfirstlane(g.whole ? (int)range_begin(blockIdx.x + 1, g.tiled_tiles, P) * ns : (int)range_begin(blockIdx.x + 1, U, P));
    if (g.lens_n && blockIdx.x == 0) advance_lens(g);
    if (u0 >= u1) return;
    const int n_my = u1 - u0;

    __shared__ __attribute__((aligned(16))) u32x4 s_x[2][4 * MT * 64];
    const size_t x_first = x_row(g, 0);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(g.x16) + x_first * K, 0, 0x7ffffff0, 0x00020000);
    uint32_t xoff[XCH];                                    // consecutive threads: consecutive 16 bytes of a row's 256
#pragma unroll
    for (int c = 0; c < XCH; ++c) {
        const int v = tid + c * NT, m = v >> 4;
        xoff[c] = v < XV && m < g.M ? (uint32_t)((x_row(g, m) - x_first) * K * 2) + (v & 15) * 16 : 0x80000000u;
    }
    u32x4 xr[R][XCH];
    int xs_step = u0 % ns, xs_n = 0;
    auto load_x = [&](int j) {
        const uint32_t dead = xs_n < n_my ? 0u : 0x80000000u;
#pragma unroll
        for (int c = 0; c < XCH; ++c) xr[j][c] = __builtin_amdgcn_raw_buffer_load_b128(rx, (xoff[c] + (uint32_t)xs_step * 256) | dead, 0, 0);
        ++xs_n;
        xs_step = xs_step + 1 == ns ? 0 : xs_step + 1;
        __builtin_amdgcn_sched_barrier(0);                 // (as in the unit kernel: the loads stay in this order)
    };
    auto store_x = [&](int j, int buf) {
#pragma unroll
        for (int c = 0; c < XCH; ++c) {
            const int v = tid + c * NT, m = v >> 4, piece = v & 15;           // piece = (half, lane group, low bit of the quarter)
            const int q = (piece >> 3) * 2 + (piece & 1), gg = (piece >> 1) & 3;
            if (v < XV) s_x[buf][(q * MT + (m >> 4)) * 64 + gg * 16 + ((m & 15) ^ (q * 4 + gg))] = xr[j][c];
        }
    };

    const uint32_t piece_w = (uint32_t)g.bands.strips * 1024u, step_w = 4 * piece_w;       // a quarter of a band's step, a step
    u32x4 A[R][4];
    int is_step = u0 % ns, is_tile = u0 / ns, is_n = 0;
    __amdgpu_buffer_rsrc_t rw;
    struct Strip { int seg, row, col0; };                  // which matrix, its first row there, the matrix' first output column
    auto strip_of = [&](int tile) {                        // this wavefront's strip of a tile
        if constexpr (GATED) return Strip{wave < NW / 2 ? 0 : 1, (tile * (NW / 2) + wave % (NW / 2)) * 16, 0};
        else {
            const TileRef t = find_tile(g, tile, 16 * NW);
            return Strip{t.seg, t.row0 + wave * 16, t.col0};
        }
    };
    auto set_tile = [&]() {                                // the buffer: the strip of the tile to request
        const Strip t = strip_of(is_tile < g.tiled_tiles ? is_tile : 0);
        const bool there = is_n < n_my && t.row < g.n[t.seg];
        const BandRef at = band_of(g.bands, g.n, t.seg, t.row);
        rw = __builtin_amdgcn_make_buffer_rsrc((char *)const_cast<void *>(g.wpack) + (there ? (size_t)at.band * ns * step_w + at.slot * 1024 : 0), 0,
                                               there ? ns * step_w - at.slot * 1024 : 0, 0x00020000);
    };
    set_tile();
    auto issue = [&](int j) {
        const uint32_t at = (lane * 16u + (uint32_t)is_step * step_w) | (is_n < n_my ? 0u : 0x80000000u);
#pragma unroll
        for (int q = 0; q < 4; ++q) A[j][q] = __builtin_amdgcn_raw_buffer_load_b128(rw, at + q * piece_w, 0, 2);       // 2: streaming
        ++is_n;
        if (++is_step == ns) { is_step = 0; ++is_tile; set_tile(); }
        __builtin_amdgcn_sched_barrier(0);
    };
    f32x4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    // acc[mt][v] = y[token mt*16 + i][row wave*16 + 4*gq + v of the tile]
    __shared__ __attribute__((aligned(16))) f32x4 s_up[GATED ? NW / 2 : 1][MT][64];
    auto flush = [&](int tile) {
        const Strip t = strip_of(tile);
        if constexpr (GATED) {
            if (wave >= NW / 2)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) s_up[wave - NW / 2][mt][lane] = acc[mt];
            __syncthreads();
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int m = mt * 16 + i;
                const f32x4 gt = acc[mt];
                acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (wave >= NW / 2 || m >= g.M || t.row >= g.n[0]) continue;
                const f32x4 up = s_up[wave][mt][lane];
                f32x4 h;
#pragma unroll
                for (int v = 0; v < 4; ++v) h[v] = gt[v] / (1.0f + expf(-gt[v])) * up[v];
                *reinterpret_cast<uint2 *>(g.swiglu16 + (size_t)m * g.n[0] + t.row + 4 * gq) =
                    make_uint2(f32_to_f16_bits(h[0]) | ((uint32_t)f32_to_f16_bits(h[1]) << 16),
                               f32_to_f16_bits(h[2]) | ((uint32_t)f32_to_f16_bits(h[3]) << 16));
            }
            // (the barrier of the next step stands before s_up is written again)
        } else {
            const int slot = g.whole ? 0 : (int)(blockIdx.x - range_owner((long)tile * ns, U, P));
            const int zero_to = (tile + 1) * ns <= u1 ? g.splitk : 0;
            const bool vec = g.N % 4 == 0 && (uintptr_t)g.partial % 16 == 0;               // (whole tiles of the head go to the caller's logits)
            const int row = t.row + 4 * gq, rows = g.n[t.seg] - row;                       // rows of the four that exist
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int m = mt * 16 + i;
                const f32x4 r = acc[mt];
                acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (m >= g.M) continue;
                float *p = g.partial + ((size_t)slot * g.M + m) * g.N + t.col0 + row;
                for (int sl = slot; sl == slot || sl < zero_to; ++sl, p += (size_t)g.M * g.N) {
                    const f32x4 o = sl == slot ? r : f32x4{0.f, 0.f, 0.f, 0.f};
                    if (rows >= 4 && vec) *reinterpret_cast<f32x4 *>(p) = o;
                    else
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            if (v < rows) p[v] = o[v];
                }
            }
        }
    };
    load_x(0);
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if (j + 1 < R) load_x(j + 1);
        issue(j);
    }
    store_x(0, 0);
    load_x(0);
    int use_step = u0 % ns, tile = u0 / ns;
    for (int base = 0; base < n_my; base += R) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if (base + j >= n_my) break;                   // the same for all wavefronts
            __syncthreads();
            store_x((j + 1) % R, (j + 1) & 1);
            load_x((j + 1) % R);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f16x8 w = __builtin_bit_cast(f16x8, bf16x8_to_f16x8(A[j][q]));
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                        w, __builtin_bit_cast(f16x8, s_x[j & 1][(q * MT + mt) * 64 + gq * 16 + (i ^ (q * 4 + gq))]), acc[mt], 0, 0, 0);
            }
            issue(j);
            if (++use_step == ns || base + j + 1 == n_my) { flush(tile); use_step = 0; ++tile; }
        }
    }
}

typedef __attribute__((ext_vector_type(2))) uint32_t uint2v;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
// 8 four-bit codes (element e in bits 4e .. 4e+3) -> 8 fp16 weights scale * (q - zero); sz = fp16 scale in the high
// half, fp16 1024 + zero in the low half
__device__ __forceinline__ u32x4 w4x8_to_f16x8(uint32_t raw, uint32_t sz) {
    const _Float16 zf = __builtin_bit_cast(_Float16, (uint16_t)(sz & 0xffffu));
    const _Float16 sf = __builtin_bit_cast(_Float16, (uint16_t)(sz >> 16));
    const f16x2 z2 = f16x2{zf, zf}, s2 = f16x2{sf, sf};
    u32x4 r;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const uint32_t t = raw >> (8 * p);
        const uint32_t pair = (t & 0xFu) | ((t & 0xF0u) << 12) | 0x64006400u;   // fp16 1024 + q of elements 2p, 2p+1
        r[p] = __builtin_bit_cast(uint32_t, (__builtin_bit_cast(f16x2, pair) - z2) * s2);
    }
    return r;
}

// ------------------------------------------------------------------------------ tiled (M > 16)
// Block tile 64 TA rows of activations x 32 TB WN rows of W x 64 of K; wavefronts in a 2 x WN grid, each on 32 TA x 32 TB
// outputs, so that per 16-wide K step a wavefront reads TA + TB operands from LDS for TA TB MFMAs.
// Both operands enter the matrix cores as fp16, one product each: the bf16 weights convert to fp16 exactly
// (8 significant bits into 11; only magnitudes below 7.6e-6 fall under the fp16 grid and are rounded to it, by at
// most 3e-8), the fp32 activations are rounded to fp16 (11 significant bits, the error of bf16 divided by 8),
// which keeps the logits of the 7B-shaped models within 2e-2 of the fp64 result at half the MFMA issue of a
// bf16 high + low pair.  Activations beyond +-65504 would overflow; none of the decoder's normalised or gated
// activations come near.  Rows are padded to 72 elements (144 B): conflict-free 16-byte reads.  LDS is dynamic.
//
// What bounds it.  With many rows: not one thing.  At 2048 x 8192 x 8192 the MFMAs and the barrier alone run at 1.57 PFLOP/s, with the LDS
// reads and stores 1.31, with the global loads too 1.12 (reading both operands from L2 only gains nothing; tiles alone enter a CU at 80
// to 99 B/ns while the blocks of an XCD are in step): about 30 % go outside the MFMAs.  The clock, which falls with what the operands make
// the chip spend, is another part: 2001 x 11008 x 4096 takes 185 us on normal operands and 129 (1.39 PFLOP/s) on all-zero ones,
// 2001 x 4096 x 22016 396 and 281.  Of 129 to 256 rows, one row of 256-row tiles, a narrow product leaves CUs without a tile (256 x 3584 x 3584:
// 112 blocks).  So the K loop is one straight line without a branch: every load is a buffer load whose range says
// what exists (rows past the end and K tiles past the last read nothing), the next tile goes into a second set of LDS
// tiles spread over three of the four MFMA groups of the current one, its registers are refilled with the tile after
// it at once, the operands of the next 16 K are read ahead of the MFMAs of the current ones, and there is one barrier
// per tile.  Measured against the branchy loop before it (2001 rows, us): 12288 x 4096 243 -> 224, 22016 x 4096 451 ->
// 364 (which also drops a SwiGLU launch of 46), 4096 x 8192 148 -> 127, 4096 x 4096 87 -> 70.
// With few rows: streaming W; the blocks take equal ranges of all the product's K tiles (unless the product is so wide that whole
// tiles are the better choice), so none of the CUs idles in a last round.  Measured (45 rows, us): 12288 x 4096 32.5 -> 25.9, 22016 x 4096 47.1 -> 42.3, 4096 x 4096 14.7 -> 10.4,
// 32000 x 4096 78.8 -> 59.1 (4.4 TB/s).  Up to 64 rows two blocks of 128 columns share a CU, so that one's loads cover the
// other's barriers and its write-out (one block of 256: 26.8 / 26.1, 41.9 / 41.0, 10.3 / 9.8, 4096 x 8192 16.5 / 15.9; two
// layers and a head of the 7B shape 384 -> 374); at 65 to 128 rows that gains nothing (128 x 12288 x 4096 35.5 / 37.3).
// Neither does a second K tile in registers (26.5), nor asking for both halves of a 256-byte row piece together (28.5),
// nor reading the weights from the packed copy in contiguous 8 KB pieces (27.3).
// Tried and not kept: an order of reads, stores and MFMAs held by scheduling barriers (1 to 5 % slower), prefetches of later K tiles into L2
// (3 %), four wavefronts of 128 x 128 with the activations straight into three stages of LDS (10 %; zeros 156 us for the 129 above),
// 256 x 160 gate|up tiles for 256 rows (96 -> 95 us); tiles shared by several blocks added up by the last of them (256 x 256 fp32 through agent-scope
// stores and loads: 140 us instead of 70 at 2001 x 4096 x 4096); an XCD-contiguous block order alone (no change: not
// bound by L2 misses); four wavefronts of 128 x 128 (5 % slower than eight of 128 x 64: one wavefront per SIMD does not
// cover its own load issue).
constexpr int kBK = 64, kLdsStride = 72;

// W4: the weights are 4-bit codes as the caller stores them (row-major, low nibble = even k) with a bf16 scale and
// a zero point per row and group of 128 k.  A thread's 8 weights of a K tile are 4 bytes of codes; on the way into
// LDS they become the fp16 numbers scale * (q - zero): (1024 + q) - (1024 + zero) is exact in fp16, the product
// with the scale (itself exact in fp16 down to 6e-5) is rounded once, to 11 significant bits.
template <int TA, int TB, int WN, bool W4>
__global__ __launch_bounds__(128 * WN, TA == 1 ? 4 : 1) void gemm_f16_tiled_kernel(GemmArgs g) {
    constexpr int BM = 64 * TA, BN = 32 * TB * WN, NT = 128 * WN;
    constexpr int XCH = BM * 8 / NT;                        // 16-byte chunks of the fp16 X tile per thread (BM x 64)
    constexpr int WCH = BN * 8 / NT;                        // 16-byte chunks of the W tile per thread (BN x 64 bf16)
    constexpr int kSet = (BM + BN) * kLdsStride;            // elements of one set of tiles
    extern __shared__ __attribute__((aligned(16))) uint16_t lds_tiled[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 31, lg = lane >> 5;
    const int wm = (wave / WN) * (BM / 2), wn = (wave % WN) * (32 * TB);   // this wavefront's corner of the block tile
    const int K = g.K, nk = K / kBK, m_tiles = (g.M + BM - 1) / BM;
    const bool moves_lens = g.lens_n > 0 && blockIdx.x == 0;
    const bool gated = g.swiglu16 != nullptr;
    // Blocks that follow each other in the work order share weight tiles: they go to the same XCD (dispatch is round
    // robin over the eight), whose L2 then serves the second reader.
    const int P = g.blocks, xcd = blockIdx.x % 8;
    const int blk = xcd * (P / 8) + min(xcd, P % 8) + (int)blockIdx.x / 8;
    const long U = (long)g.tiled_tiles * nk;
    const int u0 = __builtin_amdgcn_readfirstlane((int)range_begin(blk, U, P));
    const int u1 = __builtin_amdgcn_readfirstlane((int)range_begin(blk + 1, U, P));

    // LDS byte addresses of this thread's chunks and operands: stores go to one set of tiles, reads to the other.  They are
    // opaque to the compiler, which would otherwise keep one register per (set, chunk, K step) instead of a base and
    // an immediate offset.
    const int col = (tid & 7) * 8;
    uint32_t st_x = (uint32_t)((tid >> 3) * kLdsStride + col) * 2, st_w = st_x + BM * kLdsStride * 2;
    uint32_t rd_x = (uint32_t)(kSet + (wm + li) * kLdsStride + lg * 8) * 2;
    uint32_t rd_w = (uint32_t)(kSet + (BM + wn + li) * kLdsStride + lg * 8) * 2;
    asm volatile("" : "+v"(st_x), "+v"(st_w), "+v"(rd_x), "+v"(rd_w));
    int flip = -kSet * 2;                                   // bytes from the set that is read to the other one
    auto swap_sets = [&]() { rd_x += flip; rd_w += flip; flip = -flip; st_x += flip; st_w += flip; };
    char *lds = (char *)lds_tiled;
    constexpr int kChunkStep = NT / 8 * kLdsStride * 2;      // a thread's chunks are NT / 8 rows apart
    using WReg = std::conditional_t<W4, uint2v, u32x4>;   // what a thread holds of one 8-weight chunk
    u32x4 xr[XCH];
    WReg wr[WCH];

    for (int u = u0; u < u1;) {
        const int tile = __builtin_amdgcn_readfirstlane(u / nk), k0 = u - tile * nk, k1 = min(nk, k0 + u1 - u);
        u += k1 - k0;
        const int n_tile = __builtin_amdgcn_readfirstlane(tile / m_tiles), m_base = (tile - n_tile * m_tiles) * BM;
        // tile row r of W: row r of the segment's tile, or, gated, 32 gate rows and 32 up rows in turn, so that a lane
        // ends up with both factors of its outputs
        TileRef t;
        if (gated) t = TileRef{__builtin_amdgcn_readfirstlane(tid >> 8), n_tile * (BN / 2), 0};
        else t = find_tile(g, n_tile, BN);
        const int seg_rows = g.n[t.seg], w_rows = min(seg_rows - t.row0, gated ? BN / 2 : BN);
        const int r_first = gated ? (tid >> 3) & 31 : tid >> 3, r_step = gated ? 32 : NT / 8;
        const size_t x_first = x_row(g, m_base);
        const char *xbase = (const char *)(g.x16 + x_first * K);
        const char *wbase = (const char *)g.w[t.seg] + (size_t)t.row0 * K * (W4 ? 1 : 4) / 2;
        const int ng = K / kSkinnyStepK;
        const char *sbase = (const char *)g.w4_scale[t.seg] + (size_t)t.row0 * ng * 2;
        const char *zbase = (const char *)g.w4_zero[t.seg] + (size_t)t.row0 * ng;
        uint32_t xoff[XCH];
#pragma unroll
        for (int c = 0; c < XCH; ++c) {
            const int row = (tid + c * NT) >> 3;
            xoff[c] = m_base + row < g.M ? (uint32_t)((x_row(g, m_base + row) - x_first) * K + col) * 2u : 0x80000000u;
        }
        // chunks [C0, C1) of K tile kt: the X chunks first, then the W chunks.  Past the last K tile, and for rows past the
        // end of a matrix, nothing is read.
        auto load = [&](int kt, auto c0, auto c1) {
            constexpr int C0 = decltype(c0)::value, C1 = decltype(c1)::value;
            const bool live = kt < k1;
            const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<char *>(xbase) + (size_t)kt * (kBK * 2), 0, live ? 0x7fffffff : 0, 0x00020000);
            const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<char *>(wbase) + (size_t)kt * (W4 ? kBK / 2 : kBK * 2), 0,
                live ? (w_rows * K - kt * kBK) * (W4 ? 1 : 4) / 2 : 0, 0x00020000);
#pragma unroll
            for (int c = C0; c < C1; ++c) {
                if (c < XCH) xr[c] = __builtin_amdgcn_raw_buffer_load_b128(rx, xoff[c < XCH ? c : 0], 0, 0);
                if (c >= XCH) {
                    const int w = c >= XCH ? c - XCH : 0, row = r_first + w * r_step;
                    if constexpr (W4) {
                        const int grp = kt * kBK / kSkinnyStepK;
                        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                            const_cast<char *>(sbase) + (size_t)grp * 2, 0, live ? (w_rows * ng - grp) * 2 : 0, 0x00020000);
                        const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(
                            const_cast<char *>(zbase) + grp, 0, live ? w_rows * ng - grp : 0, 0x00020000);
                        wr[w][0] = __builtin_amdgcn_raw_buffer_load_b32(rw, (uint32_t)(row * K + col) / 2, 0, 0);
                        const uint32_t sc = __builtin_amdgcn_raw_buffer_load_b16(rs, row * ng * 2, 0, 0);
                        const uint32_t z = __builtin_amdgcn_raw_buffer_load_b8(rz, row * ng, 0, 0);
                        wr[w][1] = (sc << 16) | (z & 0xffu);
                    } else {
                        wr[w] = __builtin_amdgcn_raw_buffer_load_b128(rw, (uint32_t)(row * K + col) * 2, 0, 0);
                    }
                }
            }
        };
        auto store = [&](auto c0, auto c1) {
            constexpr int C0 = decltype(c0)::value, C1 = decltype(c1)::value;
#pragma unroll
            for (int c = C0; c < C1; ++c) {
                if (c < XCH) *reinterpret_cast<u32x4 *>(lds + st_x + c * kChunkStep) = xr[c < XCH ? c : 0];
                if (c >= XCH) {
                    const int w = c >= XCH ? c - XCH : 0;
                    if constexpr (W4) {
                        const _Float16 sc = (_Float16)__uint_as_float(wr[w][1] & 0xffff0000u);
                        const uint32_t sz = ((uint32_t)__builtin_bit_cast(uint16_t, sc) << 16) | 0x6400u | (wr[w][1] & 0xffu);
                        *reinterpret_cast<u32x4 *>(lds + st_w + w * kChunkStep) = w4x8_to_f16x8(wr[w][0], sz);
                    } else {
                        *reinterpret_cast<u32x4 *>(lds + st_w + w * kChunkStep) = bf16x8_to_f16x8(wr[w]);
                    }
                }
            }
        };
        f32x16 acc[TA][TB];
#pragma unroll
        for (int a = 0; a < TA; ++a)
#pragma unroll
            for (int b = 0; b < TB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
        // operands of one 16-wide K step, two register sets: the reads of step ks + 1 are out while step ks is multiplied
        f16x8 fa[2][TA], fb[2][TB];
        auto read_frags = [&](auto buf, int ks) {
            constexpr int q = decltype(buf)::value;
#pragma unroll
            for (int a = 0; a < TA; ++a) fa[q][a] = *reinterpret_cast<const f16x8 *>(lds + rd_x + (a * 32 * kLdsStride + ks * 16) * 2);
#pragma unroll
            for (int b = 0; b < TB; ++b) fb[q][b] = *reinterpret_cast<const f16x8 *>(lds + rd_w + (b * 32 * kLdsStride + ks * 16) * 2);
        };
        auto mma = [&](auto buf) {
            constexpr int q = decltype(buf)::value;
#pragma unroll
            for (int a = 0; a < TA; ++a)
#pragma unroll
                for (int b = 0; b < TB; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[q][a], fb[q][b], acc[a][b], 0, 0, 0);
        };
        using F0 = std::integral_constant<int, 0>;
        using F1 = std::integral_constant<int, 1>;
        // the chunks in three groups, stored in the first three of a K tile's four regions
        constexpr int kAll = XCH + WCH, kG1 = (kAll + 1) / 3, kG2 = (2 * kAll + 1) / 3;
        constexpr std::integral_constant<int, 0> c_0{};
        constexpr std::integral_constant<int, kG1> c_1{};
        constexpr std::integral_constant<int, kG2> c_2{};
        constexpr std::integral_constant<int, kAll> c_3{};
        load(k0, c_0, c_3);
        store(c_0, c_3);
        load(k0 + 1, c_0, c_3);
        swap_sets();
        __syncthreads();
        read_frags(F0{}, 0);
        for (int kt = k0; kt < k1; ++kt) {
            // (every access to the set that is read is done before the barrier, every store into the other set too)
            read_frags(F1{}, 1);
            store(c_0, c_1);
            load(kt + 2, c_0, c_1);
            mma(F0{});
            __builtin_amdgcn_sched_barrier(0);
            read_frags(F0{}, 2);
            store(c_1, c_2);
            load(kt + 2, c_1, c_2);
            mma(F1{});
            __builtin_amdgcn_sched_barrier(0);
            read_frags(F1{}, 3);
            store(c_2, c_3);
            mma(F0{});
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
            swap_sets();
            read_frags(F0{}, 0);
            load(kt + 2, c_2, c_3);
            mma(F1{});
            __builtin_amdgcn_sched_barrier(0);
        }

        // acc[a][b][v] = y[m_base + wm + a*32 + 8*(v/4) + 4*lg + v%4][tile column wn + b*32 + li] over K tiles [k0, k1)
        if (gated) {                                         // the host gives these tiles to one block each
            if constexpr (TB == 2) {
                const int c = n_tile * (BN / 2) + (wave % WN) * 32 + li;
#pragma unroll
                for (int a = 0; a < TA; ++a)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int m = m_base + wm + a * 32 + 8 * (v >> 2) + 4 * lg + (v & 3);
                        const float gt = acc[a][0][v], h = gt / (1.0f + expf(-gt)) * acc[a][1][v];
                        if (m < g.M) g.swiglu16[(size_t)m * seg_rows + c] = f32_to_f16_bits(h);
                    }
            }
            continue;
        }
        const int slot = blk - __builtin_amdgcn_readfirstlane((int)range_owner((long)tile * nk, U, P));
        const int zero_to = k1 == nk ? g.splitk : 0;         // the block that ends a tile clears the slots nobody writes
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            const int row = t.row0 + wn + b * 32 + li;
            if (row >= seg_rows) continue;
#pragma unroll
            for (int a = 0; a < TA; ++a)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int m = m_base + wm + a * 32 + 8 * (v >> 2) + 4 * lg + (v & 3);
                    if (m < g.M) store_out(g, slot, m, t.col0 + row, acc[a][b][v]);
                }
            for (int s = slot + 1; s < zero_to; ++s)
#pragma unroll
                for (int a = 0; a < TA; ++a)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int m = m_base + wm + a * 32 + 8 * (v >> 2) + 4 * lg + (v & 3);
                        if (m < g.M) store_out(g, s, m, t.col0 + row, 0.f);
                    }
        }
    }
    if (moves_lens) advance_lens(g);
}

int tiles_of(const int *n, int nseg, int rows) {
    int t = 0;
    for (int s = 0; s < nseg; ++s) t += (n[s] + rows - 1) / rows;
    return t;
}

}  // namespace

static int gemm_slots_of(int tiles, int units_per_tile, int grid);
// The rows kernel's tile width and grid.  Whole tiles need no partial slots, no zeroed ones and, in the head, no reduction; so the width
// of 96, 128 or 160 columns whose whole tiles leave the fewest CUs idle is taken, if that is at most 15 % of them; else tiles of 128
// are shared, if that gives every block ten steps (below, the tiled kernel's more and shorter blocks start and end sooner).  Measured
// (45 rows, us with the reduction; tiled kernel / this; columns x K): 32000 x 4096 66.4 / 45.0 (98 % of the CUs), 28672 x 4096 60.9 /
// 41.1 (87 %), 22016 x 4096 45.1 / 35.2 (96 columns, 90 %), 152064 x 3584 229 / 201, 12288 x 4096 shared 30.8 / 29.3, 4608 x 3584
// shared 13.6 / 18.3.  From 65 rows on the operands read from LDS, 4 MT KB a wavefront and step, weigh as much as the weights: one
// round of whole tiles still gains (96 rows, 32000 x 4096 79.1 / 60.1, 22016 x 4096 57.8 / 53.3; 128 rows, 85.4 / 70.5, 28672 x 4096
// 79.5 / 68.7), more rounds (128 x 152064 x 3584 266 / 281), shared tiles (128 x 12288 x 4096 43.8 / 45.7), ten wavefronts, whose
// registers spill (two layers and head of the Qwen2-7B shape, 88 rows 631 / 641), or, above 96 rows, six (128 x 22016 x 4096 with
// SwiGLU 67.6 / 66.9, two layers of the 7B shape 494 / 506) do not; nor do products of fewer than six K steps, most of whose time is the
// outputs, here in pieces of 64 bytes (a layer and head 32000 x 512, 96 rows 77.5 / 80.6, 128 rows 79.9 / 85.1; 32000 x 768 102.5 / 93.2).
RowsPlan gemm_rows_plan(int M, int K, const int *n, int nseg, bool gated) {
    RowsPlan p{};
    if (M <= kStreamMaxRows || M > kRowsMax) return p;
    const int ns = K / kSkinnyStepK;
    if (M > 64 && !gated && ns < 6) return p;
    double best = 0.85;
    for (int nw : {8, 6, 10}) {
        const int tiles = gated ? (n[0] + 8 * nw - 1) / (8 * nw) : tiles_of(n, nseg, 16 * nw);
        const int rounds = (tiles + kRowsBlocks - 1) / kRowsBlocks;
        const double busy = (double)tiles / (rounds * kRowsBlocks);
        if (busy < best || (M > 64 && (rounds > 1 || nw > 8)) || (M > 96 && nw < 8)) continue;
        best = busy + 0.01;                                 // (a later width has to be clearly better)
        p.used = p.whole = true;
        p.waves = nw;
        p.tiles = tiles;
        p.blocks = tiles < kRowsBlocks ? tiles : kRowsBlocks;
        p.slots = 1;
    }
    if (p.used || gated || M > 64) return p;
    p.waves = 8;
    p.tiles = tiles_of(n, nseg, 128);
    p.used = (long)p.tiles * ns >= 10 * kRowsBlocks;
    p.blocks = kRowsBlocks;
    if (p.used) p.slots = gemm_slots_of(p.tiles, ns, p.blocks);
    return p;
}
constexpr long kTallKTiles = 1600;
static int few_row_tile(int M, int K, const int *n, int nseg) {         // 64-row halves of the block tile of up to 128 rows
    return M <= 64 || (long)tiles_of(n, nseg, 256) * (K / kBK) < kTallKTiles ? 1 : 2;
}
// Whether a product of up to 128 rows leaves its tiles whole.  Sharing them fills the last round of blocks but gives most
// outputs a second partial slot, to be written, read and added.  Both losses are estimates (us) fitted to heads of 65 700 to
// 256 000 columns at K = 2048 and 4096: an idle share of the last round costs what its K tiles take, half of that from the
// third round on, where the blocks have drifted apart; a second slot costs more the more rows there are.  Tiled launch and
// reduction, shared / whole, K = 4096: 64 rows x 65 700 columns 196 / 242, x 100 352 258 / 252, x 256 000 555 / 471; 18 x
// 151 936 288 / 307; 128 x 73 448 266 / 284, x 100 352 321 / 283, x 256 000 668 / 495; K = 2048: 32 x 140 000 175 / 190,
// 64 x 110 000 170 / 158, 128 x 65 700 174 / 157.
bool gemm_tiles_whole(int M, int K, const int *n, int nseg, bool packed) {
    if (packed) {
        const RowsPlan r = gemm_rows_plan(M, K, n, nseg, false);
        if (r.used) return r.whole;
    }
    const int ta = few_row_tile(M, K, n, nseg), nk = K / kBK, tiles = tiles_of(n, nseg, 128 * ta) * (M <= 64 * ta ? 1 : 2);
    const int cap = 512 / ta, idle = (cap - tiles % cap) % cap;
    if (tiles < cap) return false;
    const double tail = (double)idle / cap * nk * (ta == 1 ? 1.6 : 1.9) * (tiles < 2 * cap ? 1.0 : 0.5);
    const double slot = ta == 1 ? (0.6 * M + 14.0) * (0.25 + 0.75 * nk / 64.0) : (0.3 * M + 52.0) * (0.36 + 0.64 * nk / 64.0);
    return tail < slot;
}
// The tile and the number of blocks of a tiled product.  Up to 128 rows it streams W: two blocks of 128 columns per CU up to
// 64 rows, one of 256 above, but at least eight K tiles each (45 rows x 4096 x 4096 in tiles of 256: 128 blocks 11.2 us and
// 16 slots less to add than 256 blocks, 11.6), tiles shared wherever the ranges fall.  Two exceptions, us of a two-layer pass'
// tiled launches and their reductions, without / with:
//   - the tiles of a wide head may be given out whole (gemm_tiles_whole);
//   - 65 to 128 rows of a product with fewer than 1600 K tiles of 256 columns, which would leave CUs idle, take 64-row tiles
//     of 128 columns and read W twice (d_model 256, 100 rows: 176 / 114; 768: 217 / 145; LLaMA3-8B shape, whose QKV and O
//     are of this kind, 540 / 527; a head of 32000 x 1024, 2000 K tiles, is 6 us slower this way).
// Above: 256 rows; the columns and the (even) K split with the least estimated
// time: rounds of 256 blocks x K tiles x the measured time of one (us: 1.15, 1.65, 1.9 for 128, 192, 256 columns) plus 4
// per round for filling and emptying the pipeline, plus a partial slot of M x N written and read at about 3 TB/s per
// split; or, where a last round would leave CUs idle, two launches: whole rounds of 256 or 192 columns, then the rest of the
// columns in narrower tiles, 3 us more for the launch (bf16).  One launch / two: 2001 x 12288 x 4096 230 / 218 us, 4096 x 6144 x
// 4096 219 / 210, 4096 x 4608 x 3584 174 / 158, 256 x 152064 x 3584 340 / 326, 1024 x 152064 x 3584 1109 / 1090; where the estimate
// is less than 2 % lower nothing is won (512 x 152064 x 3584 572 / 582, 272 x 152064 504 / 506).  gated: 128 gate and 128 up columns
// per tile, never split (the two factors meet in one lane).
// tiled_rest: the columns of each segment that are left behind the first `tiles` tiles of `cols` columns
static void tiled_rest(const int *n, int nseg, int cols, int tiles, int *rest) {
    for (int s = 0; s < nseg; ++s) {
        const int t = (n[s] + cols - 1) / cols, done = tiles < t ? tiles : t;
        rest[s] = n[s] - done * cols > 0 ? n[s] - done * cols : 0;
        tiles -= done;
    }
}
constexpr double kTileUs[3] = {1.15, 1.65, 1.9};           // a K tile of 256 rows x 128, 192, 256 columns
GemmTiledPlan gemm_tiled_plan(int M, int K, const int *n, int nseg, bool gated, bool w4) {
    GemmTiledPlan best{};
    const int nk = K / kBK;
    if (M <= 128 && !gated) {
        best.ta = few_row_tile(M, K, n, nseg);
        best.cols = best.ta == 1 ? 128 : 256;
        best.tiles = tiles_of(n, nseg, best.cols) * (M <= 64 * best.ta ? 1 : 2);
        const long cap = best.ta == 1 ? 512 : 256;
        if (gemm_tiles_whole(M, K, n, nseg, false)) {
            best.blocks = best.tiles;
            best.slots = 1;
            return best;
        }
        const long U = (long)best.tiles * nk;
        best.blocks = (int)(U / 8 < 1 ? 1 : (U / 8 < cap ? U / 8 : cap));
        best.slots = gemm_slots_of(best.tiles, nk, best.blocks);
        return best;
    }
    const int m_tiles = (M + 255) / 256;
    long N = 0;
    for (int s = 0; s < nseg; ++s) N += n[s];
    const double slot_us = 2.0 * (double)M * (double)N * 4.0 / 3.0e6;
    double least = 1e300;
    best.ta = 4;
    for (int cols = gated ? 256 : 128; cols <= 256; cols += 64) {
        const int tiles = (gated ? n[0] / 128 : tiles_of(n, nseg, cols)) * m_tiles;
        for (int c = 1; c <= (gated ? 1 : 16) && (c == 1 || nk / c >= 4); ++c) {
            const long rounds = ((long)tiles * c + 255) / 256;
            const double cost = rounds * ((nk + c - 1) / c * kTileUs[cols / 64 - 2] + 4.0) + c * slot_us;
            if (cost < least) { least = cost; best.cols = cols; best.tiles = tiles; best.blocks = tiles * c; best.slots = c; }
        }
    }
    if (gated || w4) return best;
    least *= 0.98;
    for (int cols = 192; cols <= 256; cols += 64) {
        const int strips = tiles_of(n, nseg, cols), rounds = strips * m_tiles / 256;      // tiles side by side; rounds they fill
        const int first = rounds * 256 / m_tiles;                                         // of them in the first launch
        if (rounds == 0 || first == strips) continue;
        int n2[3];
        tiled_rest(n, nseg, cols, first, n2);
        for (int cols2 = 128; cols2 < cols; cols2 += 64) {
            const int tiles2 = tiles_of(n2, nseg, cols2) * m_tiles, rounds2 = (tiles2 + 255) / 256;
            const double cost = rounds * (nk * kTileUs[cols / 64 - 2] + 4.0) + rounds2 * (nk * kTileUs[cols2 / 64 - 2] + 4.0) + 3.0 + slot_us;
            if (cost < least) {
                least = cost;
                best.cols = cols; best.tiles = best.blocks = first * m_tiles; best.slots = 1;
                best.first = first; best.cols2 = cols2; best.tiles2 = tiles2;
            }
        }
    }
    return best;
}

// from 128 tiles on (half the CUs busy) not splitting K costs less than a slot of gate and up written and read again
// (256 x 37888 x 3584, 148 tiles: 95 us; separate, 84 + 11)
bool gemm_tiled_gates(int M, int K, const int *n, bool packed) {
    return M > 128 ? gemm_tiled_plan(M, K, n, 2, true, false).tiles >= 128 : packed && gemm_rows_plan(M, K, n, 2, true).used;
}

// The bands of the projections that the band kernel runs: the width whose blocks, one a band, leave the fewest CUs idle in their last
// round, the wider one where two leave as many (a block reads all activations).
static int band_strips(int strips, int least, int most, double *busy) {
    int best = least;
    *busy = 0.;
    for (int s = least; s <= most; ++s) {
        const int blocks = (strips + s - 1) / s, rounds = (blocks + kBandBlocks - 1) / kBandBlocks;
        const double share = (double)strips / ((double)s * rounds * kBandBlocks);
        if (share > *busy - 1e-9) { *busy = share; best = s; }
    }
    return best;
}
static uint32_t inverse_of(int s) { return (uint32_t)((0xffffffffull + s) / s); }        // ceil(2^32 / s), s > 1
GemmBands gemm_gate_bands(int f) {
    double busy;
    const int s = band_strips(strips_of(f), kGateLeast, kGateMost, &busy);
    return GemmBands{s, (strips_of(f) + s - 1) / s, inverse_of(s), true};
}
// QKV: bands where they keep at least 85 % of the CUs busy, else units in equal ranges.  Two layers, us, units / bands, 1 and 16 rows: 672 strips
// (88 %, bands of 3) x 4096 127 / 124, 140 / 136; 960 (94 %, 4) x 8192 217 / 214, 256 / 247; 1344 (88 %, 6) x 4096 159 / 158, 180 / 173; below
// the line 576 strips (75 %) x 2048 100 / 96, x 4096 118 / 117, but x 8192 178 / 180 and 210 / 215; 384 (50 %) x 4096 115 / 118, 131 / 134, x 8192
// 170 / 181; 192 (25 %) x 8192 147 / 167.  The line is one for all K (a wide model has most to lose: 672 x 8192 192 / 192, 219 / 222).
// Bands of one or two strips lose, since every block reads all activations; bands of six fill the chip up to 1536 strips (24 576 columns),
// and two rounds of narrower ones do beyond.
GemmBands gemm_qkv_bands(const int *n) {
    double busy;
    const int s = band_strips(tiles_of(n, 3, kSkinnyRows) * 4, kQkvLeast, kQkvMost, &busy);
    return busy >= 0.85 ? GemmBands{s, 0, inverse_of(s), true} : kUnitBands;
}
static int gemm_stream_grid(int tiles, int K) {
    const long U = (long)tiles * (K / kSkinnyStepK);
    return (int)(U < kStreamBlocks ? (U < 1 ? 1 : U) : kStreamBlocks);
}

static int gemm_stream_slots(int tiles, int K) {
    return gemm_slots_of(tiles, K / kSkinnyStepK, gemm_stream_grid(tiles, K));
}
// Whether the down projection of up to 16 rows runs on the unit kernel, its tiles finished by the last block to arrive, and not on
// the column kernel: a property of the model, since each has a layout of its own.  A column block walks all of K beside all of its
// activations: from 257 strips of 16 columns on some CUs have two such walks one after the other; and a long one, where all strips
// together are little to read, leaves HBM waiting.  Measured, two layers, us, column / unit (1, 8, 9, 16 rows): d_model 4096, d_ffn
// 11008 217 / 220, 226 / 233, 238 / 241, 241 / 246; 4608, 12288 282 / 263, 287 / 277, 309 / 290, 306 / 290; 6144, 16384 393 / 380,
// 402 / 391, 435 / 408, 433 / 414; 8192, 28672 694 / 687, 713 / 703, 757 / 725, 761 / 724; 2048, 16384 170 / 162, 174 / 176, 193 / 189,
// 186 / 192; 4096, 28672 351 / 349, 365 / 367, 383 / 379, 383 / 392; 3584, 18944 255 / 252, 262 / 272, 279 / 279, 279 / 278; few tiles make
// many arrivals at each: 1024, 11008 122 / 123, 130 / 143, 141 / 154, 137 / 164.
bool gemm_down_by_units(int d_model, int d_ffn) { return d_model > 16 * kStreamBlocks / 2 || (d_ffn >= 16384 && d_ffn >= 7 * d_model); }

// grid of the unit kernel with the residual epilogue: one block per CU, so that few blocks share a tile (the last of them to arrive
// adds their partials).  512 blocks, us as above: 6144, 16384 379, 397, 413, 421; 4608, 12288 265, 280, 297, 305.
static int gemm_resid_grid(int tiles, int K) {
    const long U = (long)tiles * (K / kSkinnyStepK);
    return (int)(U < kStreamBlocks / 2 ? (U < 1 ? 1 : U) : kStreamBlocks / 2);
}
int gemm_resid_slots(int tiles, int K) { return gemm_slots_of(tiles, K / kSkinnyStepK, gemm_resid_grid(tiles, K)); }
// largest number of blocks that share one tile, i.e. partial slots per output element
static int gemm_slots_of(int tiles, int units_per_tile, int grid) {
    const long ns = units_per_tile, U = (long)tiles * ns, P = grid;
    long worst = 1;
    for (long t = 0; t < tiles; ++t) {
        const long span = range_owner((t + 1) * ns - 1, U, P) - range_owner(t * ns, U, P) + 1;
        if (span > worst) worst = span;
    }
    return (int)worst;
}

int gemm_pack_tiles(const int *n, int nseg) { return tiles_of(n, nseg, kSkinnyRows); }
static int gemm_band_count(const int *n, int nseg, GemmBands b) {
    if (b.paired) return 2 * b.paired;
    int strips = 0;
    for (int s = 0; s < nseg; ++s) strips += strips_of(n[s]);
    return (strips + b.strips - 1) / b.strips;
}
size_t gemm_pack_bytes(const int *n, int nseg, int K, GemmBands b) {
    return (size_t)gemm_band_count(n, nseg, b) * b.strips * 16 * K * 2;
}

void launch_gemm_pack(const void *const *w, const int *n, int nseg, int K, void *dst, GemmBands b, hipStream_t stream) {
    PackArgs p{};
    for (int s = 0; s < nseg; ++s) { p.w[s] = (const uint16_t *)w[s]; p.n[s] = n[s]; }
    p.nseg = nseg; p.K = K; p.bands = b; p.dst = (u32x4 *)dst;
    launch_kernel(gemm_pack_kernel, (unsigned)gemm_band_count(n, nseg, b) * (K / kSkinnyStepK), 256, 0, stream, p);
}
void launch_gemm_pack_strips(const void *w, int n, int K, void *dst, hipStream_t stream) {
    const size_t vecs = (size_t)((n + kSkinnyRows - 1) / kSkinnyRows) * (K / kSkinnyStepK) * kUnitVec;
    launch_kernel(gemm_pack_strip_kernel, (unsigned)((vecs + 255) / 256), 256, 0, stream, (const uint16_t *)w, n, K, (u32x4 *)dst);
}

size_t gemm_pack_w4_bytes(const int *n, int nseg, int K) {
    return (size_t)tiles_of(n, nseg, kSkinnyRows) * w4_quads(K) * kW4QuadBytes;
}

void launch_gemm_pack_w4(const void *const *q, const void *const *scale, const void *const *zero, const int *n,
                         int nseg, int K, void *dst, hipStream_t stream) {
    uint8_t *out = (uint8_t *)dst;
    const int ns4 = 4 * w4_quads(K);
    for (int s = 0; s < nseg; ++s) {
        const size_t tiles = (size_t)((n[s] + kSkinnyRows - 1) / kSkinnyRows);
        launch_kernel(gemm_pack_w4_kernel, (unsigned)(tiles * ns4), 64, 0, stream, (const uint8_t *)q[s],
                      (const uint16_t *)scale[s], (const uint8_t *)zero[s], n[s], K, out);
        out += tiles * ns4 * kW4StepBytes;
    }
}

// grid and partial slots of a 4-bit projection in equal ranges: the unit kernel's policy with the quad as the unit, except that a
// block gets at least three quads where that still leaves one block per CU (measured on the LLaMA3-8B shape: QKV,
// 768 quads, 8.0 us on 512 blocks and 7.2 us on 256; a gate|up of 3584 quads 15.3 us on 512 and 17.6 us on 256; a down projection
// with the arrival epilogue 15.4 us on 256 blocks, 16.9 us on 512, 18.9 us on 128)
static int gemm_w4_grid(int tiles, int K, bool resid) {
    const long U = (long)tiles * w4_quads(K);
    long cap = kStreamBlocks / 2;
    if (!resid && U / 3 > cap) cap = U / 3 < kStreamBlocks ? U / 3 : kStreamBlocks;
    return (int)(U < cap ? (U < 1 ? 1 : U) : cap);
}
int gemm_w4_slots(int K, const int *n, int nseg, bool resid) {
    const int tiles = tiles_of(n, nseg, kSkinnyRows);
    return gemm_slots_of(tiles, w4_quads(K), gemm_w4_grid(tiles, K, resid));
}

// Whether the gate|up projection of up to 16 rows runs by tiles, SwiGLU in it (gemm_w4_gate_kernel).  A block then walks all of K for its gate
// and its up tile, and where the last round of tiles leaves many CUs without one, the longest walk is longer than in equal ranges by more
// than the partial slots and the SwiGLU launch cost: from 18 quads on.  By ranges / by tiles, us, two layers, 1 and 9 rows, K x tiles (quads
// longer): 8192 x 264 (30) 178 / 191, 199 / 214; 6656 x 280 (22) 165 / 175, 190 / 200; 6656 x 64 (18) 116 / 123, 136 / 144; but 6656 x 336 (16) 184 /
// 186, 209 / 211; 4096 x 264 (14) 131 / 130, 147 / 148; 8192 x 400 (14) 208 / 204, 236 / 228; 4096 x 224 (2) 303 / 289 at 7 rows.
bool gemm_w4_gates(int d_model, int d_ffn) {
    const int tiles = (d_ffn + kSkinnyRows - 1) / kSkinnyRows, quads = w4_quads(d_model), cus = kStreamBlocks / 2;
    const int grid = gemm_w4_grid(2 * tiles, d_model, false), in_range = (2 * tiles * quads + grid - 1) / grid;
    return 2 * quads * ((tiles + cus - 1) / cus) - in_range * ((grid + cus - 1) / cus) < 18;
}

// whether whole tiles of a head of up to 16 rows leave at most a tenth of the blocks' time idle
bool gemm_stream_whole(const int *n, int nseg) {
    const int tiles = tiles_of(n, nseg, kSkinnyRows), rounds = (tiles + kStreamBlocks - 1) / kStreamBlocks;
    return tiles * 10 >= rounds * kStreamBlocks * 9;
}
int gemm_packed_splits(int K, const int *n, int nseg) { return gemm_stream_slots(tiles_of(n, nseg, kSkinnyRows), K); }

int gemm_pick_splitk(int dtype, int M, int K, int N, const int *n, int nseg, bool packed, bool w4) {
    (void)N;
    if (dtype != PSD_BF16) return 1;
    if (M <= kStreamMaxRows) {
        const int tiles = tiles_of(n, nseg, kSkinnyRows);
        const int nsteps = K / kSkinnyStepK;
        int want = (512 + tiles - 1) / tiles;             // aim at >= 512 blocks (2048 wavefronts)
        int cap = nsteps / 8;                             // keep >= 2 K steps per wavefront
        if (cap < 1) cap = 1;
        if (want > cap) want = cap;
        if (want > 16) want = 16;
        return want < 1 ? 1 : want;
    }
    if (packed) {
        const RowsPlan r = gemm_rows_plan(M, K, n, nseg, false);
        if (r.used) return r.slots;
    }
    return gemm_tiled_plan(M, K, n, nseg, false, w4).slots;
}

// calls go with `strips` as a constant, one of Least .. Most: the range of the rule that chose it
template <int Least, int Most, typename Go>
static void with_width(int strips, Go go) {
    if constexpr (Least < Most)
        if (strips != Least) return with_width<Least + 1, Most>(strips, go);
    go(std::integral_constant<int, Least>{});
}

bool gemm_moves_lens(int dtype, const GemmArgs &g) {
    return g.reduced || (dtype == PSD_BF16 && (g.M > kStreamMaxRows || g.whole));
}

void launch_gemm(int dtype, const GemmArgs &args, hipStream_t stream) {
    GemmArgs g = args;
    if (args.reduced) g.lens_n = 0;                        // the reduction behind it does
    if (dtype != PSD_BF16) {
        ScopedProf sp(PSD_KIND_GEMM_F32, stream);
        launch_kernel(gemm_f32_kernel, (g.N + 3) / 4, 256, 0, stream, g);
        return;
    }
    if (g.M <= kStreamMaxRows && g.wpack && g.w4) {
        // 32-bit offsets from the first activation row: these projections read M <= 16 consecutive rows
        ScopedProf sp(PSD_KIND_GEMM_W4, stream);
        if (g.swiglu16) { launch_kernel(gemm_w4_gate_kernel, g.pack_tiles / 2, 512, 0, stream, g); return; }
        if (g.x_resid && !g.tile_counter) { launch_kernel(gemm_w4_column_kernel, g.N / 16, 1024, 0, stream, g); return; }
        const bool resid = g.x_resid;
        const int grid = gemm_w4_grid(g.pack_tiles, g.K, resid);
        if (resid)
            launch_kernel(gemm_w4_unit_kernel<true>, grid, 256, 0, stream, g);
        else
            launch_kernel(gemm_w4_unit_kernel<false>, grid, 256, 0, stream, g);
        return;
    }
    if (g.M <= kStreamMaxRows && g.wpack && g.x_resid && g.tile_counter) {
        ScopedProf sp(PSD_KIND_GEMM_COLUMN, stream);
        const int grid = gemm_resid_grid(g.pack_tiles, g.K);
        if (g.op_folded) launch_kernel(gemm_bf16_unit_kernel<true, true>, grid, 256, 0, stream, g);
        else launch_kernel(gemm_bf16_unit_kernel<false, true>, grid, 256, 0, stream, g);
        return;
    }
    if (g.M <= kStreamMaxRows && g.wpack && g.x_resid) {
        ScopedProf sp(PSD_KIND_GEMM_COLUMN, stream);
        const int grid = g.N / 16;                        // every segment is a multiple of 64 wide
        if (g.op_folded) launch_kernel(gemm_bf16_column_kernel<true>, grid, 1024, 0, stream, g);
        else launch_kernel(gemm_bf16_column_kernel<false>, grid, 1024, 0, stream, g);
        return;
    }
    if (g.M <= kStreamMaxRows && g.wpack && g.bands.owned) {
        ScopedProf sp(PSD_KIND_GEMM_SKINNY, stream);
        const int bands = gemm_band_count(g.n, g.nseg, g.bands), blocks = g.bands.paired ? bands / 2 : bands;
        auto go = [&](auto strips, auto gated) {
            constexpr int S = decltype(strips)::value;
            constexpr bool G = decltype(gated)::value;
            if (g.op_folded) launch_kernel(gemm_bf16_band_kernel<true, S, G>, blocks, 512, 0, stream, g);
            else launch_kernel(gemm_bf16_band_kernel<false, S, G>, blocks, 512, 0, stream, g);
        };
        if (g.bands.paired) with_width<kGateLeast, kGateMost>(g.bands.strips, [&](auto strips) { go(strips, std::true_type{}); });
        else with_width<kQkvLeast, kQkvMost>(g.bands.strips, [&](auto strips) { go(strips, std::false_type{}); });
        return;
    }
    if (g.M <= kStreamMaxRows && g.wpack) {
        ScopedProf sp(PSD_KIND_GEMM_SKINNY, stream);
        const int grid = g.whole ? (g.pack_tiles < kStreamBlocks ? g.pack_tiles : kStreamBlocks) : gemm_stream_grid(g.pack_tiles, g.K);
        auto go = [&](auto kernel) { launch_kernel(kernel, grid, 256, 0, stream, g); };
        if (g.op_folded) go(gemm_bf16_unit_kernel<true, false>);
        else go(gemm_bf16_unit_kernel<false, false>);
    } else if (g.M <= kStreamMaxRows) {
        ScopedProf sp(PSD_KIND_GEMM_SLOT, stream);
        dim3 grid(tiles_of(g.n, g.nseg, kSkinnyRows), g.splitk);
        launch_kernel(gemm_bf16_skinny_kernel<1>, grid, 256, 0, stream, g);
    } else if (const RowsPlan rp = gemm_rows_plan(g.M, g.K, g.n, g.nseg, g.swiglu16 != nullptr); rp.used && g.wpack && !g.w4) {
        ScopedProf sp(PSD_KIND_GEMM_TILED, stream);
        GemmArgs t = g;
        t.tiled_tiles = rp.tiles;
        t.whole = rp.whole;
        auto pick = [&](auto waves, auto gated) {
            constexpr int NW = decltype(waves)::value;
            constexpr bool G = decltype(gated)::value;
            auto go = [&](auto kernel) { launch_kernel(kernel, rp.blocks, 64 * NW, 0, stream, t); };
            if (g.M <= 32) go(gemm_bf16_rows_kernel<NW, 2, G>);
            else if (g.M <= 48) go(gemm_bf16_rows_kernel<NW, 3, G>);
            else if (g.M <= 64) go(gemm_bf16_rows_kernel<NW, 4, G>);
            else if constexpr (NW <= 8) {                   // (the plan gives ten wavefronts up to 64 rows, six up to 96)
                if (g.M <= 96) go(gemm_bf16_rows_kernel<NW, 6, G>);
                else if constexpr (NW == 8) go(gemm_bf16_rows_kernel<8, 8, G>);
            }
        };
        auto widths = [&](auto gated) {
            if (rp.waves == 6) pick(std::integral_constant<int, 6>{}, gated);
            else if (rp.waves == 8) pick(std::integral_constant<int, 8>{}, gated);
            else pick(std::integral_constant<int, 10>{}, gated);
        };
        if (g.swiglu16) widths(std::true_type{});
        else widths(std::false_type{});
    } else {
        ScopedProf sp(PSD_KIND_GEMM_TILED, stream);
        const GemmTiledPlan p = gemm_tiled_plan(g.M, g.K, g.n, g.nseg, g.swiglu16 != nullptr, g.w4);
        auto run = [&](GemmArgs &t, int cols, int blocks) {
            t.blocks = blocks;
            auto go = [&](auto kernel, int threads) {
                // opt in to more than 64 KB of dynamic LDS: a property of the function on the current device, set before
                // every launch (a cheap host call) so that no process-wide flag has to remember who set it where
                const size_t lds = (size_t)(64 * p.ta + cols) * kLdsStride * sizeof(uint16_t) * 2;
                (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                          (int)lds);
                launch_kernel(kernel, blocks, threads, lds, stream, t);
            };
            auto pick = [&](auto w4) {
                constexpr bool W4 = decltype(w4)::value;
                if (p.ta == 1) go(gemm_f16_tiled_kernel<1, 1, 4, W4>, 512);
                else if (p.ta == 2) go(gemm_f16_tiled_kernel<2, 2, 4, W4>, 512);
                else if (cols == 128) go(gemm_f16_tiled_kernel<4, 1, 4, W4>, 512);
                else if (cols == 192) go(gemm_f16_tiled_kernel<4, 3, 2, W4>, 256);
                else go(gemm_f16_tiled_kernel<4, 2, 4, W4>, 512);
            };
            if (t.w4) pick(std::true_type{});
            else pick(std::false_type{});
        };
        GemmArgs t = g;
        t.tiled_tiles = p.tiles;
        if (p.first == 0) {
            run(t, p.cols, p.blocks);
        } else {                                            // the first tiles' columns of every segment, then the rest of them
            GemmArgs u = g;
            tiled_rest(g.n, g.nseg, p.cols, p.first, u.n);
            t.nseg = u.nseg = 0;                            // (both write into rows of g.N outputs)
            for (int s = 0; s < g.nseg; ++s) {
                const int done = g.n[s] - u.n[s], left = u.n[s];
                if (done > 0) { t.n[t.nseg++] = done; u.partial += done; }
                if (left > 0) {
                    u.w[u.nseg] = (const char *)g.w[s] + (size_t)done * g.K * 2;
                    u.n[u.nseg++] = left;
                }
            }
            u.lens_n = 0;
            u.tiled_tiles = p.tiles2;
            run(t, p.cols, p.blocks);
            run(u, p.cols2, p.tiles2);
        }
    }
    if (args.reduced) {
        const dim3 grid((unsigned)((g.N + 255) / 256), (unsigned)g.M);
        ScopedProf sp(PSD_KIND_GEMM_REDUCE, stream);
        launch_kernel(gemm_splitk_reduce_kernel, grid, 256, 0, stream, args);
    }
}

}  // namespace psd
