// Row-wise pieces of the decoder forward pass on gfx950: embedding gather, RMSNorm, rotary
// embedding + KV append, SwiGLU, and the KV-length bookkeeping (the rollback of Sec. 3.3).
// All are bandwidth-trivial next to the weight streaming of the GEMMs; they exist so that no
// step of the forward pass leaves the GPU.
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "prof.h"
#include "../../include/psd.h"

namespace psd {
namespace {

constexpr int kMaxRowV4 = 2048;        // float4 per row kept in registers: rows up to 8192 wide

// fixed-order block sum: butterfly inside each wavefront, then the wavefronts' totals left to right
template <int NT = 256>
__device__ __forceinline__ float block_sum4(float v, float *red) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = red[0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) t += red[w];
    return t;
}

__device__ __forceinline__ f32x4 load_gain4(const float *g, int i4) { return reinterpret_cast<const f32x4 *>(g)[i4]; }
__device__ __forceinline__ f32x4 load_gain4(const uint16_t *g, int i4) {
    const uint2 raw = reinterpret_cast<const uint2 *>(g)[i4];
    return f32x4{bf16_bits_to_f32(raw.x & 0xffffu), __uint_as_float(raw.x & 0xffff0000u),
                 bf16_bits_to_f32(raw.y & 0xffffu), __uint_as_float(raw.y & 0xffff0000u)};
}
__device__ __forceinline__ f32x4 load_row4(const float *row, int i4) { return reinterpret_cast<const f32x4 *>(row)[i4]; }
__device__ __forceinline__ f32x4 load_row4(const uint16_t *row, int i4) { return load_gain4(row, i4); }

// One block per row: x (+)= source, then xn = x * rsqrt(mean(x^2) + eps) * gain.  The source is either
// an embedding row (EMBED) or the split-K partial sums of the projection that feeds the residual
// stream, added in split order.  All loads of a row are issued before the first use.  xn NULL: only the fp16 copy is read.
// What bounds it: a block's own loads in flight.  1024 threads hold a whole row of a split at once, in few registers, so that two blocks
// a CU are full (us a launch, 256 threads / 1024: 45 rows x 4096, 8 splits 9.6 / 5.2; 256 rows x 3584 10.1 / 7.0; 2001 rows x 4096, one split
// 35.6 / 21.3 = 5.4 TB/s, two splits 40.4 / 24.8; 512 threads 24.7 and 28.2).  The embedding, whose first wavefront or two work out angles in
// fp64 meanwhile, so only for as many rows as are resident at once (1 row 6.2 / 5.0, 15 rows 7.2 / 5.1, 256 rows 8.9 / 6.6, 2001 rows 20.1 / 26.3).
template <typename TW, bool EMBED, int kRowThreads, bool OP = false>
__global__ __launch_bounds__(kRowThreads) void residual_norm_kernel(const TW *embed, const int32_t *tokens, int vocab,
                                                                    const float *partial, int S, size_t split_stride,
                                                                    float *x, const TW *gain, float *xn, float *sumsq_out,
                                                                    int d, float eps, RopeTable rt, uint16_t *xn16,
                                                                    ZeroFill zf, TreeShape tree, uint32_t *tree_anc, OpRows op) {
    constexpr int kMaxV4 = kMaxRowV4 / kRowThreads;
    __shared__ float red[kRowThreads / 64];
    const int m = blockIdx.x, tid = threadIdx.x, n4 = d >> 2;
    if constexpr (EMBED) {
        // counters that later kernels of this forward pass expect at zero
        if (m == 0)
            for (int j = tid; j < zf.n; j += kRowThreads) zf.words[j] = 0u;
        if (m < tree.n && tid == 0) tree_anc[m] = tree.anc[m];                  // m: the same for the block
        // (cos, sin) of this row's position at every rotation frequency, once per forward pass for all layers;
        // the angle position * theta^(-2i/d_h) is evaluated in fp64
        if (rt.cs && tid < rt.d_h / 2) {
            const int pos = rt.lens[m / rt.R] + (tree.n ? tree.depth[m % rt.R] : m % rt.R);
            const double inv_freq = exp2(-2.0 * (double)tid / (double)rt.d_h * log2((double)rt.theta));
            double sn, cs;
            sincos((double)pos * inv_freq, &sn, &cs);
            rt.cs[(size_t)m * (rt.d_h / 2) + tid] = make_float2((float)cs, (float)sn);
        }
    }
    f32x4 v[kMaxV4];
    float ss = 0.f;
    f32x4 *__restrict__ xrow = reinterpret_cast<f32x4 *>(x + (size_t)m * d);
    const TW *erow = nullptr;
    if constexpr (EMBED) {
        int tok = tokens[m];
        tok = min(max(tok, 0), vocab - 1);
        erow = embed + (size_t)tok * d;
    }
    // issue every load of the row first (x or the embedding row, then the partials four splits at a
    // time), add in split order, store afterwards
    const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < kMaxV4; ++j) {
        const int i4 = tid + j * kRowThreads;
        v[j] = zero;
        if (i4 < n4) {
            if constexpr (EMBED) v[j] = load_row4(erow, i4);
            else v[j] = xrow[i4];
        }
    }
    if constexpr (!EMBED) {
        const f32x4 *prow = reinterpret_cast<const f32x4 *>(partial + (size_t)m * d);
        const size_t stride4 = split_stride >> 2;
        int sp = 0;
        for (; sp + 4 <= S; sp += 4) {
            f32x4 t[4][kMaxV4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int j = 0; j < kMaxV4; ++j) {
                    const int i4 = tid + j * kRowThreads;
                    t[u][j] = i4 < n4 ? prow[(sp + u) * stride4 + i4] : zero;
                }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int j = 0; j < kMaxV4; ++j) v[j] += t[u][j];
        }
        for (; sp < S; ++sp) {
#pragma unroll
            for (int j = 0; j < kMaxV4; ++j) {
                const int i4 = tid + j * kRowThreads;
                if (i4 < n4) v[j] += prow[sp * stride4 + i4];
            }
        }
    }
#pragma unroll
    for (int j = 0; j < kMaxV4; ++j) {
        const int i4 = tid + j * kRowThreads;
        if (i4 < n4) {
            const f32x4 a = v[j];
            xrow[i4] = a;
            ss += a[0] * a[0] + a[1] * a[1] + a[2] * a[2] + a[3] * a[3];
        }
    }
    const float tot = block_sum4<kRowThreads>(ss, red);
    float scale = 1.0f / sqrtf(tot / (float)d + eps);
    if (sumsq_out) {                       // the norm scale is applied by the consumer of the next projection
        if (tid == 0) sumsq_out[m] = tot;
        scale = 1.0f;
    }
    f32x4 *orow = reinterpret_cast<f32x4 *>(xn + (size_t)m * d);
    const int op_r = OP ? m % op.per_group - op.first : -1, op_row = OP ? m / op.per_group * (op.per_group - op.first) + op_r : 0;
#pragma unroll
    for (int j = 0; j < kMaxV4; ++j) {
        const int i4 = tid + j * kRowThreads;
        if (i4 < n4) {
            const f32x4 r = v[j] * scale * load_gain4(gain, i4);
            if (xn) orow[i4] = r;
            if (OP && op_r >= 0) op_store4(op.op, op_row, 4 * i4, op.folded, r);
            if (xn16)              // the same row rounded to fp16: the operand of the tiled projections
                reinterpret_cast<uint2 *>(xn16 + (size_t)m * d)[i4] =
                    make_uint2(f32_to_f16_bits(r[0]) | ((uint32_t)f32_to_f16_bits(r[1]) << 16),
                               f32_to_f16_bits(r[2]) | ((uint32_t)f32_to_f16_bits(r[3]) << 16));
        }
    }
}

// One block per (new row, head slot): slots 0..h_q-1 rotate a query head, the next h_kv rotate a
// key head into the cache, the last h_kv copy a value head into the transposed V cache.  The
// projection arrives as split-K partials and is summed here, in split order.  Thread i < d_h/2
// owns the rotation pair (i, i + d_h/2); the angle position * theta^(-2i/d_h) is evaluated in fp64.
template <typename TC>
__global__ __launch_bounds__(64) void reduce_rope_append_kernel(const float *partial, int S, size_t split_stride,
                                                                RowScale rs, float *q_out, TC *k_cache, TC *v_cache,
                                                                const int32_t *lens, int R, int h_q, int h_kv, int d_h,
                                                                int max_len, float theta, const float2 *cs_table) {
    const int m = blockIdx.x, slot = blockIdx.y, b = m / R, r = m % R;
    const int pos = lens[b] + r;
    if (pos >= max_len) return;            // capacity was checked on the host; never write outside
    // the sums of squares first, the projection's partials next, the reduction after both are in flight
    float ssq = 0.f;
    if (rs.sumsq)
        for (int t = threadIdx.x; t < rs.tiles; t += 64) ssq += rs.sumsq[(size_t)t * gridDim.x + m];
    const int half = d_h / 2;
    const int width = (h_q + 2 * h_kv) * d_h;
    const float *src = partial + (size_t)m * width + (size_t)slot * d_h;
    const int i = threadIdx.x;
    auto value = [&](int e) {                  // loads four splits at a time, adds in split order
        float a = 0.f;
        int sp = 0;
        for (; sp + 4 <= S; sp += 4) {
            const float t0 = src[sp * split_stride + e], t1 = src[(sp + 1) * split_stride + e];
            const float t2 = src[(sp + 2) * split_stride + e], t3 = src[(sp + 3) * split_stride + e];
            a += t0; a += t1; a += t2; a += t3;
        }
        for (; sp < S; ++sp) a += src[sp * split_stride + e];
        return a;
    };
    auto scale_of = [&]() { return rs.sumsq ? 1.0f / sqrtf(wave_sum(ssq) * rs.inv_d + rs.eps) : 1.0f; };
    if (slot < h_q + h_kv) {
        const float r1 = i < half ? value(i) : 0.f, r2 = i < half ? value(half + i) : 0.f;
        const float sc = scale_of();
        if (i >= half) return;
        float c, s;
        if (cs_table) {
            const float2 t = cs_table[(size_t)m * half + i];
            c = t.x;
            s = t.y;
        } else {
            const double inv_freq = exp2(-2.0 * (double)i / (double)d_h * log2((double)theta));
            double sn, cs;
            sincos((double)pos * inv_freq, &sn, &cs);
            c = (float)cs;
            s = (float)sn;
        }
        const float x1 = r1 * sc, x2 = r2 * sc;
        const float y1 = x1 * c - x2 * s, y2 = x2 * c + x1 * s;
        if (slot < h_q) {
            float *dst = q_out + ((size_t)m * h_q + slot) * d_h;
            dst[i] = y1;
            dst[half + i] = y2;
        } else {
            TC *dst = k_cache + (((size_t)b * h_kv + (slot - h_q)) * max_len + pos) * d_h;
            store_elem(dst, i, y1);
            store_elem(dst, half + i, y2);
        }
    } else {
        // V is stored transposed: v_cache[b][h][d][pos]
        const int h = slot - h_q - h_kv;
        const float v0 = i < d_h ? value(i) : 0.f, v1 = i + 64 < d_h ? value(i + 64) : 0.f;     // d_h <= 128
        const float sc = scale_of();
        if (i < d_h) store_elem(v_cache, (((size_t)b * h_kv + h) * d_h + i) * max_len + pos, v0 * sc);
        if (i + 64 < d_h) store_elem(v_cache, (((size_t)b * h_kv + h) * d_h + i + 64) * max_len + pos, v1 * sc);
    }
}

// The same for a bf16 model without a row scale (more than 16 rows in all, or no packed weights).  Bound by the bytes with
// many rows, by the trips to the partial sums with few: the first blocks take one row and 2048 / d_head query and key heads
// each, four rotation pairs per thread; the others take kAppendRows rows of the values of one head through LDS, so that the
// transposed cache is written along the positions; four splits of every sum are in flight.  The kernel above (one wavefront
// per row and head, each value into a line of its own) and the present one, us: one sequence of the LLaMA3-8B shape (8 KV
// heads) 20 rows 5.2 / 4.1, 64 rows 5.5 / 4.8, 256 rows 10.2 / 7.2; of the 7B shape 64 rows 7.9 / 5.9, 1800 rows 103 / 29;
// 16 x 16 rows of the Qwen2-7B shape 9.8 / 6.1.  64 rows a value block and one split in flight left too few loads under
// way: 20 rows 11.0, 64 rows 23.9, 16 x 16 rows 8.3; 8 and 32 rows a block with four in flight: 64 rows 4.5 and 6.9, 1800
// rows 31.6 and 29.3.
constexpr int kAppendRows = 16;
__global__ __launch_bounds__(256) void reduce_rope_append_tiled_kernel(const float *partial, int S, size_t split_stride,
                                                                       float *q_out, uint16_t *k_cache, uint16_t *v_cache,
                                                                       const int32_t *lens, int B, int R, int h_q, int h_kv,
                                                                       int d_h, int max_len, const float2 *cs_table, int qk_blocks) {
    __shared__ float tile[kAppendRows][129];
    const int half = d_h / 2, width = (h_q + 2 * h_kv) * d_h, tid = threadIdx.x;
    // sums of N groups of four columns, four splits of each in flight, added in split order
    auto sums = [&](auto &v, const size_t (&at)[std::extent<std::remove_reference_t<decltype(v)>>::value]) {
        constexpr int N = std::extent<std::remove_reference_t<decltype(v)>>::value;
        auto get = [&](int sp, int k) { return *reinterpret_cast<const f32x4 *>(partial + sp * split_stride + at[k]); };
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = f32x4{0.f, 0.f, 0.f, 0.f};
        int sp = 0;
        for (; sp + 4 <= S; sp += 4) {
            f32x4 t[4][N];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int k = 0; k < N; ++k) t[u][k] = get(sp + u, k);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int k = 0; k < N; ++k) v[k] += t[u][k];
        }
        for (; sp < S; ++sp)
#pragma unroll
            for (int k = 0; k < N; ++k) v[k] += get(sp, k);
    };
    if ((int)blockIdx.x < qk_blocks) {
        const int per = 1024 / half, groups = (h_q + h_kv + per - 1) / per;                       // heads per block
        const int m = blockIdx.x / groups, b = m / R, pos = lens[b] + m % R;
        const int head = (blockIdx.x % groups) * per + tid * 4 / half, i = tid * 4 % half;
        if (head >= h_q + h_kv || pos >= max_len) return;           // capacity was checked on the host; never write outside
        const size_t at = (size_t)m * width + (size_t)head * d_h + i;
        f32x4 x[2];
        sums(x, {at, at + half});
        const f32x4 x1 = x[0], x2 = x[1];
        const f32x4 t0 = reinterpret_cast<const f32x4 *>(cs_table + (size_t)m * half + i)[0];
        const f32x4 t1 = reinterpret_cast<const f32x4 *>(cs_table + (size_t)m * half + i)[1];
        const f32x4 c = f32x4{t0[0], t0[2], t1[0], t1[2]}, s = f32x4{t0[1], t0[3], t1[1], t1[3]};
        const f32x4 y1 = x1 * c - x2 * s, y2 = x2 * c + x1 * s;
        if (head < h_q) {
            float *dst = q_out + ((size_t)m * h_q + head) * d_h + i;
            *reinterpret_cast<f32x4 *>(dst) = y1;
            *reinterpret_cast<f32x4 *>(dst + half) = y2;
        } else {
            uint16_t *dst = k_cache + (((size_t)b * h_kv + (head - h_q)) * max_len + pos) * d_h + i;
            *reinterpret_cast<uint2 *>(dst) = make_uint2(pack_bf16x2(y1[0], y1[1]), pack_bf16x2(y1[2], y1[3]));
            *reinterpret_cast<uint2 *>(dst + half) = make_uint2(pack_bf16x2(y2[0], y2[1]), pack_bf16x2(y2[2], y2[3]));
        }
        return;
    }
    const int vb = blockIdx.x - qk_blocks, h = vb % h_kv, tiles = (R + kAppendRows - 1) / kAppendRows;
    const int b = vb / h_kv / tiles, r0 = vb / h_kv % tiles * kAppendRows, rows = min(kAppendRows, R - r0);
    const int n4 = rows * (d_h / 4);
    for (int e0 = tid; e0 < n4; e0 += 512) {
        size_t at[2];
        f32x4 v[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int e = min(e0 + k * 256, n4 - 1);
            at[k] = (size_t)(b * R + r0 + e / (d_h / 4)) * width + (size_t)(h_q + h_kv + h) * d_h + e % (d_h / 4) * 4;
        }
        sums(v, {at[0], at[1]});
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (e0 + k * 256 < n4) {
                const int r = (e0 + k * 256) / (d_h / 4), d = (e0 + k * 256) % (d_h / 4) * 4;
#pragma unroll
                for (int j = 0; j < 4; ++j) tile[r][d + j] = v[k][j];
            }
    }
    __syncthreads();
    const int r = tid & (kAppendRows - 1), pos = lens[b] + r0 + r;
    if (r >= rows || pos >= max_len) return;
    for (int d = tid / kAppendRows; d < d_h; d += 256 / kAppendRows)
        v_cache[(((size_t)b * h_kv + h) * d_h + d) * max_len + pos] = (uint16_t)f32_to_bf16_bits(tile[r][d]);
}

// h = silu(g) * u, four columns per thread, one row per blockIdx.y; [g | u] arrive as split-K partials of
// the gate|up projection, to be scaled by the row's factor where its norm is folded into the projection
__global__ __launch_bounds__(256) void reduce_swiglu_kernel(const float *partial, int S, size_t split_stride, RowScale rs, float *h, int f,
                                                            uint16_t *h16) {
    __shared__ float red[4];
    const int m = blockIdx.y, f4 = f >> 2;
    const int j4 = blockIdx.x * 256 + threadIdx.x;
    float ssq = 0.f;
    if (rs.sumsq)
        for (int t = threadIdx.x; t < rs.tiles; t += 256) ssq += rs.sumsq[(size_t)t * gridDim.y + m];
    f32x4 g = f32x4{0.f, 0.f, 0.f, 0.f}, u = g;
    if (j4 < f4)
        for (int sp = 0; sp < S; ++sp) {
            const f32x4 *row = reinterpret_cast<const f32x4 *>(partial + sp * split_stride + (size_t)m * 2 * f);
            g += row[j4];
            u += row[f4 + j4];
        }
    if (rs.sumsq) {
        const float sc = 1.0f / sqrtf(block_sum4(ssq, red) * rs.inv_d + rs.eps);
        g *= sc;
        u *= sc;
    }
    if (j4 >= f4) return;
    f32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = g[e] / (1.0f + expf(-g[e])) * u[e];
    if (h) reinterpret_cast<f32x4 *>(h + (size_t)m * f)[j4] = o;
    if (h16)
        reinterpret_cast<uint2 *>(h16 + (size_t)m * f)[j4] =
            make_uint2(f32_to_f16_bits(o[0]) | ((uint32_t)f32_to_f16_bits(o[1]) << 16),
                       f32_to_f16_bits(o[2]) | ((uint32_t)f32_to_f16_bits(o[3]) << 16));
}

__global__ void advance_lens_kernel(int32_t *lens, int B, int delta, int max_len) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < B) lens[b] = min(lens[b] + delta, max_len);
}

__global__ void truncate_kernel(int32_t *lens, const int32_t *base, const int32_t *keep, int offset, int cap, int B) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < B) lens[b] = max(0, min(min(lens[b], cap), base[b] + keep[b] + offset));
}

__global__ void truncate_to_kernel(int32_t *lens, int new_len, int B) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < B) lens[b] = max(0, min(lens[b], new_len));
}

}  // namespace

constexpr int kWideEmbedMax = 512;     // rows of an embedding launch up to which a block has 1024 threads: all of them fit the chip at once
void launch_embed_norm(int dtype, const void *embed, const int32_t *tokens, float *x, const void *gain, float *xn,
                       float *sumsq_out, int M, int d, int vocab, float eps, RopeTable rt, uint16_t *xn16, OpRows op, ZeroFill zf,
                       const TreeShape *tree, uint32_t *tree_anc, hipStream_t stream) {
    ScopedProf sp(PSD_KIND_EMBED, stream);
    const TreeShape ts = tree ? *tree : TreeShape{};
    if (dtype == PSD_BF16) {
        auto go = [&](auto kernel, int threads) {
            launch_kernel(kernel, M, threads, 0, stream, (const uint16_t *)embed, tokens, vocab, nullptr, 0, 0, x, (const uint16_t *)gain, xn, sumsq_out,
                          d, eps, rt, xn16, zf, ts, tree_anc, op);
        };
        auto pick = [&](auto with_op) {
            constexpr bool OP = decltype(with_op)::value;
            if (M <= kWideEmbedMax) go(residual_norm_kernel<uint16_t, true, 1024, OP>, 1024);
            else go(residual_norm_kernel<uint16_t, true, 256, OP>, 256);
        };
        if (op.op) pick(std::true_type{});
        else pick(std::false_type{});
    } else
        launch_kernel(residual_norm_kernel<float, true, 256>, M, 256, 0, stream, (const float *)embed, tokens, vocab, nullptr, 0, 0, x,
                                                                        (const float *)gain, xn, sumsq_out, d, eps, rt, xn16, zf, ts, tree_anc, op);
}

void launch_reduce_residual_norm(int dtype, const float *partial, int S, float *x, const void *gain, float *xn,
                                 int M, int d, float eps, uint16_t *xn16, OpRows op, hipStream_t stream) {
    ScopedProf sp(PSD_KIND_RMSNORM, stream);
    const size_t stride = (size_t)M * d;
    if (dtype == PSD_BF16) {
        auto go = [&](auto kernel, int threads) {
            launch_kernel(kernel, M, threads, 0, stream, nullptr, nullptr, 0, partial, S, stride, x, (const uint16_t *)gain, xn, nullptr, d, eps,
                          RopeTable{}, xn16, ZeroFill{}, TreeShape{}, nullptr, op);
        };
        if (op.op) go(residual_norm_kernel<uint16_t, false, 1024, true>, 1024);
        else go(residual_norm_kernel<uint16_t, false, 1024, false>, 1024);
    } else
        launch_kernel(residual_norm_kernel<float, false, 256>, M, 256, 0, stream, nullptr, nullptr, 0, partial, S, stride, x,
                      (const float *)gain, xn, nullptr, d, eps, RopeTable{}, xn16, ZeroFill{}, TreeShape{}, nullptr, op);
}

void launch_reduce_rope_append(int dtype, const float *partial, int S, RowScale rs, float *q_out, void *k_cache,
                               void *v_cache, const int32_t *lens, int B, int R, int h_q, int h_kv, int d_h,
                               int max_len, float theta, const float2 *cs_table, hipStream_t stream) {
    ScopedProf sp(PSD_KIND_ROPE_APPEND, stream);
    const size_t stride = (size_t)B * R * (h_q + 2 * h_kv) * d_h;
    const dim3 grid(B * R, h_q + 2 * h_kv);
    if (dtype == PSD_BF16 && !rs.sumsq && cs_table) {
        const int per = 1024 / (d_h / 2);                                   // query and key heads per block
        const int qk = B * R * ((h_q + h_kv + per - 1) / per);
        const int vb = B * ((R + kAppendRows - 1) / kAppendRows) * h_kv;
        launch_kernel(reduce_rope_append_tiled_kernel, qk + vb, 256, 0, stream, partial, S, stride, q_out, (uint16_t *)k_cache,
                      (uint16_t *)v_cache, lens, B, R, h_q, h_kv, d_h, max_len, cs_table, qk);
        return;
    }
    if (dtype == PSD_BF16)
        launch_kernel(reduce_rope_append_kernel<uint16_t>, grid, 64, 0, stream, partial, S, stride, rs, q_out, (uint16_t *)k_cache,
                                                                     (uint16_t *)v_cache, lens, R, h_q, h_kv, d_h, max_len, theta, cs_table);
    else
        launch_kernel(reduce_rope_append_kernel<float>, grid, 64, 0, stream, partial, S, stride, rs, q_out, (float *)k_cache, (float *)v_cache,
                                                                  lens, R, h_q, h_kv, d_h, max_len, theta, cs_table);
}

void launch_reduce_swiglu(const float *partial, int S, RowScale rs, float *h, int M, int f, uint16_t *h16, hipStream_t stream) {
    ScopedProf sp(PSD_KIND_SWIGLU, stream);
    const dim3 grid((unsigned)((f / 4 + 255) / 256), (unsigned)M);
    launch_kernel(reduce_swiglu_kernel, grid, 256, 0, stream, partial, S, (size_t)M * 2 * f, rs, h, f, h16);
}

void launch_advance_lens(int32_t *lens, int B, int delta, int max_len, hipStream_t stream) {
    ScopedProf sp(PSD_KIND_LENS, stream);
    launch_kernel(advance_lens_kernel, (B + 63) / 64, 64, 0, stream, lens, B, delta, max_len);
}
void launch_truncate(int32_t *lens, const int32_t *base, const int32_t *keep, int offset, int cap, int B,
                     hipStream_t stream) {
    ScopedProf sp(PSD_KIND_LENS, stream);
    launch_kernel(truncate_kernel, (B + 63) / 64, 64, 0, stream, lens, base, keep, offset, cap, B);
}
void launch_truncate_to(int32_t *lens, int new_len, int B, hipStream_t stream) {
    ScopedProf sp(PSD_KIND_LENS, stream);
    launch_kernel(truncate_to_kernel, (B + 63) / 64, 64, 0, stream, lens, new_len, B);
}

}  // namespace psd
