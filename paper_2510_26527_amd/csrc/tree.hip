// Token-tree verification (Related Work, "Verification Mechanisms": token-tree-based verification; Sec. 4.6 names
// deeper and wider drafting as the next step).  The paper prints no rule; the one used is multi-round speculative
// sampling for sibling tokens drawn independently from the drafter's distribution at their parent, which leaves the
// verifier's distribution unchanged (Abstract; Sec. 3.1).
//
//   tree_stats / mass / draw_kernel  the walk from the root: at a node the children are tried in index order against the
//                            running residual of the verifier's distribution, the first accepted child is descended
//                            into, and where none is accepted one token is drawn from what is left; every pass over
//                            the vocabulary is spread over the chip;
//   tree_accept_alone_kernel the same by one block per sequence: greedy matching, small calls, captured ones;
//   kv_compact_tree_kernel   after acceptance: the accepted nodes' K/V rows move to consecutive cache positions.
//
// The residual after j refusals at one node needs no vector: with p, q the two distributions at the node,
//   r_0 = p,  r_{j+1} = norm(max(0, r_j - q))   =>   r_j is proportional to R_j = max(0, p - c_j q),
//   c_0 = 0,  c_{j+1} = c_j + M_j,  M_j = sum_i R_j[i]  (M_0 = 1),
// (induction: max(0, R_j / M_j - q) = max(0, p - (c_j + M_j) q) / M_j), so a refusal costs one pass over the
// vocabulary for M_{j+1}, and child j + 1 with token x is accepted with probability min(1, R_j[x] / (M_j q[x])).
// Everything that decides a token runs in fp64 with a fixed summation order.
#include <atomic>

#include "common.h"
#include "kernels.h"
#include "exp64.h"
#include "prof.h"
#include "../../include/psd.h"

namespace psd {
namespace {

constexpr int kTreeThreads = 1024;
constexpr int kTreeWaves = kTreeThreads / 64;

// block-wide sum in a fixed order: butterfly inside each wavefront, wavefronts added in order; every thread gets it
__device__ __forceinline__ double block_sum_d(double v, double *s_w) {
    v = wave_sum(v);
    __syncthreads();                                       // s_w may still be read from the previous call
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kTreeWaves; ++w) t += s_w[w];
    return t;
}

// The vocabulary is cut into chunks of kTreeChunk entries and these into pieces of kPiece, one wavefront's work: lane l has
// the entries l, l + 64, ... of a piece.  Every sum over a row adds in the same order whoever takes it: over a lane's
// entries, over the lanes, over the pieces of a chunk, over the chunks (one a lane).  So a call's result does not depend
// on which of the two ways of walking the tree it gets.
constexpr int kTreeChunk = 4096, kPiece = 256, kPieces = kTreeChunk / kPiece, kPerLane = kPiece / 64;
constexpr int kTreeMaxChunks = 64;                // per row: one per lane
constexpr int kMassPasses = 3;                    // refusals at one node whose masses are added piece by piece (all of them at a
                                                  //   node of up to four children: the last refusal needs none)
static_assert(kPieces == 16, "a chunk's pieces are joined by 16 lanes");

struct TreeStat { double zp, zq; float mp, mq; };                  // sums of exp((l - max) / T), maxima

// this lane's entries of the piece that begins at `first` (-infinity past the end of the row)
template <typename T>
__device__ __forceinline__ void load_piece(const T *row, int first, int V, float (&x)[kPerLane]) {
    const T *at = row + first;
    const int lane = threadIdx.x & 63, left = __builtin_amdgcn_readfirstlane(V - first);
    if (left >= kPiece) {
#pragma unroll
        for (int i = 0; i < kPerLane; ++i) x[i] = load_elem(at, (size_t)(lane + i * 64));
    } else {
#pragma unroll
        for (int i = 0; i < kPerLane; ++i) x[i] = lane + i * 64 < left ? load_elem(at, (size_t)(lane + i * 64)) : -INFINITY;
    }
}
// a lane's share of a piece's denominators, against maxima taken over the whole wavefront
__device__ __forceinline__ TreeStat piece_stat(const float (&p)[kPerLane], const float (&q)[kPerLane], double inv_t, const double *exp2tab) {
    TreeStat t{0.0, 0.0, p[0], q[0]};
#pragma unroll
    for (int i = 1; i < kPerLane; ++i) { t.mp = fmaxf(t.mp, p[i]); t.mq = fmaxf(t.mq, q[i]); }
    t.mp = wave_top_f(t.mp);
    t.mq = wave_top_f(t.mq);
    const double dp = (double)t.mp * inv_t, dq = (double)t.mq * inv_t;
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) {
        t.zp += exp_nonpos(fma((double)p[i], inv_t, -dp), exp2tab);
        t.zq += exp_nonpos(fma((double)q[i], inv_t, -dq), exp2tab);
    }
    return t;
}
// z against the maximum m, now against `top`; a piece or chunk of -infinities contributes nothing
__device__ __forceinline__ double against(double z, float m, float top, double inv_t, const double *exp2tab) {
    return m > -INFINITY ? z * exp_nonpos(fma((double)m, inv_t, -(double)top * inv_t), exp2tab) : 0.0;
}
// over the 16 lanes that hold a chunk's pieces
__device__ __forceinline__ double join_pieces(double v) {
#pragma unroll
    for (int o = kPieces / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ TreeStat join_pieces(const TreeStat &t, double inv_t, const double *exp2tab) {
    float mp = t.mp, mq = t.mq;
#pragma unroll
    for (int o = kPieces / 2; o > 0; o >>= 1) {
        mp = fmaxf(mp, __shfl_xor(mp, o, 64));
        mq = fmaxf(mq, __shfl_xor(mq, o, 64));
    }
    return TreeStat{join_pieces(against(t.zp, t.mp, mp, inv_t, exp2tab)), join_pieces(against(t.zq, t.mq, mq, inv_t, exp2tab)), mp, mq};
}

struct NodeStat { double mp, mq, inv_zp, inv_zq; };                // scaled maxima, reciprocals of the denominators
// one wavefront, lane = chunk
__device__ __forceinline__ NodeStat node_stat(const TreeStat *st, int chunks, double inv_t, const double *exp2tab) {
    const int lane = threadIdx.x & 63;
    TreeStat t = st[min(lane, chunks - 1)];
    if (lane >= chunks) t.mp = t.mq = -INFINITY;
    const float mp = wave_top_f(t.mp), mq = wave_top_f(t.mq);
    NodeStat s;
    s.mp = (double)mp * inv_t;
    s.mq = (double)mq * inv_t;
    s.inv_zp = 1.0 / wave_total_d(against(t.zp, t.mp, mp, inv_t, exp2tab));
    s.inv_zq = 1.0 / wave_total_d(against(t.zq, t.mq, mq, inv_t, exp2tab));
    return s;
}
// weight of one entry in the residual max(0, p - c q)
__device__ __forceinline__ double residual(const NodeStat &s, float lp, float lq, double c, double inv_t, const double *exp2tab) {
    const double pi = exp_nonpos(fma((double)lp, inv_t, -s.mp), exp2tab) * s.inv_zp;
    const double qi = exp_nonpos(fma((double)lq, inv_t, -s.mq), exp2tab) * s.inv_zq;
    return fmax(fma(-c, qi, pi), 0.0);
}
// a lane's share of a piece's residual mass
__device__ __forceinline__ double piece_mass(const NodeStat &s, const float (&p)[kPerLane], const float (&q)[kPerLane], double c,
                                             double inv_t, const double *exp2tab) {
    double m = 0.0;
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) m += residual(s, p[i], q[i], c, inv_t, exp2tab);
    return m;
}
// (c, mass) of the residual max(0, p - c q) / mass, taken one refusal further: mass 0 means that the residual equalled q,
// where no refusal can happen
__device__ __forceinline__ void refuse(double m, double *c, double *mass) {
    if (m > 0.0) { *c += *mass; *mass = m; }
}
// (order-preserving bits of the logit) << 32 | ~index: the largest is the likeliest token, the lowest index among equals
__device__ __forceinline__ unsigned long long argmax_key(float x, int i) {
    uint32_t b = __float_as_uint(x);
    b = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
    return ((unsigned long long)b << 32) | (uint32_t)(~(uint32_t)i);
}

// ---- the same walk spread over the chip.  What a node's decisions need is taken for all nodes at once, chunk by chunk:
// tree_stats_kernel (softmax statistics) and, for nodes with more than j children, tree_mass_kernel j (the residual mass M_j
// after j refusals, j = 1 .. kMassPasses); then every block of tree_draw_kernel walks the tree on those numbers, sums the
// weights of its chunk of the row the draw reads, and the block of a sequence that arrives last finds the token.  Bound by
// fp64 arithmetic (2 exponentials per entry and pass: one block needs about 15 us per pass of 32 000 entries) and by the
// launches.  Four sequences x 15 nodes x 32 000 entries (fp32 logits): 127 us with a block per sequence, 41 us this way;
// which way a call goes: spread_pays.
//
// The statistics travel through a slot of a static array, so that the call needs no workspace.  Calls on different
// streams may overlap: a call has a number of its own (the host counts them) and tree_claim_kernel takes the slot that
// number selects, by compare-and-swap, if it is free.  A call that did not get it falls back to walk_alone, decided on the
// device by the same test in every later block.  Nothing waits.  The last block of the last kernel frees the slot.
// (Claimed by the 480 blocks of the statistics kernel themselves, the same-address atomics took 13 us.)  Calls under graph
// capture, vocabularies above 262 144 entries and calls whose statistics exceed a slot (64 sequences x 8 nodes x 32 000
// entries need 213 KB, 24 bytes and kMassPasses times 8 a chunk and node) run walk_alone from the start.
constexpr int kTreeSlots = 4;
constexpr size_t kTreeSlotBytes = 512 << 10;
struct TreeSlotHead { uint32_t owner, done, pad[62]; };
__device__ __align__(256) unsigned char g_tree_slots[kTreeSlots * kTreeSlotBytes];

struct TreeShare {
    uint32_t id;                                  // this call's number, never 0
    int n_chunks;
    int n_inner[kMassPasses];                     // nodes with more than j + 1 children ...
    uint8_t inner[kMassPasses][kTreeMaxAcceptNodes];   // ... and which
};
struct SlotView {
    TreeSlotHead *head;
    uint32_t *count;                              // [rows] chunks of the draw done
    TreeStat *stat;                               // [rows][n][chunks]
    double *mass;                                 // [kMassPasses][rows][n][chunks]
    double *part;                                 // [rows][chunks]
};
__host__ __device__ inline size_t slot_layout(int rows, int n, int chunks, size_t *stat, size_t *mass, size_t *part) {
    size_t at = sizeof(TreeSlotHead) + ((size_t)rows * 4 + 255) / 256 * 256;
    *stat = at; at += (size_t)rows * n * chunks * sizeof(TreeStat);
    *mass = at; at += (size_t)kMassPasses * rows * n * chunks * 8;
    *part = at; at += (size_t)rows * chunks * 8;
    return at;
}
__device__ __forceinline__ SlotView slot_of(const TreeAcceptArgs &a, const TreeShare &sh) {
    unsigned char *base = g_tree_slots + (sh.id % kTreeSlots) * kTreeSlotBytes;
    size_t st, ms, pt;
    slot_layout(a.rows, a.n_nodes, sh.n_chunks, &st, &ms, &pt);
    return SlotView{(TreeSlotHead *)base, (uint32_t *)(base + sizeof(TreeSlotHead)), (TreeStat *)(base + st), (double *)(base + ms),
                    (double *)(base + pt)};
}
__device__ __forceinline__ bool slot_is_mine(const SlotView &s, const TreeShare &sh) {
    return __hip_atomic_load(&s.head->owner, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == sh.id;
}
__global__ void tree_claim_kernel(TreeAcceptArgs a, TreeShare sh) {
    const SlotView sv = slot_of(a, sh);
    int mine = 0;
    if (threadIdx.x == 0) {
        uint32_t was = 0;
        mine = __hip_atomic_compare_exchange_strong(&sv.head->owner, &was, sh.id, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
    }
    if (__shfl(mine, 0, 64))
        for (int i = threadIdx.x; i < a.rows; i += 64) sv.count[i] = 0u;
}

// Measured (us a call, 256 / 512 / 1024 threads; in the same order of sums): 4 sequences x 15 nodes x 32 000 entries about
// 41 / 40 / 38, 64 x 7 x 32 000 in bf16 136 / 119 / 130, 8 x 15 x 128 256 101 / 98 / 106.
constexpr int kStatThreads = 512, kStatWaves = kStatThreads / 64, kWavePieces = kPieces / kStatWaves;

// Grid: rows x nodes x chunks; a wavefront takes kWavePieces pieces of its chunk.
template <typename T>
__global__ __launch_bounds__(kStatThreads) void tree_stats_kernel(TreeAcceptArgs a, TreeShare sh) {
    __shared__ double s_exp2[64];
    __shared__ TreeStat s_piece[kPieces];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, V = a.vocab;
    const SlotView sv = slot_of(a, sh);
    if (!slot_is_mine(sv, sh)) return;
    if (tid < 64) s_exp2[tid] = kExp2Table[tid];
    const int c = blockIdx.x % sh.n_chunks, rn = blockIdx.x / sh.n_chunks, node = rn % a.n_nodes, row = rn / a.n_nodes;
    const T *lp = (const T *)a.p + (size_t)row * a.p_stride + (size_t)node * V;
    const T *lq = (const T *)a.q + (size_t)row * a.q_stride + (size_t)node * V;
    const int first = c * kTreeChunk + wave * kWavePieces * kPiece;
    float p[kWavePieces][kPerLane], q[kWavePieces][kPerLane];
#pragma unroll
    for (int k = 0; k < kWavePieces; ++k) {
        load_piece(lp, first + k * kPiece, V, p[k]);
        load_piece(lq, first + k * kPiece, V, q[k]);
    }
    __syncthreads();
    const double inv_t = 1.0 / (double)a.temperature;
    TreeStat t[kWavePieces];
#pragma unroll
    for (int k = 0; k < kWavePieces; ++k) {
        t[k] = piece_stat(p[k], q[k], inv_t, s_exp2);
        t[k].zp = wave_total_d(t[k].zp);
        t[k].zq = wave_total_d(t[k].zq);
    }
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < kWavePieces; ++k) s_piece[wave * kWavePieces + k] = t[k];
    __syncthreads();
    if (wave != 0) return;
    const TreeStat all = join_pieces(s_piece[lane % kPieces], inv_t, s_exp2);
    if (lane == 0) sv.stat[(size_t)rn * sh.n_chunks + c] = all;
}

// M_{j+1} = sum max(0, p - c q) of one chunk of one node, c after j refusals and the next
template <typename T>
__global__ __launch_bounds__(kStatThreads) void tree_mass_kernel(TreeAcceptArgs a, TreeShare sh, int j) {
    __shared__ double s_exp2[64];
    __shared__ double s_piece[kPieces];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, V = a.vocab;
    const SlotView sv = slot_of(a, sh);
    if (!slot_is_mine(sv, sh)) return;
    if (tid < 64) s_exp2[tid] = kExp2Table[tid];
    const int ch = sh.n_chunks, c = blockIdx.x % ch, rn = blockIdx.x / ch, row = rn / sh.n_inner[j];
    const int node = sh.inner[j][rn % sh.n_inner[j]];
    const int first = c * kTreeChunk + wave * kWavePieces * kPiece;
    float p[kWavePieces][kPerLane], q[kWavePieces][kPerLane];
#pragma unroll
    for (int k = 0; k < kWavePieces; ++k) {
        load_piece((const T *)a.p + (size_t)row * a.p_stride + (size_t)node * V, first + k * kPiece, V, p[k]);
        load_piece((const T *)a.q + (size_t)row * a.q_stride + (size_t)node * V, first + k * kPiece, V, q[k]);
    }
    __syncthreads();
    const double inv_t = 1.0 / (double)a.temperature;
    const size_t at = ((size_t)row * a.n_nodes + node) * ch, pass = (size_t)a.rows * a.n_nodes * ch;
    const NodeStat s = node_stat(sv.stat + at, ch, inv_t, s_exp2);
    double cc = 0.0, mass = 1.0;
    for (int t = 0; t < j; ++t) refuse(wave_total_d(lane < ch ? sv.mass[t * pass + at + lane] : 0.0), &cc, &mass);
    double m[kWavePieces];
#pragma unroll
    for (int k = 0; k < kWavePieces; ++k) m[k] = wave_total_d(piece_mass(s, p[k], q[k], cc + mass, inv_t, s_exp2));
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < kWavePieces; ++k) s_piece[wave * kWavePieces + k] = m[k];
    __syncthreads();
    if (wave != 0) return;
    const double all = join_pieces(s_piece[lane % kPieces]);
    if (lane == 0) sv.mass[j * pass + at + c] = all;
}

// this call's last access to the slot: whoever counts last hands it back
__device__ __forceinline__ void slot_leave(const SlotView &s, unsigned blocks) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x != 0) return;
    if (__hip_atomic_fetch_add(&s.head->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != blocks - 1) return;
    __hip_atomic_store(&s.head->done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __hip_atomic_store(&s.head->owner, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Greedy matching of one sequence by one block.
template <typename T>
__device__ void walk_alone_greedy(const TreeAcceptArgs &a, int row) {
    __shared__ int s_par[kTreeMaxAcceptNodes];
    __shared__ unsigned long long s_best;
    const int tid = threadIdx.x, n = a.n_nodes, V = a.vocab;
    for (int j = tid; j < n; j += kTreeThreads) s_par[j] = a.parents[j];
    __syncthreads();
    const T *P = (const T *)a.p + (size_t)row * a.p_stride;
    const int32_t *tok = a.tokens + (size_t)row * n;
    int32_t *path = a.out_path + (size_t)row * n;
    int node = 0, plen = 0;
    while (true) {                                          // every descent moves to a larger node index: at most n rounds
        const T *lp = P + (size_t)node * V;
        unsigned long long best = 0ull;
        for (int i = tid; i < V; i += kTreeThreads) {
            const unsigned long long key = argmax_key(load_elem(lp, (size_t)i), i);
            best = key > best ? key : best;
        }
        best = wave_max(best);
        if (tid == 0) s_best = 0ull;
        __syncthreads();
        if ((tid & 63) == 0) atomicMax(&s_best, best);
        __syncthreads();
        const int top = (int)(~(uint32_t)(s_best & 0xffffffffull));
        int next = -1;
        for (int c = node + 1; c < n && next < 0; ++c)
            if (s_par[c] == node && tok[c] == top) next = c;
        __syncthreads();                                    // s_best is reset by the next round
        if (next < 0) {
            if (tid == 0) { a.out_path_len[row] = plen; a.out_token[row] = top; if (a.out_flags) a.out_flags[row] = 0; }
            return;
        }
        if (tid == 0) path[plen] = next;
        ++plen;
        node = next;
    }
}

// The walk of one sequence.  ALONE: by one block, which takes the statistics of the nodes it visits itself and needs no
// memory to share (more than kTreeMaxChunks chunks: longer ones, of `sub` times kTreeChunk entries).  Otherwise by
// `chunks` blocks on what the kernels above left in the slot: block `chunk` sums the draw's weights over its chunk, and
// the one that counts itself in last finds the token.
template <typename T, bool ALONE>
__device__ void walk(const TreeAcceptArgs &a, const SlotView &sv, int row, int chunk, int chunks, int sub) {
    constexpr int E = kTreeChunk / kTreeThreads;
    __shared__ double s_wd[kTreeWaves], s_exp2[64];
    __shared__ NodeStat s_node[ALONE ? 1 : kTreeMaxAcceptNodes];
    __shared__ double s_mass[ALONE ? 1 : kMassPasses][kTreeMaxAcceptNodes], s_px[kTreeMaxAcceptNodes], s_qx[kTreeMaxAcceptNodes];
    __shared__ float s_u[kTreeMaxAcceptNodes + 1];
    __shared__ int s_par[kTreeMaxAcceptNodes], s_tok[kTreeMaxAcceptNodes], s_kids[kTreeMaxAcceptNodes];
    __shared__ int s_pick, s_lastpos, s_chunk, s_last;
    __shared__ double s_target, s_base;
    __shared__ TreeStat s_piece[ALONE ? kTreeMaxChunks * kPieces : 1], s_chunk_stat[ALONE ? kTreeMaxChunks : 1];
    __shared__ double s_part[ALONE ? kTreeMaxChunks : 1][kPieces + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = a.n_nodes, V = a.vocab, length = sub * kTreeChunk;
    const T *P = (const T *)a.p + (size_t)row * a.p_stride;
    const T *Q = (const T *)a.q + (size_t)row * a.q_stride;
    const double inv_t = 1.0 / (double)a.temperature;
    int32_t *path = a.out_path + (size_t)row * n;
    if (tid < 64) s_exp2[tid] = kExp2Table[tid];
    if (tid < n) {
        s_par[tid] = a.parents[tid];
        s_tok[tid] = a.tokens[(size_t)row * n + tid];
        s_kids[tid] = 0;
    }
    if (tid <= n) s_u[tid] = a.uniforms[(size_t)row * (n + 1) + tid];
    __syncthreads();
    if (tid > 0 && tid < n) atomicAdd(&s_kids[s_par[tid]], 1);
    __syncthreads();
    NodeStat here;                                              // alone: of the node the walk is at
    auto stat_of = [&](int v) {
        if constexpr (ALONE) return here;
        else return s_node[v];
    };
    // the probabilities at its parent of the token that node v carries
    auto probe = [&](int v) {
        const NodeStat s = stat_of(s_par[v]);
        const size_t at = (size_t)s_par[v] * V + min(max(s_tok[v], 0), V - 1);
        s_px[v] = exp_nonpos(fma((double)load_elem(P, at), inv_t, -s.mp), s_exp2) * s.inv_zp;
        s_qx[v] = exp_nonpos(fma((double)load_elem(Q, at), inv_t, -s.mq), s_exp2) * s.inv_zq;
    };
    if constexpr (!ALONE) {
        // every node's statistics and masses, then every child's probabilities, all at once
        const size_t row_at = (size_t)row * n * chunks;
        for (int v = wave; v < n; v += kTreeWaves) {
            const NodeStat s = node_stat(sv.stat + row_at + (size_t)v * chunks, chunks, inv_t, s_exp2);
            double m[kMassPasses];
#pragma unroll
            for (int j = 0; j < kMassPasses; ++j) {
                const bool there = s_kids[v] > j + 1 && lane < chunks;
                m[j] = wave_total_d(there ? sv.mass[((size_t)j * a.rows * n + (size_t)row * n + v) * chunks + lane] : 0.0);
            }
            if (lane == 0) {
                s_node[v] = s;
#pragma unroll
                for (int j = 0; j < kMassPasses; ++j) s_mass[j][v] = m[j];
            }
        }
        __syncthreads();
        if (tid > 0 && tid < n) probe(tid);
        __syncthreads();
    }
    // alone: statistics of a node, then its children's probabilities
    auto visit = [&](int v) {
        const T *lp = P + (size_t)v * V, *lq = Q + (size_t)v * V;
        for (int c = 0; c < chunks; ++c) {
            TreeStat all{0.0, 0.0, -INFINITY, -INFINITY};
            for (int k = 0; k < sub; ++k) {
                const int first = c * length + k * kTreeChunk + wave * kPiece;
                if (first >= V) break;                          // the same for the wavefront
                float p[kPerLane], q[kPerLane];
                load_piece(lp, first, V, p);
                load_piece(lq, first, V, q);
                const TreeStat t = piece_stat(p, q, inv_t, s_exp2);
                if (k == 0) {
                    all = t;
                } else {
                    const float mp = fmaxf(all.mp, t.mp), mq = fmaxf(all.mq, t.mq);
                    all.zp = against(all.zp, all.mp, mp, inv_t, s_exp2) + against(t.zp, t.mp, mp, inv_t, s_exp2);
                    all.zq = against(all.zq, all.mq, mq, inv_t, s_exp2) + against(t.zq, t.mq, mq, inv_t, s_exp2);
                    all.mp = mp;
                    all.mq = mq;
                }
            }
            all.zp = wave_total_d(all.zp);
            all.zq = wave_total_d(all.zq);
            if (lane == 0) s_piece[c * kPieces + wave] = all;
        }
        __syncthreads();
        if (wave * 64 < chunks * kPieces) {                     // one piece a lane
            const TreeStat t = join_pieces(s_piece[min(tid, chunks * kPieces - 1)], inv_t, s_exp2);
            if (tid % kPieces == 0 && tid < chunks * kPieces) s_chunk_stat[tid / kPieces] = t;
        }
        __syncthreads();
        if (wave == 0) {
            const NodeStat t = node_stat(s_chunk_stat, chunks, inv_t, s_exp2);
            if (lane == 0) s_node[0] = t;
        }
        __syncthreads();
        here = s_node[0];
        if (tid > v && tid < n && s_par[tid] == v) probe(tid);
        __syncthreads();
    };
    // alone: the sums over the chunks of what f(chunk) gives each lane, chunk l in lane l
    auto by_chunks = [&](auto f) {
        for (int c = 0; c < chunks; ++c) {
            const double m = wave_total_d(f(c));
            if (lane == 0) s_part[c][wave] = m;
        }
        __syncthreads();
        double v[kPieces];                                      // added in join_pieces' order
#pragma unroll
        for (int k = 0; k < kPieces; ++k) v[k] = s_part[min(lane, chunks - 1)][k];
#pragma unroll
        for (int o = kPieces / 2; o > 0; o >>= 1)
#pragma unroll
            for (int k = 0; k < o; ++k) v[k] += v[k + o];
        __syncthreads();                                        // s_part: read before the next pass writes it
        return lane < chunks ? v[0] : 0.0;
    };
    auto mass_by_chunks = [&](int v, double c) {
        const T *lp = P + (size_t)v * V, *lq = Q + (size_t)v * V;
        const NodeStat s = stat_of(v);
        return wave_total_d(by_chunks([&](int ch) {
            double m = 0.0;
            for (int first = ch * length + wave * kPiece; first < min(ch * length + length, V); first += kTreeChunk) {
                float p[kPerLane], q[kPerLane];
                load_piece(lp, first, V, p);
                load_piece(lq, first, V, q);
                m += piece_mass(s, p, q, c, inv_t, s_exp2);
            }
            return m;
        }));
    };
    auto mass_of_row = [&](int v, double c) {                   // past the first kMassPasses refusals
        const NodeStat s = stat_of(v);
        double m = 0.0;
        for (int e = tid; e < V; e += kTreeThreads)
            m += residual(s, load_elem(P, (size_t)v * V + e), load_elem(Q, (size_t)v * V + e), c, inv_t, s_exp2);
        return block_sum_d(m, s_wd);
    };
    // the walk (every thread alike): at a node the children are tried in index order
    const bool writer = chunk == 0 && tid == 0;
    int node = 0, plen = 0, flags = 0;
    double c = 0.0, mass = 1.0, c_before = 0.0;
    while (true) {                                              // every descent moves to a larger node index: at most n rounds
        if constexpr (ALONE) visit(node);
        int next = -1, tried = 0;
        c = 0.0; mass = 1.0; c_before = 0.0;                    // the residual here is max(0, p - c q) / mass
        for (int k = node + 1; k < n; ++k) {
            if (s_par[k] != node) continue;
            ++tried;
            const double rx = fmax(s_px[k] - c * s_qx[k], 0.0);
            const double ratio = s_qx[k] == 0.0 ? INFINITY : rx / (mass * s_qx[k]);
            const double thr = fmin(1.0, ratio), uu = (double)s_u[k];
            if (fabs(uu - thr) < 1e-5) flags |= PSD_FLAG_NEAR_TIE;
            if (uu < thr) { next = k; break; }
            c_before = c;
            if (tried == s_kids[node]) { c += mass; continue; } // the draw's own sums say whether anything is left
            double m;
            if (tried > kMassPasses) m = mass_of_row(node, c + mass);
            else if constexpr (ALONE) m = mass_by_chunks(node, c + mass);
            else m = s_mass[tried - 1][node];
            refuse(m, &c, &mass);
        }
        if (next < 0) break;
        if (writer) path[plen] = next;
        ++plen;
        node = next;
    }
    // one draw from max(0, p - c q) by inverse CDF in index order: first the weight of every chunk
    const NodeStat s = stat_of(node);
    const T *lp = P + (size_t)node * V, *lq = Q + (size_t)node * V;
    auto entry = [&](int e, double at_c) {
        return residual(s, load_elem(lp, (size_t)e), load_elem(lq, (size_t)e), at_c, inv_t, s_exp2);
    };
    auto my_share = [&](int ch) {                               // of chunk ch: E consecutive entries of every kTreeChunk
        double w = 0.0;
        for (int t0 = ch * length; t0 < min(ch * length + length, V); t0 += kTreeChunk) {
            const int i0 = min(t0 + tid * E, V), i1 = min(i0 + E, V);
#pragma unroll
            for (int k = 0; k < E; ++k)
                if (i0 + k < i1) w += entry(i0 + k, c);
        }
        return w;
    };
    double mine = 0.0;                                          // first wavefront: the weight of chunk `lane`
    if constexpr (ALONE) {
        mine = by_chunks(my_share);
    } else {
        const double part = wave_total_d(my_share(chunk));
        __syncthreads();                                        // s_wd: a refusal's pass may still be read
        if (lane == 0) s_wd[wave] = part;
        __syncthreads();
        if (wave == 0) {
            const double w = join_pieces(s_wd[lane % kPieces]);
            if (lane == 0) {
                __hip_atomic_store(sv.part + (size_t)row * chunks + chunk, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                s_last = __hip_atomic_fetch_add(sv.count + row, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)chunks - 1u;
            }
        }
        __syncthreads();
        if (!s_last) return;
        if (wave == 0 && lane < chunks)
            mine = __hip_atomic_load(sv.part + (size_t)row * chunks + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (wave == 0) {
        double incl = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        const double total = __shfl(incl, 63, 64), target = (double)s_u[n] * total;
        const unsigned long long over = __ballot(mine > 0.0 && incl > target), any = __ballot(mine > 0.0);
        // no crossing through rounding: the last chunk that holds weight, whose walk then ends at its last positive entry
        const int pick = over ? __ffsll(over) - 1 : (any ? 63 - __clzll(any) : -1);
        if (lane == (pick < 0 ? 0 : pick)) {
            s_chunk = pick;
            s_base = incl - mine;
            s_target = target;
        }
    }
    if (tid == 0) { s_pick = kTreeThreads; s_lastpos = -1; }
    __syncthreads();
    int first = s_chunk * length, last = min(first + length, V);
    double base = s_base, target = s_target;
    if (s_chunk < 0 && c != c_before) {
        // the last refusal left a mass of exactly 0 (the residual equalled q): the draw is from what was there before it
        c = c_before;
        target = (double)s_u[n] * mass_of_row(node, c);
    }
    if (s_chunk < 0) { first = 0; last = V; base = 0.0; }       // all of the row
    __syncthreads();
    for (int t0 = first; t0 < last; t0 += kTreeChunk) {
        const int j0 = min(t0 + tid * E, last), j1 = min(j0 + E, last);
        double wv[E], sum = 0.0;
        int lastpos = -1;
#pragma unroll
        for (int k = 0; k < E; ++k) {
            wv[k] = j0 + k < j1 ? entry(j0 + k, c) : 0.0;
            if (wv[k] > 0.0) lastpos = j0 + k;
            sum += wv[k];
        }
        double incl = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        __syncthreads();                                        // s_wd: earlier readers are done
        if (lane == 63) s_wd[wave] = incl;
        __syncthreads();
        double before = base, total = 0.0;
#pragma unroll
        for (int v = 0; v < kTreeWaves; ++v) {
            if (v < wave) before += s_wd[v];
            total += s_wd[v];
        }
        if (sum > 0.0 && before + incl > target) atomicMin(&s_pick, tid);
        if (lastpos >= 0) atomicMax(&s_lastpos, lastpos);
        __syncthreads();
        if (s_pick < kTreeThreads) {
            if (tid == s_pick) {
                double cum = before + incl - sum;
                int token = lastpos;                            // rounding left no crossing inside: the last positive entry
                bool found = false;
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    cum += wv[k];
                    if (!found && j0 + k < j1 && cum > target) { token = j0 + k; found = true; }
                }
                a.out_token[row] = token;
            }
            break;                                              // the same for the whole block
        }
        base += total;
    }
    if (tid == 0) {
        if (s_pick == kTreeThreads) a.out_token[row] = s_lastpos;
        a.out_path_len[row] = plen;
        if (a.out_flags) a.out_flags[row] = flags;
    }
}

template <typename T>
__device__ __forceinline__ void walk_alone(const TreeAcceptArgs &a, int row) {
    if (a.temperature == 0.f) return walk_alone_greedy<T>(a, row);
    const int tiles = (a.vocab + kTreeChunk - 1) / kTreeChunk, sub = (tiles + kTreeMaxChunks - 1) / kTreeMaxChunks;
    walk<T, true>(a, SlotView{}, row, 0, (tiles + sub - 1) / sub, sub);
}
template <typename T>
__global__ __launch_bounds__(kTreeThreads) void tree_accept_alone_kernel(TreeAcceptArgs a) { walk_alone<T>(a, blockIdx.x); }

// Grid: rows x chunks.
template <typename T>
__global__ __launch_bounds__(kTreeThreads) void tree_draw_kernel(TreeAcceptArgs a, TreeShare sh) {
    const SlotView sv = slot_of(a, sh);
    const bool mine = slot_is_mine(sv, sh);                 // only this call's blocks can end that, after all have counted
    const int chunk = blockIdx.x % sh.n_chunks, row = blockIdx.x / sh.n_chunks;
    if (mine) {
        walk<T, false>(a, sv, row, chunk, sh.n_chunks, 1);
        slot_leave(sv, gridDim.x);
    } else if (chunk == 0) {
        walk_alone<T>(a, row);
    }
}

// One block per (layer, sequence, KV head).  Thread t moves element t of the d_h-long K row and of the V^T column of
// every accepted node, in path order: destination j is never a later source (sources grow along a path and a
// source is never below its destination), and each element has one thread, so no synchronisation is needed.
template <typename T>
__global__ __launch_bounds__(128) void kv_compact_tree_kernel(T *k, T *v, int32_t *lens, const int32_t *base,
                                                              const int32_t *path, const int32_t *path_len, int path_stride,
                                                              int n_nodes, int B, int h_kv, int d_h, int max_len, int cap) {
    const int hk = blockIdx.x % h_kv, b = (blockIdx.x / h_kv) % B;
    const size_t head = (size_t)blockIdx.x * max_len * d_h;           // blockIdx.x = (l * B + b) * h_kv + hk
    T *kh = k + head, *vh = v + head;
    const int s0 = base[b];
    int plen = path_len[b];
    plen = min(max(plen, 0), n_nodes - 1);
    for (int j = 0; j < plen; ++j) {
        const int node = path[(size_t)b * path_stride + j];
        const int src = s0 + node, dst = s0 + 1 + j;
        if (node < 1 || node >= n_nodes || src >= max_len || src == dst) continue;
        for (int t = threadIdx.x; t < d_h; t += blockDim.x) {
            kh[(size_t)dst * d_h + t] = kh[(size_t)src * d_h + t];
            vh[(size_t)t * max_len + dst] = vh[(size_t)t * max_len + src];
        }
    }
    if (blockIdx.x / (h_kv * B) == 0 && hk == 0 && threadIdx.x == 0) lens[b] = max(0, min(min(lens[b], cap), s0 + 1 + plen));
}

}  // namespace

// This call's number, never 0.  One count for all element types: the number says which slot a call takes and whether a
// slot is its own, and calls of both types share the slots.
static uint32_t tree_call_number() {
    static std::atomic<uint32_t> tree_calls{0};
    uint32_t id;
    do id = tree_calls.fetch_add(1, std::memory_order_relaxed) + 1;
    while (id == 0);
    return id;
}

// Whether spreading a call over the chip is the faster way.  Both times are estimates (us) fitted to calls of 1 to 128
// sequences, 1 to 41 nodes and 512 to 128 256 entries.  Spread: the launches; 9 a mass pass; 12 a round of the draw's blocks
// (one per CU); 2.4 per million entries that the statistics and mass passes read, those of every node whether the walk
// gets there or not.  One block per sequence: 0.5 per thousand entries and pass; about 1.2 passes a level of the tree, and
// more the more sequences there are, since the longest walk counts.  Measured, spread / one block: 1 x 15 x 4096 34.9 / 33.8,
// 1 x 15 x 10 000 35.7 / 53.8, 1 x 31 x 10 000 (four children) 55.6 / 56.5, 4 x 15 x 32 000 40.8 / 127, 64 x 7 x 32 000 102 /
// 123, 64 x 15 x 32 000 161 / 147, 128 x 7 x 32 000 182 / 123, 32 x 7 x 128 256 176 / 363.
static bool spread_pays(const TreeAcceptArgs &a, const TreeShare &sh) {
    double entries = (double)a.rows * a.n_nodes, passes = 0.0, rows_pow = 0.0;
    for (int j = 0; j < kMassPasses && sh.n_inner[j] > 0; ++j) { entries += (double)a.rows * sh.n_inner[j]; ++passes; }
    int depth[kTreeMaxAcceptNodes] = {}, deepest = 0;
    for (int i = 1; i < a.n_nodes; ++i) {
        depth[i] = depth[a.parents[i]] + 1;
        deepest = depth[i] > deepest ? depth[i] : deepest;
    }
    for (int r = 1; r < a.rows; r *= 2) ++rows_pow;
    const double rounds = (double)(((long)a.rows * sh.n_chunks + 255) / 256);
    const double spread = 17.0 + 9.0 * passes + 12.0 * rounds + 2.4e-6 * entries * a.vocab;
    const double alone = 17.0 + 0.5e-3 * a.vocab * (2.0 + 1.2 * deepest + 0.4 * rows_pow);
    return spread < alone;
}

template <typename T>
static void launch_tree_accept_t(const TreeAcceptArgs &a, hipStream_t stream) {
    auto alone = [&]() { launch_kernel(tree_accept_alone_kernel<T>, a.rows, kTreeThreads, 0, stream, a); };
    // greedy: one launch that reads each visited node once is faster at every size measured but the largest (a path of
    // two nodes, 128 256 entries: 21 us, spread 22; 32 sequences of them 42 / 33)
    if (a.temperature == 0.f) return alone();
    TreeShare sh{};
    sh.n_chunks = (a.vocab + kTreeChunk - 1) / kTreeChunk;
    size_t st, ms, pt;
    if (sh.n_chunks > kTreeMaxChunks || slot_layout(a.rows, a.n_nodes, sh.n_chunks, &st, &ms, &pt) > kTreeSlotBytes) return alone();
    int kids[kTreeMaxAcceptNodes] = {};
    for (int i = 1; i < a.n_nodes; ++i) ++kids[a.parents[i]];
    for (int j = 0; j < kMassPasses; ++j)
        for (int i = 0; i < a.n_nodes; ++i)
            if (kids[i] > j + 1) sh.inner[j][sh.n_inner[j]++] = (uint8_t)i;
    if (!spread_pays(a, sh)) return alone();
    // a captured call would keep its number in every copy of its graph, and two copies may run at once
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    const bool captured = hipStreamIsCapturing(stream, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    if (captured) return alone();
    sh.id = tree_call_number();
    launch_kernel(tree_claim_kernel, 1, 64, 0, stream, a, sh);
    launch_kernel(tree_stats_kernel<T>, (unsigned)(a.rows * a.n_nodes * sh.n_chunks), kStatThreads, 0, stream, a, sh);
    for (int j = 0; j < kMassPasses && sh.n_inner[j] > 0; ++j)
        launch_kernel(tree_mass_kernel<T>, (unsigned)(a.rows * sh.n_inner[j] * sh.n_chunks), kStatThreads, 0, stream, a, sh, j);
    launch_kernel(tree_draw_kernel<T>, (unsigned)(a.rows * sh.n_chunks), kTreeThreads, 0, stream, a, sh);
}

void launch_tree_accept(int dtype, const TreeAcceptArgs &a, hipStream_t stream) {
    ScopedProf sp(PSD_KIND_ACCEPT_DRAW, stream);
    if (dtype == PSD_BF16) launch_tree_accept_t<uint16_t>(a, stream);
    else launch_tree_accept_t<float>(a, stream);
}

void launch_kv_compact_tree(int dtype, void *k, void *v, int32_t *lens, const int32_t *base, const int32_t *path,
                            const int32_t *path_len, int path_stride, int n_nodes, int L, int B, int h_kv, int d_h,
                            int max_len, int cap, hipStream_t stream) {
    ScopedProf sp(PSD_KIND_LENS, stream);
    const unsigned grid = (unsigned)((size_t)L * B * h_kv);
    if (dtype == PSD_BF16)
        launch_kernel(kv_compact_tree_kernel<uint16_t>, grid, 128, 0, stream, (uint16_t *)k, (uint16_t *)v, lens, base, path,
                      path_len, path_stride, n_nodes, B, h_kv, d_h, max_len, cap);
    else
        launch_kernel(kv_compact_tree_kernel<float>, grid, 128, 0, stream, (float *)k, (float *)v, lens, base, path,
                      path_len, path_stride, n_nodes, B, h_kv, d_h, max_len, cap);
}

}  // namespace psd
