// Token-tree verification (Related Work, "Verification Mechanisms": token-tree-based verification; Sec. 4.6 names
// deeper and wider drafting as the next step).  The paper prints no rule; the one used is multi-round speculative
// sampling for sibling tokens drawn independently from the drafter's distribution at their parent, which leaves the
// verifier's distribution unchanged (Abstract; Sec. 3.1).
//
//   tree_stats / mass / draw_kernel  the walk from the root: at a node the children are tried in index order against the
//                            running residual of the verifier's distribution, the first accepted child is descended
//                            into, and where none is accepted one token is drawn from what is left; every pass over
//                            the vocabulary is spread over the chip (tree_accept_alone_kernel: by one block per sequence);
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
__device__ __forceinline__ float block_max_f(float v, float *s_w) {
    v = wave_max(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = s_w[0];
#pragma unroll
    for (int w = 1; w < kTreeWaves; ++w) t = fmaxf(t, s_w[w]);
    return t;
}

// The whole walk by one block, which needs no memory to share: calls whose statistics do not fit a scratch slot (below),
// or that find theirs taken.
template <typename T>
__device__ void walk_alone(const TreeAcceptArgs &a, int row) {
    __shared__ double s_wd[kTreeWaves];
    __shared__ float s_wf[kTreeWaves];
    __shared__ int s_par[kTreeMaxAcceptNodes];
    __shared__ int s_pick, s_lastpos;
    __shared__ unsigned long long s_best;
    __shared__ double s_exp2[64];                           // kExp2Table, for exp_nonpos
    const int tid = threadIdx.x, n = a.n_nodes, V = a.vocab;
    for (int j = tid; j < n; j += kTreeThreads) s_par[j] = a.parents[j];
    if (tid < 64) s_exp2[tid] = kExp2Table[tid];
    __syncthreads();
    const T *P = (const T *)a.p + (size_t)row * a.p_stride;
    const T *Q = (const T *)a.q + (size_t)row * a.q_stride;
    const int32_t *tok = a.tokens + (size_t)row * n;
    const float *u = a.uniforms ? a.uniforms + (size_t)row * (n + 1) : nullptr;
    const bool greedy = a.temperature == 0.f;
    const double Tm = (double)a.temperature, inv_t = 1.0 / Tm;
    // exp(logit / T - max / T): the scaled logit minus the row's scaled maximum is never positive
    auto ex = [&](float logit, double m) { return exp_nonpos(fma((double)logit, inv_t, -m), s_exp2); };
    int32_t *path = a.out_path + (size_t)row * n;
    int node = 0, plen = 0, flags = 0;

    while (true) {                                          // every descent moves to a larger node index: at most n rounds
        const T *lp = P + (size_t)node * V;
        const T *lq = Q + (size_t)node * V;
        if (greedy) {
            // the verifier's most likely token, lowest index among equals
            unsigned long long best = 0ull;                 // (order-preserving bits of the logit) << 32 | ~index
            for (int i = tid; i < V; i += kTreeThreads) {
                const float x = load_elem(lp, (size_t)i);
                uint32_t b = __float_as_uint(x);
                b = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
                const unsigned long long key = ((unsigned long long)b << 32) | (uint32_t)(~(uint32_t)i);
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
            __syncthreads();                                // s_best is reset by the next round
            if (next < 0) {
                if (tid == 0) { a.out_path_len[row] = plen; a.out_token[row] = top; if (a.out_flags) a.out_flags[row] = 0; }
                return;
            }
            if (tid == 0) path[plen] = next;
            ++plen;
            node = next;
            continue;
        }

        // ---- softmax statistics of the two rows at this node: s_i = logit_i / T, max, sum of exp(s_i - max)
        float mpf = -INFINITY, mqf = -INFINITY;
        for (int i = tid; i < V; i += kTreeThreads) {
            mpf = fmaxf(mpf, load_elem(lp, (size_t)i));
            mqf = fmaxf(mqf, load_elem(lq, (size_t)i));
        }
        const double mp = (double)block_max_f(mpf, s_wf) * inv_t, mq = (double)block_max_f(mqf, s_wf) * inv_t;
        double zp = 0.0, zq = 0.0;
        for (int i = tid; i < V; i += kTreeThreads) {
            zp += ex(load_elem(lp, (size_t)i), mp);
            zq += ex(load_elem(lq, (size_t)i), mq);
        }
        const double Zp = block_sum_d(zp, s_wd), Zq = block_sum_d(zq, s_wd);
        const double inv_zp = 1.0 / Zp, inv_zq = 1.0 / Zq;       // one division per row, not one per entry
        double c = 0.0, mass = 1.0;                         // the residual here is max(0, p - c q) / mass

        int next = -1;
        for (int ch = node + 1; ch < n; ++ch) {
            if (s_par[ch] != node) continue;
            int x = tok[ch];
            x = min(max(x, 0), V - 1);
            const double px = ex(load_elem(lp, (size_t)x), mp) * inv_zp;
            const double qx = ex(load_elem(lq, (size_t)x), mq) * inv_zq;
            const double rx = fmax(px - c * qx, 0.0);
            const double ratio = qx == 0.0 ? INFINITY : rx / (mass * qx);
            const double thr = fmin(1.0, ratio), uu = (double)u[ch];
            if (fabs(uu - thr) < 1e-5) flags |= PSD_FLAG_NEAR_TIE;
            if (uu < thr) { next = ch; break; }
            // refused: take the drafter's share out of what is left
            const double c2 = c + mass;
            double m2 = 0.0;
            for (int i = tid; i < V; i += kTreeThreads) {
                const double pi = ex(load_elem(lp, (size_t)i), mp) * inv_zp;
                const double qi = ex(load_elem(lq, (size_t)i), mq) * inv_zq;
                m2 += fmax(pi - c2 * qi, 0.0);
            }
            m2 = block_sum_d(m2, s_wd);
            if (m2 > 0.0) { c = c2; mass = m2; }            // mass 0: the residual equalled q, where no refusal can happen
        }
        if (next >= 0) {
            if (tid == 0) path[plen] = next;
            ++plen;
            node = next;
            continue;
        }

        // ---- no child accepted: one draw from max(0, p - c q) by inverse CDF in index order.  Thread t owns the
        // contiguous entries [t * per, (t + 1) * per); prefix sums over threads in a fixed order.
        const int per = (V + kTreeThreads - 1) / kTreeThreads;
        const int i0 = min(tid * per, V), i1 = min(i0 + per, V);
        double w = 0.0;
        int lastpos = -1;
        for (int i = i0; i < i1; ++i) {
            const double pi = ex(load_elem(lp, (size_t)i), mp) * inv_zp;
            const double qi = ex(load_elem(lq, (size_t)i), mq) * inv_zq;
            const double r = fmax(pi - c * qi, 0.0);
            if (r > 0.0) lastpos = i;
            w += r;
        }
        // inclusive prefix inside the wavefront, then the wavefronts before it
        double incl = w;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double up = __shfl_up(incl, o, 64);
            if ((tid & 63) >= o) incl += up;
        }
        __syncthreads();
        if ((tid & 63) == 63) s_wd[tid >> 6] = incl;
        if (tid == 0) { s_pick = kTreeThreads; s_lastpos = -1; }
        __syncthreads();
        double before = 0.0, total = 0.0;
#pragma unroll
        for (int wv = 0; wv < kTreeWaves; ++wv) {
            if (wv < (tid >> 6)) before += s_wd[wv];
            total += s_wd[wv];
        }
        const double target = (double)u[n] * total;
        if (w > 0.0 && before + incl > target) atomicMin(&s_pick, tid);
        if (lastpos >= 0) atomicMax(&s_lastpos, lastpos);
        __syncthreads();
        if (tid == s_pick) {
            double cum = before + incl - w;
            int token = lastpos;                            // rounding left no crossing inside: the last positive entry
            for (int i = i0; i < i1; ++i) {
                const double pi = ex(load_elem(lp, (size_t)i), mp) * inv_zp;
                const double qi = ex(load_elem(lq, (size_t)i), mq) * inv_zq;
                cum += fmax(pi - c * qi, 0.0);
                if (cum > target) { token = i; break; }
            }
            a.out_token[row] = token;
        }
        if (tid == 0) {
            if (s_pick == kTreeThreads) a.out_token[row] = s_lastpos;      // no crossing at all: last positive entry
            a.out_path_len[row] = plen;
            if (a.out_flags) a.out_flags[row] = flags;
        }
        return;
    }
}

template <typename T>
__global__ __launch_bounds__(kTreeThreads) void tree_accept_alone_kernel(TreeAcceptArgs a) { walk_alone<T>(a, blockIdx.x); }

// ---- the same walk spread over the chip.  What a node's decisions need is taken for all nodes at once, chunk by chunk:
// tree_stats_kernel (softmax statistics, or the argmax when greedy) and, for nodes with more than j children,
// tree_mass_kernel j (the residual mass M_j after j refusals, j = 1 .. kMassPasses); then every block of
// tree_draw_kernel walks the tree on those numbers, sums the weights of its chunk of the row the draw reads, and the
// block of a sequence that arrives last finds the token.  Bound by fp64 arithmetic (2 exponentials per entry and pass):
// one block needs about 15 us per pass of 32 000 entries and makes ten of them.  Four sequences x 15 nodes x 32 000
// entries (fp32 logits): 128 us with a block per sequence, 44 us this way
// (2 + 9 + 10 + 24 for claim, statistics, one mass pass and the draw).
//
// The statistics travel through a slot of a static array, so that the call needs no workspace.  Calls on different
// streams may overlap: a call has a number of its own (the host counts them) and tree_claim_kernel takes the slot that
// number selects, by compare-and-swap, if it is free.  A call that did not get it falls back to walk_alone, decided on the
// device by the same test in every later block.  Nothing waits.  The last block of the last kernel frees the slot.
// (Claimed by the 480 blocks of the statistics kernel themselves, the same-address atomics took 13 us.)  Calls under graph capture, vocabularies above 262 144 entries and calls whose
// statistics exceed a slot (64 sequences x 8 nodes x 32 000 entries need 205 KB) run walk_alone from the start.
constexpr int kTreeChunk = 4096;                  // entries of one chunk
constexpr int kTreeMaxChunks = 64;                // per row: one per lane
constexpr int kMassPasses = 3;                    // further refusals at one node are summed by walk-time passes
constexpr int kTreeSlots = 4;
constexpr size_t kTreeSlotBytes = 512 << 10;
struct TreeSlotHead { uint32_t owner, done, pad[62]; };
struct TreeStat { double zp, zq; float mp, mq; };                  // sums of exp((l - chunk max) / T), chunk maxima
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

constexpr int kStatThreads = 256, kPerThread = kTreeChunk / kStatThreads;

template <typename T>
__global__ __launch_bounds__(kStatThreads) void tree_stats_kernel(TreeAcceptArgs a, TreeShare sh) {
    __shared__ double s_exp2[64];
    __shared__ double s_z[2][kStatThreads / 64];
    __shared__ float s_m[2][kStatThreads / 64];
    __shared__ unsigned long long s_k[kStatThreads / 64];
    const int tid = threadIdx.x, wave = tid >> 6, V = a.vocab;
    const SlotView sv = slot_of(a, sh);
    if (!slot_is_mine(sv, sh)) return;
    if (tid < 64) s_exp2[tid] = kExp2Table[tid];
    const int c = blockIdx.x % sh.n_chunks, rn = blockIdx.x / sh.n_chunks, node = rn % a.n_nodes, row = rn / a.n_nodes;
    const bool greedy = a.temperature == 0.f;
    const T *lp = (const T *)a.p + (size_t)row * a.p_stride + (size_t)node * V;
    const T *lq = (const T *)a.q + (size_t)row * a.q_stride + (size_t)node * V;
    const int e0 = c * kTreeChunk + tid;
    float p[kPerThread], q[kPerThread];
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
        const int e = e0 + i * kStatThreads;
        p[i] = e < V ? load_elem(lp, (size_t)e) : -INFINITY;
        q[i] = e < V && !greedy ? load_elem(lq, (size_t)e) : -INFINITY;
    }
    __syncthreads();
    if (greedy) {
        unsigned long long best = 0ull;                        // (order-preserving bits of the logit) << 32 | ~index
#pragma unroll
        for (int i = 0; i < kPerThread; ++i) {
            const int e = e0 + i * kStatThreads;
            uint32_t b = __float_as_uint(p[i]);
            b = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
            const unsigned long long key = ((unsigned long long)b << 32) | (uint32_t)(~(uint32_t)e);
            if (e < V && key > best) best = key;
        }
        best = wave_max(best);
        if ((tid & 63) == 0) s_k[wave] = best;
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < kStatThreads / 64; ++w) best = s_k[w] > best ? s_k[w] : best;
            *reinterpret_cast<unsigned long long *>(&sv.stat[(size_t)rn * sh.n_chunks + c]) = best;
        }
        return;
    }
    float mp = -INFINITY, mq = -INFINITY;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) { mp = fmaxf(mp, p[i]); mq = fmaxf(mq, q[i]); }
    mp = wave_max(mp);
    mq = wave_max(mq);
    if ((tid & 63) == 0) { s_m[0][wave] = mp; s_m[1][wave] = mq; }
    __syncthreads();
    mp = fmaxf(fmaxf(s_m[0][0], s_m[0][1]), fmaxf(s_m[0][2], s_m[0][3]));
    mq = fmaxf(fmaxf(s_m[1][0], s_m[1][1]), fmaxf(s_m[1][2], s_m[1][3]));
    const double inv_t = 1.0 / (double)a.temperature, dp = (double)mp * inv_t, dq = (double)mq * inv_t;
    double zp = 0.0, zq = 0.0;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
        zp += exp_nonpos(fma((double)p[i], inv_t, -dp), s_exp2);
        zq += exp_nonpos(fma((double)q[i], inv_t, -dq), s_exp2);
    }
    zp = wave_sum(zp);
    zq = wave_sum(zq);
    if ((tid & 63) == 0) { s_z[0][wave] = zp; s_z[1][wave] = zq; }
    __syncthreads();
    if (tid == 0)
        sv.stat[(size_t)rn * sh.n_chunks + c] = TreeStat{((s_z[0][0] + s_z[0][1]) + s_z[0][2]) + s_z[0][3],
                                                         ((s_z[1][0] + s_z[1][1]) + s_z[1][2]) + s_z[1][3], mp, mq};
}

struct NodeStat { double mp, mq, inv_zp, inv_zq; };                // scaled maxima, reciprocals of the denominators
// one wavefront, lane = chunk
__device__ __forceinline__ NodeStat node_stat(const TreeStat *st, int chunks, double inv_t, const double *exp2tab) {
    const int lane = threadIdx.x & 63;
    const TreeStat t = st[min(lane, chunks - 1)];
    const float mp = wave_max(t.mp), mq = wave_max(t.mq);
    NodeStat s;
    s.mp = (double)mp * inv_t;
    s.mq = (double)mq * inv_t;
    // a chunk of -infinities contributes nothing
    const bool in = lane < chunks;
    const double zp = in && t.mp > -INFINITY ? t.zp * exp_nonpos(fma((double)t.mp, inv_t, -s.mp), exp2tab) : 0.0;
    const double zq = in && t.mq > -INFINITY ? t.zq * exp_nonpos(fma((double)t.mq, inv_t, -s.mq), exp2tab) : 0.0;
    s.inv_zp = 1.0 / wave_sum(zp);
    s.inv_zq = 1.0 / wave_sum(zq);
    return s;
}
// (c, mass) of the residual max(0, p - c q) / mass, taken one refusal further: mass 0 means that the residual equalled q,
// where no refusal can happen
__device__ __forceinline__ void refuse(double m, double *c, double *mass) {
    if (m > 0.0) { *c += *mass; *mass = m; }
}

// M_{j+1} = sum max(0, p - c q) of one chunk of one node, c after j refusals and the next
template <typename T>
__global__ __launch_bounds__(kStatThreads) void tree_mass_kernel(TreeAcceptArgs a, TreeShare sh, int j) {
    __shared__ double s_exp2[64];
    __shared__ double s_w[kStatThreads / 64];
    const int tid = threadIdx.x, wave = tid >> 6, V = a.vocab;
    const SlotView sv = slot_of(a, sh);
    if (!slot_is_mine(sv, sh)) return;
    if (tid < 64) s_exp2[tid] = kExp2Table[tid];
    const int ch = sh.n_chunks, c = blockIdx.x % ch, rn = blockIdx.x / ch, row = rn / sh.n_inner[j];
    const int node = sh.inner[j][rn % sh.n_inner[j]];
    const T *lp = (const T *)a.p + (size_t)row * a.p_stride + (size_t)node * V;
    const T *lq = (const T *)a.q + (size_t)row * a.q_stride + (size_t)node * V;
    const int e0 = c * kTreeChunk + tid;
    float p[kPerThread], q[kPerThread];
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
        const int e = e0 + i * kStatThreads;
        p[i] = e < V ? load_elem(lp, (size_t)e) : -INFINITY;
        q[i] = e < V ? load_elem(lq, (size_t)e) : -INFINITY;
    }
    __syncthreads();
    const double inv_t = 1.0 / (double)a.temperature;
    const size_t at = ((size_t)row * a.n_nodes + node) * ch, pass = (size_t)a.rows * a.n_nodes * ch;
    const NodeStat s = node_stat(sv.stat + at, ch, inv_t, s_exp2);
    double cc = 0.0, mass = 1.0;
    for (int t = 0; t < j; ++t) {
        const int lane = tid & 63;
        refuse(wave_sum(lane < ch ? sv.mass[t * pass + at + lane] : 0.0), &cc, &mass);
    }
    cc += mass;
    double m = 0.0;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
        const double pi = exp_nonpos(fma((double)p[i], inv_t, -s.mp), s_exp2) * s.inv_zp;
        const double qi = exp_nonpos(fma((double)q[i], inv_t, -s.mq), s_exp2) * s.inv_zq;
        m += fmax(pi - cc * qi, 0.0);
    }
    m = wave_sum(m);
    if ((tid & 63) == 0) s_w[wave] = m;
    __syncthreads();
    if (tid == 0) sv.mass[j * pass + at + c] = ((s_w[0] + s_w[1]) + s_w[2]) + s_w[3];
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

// Grid: rows x chunks (greedy: rows).  kTreeThreads threads, each on kTreeChunk / kTreeThreads consecutive entries.
template <typename T>
__device__ void shared_walk(const TreeAcceptArgs &a, const TreeShare &sh, const SlotView &sv, int row, int chunk, int chunks) {
    constexpr int E = kTreeChunk / kTreeThreads;
    __shared__ double s_wd[kTreeWaves], s_exp2[64];
    __shared__ NodeStat s_node[kTreeMaxAcceptNodes];
    __shared__ double s_mass[kMassPasses][kTreeMaxAcceptNodes], s_px[kTreeMaxAcceptNodes], s_qx[kTreeMaxAcceptNodes];
    __shared__ float s_u[kTreeMaxAcceptNodes + 1];
    __shared__ int s_par[kTreeMaxAcceptNodes], s_tok[kTreeMaxAcceptNodes], s_top[kTreeMaxAcceptNodes], s_kids[kTreeMaxAcceptNodes];
    __shared__ int s_pick, s_lastpos, s_chunk, s_last;
    __shared__ double s_c, s_base;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = a.n_nodes, V = a.vocab;
    const T *P = (const T *)a.p + (size_t)row * a.p_stride;
    const T *Q = (const T *)a.q + (size_t)row * a.q_stride;
    const bool greedy = a.temperature == 0.f;
    const double inv_t = 1.0 / (double)a.temperature;
    int32_t *path = a.out_path + (size_t)row * n;
    if (tid < 64) s_exp2[tid] = kExp2Table[tid];
    if (tid < n) {
        s_par[tid] = a.parents[tid];
        s_tok[tid] = a.tokens[(size_t)row * n + tid];
        s_kids[tid] = 0;
    }
    if (!greedy && tid <= n) s_u[tid] = a.uniforms[(size_t)row * (n + 1) + tid];
    __syncthreads();
    if (tid > 0 && tid < n) atomicAdd(&s_kids[s_par[tid]], 1);
    const size_t row_at = (size_t)row * n * chunks;
    if (greedy) {
        for (int v = wave; v < n; v += kTreeWaves) {
            const unsigned long long k = *reinterpret_cast<const unsigned long long *>(&sv.stat[row_at + (size_t)v * chunks + min(lane, chunks - 1)]);
            const unsigned long long best = wave_max(k);
            if (lane == 0) s_top[v] = (int)(~(uint32_t)(best & 0xffffffffull));
        }
        __syncthreads();
        if (tid == 0) {
            int node = 0, plen = 0;
            for (int c = 1; c < n; ++c)                       // a node's children follow it, so one sweep walks the path
                if (s_par[c] == node && s_tok[c] == s_top[node]) { path[plen++] = c; node = c; }
            a.out_path_len[row] = plen;
            a.out_token[row] = s_top[node];
            if (a.out_flags) a.out_flags[row] = 0;
        }
        return;
    }
    // every node's statistics and masses, then every child's probabilities at its parent, all at once
    __syncthreads();
    for (int v = wave; v < n; v += kTreeWaves) {
        const NodeStat s = node_stat(sv.stat + row_at + (size_t)v * chunks, chunks, inv_t, s_exp2);
        double m[kMassPasses];
#pragma unroll
        for (int j = 0; j < kMassPasses; ++j) {
            const bool there = s_kids[v] > j + 1 && lane < chunks;
            m[j] = wave_sum(there ? sv.mass[((size_t)j * a.rows * n + (size_t)row * n + v) * chunks + lane] : 0.0);
        }
        if (lane == 0) {
            s_node[v] = s;
#pragma unroll
            for (int j = 0; j < kMassPasses; ++j) s_mass[j][v] = m[j];
        }
    }
    __syncthreads();
    if (tid > 0 && tid < n) {
        const NodeStat s = s_node[s_par[tid]];
        const int x = min(max(s_tok[tid], 0), V - 1);
        const size_t at = (size_t)s_par[tid] * V + x;
        s_px[tid] = exp_nonpos(fma((double)load_elem(P, at), inv_t, -s.mp), s_exp2) * s.inv_zp;
        s_qx[tid] = exp_nonpos(fma((double)load_elem(Q, at), inv_t, -s.mq), s_exp2) * s.inv_zq;
    }
    __syncthreads();
    // the walk (every thread alike): at a node the children are tried in index order
    auto entry = [&](const NodeStat &s, const T *lp, const T *lq, int e, double c) {
        const double pi = exp_nonpos(fma((double)load_elem(lp, (size_t)e), inv_t, -s.mp), s_exp2) * s.inv_zp;
        const double qi = exp_nonpos(fma((double)load_elem(lq, (size_t)e), inv_t, -s.mq), s_exp2) * s.inv_zq;
        return fmax(pi - c * qi, 0.0);
    };
    auto mass_of_row = [&](int node, double c) {                // a pass by this block: past the precomputed refusals
        double m = 0.0;
        for (int e = tid; e < V; e += kTreeThreads) m += entry(s_node[node], P + (size_t)node * V, Q + (size_t)node * V, e, c);
        return block_sum_d(m, s_wd);
    };
    const bool writer = chunk == 0 && tid == 0;
    int node = 0, plen = 0, flags = 0;
    double c = 0.0, mass = 1.0, c_before = 0.0;
    while (true) {
        int next = -1, tried = 0;
        c = 0.0; mass = 1.0; c_before = 0.0;
        for (int k = node + 1; k < n; ++k) {
            if (s_par[k] != node) continue;
            ++tried;
            const double rx = fmax(s_px[k] - c * s_qx[k], 0.0);
            const double ratio = s_qx[k] == 0.0 ? INFINITY : rx / (mass * s_qx[k]);
            const double thr = fmin(1.0, ratio), uu = (double)s_u[k];
            if (fabs(uu - thr) < 1e-5) flags |= PSD_FLAG_NEAR_TIE;
            if (uu < thr) { next = k; break; }
            c_before = c;
            if (tried == s_kids[node]) c += mass;             // the draw's own sums say whether anything is left
            else refuse(tried <= kMassPasses ? s_mass[tried - 1][node] : mass_of_row(node, c + mass), &c, &mass);
        }
        if (next < 0) break;
        if (writer) path[plen] = next;
        ++plen;
        node = next;
    }
    // one draw from max(0, p - c q): this block's chunk
    const NodeStat s = s_node[node];
    const T *lp = P + (size_t)node * V, *lq = Q + (size_t)node * V;
    const int i0 = min(chunk * kTreeChunk + tid * E, V), i1 = min(i0 + E, V);
    double w = 0.0;
#pragma unroll
    for (int k = 0; k < E; ++k)
        if (i0 + k < i1) w += entry(s, lp, lq, i0 + k, c);
    w = block_sum_d(w, s_wd);
    if (tid == 0) {
        __hip_atomic_store(sv.part + (size_t)row * chunks + chunk, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        s_last = __hip_atomic_fetch_add(sv.count + row, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)chunks - 1u;
    }
    __syncthreads();
    if (!s_last) return;
    if (wave == 0) {
        const double mine = lane < chunks ? __hip_atomic_load(sv.part + (size_t)row * chunks + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0;
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
            s_c = target;
        }
    }
    if (tid == 0) { s_pick = kTreeThreads; s_lastpos = -1; }
    __syncthreads();
    int first = s_chunk * kTreeChunk, last = min(first + kTreeChunk, V);
    double base = s_base, target = s_c;
    if (s_chunk < 0 && c != c_before) {
        // the last refusal left a mass of exactly 0 (the residual equalled q): the draw is from what was there before it
        c = c_before;
        target = (double)s_u[n] * mass_of_row(node, c);
    }
    if (s_chunk < 0) { first = 0; last = V; base = 0.0; }       // all of the row, a chunk at a time
    __syncthreads();
    for (int t0 = first; t0 < last; t0 += kTreeChunk) {
        const int j0 = min(t0 + tid * E, last), j1 = min(j0 + E, last);
        double wv[E], mine = 0.0;
        int lastpos = -1;
#pragma unroll
        for (int k = 0; k < E; ++k) {
            wv[k] = j0 + k < j1 ? entry(s, lp, lq, j0 + k, c) : 0.0;
            if (wv[k] > 0.0) lastpos = j0 + k;
            mine += wv[k];
        }
        double incl = mine;
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
        if (mine > 0.0 && before + incl > target) atomicMin(&s_pick, tid);
        if (lastpos >= 0) atomicMax(&s_lastpos, lastpos);
        __syncthreads();
        if (s_pick < kTreeThreads) {
            if (tid == s_pick) {
                double cum = before + incl - mine;
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
__global__ __launch_bounds__(kTreeThreads) void tree_draw_kernel(TreeAcceptArgs a, TreeShare sh) {
    const SlotView sv = slot_of(a, sh);
    const bool mine = slot_is_mine(sv, sh);                 // only this call's blocks can end that, after all have counted
    const int chunks = sh.n_chunks, per_row = a.temperature == 0.f ? 1 : chunks;
    const int chunk = blockIdx.x % per_row, row = blockIdx.x / per_row;
    if (mine) shared_walk<T>(a, sh, sv, row, chunk, chunks);
    else if (chunk == 0) walk_alone<T>(a, row);
    if (mine) slot_leave(sv, gridDim.x);
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

template <typename T>
static void launch_tree_accept_t(const TreeAcceptArgs &a, hipStream_t stream) {
    TreeShare sh{};
    sh.n_chunks = (a.vocab + kTreeChunk - 1) / kTreeChunk;
    size_t st, ms, pt;
    // a captured call would keep its number in every copy of its graph, and two copies may run at once
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    const bool captured = hipStreamIsCapturing(stream, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    if (captured || sh.n_chunks > kTreeMaxChunks || slot_layout(a.rows, a.n_nodes, sh.n_chunks, &st, &ms, &pt) > kTreeSlotBytes) {
        launch_kernel(tree_accept_alone_kernel<T>, a.rows, kTreeThreads, 0, stream, a);
        return;
    }
    sh.id = tree_call_number();
    const bool greedy = a.temperature == 0.f;
    launch_kernel(tree_claim_kernel, 1, 64, 0, stream, a, sh);
    launch_kernel(tree_stats_kernel<T>, (unsigned)(a.rows * a.n_nodes * sh.n_chunks), kStatThreads, 0, stream, a, sh);
    int kids[kTreeMaxAcceptNodes] = {};
    for (int i = 1; i < a.n_nodes; ++i) ++kids[a.parents[i]];
    for (int j = 0; j < kMassPasses && !greedy; ++j)
        for (int i = 0; i < a.n_nodes; ++i)
            if (kids[i] > j + 1) sh.inner[j][sh.n_inner[j]++] = (uint8_t)i;
    for (int j = 0; j < kMassPasses && sh.n_inner[j] > 0; ++j)
        launch_kernel(tree_mass_kernel<T>, (unsigned)(a.rows * sh.n_inner[j] * sh.n_chunks), kStatThreads, 0, stream, a, sh, j);
    launch_kernel(tree_draw_kernel<T>, (unsigned)(a.rows * (greedy ? 1 : sh.n_chunks)), kTreeThreads, 0, stream, a, sh);
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
