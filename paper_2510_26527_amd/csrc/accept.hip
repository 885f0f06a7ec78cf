// Speculative-sampling acceptance on gfx950 (the VERIFY loop of Algorithm 1 and the residual
// draw that keeps the verifier's distribution, Sec. 3.1).
//
// Two launches per call, no host round trip:
//   1. accept_stats_kernel  one pass over every logits row of p and q (the HBM-bound part):
//      per (row, chunk) the max raw logit and sum exp((l - max)/T), fp32, wavefront
//      reductions, 8 x 16-byte loads in flight per lane.  The block whose chunk holds the
//      draft token of its position also hands on that one logit, so the ratio test later
//      needs no dependent load.
//   2. accept_draw_kernel   bound by a chain of dependent steps (its fp64 instructions, two exponentials per entry of the
//      one position, fill about a fifth of its time): reductions and scans run on lane moves in registers, and the finishing
//      block's chunk sums in one wavefront without a barrier.  Several blocks per sequence.  Each re-derives the first
//      rejection n of its sequence from the statistics (ratio test against the supplied uniforms, scan over <= 64
//      flags) and accumulates, in fp64 and for the ONE position the draw needs, the
//      softmax denominators and the residual mass of its chunk.  The block of a sequence that
//      finishes last (one counter per sequence; partial sums travel as agent-scope atomic
//      stores / loads, so no cache write-back fence is needed and nothing ever waits) sums the
//      chunks in index order and locates the inverse-CDF crossing, first among the chunks,
//      then among the entries of that chunk.
// All sums are taken in a fixed order, so results do not depend on block scheduling.
#include "common.h"
#include "kernels.h"
#include "exp64.h"
#include "prof.h"
#include "../../include/psd.h"

namespace psd {

namespace {

constexpr int kThreads = 256;
constexpr int kLoadsPerLane = 8;
constexpr double kTieEps = 1e-5;
constexpr int kMaxChunksE = 128;      // draw-pass chunks per logits row: two per lane of the wavefront that finishes a sequence
constexpr int kMaxQuarters = 64;      // ... or quarters of chunks, one per lane
constexpr int kMaxGroup = 8;          // consecutive entries a thread of the draw kernel takes at a time (2 or 8)

template <typename T>
__device__ __forceinline__ const T *logits_row(const AcceptArgs &a, int b, bool is_q, int j) {
    const T *base = is_q ? (const T *)a.q + (int64_t)b * a.q_stride : (const T *)a.p + (int64_t)b * a.p_stride;
    return base + (int64_t)j * a.V;
}

template <typename T, bool VEC>
__global__ __launch_bounds__(kThreads) void accept_stats_kernel(AcceptArgs a) {
    constexpr int EPL = VEC ? (int)(16 / sizeof(T)) : 1;
    const int tid = threadIdx.x;
    const int per_seq = a.n_p_rows + a.gamma;
    const int vec = blockIdx.x / a.n_chunksA, c = blockIdx.x % a.n_chunksA;
    const int b = vec / per_seq, r = vec % per_seq;
    const bool is_q = r >= a.n_p_rows;
    const int j = is_q ? r - a.n_p_rows : r;           // position of this row inside the block of draft tokens
    const T *row = logits_row<T>(a, b, is_q, j);
    const int e0 = c * a.chunkA;
    const int e1 = min(a.V, e0 + a.chunkA);
    // the draft token of this position (none for the bonus row): its logit passes through this block's
    // registers if it lies in [e0, e1)
    int xj = -1;
    if (j < a.gamma) xj = min(max(a.x[(size_t)b * a.gamma + j], 0), a.V - 1);
    // the per-sequence arrival counters of the draw kernel start every call at zero
    if (blockIdx.x == 0)
        for (int i = tid; i < a.rows; i += kThreads) a.counter[i] = 0u;

    // keep the loaded 16-byte vectors as they are (32 registers) and unpack them twice, once for
    // the max and once for the exponentials: the small footprint keeps 8 blocks resident per CU
    u32x4 raw[kLoadsPerLane];
    float sc[kLoadsPerLane];               // scalar path
    bool have[kLoadsPerLane];
#pragma unroll
    for (int i = 0; i < kLoadsPerLane; ++i) {
        const int idx = e0 + (i * kThreads + tid) * EPL;
        have[i] = idx < e1;                // chunk bounds and V are multiples of EPL: a vector load is whole
        if constexpr (VEC) {
            raw[i] = have[i] ? __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(row + idx)) : u32x4{0u, 0u, 0u, 0u};
        } else {
            sc[i] = have[i] ? load_elem(row, idx) : -INFINITY;
        }
    }
    auto elem = [&](int i, int e) -> float {
        if constexpr (!VEC) return sc[i];
        else if constexpr (sizeof(T) == 2)
            return (e & 1) ? __uint_as_float(raw[i][e >> 1] & 0xffff0000u) : __uint_as_float(raw[i][e >> 1] << 16);
        else return __uint_as_float(raw[i][e]);
    };
    if (xj >= e0 && xj < e1) {
        // vector v = i * kThreads + tid of the chunk holds the token's logit as its element e
        const int rel = xj - e0, v = rel / EPL, e = rel % EPL;
        if (tid == v % kThreads) {
            const int iv = v / kThreads;
            float val = 0.f;
#pragma unroll
            for (int i = 0; i < kLoadsPerLane; ++i)
#pragma unroll
                for (int ee = 0; ee < EPL; ++ee)
                    if (i == iv && ee == e) val = elem(i, ee);
            a.xlogit[((size_t)b * a.gamma + j) * 2 + (is_q ? 1 : 0)] = val;
        }
    }
    float m = -INFINITY;
#pragma unroll
    for (int i = 0; i < kLoadsPerLane; ++i)
        if (have[i]) {
#pragma unroll
            for (int e = 0; e < EPL; ++e) m = fmaxf(m, elem(i, e));
        }
    __shared__ float sm[kThreads / 64];
    __shared__ float ss[kThreads / 64];
    m = wave_max(m);
    if ((tid & 63) == 0) sm[tid >> 6] = m;
    __syncthreads();
    m = fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
    float s = 0.f;
    if (m > -INFINITY) {
        const float k2 = 1.4426950408889634f / a.temperature;
#pragma unroll
        for (int i = 0; i < kLoadsPerLane; ++i)
            if (have[i]) {
#pragma unroll
                for (int e = 0; e < EPL; ++e) s += __builtin_amdgcn_exp2f((elem(i, e) - m) * k2);
            }
    }
    s = wave_sum(s);
    if ((tid & 63) == 0) ss[tid >> 6] = s;
    __syncthreads();
    if (tid == 0) a.stats[(size_t)vec * a.n_chunksA + c] = make_float2(m, ((ss[0] + ss[1]) + ss[2]) + ss[3]);
}

// fp32 statistics of every position of one sequence, kept in LDS by the block that decides it
struct SeqStats {
    float mp[65], mq[64];
    double zp[65], zq[64];
    double exp2tab[64];           // kExp2Table, for exp_core
    double inv_t;
    int n, flags;
};

// Ratio tests of sequence b and the scan to the first rejection.  Called by a whole block; every thread returns the same
// n and flags.  The per-chunk statistics of a logits row (max raw logit, sum exp((l - max)/T)) are combined by eight lanes
// per row, all rows at once: first the row's maximum, then every chunk's sum against it, so that a sum (an fp32 quantity)
// meets one fp32 exponential on its way; the sums add in fp64.  Then the first wavefront tests all positions, one per lane, and the first rejection is a bit scan.
__device__ __forceinline__ void decide(const AcceptArgs &a, int b, SeqStats *ss, int *n_out, int *flags_out) {
    const int tid = threadIdx.x, lane = tid & 63, sub = tid & 7;
    const double tabv = tid < 64 ? kExp2Table[tid] : 0.0;      // requested first, stored once the other loads are out
    double u = 0.0;
    float lpx = 0.f, lqx = 0.f;
    if (tid < a.gamma) {
        u = (double)a.u[(size_t)b * (a.gamma + 1) + lane];
        lpx = a.xlogit[((size_t)b * a.gamma + lane) * 2];
        lqx = a.xlogit[((size_t)b * a.gamma + lane) * 2 + 1];
    }
    const float k2 = 1.4426950408889634f / a.temperature;
    const int rows = a.n_p_rows + a.gamma, nA = a.n_chunksA;
    for (int r0 = 0; r0 < rows; r0 += kThreads / 8) {          // the same number of rounds for the whole block
        const int r = r0 + (tid >> 3);
        const float2 *st = a.stats + ((size_t)b * rows + min(r, rows - 1)) * nA;
        float2 t[4];                                           // up to four chunks per lane in flight
        auto load = [&](int c0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) t[i] = st[min(c0 + sub + 8 * i, nA - 1)];
        };
        float top = -INFINITY;
        for (int c0 = 0; c0 < nA; c0 += 32) {
            load(c0);
#pragma unroll
            for (int i = 0; i < 4; ++i) top = fmaxf(top, t[i].x);      // past the end: the last chunk again
        }
        top = fmaxf(top, __shfl_xor(top, 1, 64));
        top = fmaxf(top, __shfl_xor(top, 2, 64));
        top = fmaxf(top, __shfl_xor(top, 4, 64));
        double z = 0.0;
        for (int c0 = 0; c0 < nA; c0 += 32) {
            if (nA > 32) load(c0);                             // else they are still there
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (c0 + sub + 8 * i < nA && t[i].x > -INFINITY) z += (double)(t[i].y * __builtin_amdgcn_exp2f((t[i].x - top) * k2));
        }
        z += __shfl_xor(z, 1, 64);
        z += __shfl_xor(z, 2, 64);
        z += __shfl_xor(z, 4, 64);
        if (sub == 0 && r < rows) {
            if (r < a.n_p_rows) { ss->mp[r] = top; ss->zp[r] = z; }
            else { ss->mq[r - a.n_p_rows] = top; ss->zq[r - a.n_p_rows] = z; }
        }
    }
    if (tid < 64) ss->exp2tab[tid] = tabv;
    __syncthreads();
    if (tid < 64) {
        bool acc = true, tie = false;
        if (lane < a.gamma) {
            const float Mp = ss->mp[lane], Mq = ss->mq[lane];
            double rho;
            if (lqx == -INFINITY) {
                rho = INFINITY;             // q[x] = 0: the token could not have been drafted; accept
            } else {
                rho = exp_any((((double)lpx - (double)Mp) - ((double)lqx - (double)Mq)) / (double)a.temperature, ss->exp2tab) *
                      (ss->zq[lane] / ss->zp[lane]);
            }
            acc = u < fmin(1.0, rho);
            tie = fabs(u - rho) < kTieEps;
        }
        const unsigned long long refused = __ballot(!acc), ties = __ballot(tie);       // lanes from gamma on: neither
        const int n = refused ? __ffsll(refused) - 1 : a.gamma;
        const unsigned long long tested = n >= 63 ? ~0ull : (2ull << n) - 1;           // positions up to the first rejection
        if (lane == 0) {
            ss->n = n;
            ss->flags = (ties & tested) ? PSD_FLAG_NEAR_TIE : 0;
            ss->inv_t = 1.0 / (double)a.temperature;
        }
    }
    __syncthreads();
    *n_out = ss->n;
    *flags_out = ss->flags;
}

// which position the draw reads: the rejected one (p and q) or the bonus row (p only)
struct DrawRows {
    int p_row;      // row index within p, -1: nothing to draw
    bool have_q;
};
__device__ __forceinline__ DrawRows draw_rows(const AcceptArgs &a, int n) {
    DrawRows d;
    if (n < a.gamma) { d.p_row = n; d.have_q = true; }
    else if (a.n_p_rows > a.gamma) { d.p_row = a.gamma; d.have_q = false; }
    else { d.p_row = -1; d.have_q = false; }
    return d;
}

// The draw position of one sequence.  With a_i = exp(lp_i/T - mp), b_i = exp(lq_i/T - mq) (fp64) and
// Zp = sum a, Zq = sum b, the residual weight of entry i is a_i/Zp - b_i/Zq where that is positive, i.e.
// where d_i = (lp_i/T - mp) - (lq_i/T - mq) exceeds log(Zp/Zq).  The chunk pass runs before the fp64
// Zp, Zq exist; it decides the sign against the fp32 estimate `delta` of log(Zp/Zq) from the statistics
// pass (t_i = d_i - delta > 0) and records, per chunk, the smallest positive and the largest non-positive
// t_i.  The block that finishes the sequence knows eps = log(Zp/Zq) - delta; a chunk with no t_i between
// 0 and eps was classified exactly as the fp64 residual would have been, any other chunk is summed again
// with the sign taken from a_i/Zp - b_i/Zq itself.  Nothing rests on how good the estimate is.
constexpr double kSignTol = 1e-11;      // rounding of t_i and of eps (|d_i| stays below ~1e3)

template <typename T>
struct DrawPos {
    const T *prow, *qrow;
    const double *tab;             // the block's copy of kExp2Table
    double inv_t, mp, mq, delta;
    bool have_q;
    __device__ __forceinline__ void init(const AcceptArgs &a, int b, int n, const DrawRows &d, const SeqStats &ss) {
        const float Mp = ss.mp[d.p_row], Mq = d.have_q ? ss.mq[n] : 0.f;
        const double Zp32 = ss.zp[d.p_row], Zq32 = d.have_q ? ss.zq[n] : 1.0;
        tab = ss.exp2tab;
        prow = logits_row<T>(a, b, false, d.p_row);
        qrow = logits_row<T>(a, b, true, d.have_q ? n : 0);
        inv_t = ss.inv_t;
        mp = (double)Mp * inv_t;
        mq = (double)Mq * inv_t;
        const float est = __logf((float)Zp32) - __logf((float)Zq32);
        delta = d.have_q && est == est ? (double)est : 0.0;       // any finite value will do
        have_q = d.have_q;
    }
    // raw logits of the G consecutive entries i0 .. i0 + G - 1 (those at or past i_end: entry i0 again,
    // q's are 0 when there is no q row).  VEC: rows are 16-byte aligned, i0 and V are multiples of the elements
    // per 16-byte load, so whole vectors are inside the row (fewer than a vector's entries are loaded one by one)
    template <bool VEC, int G>
    __device__ __forceinline__ void load_group(int i0, int i_end, float (&lp)[G], float (&lq)[G]) const {
        if constexpr (VEC && G % (int)(16 / sizeof(T)) == 0) {
            constexpr int EPL = (int)(16 / sizeof(T)), NV = G / EPL;
            u32x4 rp[NV], rq[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const int i = i0 + v * EPL < i_end ? i0 + v * EPL : i0;
                rp[v] = *reinterpret_cast<const u32x4 *>(prow + i);
                rq[v] = have_q ? *reinterpret_cast<const u32x4 *>(qrow + i) : u32x4{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int j = 0; j < G; ++j) {
                if constexpr (sizeof(T) == 2) {
                    const uint32_t wp = rp[j / EPL][(j % EPL) >> 1], wq = rq[j / EPL][(j % EPL) >> 1];
                    lp[j] = (j & 1) ? __uint_as_float(wp & 0xffff0000u) : __uint_as_float(wp << 16);
                    lq[j] = (j & 1) ? __uint_as_float(wq & 0xffff0000u) : __uint_as_float(wq << 16);
                } else {
                    lp[j] = __uint_as_float(rp[j / EPL][j % EPL]);
                    lq[j] = __uint_as_float(rq[j / EPL][j % EPL]);
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < G; ++j) {
                const int i = i0 + j < i_end ? i0 + j : i0;
                lp[j] = load_elem(prow, i);
                lq[j] = have_q ? load_elem(qrow, i) : 0.f;
            }
        }
    }
    // (a_i, b_i, t_i) from the raw logits; without a q row b_i = 0 and t_i = +inf (every entry counts)
    __device__ __forceinline__ void eval(float lp, float lq, double *ea, double *eb, double *t) const {
        const double xa = fma((double)lp, inv_t, -mp);
        const double xb = fma((double)lq, inv_t, -mq);
        *ea = exp_nonpos(xa, tab);
        const double e = exp_nonpos(xb, tab);
        *eb = have_q ? e : 0.0;
        *t = have_q ? (xa - xb) - delta : INFINITY;
    }
};

// per (sequence, piece): sum a, sum b, both over the entries with t_i > 0, the smallest positive t_i and the
// largest non-positive t_i
constexpr int kPartStride = 6;

// Grid: rows x n_chunksE blocks.  Every block: first rejection of its sequence, fp64 sums of the pieces of its chunk of
// the draw position; the block that arrives last at the sequence's counter finishes the draw (one or
// two pieces per lane of its first wavefront).  A piece is the chunk, or, where chunks are of
// 4096 entries and more and a row has at most 64 pieces, a wavefront's quarter of it (pieceE = chunkE / 4): the walk that finds the entry,
// two exponentials an entry again, then has a quarter of the chunk to go through.  Draw kernel, us, whole chunks / quarters: 64 x
// 32 000 entries 22.0 / 19.1 (bf16), 128 x 32 000 34.9 / 27.2, 64 x 32 001 28.8 / 22.8; more pieces cost more to gather than the
// walk saves: 16 x 152 064 (152 pieces) 30.6 / 34.6, 8 x 128 256 (252) 22.0 / 26.0, 16 x 32 000 (64 of 512) 16.9 / 17.5.
template <typename T, bool VEC, int G, bool QUARTERS>
__global__ __launch_bounds__(kThreads) void accept_draw_kernel(AcceptArgs a) {
    constexpr int kWaves = kThreads / 64;
    __shared__ SeqStats s_seq;
    __shared__ double s_red[6][kWaves], s_scan[2][kWaves];
    __shared__ int s_redo[kMaxChunksE];            // pieces whose sign classification has to be redone
    __shared__ double s_again[kMaxChunksE];        // ... and their weight then
    __shared__ int s_last, s_any, s_cstar, s_best, s_lastpos, s_fall;
    __shared__ double s_base, s_target, s_inv[2];
    const int nE = a.n_chunksE, nP = QUARTERS ? a.n_piecesE : nE, pieceE = QUARTERS ? a.pieceE : a.chunkE;
    const int b = blockIdx.x / nE, c = blockIdx.x % nE, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int n, flags;
    decide(a, b, &s_seq, &n, &flags);
    const DrawRows d = draw_rows(a, n);
    if (d.p_row < 0) {                            // every token accepted and no bonus row
        if (c == 0 && tid == 0) { a.out_n[b] = n; a.flags[b] = flags; a.out_tok[b] = -1; }
        return;
    }
    DrawPos<T> w;
    w.init(a, b, n, d, s_seq);
    const auto add = [](double x, double y) { return x + y; };
    const auto lower = [](double x, double y) { return fmin(x, y); };
    const auto upper = [](double x, double y) { return fmax(x, y); };

    // ---- this block's chunk
    {
        const int e0 = c * a.chunkE + (QUARTERS ? wave * pieceE : 0), e1 = min(a.V, e0 + pieceE);
        const int step = QUARTERS ? 64 * G : kThreads * G;
        double acc[4] = {0.0, 0.0, 0.0, 0.0};               // sum a, sum b, positive a, positive b
        double tpos = INFINITY, tneg = -INFINITY;
        for (int i0 = e0 + (QUARTERS ? lane : tid) * G; i0 < e1; i0 += step) {
            float lp[G], lq[G];
            w.template load_group<VEC>(i0, e1, lp, lq);
            double ea[G], eb[G], t[G];
#pragma unroll
            for (int j = 0; j < G; ++j) w.eval(lp[j], lq[j], &ea[j], &eb[j], &t[j]);
#pragma unroll
            for (int j = 0; j < G; ++j) {
                if (i0 + j < e1) {
                    acc[0] += ea[j];
                    acc[1] += eb[j];
                    if (t[j] > 0.0) { acc[2] += ea[j]; acc[3] += eb[j]; tpos = fmin(tpos, t[j]); }
                    if (t[j] <= 0.0) tneg = fmax(tneg, t[j]);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] = wave_scan_d(acc[k], 0.0, add);
        tpos = wave_scan_d(tpos, INFINITY, lower);
        tneg = wave_scan_d(tneg, -INFINITY, upper);
        // Hand the results on as write-through stores, wait for them to be performed, then count this block in; whoever counts
        // last reads all of them back with loads of the same scope.
        auto publish = [&](int piece) {
            double *dst = a.part + ((size_t)b * nP + piece) * kPartStride;
#pragma unroll
            for (int k = 0; k < 4; ++k) __hip_atomic_store(dst + k, acc[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(dst + 4, tpos, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(dst + 5, tneg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        };
        if constexpr (QUARTERS) {
            if (lane == 63) publish(c * kWaves + wave);
            __syncthreads();
        } else {
            // one value per wavefront into LDS, thread 0 folds the four in wavefront order
            if (lane == 63) {
#pragma unroll
                for (int k = 0; k < 4; ++k) s_red[k][wave] = acc[k];
                s_red[4][wave] = tpos;
                s_red[5][wave] = tneg;
            }
            __syncthreads();
            if (tid == 0) {
#pragma unroll
                for (int k = 0; k < 4; ++k) acc[k] = ((s_red[k][0] + s_red[k][1]) + s_red[k][2]) + s_red[k][3];
                tpos = fmin(fmin(s_red[4][0], s_red[4][1]), fmin(s_red[4][2], s_red[4][3]));
                tneg = fmax(fmax(s_red[5][0], s_red[5][1]), fmax(s_red[5][2], s_red[5][3]));
                publish(c);
            }
        }
        if (tid == 0) {
            const unsigned old = __hip_atomic_fetch_add(a.counter + b, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_last = old == (unsigned)nE - 1u;
        }
        __syncthreads();
        if (!s_last) return;
    }

    // ---- the last block of the sequence: its first wavefront takes all pieces' results, one or two per lane (one round of loads)
    const double u = (double)a.u[(size_t)b * (a.gamma + 1) + a.gamma];
    constexpr int kPiecesPerLane = QUARTERS ? 1 : 2;         // lane l has the pieces kPiecesPerLane l + h
    auto sum_of = [](auto term) { return QUARTERS ? term(0) : term(0) + term(kPiecesPerLane - 1); };
    double pk[kPiecesPerLane][kPartStride];
    if (wave == 0) {
#pragma unroll
        for (int h = 0; h < kPiecesPerLane; ++h) {
            const int k = kPiecesPerLane * lane + h;
            const double *src = a.part + ((size_t)b * nP + min(k, nP - 1)) * kPartStride;
#pragma unroll
            for (int e = 0; e < kPartStride; ++e) {
                const double v = __hip_atomic_load(src + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                pk[h][e] = k < nP ? v : (e < 4 ? 0.0 : (e == 4 ? (double)INFINITY : -(double)INFINITY));
            }
        }
        const double zp = wave_total_d(sum_of([&](int h) { return pk[h][0]; }));
        const double zq = wave_total_d(sum_of([&](int h) { return pk[h][1]; }));
        // pieces with a t_i between 0 and eps (or too close to tell): every entry's sign again, from the fp64 weights
        bool redo = false;
        if (d.have_q) {
            const double eps = log(zp / zq) - w.delta;
            const double lo = fmin(0.0, eps) - kSignTol, hi = fmax(0.0, eps) + kSignTol;
#pragma unroll
            for (int h = 0; h < kPiecesPerLane; ++h) {
                const int k = kPiecesPerLane * lane + h;
                const bool r = k < nP && (!(eps == eps) || pk[h][5] >= lo || pk[h][4] <= hi);
                if (k < nP) s_redo[k] = r ? 1 : 0;
                redo = redo || r;
            }
        }
        const bool any = __ballot(redo) != 0;
        if (lane == 0) {
            s_inv[0] = 1.0 / zp;
            s_inv[1] = d.have_q ? 1.0 / zq : 0.0;
            s_any = any ? 1 : 0;
            s_best = 0x7fffffff;
            s_lastpos = -1;
        }
    }
    __syncthreads();
    const double inv_zp = s_inv[0], inv_zq = s_inv[1];
    if (s_any) {                                                 // the same for the whole block
        for (int k = 0; k < nP; ++k) {
            if (!s_redo[k]) continue;
            const int f0 = k * pieceE, f1 = min(a.V, f0 + pieceE);
            double pa = 0.0, pb = 0.0;
            for (int i0 = f0 + tid * G; i0 < f1; i0 += G * kThreads) {
                float lp[G], lq[G];
                w.template load_group<VEC>(i0, f1, lp, lq);
#pragma unroll
                for (int j = 0; j < G; ++j) {
                    double ea, eb, t;
                    w.eval(lp[j], lq[j], &ea, &eb, &t);
                    if (i0 + j < f1 && ea * inv_zp - eb * inv_zq > 0.0) { pa += ea; pb += eb; }
                }
            }
            pa = wave_total_d(pa);
            pb = wave_total_d(pb);
            __syncthreads();                                     // s_red: earlier readers are done
            if (lane == 0) { s_red[0][wave] = pa; s_red[1][wave] = pb; }
            __syncthreads();
            if (tid == 0)
                s_again[k] = (((s_red[0][0] + s_red[0][1]) + s_red[0][2]) + s_red[0][3]) * inv_zp -
                             (((s_red[1][0] + s_red[1][1]) + s_red[1][2]) + s_red[1][3]) * inv_zq;
        }
        __syncthreads();
    }
    if (wave == 0) {
        double wk[kPiecesPerLane];
        auto sum = [&]() { return sum_of([&](int h) { return wk[h]; }); };
#pragma unroll
        for (int h = 0; h < kPiecesPerLane; ++h) {
            const int k = kPiecesPerLane * lane + h;
            wk[h] = pk[h][2] * inv_zp - pk[h][3] * inv_zq;
            if (s_any && k < nP && s_redo[k]) wk[h] = s_again[k];
        }
        double incl = wave_prefix_sum_d(sum()), mass = lane_value_d(incl, 63);
        const bool fall = d.have_q && !(mass > 0.0);             // residual mass 0: draw from p itself
        if (fall) {
#pragma unroll
            for (int h = 0; h < kPiecesPerLane; ++h) wk[h] = pk[h][0] * inv_zp;
            incl = wave_prefix_sum_d(sum());
            mass = 1.0;                                          // sum of a_i / Zp
        }
        // first piece whose inclusive prefix exceeds t
        const double t = u * mass;
        double base[kPiecesPerLane];
        base[0] = incl - sum();
#pragma unroll
        for (int h = 1; h < kPiecesPerLane; ++h) base[h] = base[h - 1] + wk[h - 1];
        int over = kPiecesPerLane, held = -1;                    // this lane's first piece beyond t, its last one with weight
#pragma unroll
        for (int h = kPiecesPerLane - 1; h >= 0; --h)
            if (kPiecesPerLane * lane + h < nP && base[h] + wk[h] > t) over = h;
#pragma unroll
        for (int h = 0; h < kPiecesPerLane; ++h)
            if (wk[h] > 0.0) held = h;
        const unsigned long long overs = __ballot(over < kPiecesPerLane), helds = __ballot(held >= 0);
        const bool crossing = overs != 0;
        // rounding left no crossing: last piece with weight, whose walk then only looks for its last entry with weight
        const int pick = crossing ? __ffsll(overs) - 1 : (helds ? 63 - __clzll(helds) : 0);
        if (lane == pick) {
            const int h = crossing ? over : (held > 0 ? held : 0);
            double at = base[0];
#pragma unroll
            for (int k = 1; k < kPiecesPerLane; ++k)
                if (h == k) at = base[k];
            s_cstar = kPiecesPerLane * lane + h;
            s_base = crossing ? at : -(double)INFINITY;
            s_target = t;
            s_fall = fall ? 1 : 0;
        }
    }
    __syncthreads();
    const int cs = s_cstar;
    const bool no_crossing = s_base == -INFINITY, fall_back_to_p = s_fall != 0;
    const double t = s_target;
    const int f0 = cs * pieceE, f1 = min(a.V, f0 + pieceE);
    // walk the piece in tiles of 256 x GW entries, GW consecutive entries per thread, carrying the prefix
    double before = no_crossing ? 0.0 : s_base;    // weight in front of the current tile
    int found = 0x7fffffff, lastpos = -1, turn = 0;
    constexpr int GW = QUARTERS ? 4 : G;                   // (a quarter of a chunk: more threads with fewer entries each)
    for (int t0 = f0; t0 < f1; t0 += kThreads * GW, turn ^= 1) {
        const int g0 = t0 + tid * GW;
        const bool active = g0 < f1;              // idle threads re-read the piece's first group and count nothing
        const int i0 = active ? g0 : f0, i1 = active ? min(f1, g0 + GW) : f0;
        double wv[GW];
        double local = 0.0;
        float lp[GW], lq[GW];
        w.template load_group<VEC>(i0, active ? i1 : f1, lp, lq);
#pragma unroll
        for (int j = 0; j < GW; ++j) {
            double ea, eb, tt;
            w.eval(lp[j], lq[j], &ea, &eb, &tt);
            const double r = ea * inv_zp - eb * inv_zq;
            const double wj = fall_back_to_p ? ea * inv_zp : (r > 0.0 ? r : 0.0);
            wv[j] = i0 + j < i1 ? wj : 0.0;
            local += wv[j];
        }
        // exclusive prefix of `local` over threads, in thread order
        const double incl = wave_prefix_sum_d(local);
        if (lane == 63) s_scan[turn][wave] = incl;  // two sets: the previous tile's may still be read
        __syncthreads();
        double run = before;
        for (int wvi = 0; wvi < wave; ++wvi) run += s_scan[turn][wvi];
        run += incl - local;
#pragma unroll
        for (int j = 0; j < GW; ++j) {
            if (i0 + j < i1) {
                if (wv[j] > 0.0) lastpos = i0 + j;
                run += wv[j];
                if (!no_crossing && run > t && found == 0x7fffffff) found = i0 + j;
            }
        }
        before += ((s_scan[turn][0] + s_scan[turn][1]) + s_scan[turn][2]) + s_scan[turn][3];
    }
    if (found != 0x7fffffff) atomicMin(&s_best, found);
    if (lastpos >= 0) atomicMax(&s_lastpos, lastpos);
    __syncthreads();
    if (tid == 0) {
        int tok = s_best;
        if (tok == 0x7fffffff) tok = s_lastpos >= 0 ? s_lastpos : f1 - 1;
        a.out_tok[b] = tok;
        a.out_n[b] = n;
        a.flags[b] = flags | (fall_back_to_p ? PSD_FLAG_ZERO_RESIDUAL : 0);
    }
}

inline int round_up(int v, int m) { return (v + m - 1) / m * m; }

}  // namespace

static size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// workspace layout: statistics | the draft tokens' logits | chunk sums of the draw | arrival counters | flags
struct WsLayout { size_t stats, xlogit, part, counter, flags, total; };
static WsLayout ws_layout(const AcceptArgs &a) {
    const size_t rows = a.rows > 0 ? a.rows : 1;
    WsLayout l;
    size_t at = 0;
    l.stats = at;   at += align256(rows * (a.n_p_rows + a.gamma) * a.n_chunksA * sizeof(float2));
    l.xlogit = at;  at += align256(rows * (a.gamma > 0 ? a.gamma : 1) * 2 * sizeof(float));
    l.part = at;    at += align256(rows * a.n_piecesE * kPartStride * sizeof(double));
    l.counter = at; at += align256(rows * sizeof(uint32_t));
    l.flags = at;   at += align256(rows * sizeof(int32_t));
    l.total = at;
    return l;
}

size_t accept_workspace_bytes(const AcceptArgs &a) { return ws_layout(a).total; }

// Draw pass chunking.  Every block repeats its sequence's decision (about 10 us of dependent steps) and one of them finishes
// the draw from the chunk sums; three blocks fit a CU, and the fewer of them share it the faster each.  So: chunks of 512
// entries (two per thread, once) while that makes at most 256 blocks; of 2048 (eight per thread, once) up to 512 blocks; of
// 4096 (twice); and of 8192 for 96 sequences and more of aligned rows once chunks of 4096 no longer fit in one round of the
// chip, or from 2048 blocks on.  Measured (us, draw kernel, fp32; chunks of 512 / 2048 / 4096 / 8192): 1 sequence x 32 000 entries 11.7 /
// 13.5 / 16.7 / 22.3, 4 x 32 000 13.7 / 13.4 / 16.9 / 22.7, 9 x 32 000 17.7 / 14.3 / 16.8 / 22.6, 1 x 128 256 (chunks of 1024
// at least: 128 a row) 13.7 / 12.6 / 16.3 / 22.3, 4 x 152 064 19.4 / 16.7 / 17.5 / 23.0, 32 x 32 000 34.7 / 17.5 / 18.0 / 24.7,
// 96 x 10 000 23.8 / 16.0 / 19.9 / 24.2, 64 x 32 000 45 / 25.9 / 21.7 / 26.1, 128 x 32 000 68 / 42.5 / 37.5 / 34.7, 192 x
// 32 000 91 / 60 / 47.7 / 39.5, 32 x 152 064 66 / 48 / 37.5 / 41.7; unaligned rows, 128 x 32 001 70 / 50 / 44.6 / 47.9.  The last form needs the least workspace: it is
// also taken where the finer one would not fit the built-in scratch buffer.
// pieces: whether the sums of a chunk's quarters may be kept (where it pays: accept_draw_kernel)
static void accept_draw_chunks(AcceptArgs *a, bool vec, bool coarse, bool pieces) {
    const long rows = a->rows > 0 ? a->rows : 1;
    const int V = a->V;
    auto blocks = [&](int ce) { return rows * ((V + ce - 1) / ce); };
    a->groupE = kMaxGroup;
    int ce = 4096;
    if (V <= 512 * kMaxChunksE && blocks(512) <= 256) {
        a->groupE = 2;
        ce = 512;
    } else if (blocks(2048) <= 512) {
        ce = 2048;
    } else if (vec && rows >= 96 && blocks(4096) >= 1024) {
        ce = 8192;
    } else if (blocks(4096) > 2048) {
        coarse = true;
    }
    if (coarse) {
        const long want = ((long)V * rows + 511) / 512;
        a->groupE = kMaxGroup;
        ce = round_up((int)(want < 512 ? 512 : (want > 8192 ? 8192 : want)), 256);
    }
    if ((V + ce - 1) / ce > kMaxChunksE) ce = round_up((V + kMaxChunksE - 1) / kMaxChunksE, 256);
    a->chunkE = ce;
    a->n_chunksE = (V + ce - 1) / ce;
    const bool quarters = pieces && ce >= 4096 && a->n_chunksE * 4 <= kMaxQuarters;
    a->pieceE = quarters ? ce / 4 : ce;
    a->n_piecesE = quarters ? a->n_chunksE * 4 : a->n_chunksE;
}

void accept_plan(int rows, int gamma, int n_p_rows, int V, int dtype, bool vec, AcceptArgs *a) {
    a->rows = rows; a->gamma = gamma; a->n_p_rows = n_p_rows; a->V = V; a->dtype = dtype;
    // whether the finer division of the draw is taken rests on the plan that needs the most workspace (unaligned rows),
    // whatever these rows are: a workspace sized for that plan serves every other
    const int nU = (V + kThreads * kLoadsPerLane - 1) / (kThreads * kLoadsPerLane);
    a->chunkA = (V + nU - 1) / nU;
    a->n_chunksA = (V + a->chunkA - 1) / a->chunkA;
    accept_draw_chunks(a, false, false, false);
    const bool coarse = accept_workspace_bytes(*a) > PSD_STATIC_SCRATCH_BYTES;
    accept_draw_chunks(a, false, coarse, true);                  // and so does whether the chunks come in pieces
    const bool pieces = a->pieceE < a->chunkE && accept_workspace_bytes(*a) <= PSD_STATIC_SCRATCH_BYTES;
    accept_draw_chunks(a, vec, coarse, pieces);
    const int epl = !vec ? 1 : (dtype == PSD_BF16 ? 8 : 4);
    const int cap = kThreads * kLoadsPerLane * epl;            // elements one block can hold
    const int nA = (V + cap - 1) / cap;
    a->chunkA = round_up((V + nA - 1) / nA, epl);
    a->n_chunksA = (V + a->chunkA - 1) / a->chunkA;
}

void accept_bind_workspace(AcceptArgs *a, void *ws, int32_t *out_flags) {
    const WsLayout l = ws_layout(*a);
    char *p = (char *)ws;
    a->stats = (float2 *)(p + l.stats);
    a->xlogit = (float *)(p + l.xlogit);
    a->part = (double *)(p + l.part);
    a->counter = (uint32_t *)(p + l.counter);
    a->flags = out_flags ? out_flags : (int32_t *)(p + l.flags);
}

template <typename T>
static void launch_accept_t(const AcceptArgs &a, bool vec_ok, hipStream_t stream) {
    const int vecs = a.rows * (a.n_p_rows + a.gamma);
    if (vecs > 0) {
        dim3 grid((unsigned)vecs * a.n_chunksA);
        ScopedProf sp(PSD_KIND_ACCEPT_STATS, stream);
        if (vec_ok) launch_kernel(accept_stats_kernel<T, true>, grid, kThreads, 0, stream, a);
        else launch_kernel(accept_stats_kernel<T, false>, grid, kThreads, 0, stream, a);
    }
    dim3 gridE((unsigned)a.rows * a.n_chunksE);
    ScopedProf sp(PSD_KIND_ACCEPT_DRAW, stream);
    auto go = [&](auto kernel) { launch_kernel(kernel, gridE, kThreads, 0, stream, a); };
    auto pick = [&](auto vec) {
        constexpr bool VEC = decltype(vec)::value != 0;
        if (a.groupE == 2) go(accept_draw_kernel<T, VEC, 2, false>);
        else if (a.pieceE < a.chunkE) go(accept_draw_kernel<T, VEC, kMaxGroup, true>);
        else go(accept_draw_kernel<T, VEC, kMaxGroup, false>);
    };
    if (vec_ok) pick(Int<1>{});
    else pick(Int<0>{});
}

void launch_accept(const AcceptArgs &a, bool vec_ok, hipStream_t stream) {
    if (a.dtype == PSD_BF16) launch_accept_t<uint16_t>(a, vec_ok, stream);
    else launch_accept_t<float>(a, vec_ok, stream);
}

}  // namespace psd
