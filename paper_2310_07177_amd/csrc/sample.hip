// sample.hip -- token sampling on gfx950: the draft's proposals y ~ q
// (Algorithm 1 of arXiv:2310.07177) and the mixed sampling
// y ~ beta p + (1 - beta) q that Section 4.1 uses to generate distillation
// data, at temperature T (T = 0: argmax).
//
// Work layout: one workgroup per sampled row n, the row (or the row pair of a
// mixture) read once from HBM into registers; the softmax statistics (K, S) are
// folded in chunk by chunk and merged over lanes and waves; the token is drawn
// with the exact fixed-point inverse CDF of row_draw.hpp.  Masses:
//   one row:  2^(x c2 - K), in units of S (the verification's bonus draw);
//   mixture:  beta 2^(t c2 - K_p)/S_p + (1 - beta) 2^(d c2 - K_q)/S_q, in
//             probability units (the row's total is 1).
// Both are linear in the exponentials, so the draw takes a chunk's mass from
// the sums that the statistics pass kept, and only the winning chunk's elements
// are evaluated again (instruction issue bounded the kernels while every
// element's exponentials were taken twice).  Where the rows fill the chip they
// are streamed (sample_stream_kernel); few rows keep their chunks in registers
// (sample_kernel: 300 pairs of V = 32000 bf16 23.9 -> 18.0 us) or are split
// over workgroups (sample_split_kernel).
#include <stdlib.h>

#include "osd.h"
#include "osd_device.hpp"
#include "osd_internal.hpp"
#include "row_draw.hpp"
#include "stream_device.hpp"

namespace osd {
namespace {

constexpr int kShiftOne = 44;  // units of S: elements <= 1, row total <= V
constexpr int kShiftMix = 52;  // probability units: total 1

enum : int { kModeGreedy = 0, kModeOne = 1, kModeMix = 2 };

struct SampleArgs {
    const char* p;        // the row with weight beta (one-row modes: the row sampled)
    const char* q;        // the row with weight 1 - beta (mixture only)
    int64_t p_stride;     // row strides, bytes
    int64_t q_stride;
    int N, V;
    float c2;             // log2(e) / T
    float beta;
    const float* u;       // [N]
    int32_t* out;         // [N]
};

// One chunk's sum of exponentials and the shift it is relative to.
struct ChunkSum {
    float s, k;
};

// fold_chunk in fp32 that also yields the chunk's own sum, taken left to right.
template <typename Fmt>
__device__ inline ChunkSum fold_chunk_sum(const chunk_t& x, float c2, float& K, float& S) {
    const float kn = fmaxf(K, ceilf(chunk_max<Fmt>(x) * c2));
    S = rescale(S, K, kn);
    K = kn;
    const float kx = fmaxf(K, -3.0e38f);  // see fold_chunk
    float s = exp2_fast(__builtin_fmaf(Fmt::get(x, 0), c2, -kx));
#pragma unroll
    for (int e = 1; e < Fmt::kPerChunk; ++e) s = s + exp2_fast(__builtin_fmaf(Fmt::get(x, e), c2, -kx));
    S = S + s;
    return ChunkSum{s, kx};
}

// The masses of a row (pair) in the terms of the file's header, from the merged
// statistics: a chunk's from its sums, an element's from its logits.
template <bool MIX>
struct SampleMass {
    float c2, Kp, Kq, wp, wq;
    __device__ SampleMass(float c2_, float beta, float Kp_, double Sp, float Kq_, double Sq)
        : c2(c2_), Kp(Kp_), Kq(Kq_), wp(MIX ? float(double(beta) / Sp) : 1.0f),
          wq(MIX ? float((1.0 - double(beta)) / Sq) : 0.0f) {}
    __device__ float chunk(const ChunkSum& p, const ChunkSum& q) const {
        if constexpr (!MIX) return rescale(p.s, p.k, Kp);
        return __builtin_fmaf(rescale(wp, p.k, Kp), p.s, rescale(wq, q.k, Kq) * q.s);
    }
    template <typename Fmt>
    __device__ void elements(const chunk_t& t, const chunk_t& d, float kp, float kq, float (&m)[Fmt::kPerChunk]) const {
        const float sp = rescale(wp, kp, Kp), sq = MIX ? rescale(wq, kq, Kq) : 0.0f;
#pragma unroll
        for (int e = 0; e < Fmt::kPerChunk; ++e) {
            const float et = exp2_fast(__builtin_fmaf(Fmt::get(t, e), c2, -kp));
            if constexpr (!MIX) {
                m[e] = et * sp;
            } else {
                const float ed = exp2_fast(__builtin_fmaf(Fmt::get(d, e), c2, -kq));
                m[e] = __builtin_fmaf(sp, et, sq * ed);
            }
        }
    }
};

template <typename Fmt, int W, int CPT, bool VEC, int MODE>
__global__ __launch_bounds__(W, min_waves_per_simd(W, CPT)) void sample_kernel(SampleArgs a) {
    constexpr int NW = W / kWave;
    constexpr int EPC = Fmt::kPerChunk;
    constexpr bool MIX = MODE == kModeMix;
    __shared__ float s_max[2 * NW];
    __shared__ double s_sum[2 * NW];
    __shared__ int s_idx[NW];
    __shared__ int s_tok;
    __shared__ unsigned long long s_tot[CPT * NW];
    __shared__ DrawShared s_draw;

    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const int n = blockIdx.x;
    chunk_t tv[CPT], dv[CPT];
    // The rows are loaded without padding (a row pair interleaved chunk by
    // chunk) and the statistics pad each chunk as they take it, so they fold
    // in as the loads land.
    const RowCut<Fmt> cut(a.V);
    if constexpr (VEC && MIX) {
        load_rows_interleaved<Fmt, W, CPT>(tv, dv, a.p + int64_t(n) * a.p_stride, a.q + int64_t(n) * a.q_stride, cut);
    } else {
        load_row<Fmt, W, CPT, VEC>(tv, a.p + int64_t(n) * a.p_stride, cut, a.V);
        if constexpr (MIX) load_row<Fmt, W, CPT, VEC>(dv, a.q + int64_t(n) * a.q_stride, cut, a.V);
    }

    if constexpr (MODE == kModeGreedy) {
        // Argmax, lowest index on ties: within a thread indices grow with
        // (round, element), so a strict ">" keeps the first maximum.
        if constexpr (VEC) pad_row_tail<Fmt, W, CPT>(tv, cut);
        float best = kNegInf;
        int bi = 0x7FFFFFFF;
#pragma unroll
        for (int r = 0; r < CPT; ++r)
#pragma unroll
            for (int e = 0; e < EPC; ++e) {
                const float x = Fmt::get(tv[r], e);
                if (x > best) {
                    best = x;
                    bi = (r * W + tid) * EPC + e;
                }
            }
        wave_argmax(best, bi);
        if (lane == 0) {
            s_max[wid] = best;
            s_idx[wid] = bi;
        }
        __syncthreads();
        if (tid == 0) {
            float bv = s_max[0];
            int g = s_idx[0];
            for (int w = 1; w < NW; ++w)
                if (s_max[w] > bv || (s_max[w] == bv && s_idx[w] < g)) {
                    bv = s_max[w];
                    g = s_idx[w];
                }
            a.out[n] = (bv > kNegInf && bv < -kNegInf) ? (VEC ? cut.token(g) : g) : -1;
        }
        return;
    } else {
        const float c2 = a.c2;
        const float u = a.u[n];
        ChunkSum cp[CPT], cq[MIX ? CPT : 1];
        float Kp = kNegInf, Kq = kNegInf, fp = 0.0f, fq = 0.0f;
        if constexpr (VEC) {
            pad_shared_head<Fmt, W, CPT>(tv, cut);
            if constexpr (MIX) pad_shared_head<Fmt, W, CPT>(dv, cut);
        }
#pragma unroll
        for (int r = 0; r < CPT; ++r) {
            if constexpr (VEC) tv[r] = chunk_or_pad<Fmt, W>(tv[r], r, cut);
            cp[r] = fold_chunk_sum<Fmt>(tv[r], c2, Kp, fp);
            if constexpr (MIX) {
                if constexpr (VEC) dv[r] = chunk_or_pad<Fmt, W>(dv[r], r, cut);
                cq[r] = fold_chunk_sum<Fmt>(dv[r], c2, Kq, fq);
            }
            __builtin_amdgcn_sched_barrier(0);  // one chunk pair in flight: bounded VGPRs
        }
        double Sp = fp, Sq = fq;
        if (tid == 0) s_tok = -1;
        block_merge2<NW>(Kp, Sp, Kq, Sq, s_max, s_sum);
        const bool bad = !(Kp > kNegInf && Kp < -kNegInf) || !usable_sum(Sp) ||
                         (MIX && (!(Kq > kNegInf && Kq < -kNegInf) || !usable_sum(Sq)));
        if (bad) {
            if (tid == 0) a.out[n] = -1;
            return;
        }
        const SampleMass<MIX> mass(c2, a.beta, Kp, Sp, Kq, Sq);
        float cm[CPT];
#pragma unroll
        for (int r = 0; r < CPT; ++r) cm[r] = mass.chunk(cp[r], cq[MIX ? r : 0]);
        const auto element = [&](int nstar, float (&m)[EPC]) {
#pragma unroll
            for (int r = 0; r < CPT; ++r)
                if (r == nstar) mass.template elements<Fmt>(tv[r], MIX ? dv[r] : tv[r], cp[r].k, cq[MIX ? r : 0].k, m);
        };
        const int at = draw_from_sums<MIX ? kShiftMix : kShiftOne, W, CPT, EPC>(cm, element, u, s_tot, &s_draw);
        if (at >= 0) s_tok = VEC ? cut.token(at) : at;
        __syncthreads();
        if (tid == 0) a.out[n] = s_tok;  // -1 when no element carries mass
    }
}

template <typename Fmt, int W, int CPT, bool VEC, int MODE>
hipError_t launch_mode(const SampleLaunch& L, const SampleArgs& a) {
    return launch_kernel(&sample_kernel<Fmt, W, CPT, VEC, MODE>, dim3(unsigned(L.N)), dim3(W), 0, L.stream, a);
}

// sample_kernel with the rows streamed, U rounds of loads at a time: only the
// chunk sums are held (63 VGPRs at 8 chunks per thread of a pair instead of 102,
// so twice the waves hide the loads), and the winning wave reads its chunk
// again.  Mixtures of 4096 row pairs of V = 32000 bf16: 131 -> 90 us (5.8 TB/s;
// 32000 fp32 254 -> 160, 6.6 TB/s), of 2048 pairs of V = 128256: 346 -> 215 (the
// rows were read twice before).  Four rounds at a time beat two by up to 6 %.
constexpr int kStreamUnroll = 4;

template <typename Fmt, int W, int CPT, int U, bool MIX>
__global__ __launch_bounds__(W, 1) void sample_stream_kernel(SampleArgs a) {
    constexpr int NW = W / kWave, EPC = Fmt::kPerChunk;
    __shared__ float s_max[2 * NW];
    __shared__ double s_sum[2 * NW];
    __shared__ int s_tok;
    __shared__ unsigned long long s_tot[CPT * NW];
    __shared__ DrawShared s_draw;

    const int tid = threadIdx.x;
    const int n = blockIdx.x;
    const char* prow = a.p + int64_t(n) * a.p_stride;
    const char* qrow = MIX ? a.q + int64_t(n) * a.q_stride : prow;
    const RowCut<Fmt> cut(a.V);
    const int R = (cut.nchunks + W - 1) / W;
    const float c2 = a.c2;
    const float u = a.u[n];
    ChunkSum cp[CPT], cq[MIX ? CPT : 1];
    float Kp = kNegInf, Kq = kNegInf, fp = 0.0f, fq = 0.0f;
    cq[0] = ChunkSum{0.0f, kNegInf};
#pragma unroll
    for (int g = 0; g < CPT; g += U) {
        if (g < R) {
            chunk_t xp[U], xq[U];
#pragma unroll
            for (int r = 0; r < U; ++r) {
                const int off = cut.off((g + r) * W + tid);
                xp[r] = load_off(prow, off);
                if constexpr (MIX) xq[r] = load_off(qrow, off);
            }
            pad_shared_head<Fmt, W, U>(xp, cut, g);
            if constexpr (MIX) pad_shared_head<Fmt, W, U>(xq, cut, g);
#pragma unroll
            for (int r = 0; r < U; ++r) {
                cp[g + r] = fold_chunk_sum<Fmt>(chunk_or_pad<Fmt, W>(xp[r], g + r, cut), c2, Kp, fp);
                if constexpr (MIX)
                    cq[g + r] = fold_chunk_sum<Fmt>(chunk_or_pad<Fmt, W>(xq[r], g + r, cut), c2, Kq, fq);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            // Rounds past the row, as a chunk of padding: a shift above the row's (0, where
            // every logit lies far below) would scale the absent mass up to infinity.
#pragma unroll
            for (int r = 0; r < U; ++r) cp[g + r] = cq[MIX ? g + r : 0] = ChunkSum{0.0f, kNegInf};
        }
    }
    double Sp = fp, Sq = fq;
    if (tid == 0) s_tok = -1;
    block_merge2<NW>(Kp, Sp, Kq, Sq, s_max, s_sum);
    const bool bad = !(Kp > kNegInf && Kp < -kNegInf) || !usable_sum(Sp) ||
                     (MIX && (!(Kq > kNegInf && Kq < -kNegInf) || !usable_sum(Sq)));
    if (bad) {
        if (tid == 0) a.out[n] = -1;
        return;
    }
    const SampleMass<MIX> mass(c2, a.beta, Kp, Sp, Kq, Sq);
    float cm[CPT];
#pragma unroll
    for (int r = 0; r < CPT; ++r) cm[r] = mass.chunk(cp[r], cq[MIX ? r : 0]);
    const auto element = [&](int nstar, float (&m)[EPC]) {
        float kp = 0.0f, kq = 0.0f;
#pragma unroll
        for (int r = 0; r < CPT; ++r)
            if (r == nstar) {
                kp = cp[r].k;
                kq = cq[MIX ? r : 0].k;
            }
        const chunk_t tc = stream_chunk<Fmt, W>(prow, nstar, cut);
        mass.template elements<Fmt>(tc, MIX ? stream_chunk<Fmt, W>(qrow, nstar, cut) : tc, kp, kq, m);
    };
    const int at = draw_from_sums<MIX ? kShiftMix : kShiftOne, W, CPT, EPC>(cm, element, u, s_tot, &s_draw);
    if (at >= 0) s_tok = cut.token(at);
    __syncthreads();
    if (tid == 0) a.out[n] = s_tok;
}

// One-row sampling of few rows (fewer than two per CU), each row split over S
// segment workgroups of 256 threads (CPT chunks per thread, SEG = CPT*256
// chunks per segment).  The inverse CDF needs no global normaliser: for any
// common shift K, token j is the first whose running sum of 2^(x c2 - K)
// exceeds u times the total.  Each segment therefore works alone:
//   1. shift k_s = ceil(max over the segment * c2); masses 2^(x c2 - k_s);
//      each thread's chunk sums become 2^-40 fixed point (whole numbers in
//      fp64, exact below 2^53), summed into cells (round, wave) and the
//      segment total T_s;
//   2. it publishes (k_s, T_s) and reads its siblings' (bounded polls; a
//      workgroup that runs out of polls computes the missing records itself
//      from the rows in memory, bit for bit as their owners do);
//   3. every segment combines the S records in segment order, identically:
//      K = max k_s over segments with a finite logit, weights
//      W_s = floor(T_s 2^(k_s - K)) (u64), Z = sum W_s, the point
//      c = floor(u Z), and the segment s* whose weight interval holds c;
//   4. s* maps c into its own units (an exact shift: the local offset stays
//      below T_s*) and walks its cells, its lanes and its elements.
// The cells partition [0, Z) exactly, so the token is always one with mass;
// it can differ from the one-workgroup kernel's only where u*Z lies within
// the fp32 rounding of a boundary.  Records are two never-zero words per
// segment (the shift's bits with the top bit set; the total's bits
// inverted); each workgroup arrives at its row's counter once it holds all
// S records, and the last to arrive clears the row's words and counter.
constexpr int kSegSampleW = 256;
constexpr int kMaxSampleSegments = 16;
constexpr int kSamplePolls = 256;

struct SplitSampleArgs {
    const char* row;   // row 0 of the sampled rows
    int64_t stride;    // bytes between rows
    int N, V, S, polls;
    float c2;
    const float* u;
    int32_t* out;
    uint64_t* rec;     // [N, kMaxSampleSegments, 2], zero between calls
    uint32_t* cnt;     // [N, 4] (word 0: arrivals), zero between calls
};

__device__ inline double fixed40(float x) { return floor(double(x) * 0x1p40); }

// Statistics of one segment held in x (chunk r of this thread is segment
// chunk r*W + tid): the shift, the cell totals (s_cell[r*NW + w]) and their
// exclusive prefix in segment order (s_excl), the total and whether the
// segment has any finite logit.  Each thread also keeps what a walk to a
// point inside its chunks needs: the chunk masses m, their fixed-point sums
// f and the sum of the lower lanes' sums in the same cell (off).  All
// threads call it; it ends with the cell values visible to every thread.
template <typename Fmt, int CPT>
__device__ void segment_stats(const chunk_t (&x)[CPT], float c2, float* s_mx, double* s_cell, double* s_excl,
                              double* s_tot, float& k, double& T, bool& empty, float (&m)[CPT][Fmt::kPerChunk],
                              double (&f)[CPT], double (&off)[CPT]) {
    constexpr int W = kSegSampleW, NW = W / kWave, EPC = Fmt::kPerChunk, CELLS = CPT * NW;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    float mx = chunk_max<Fmt>(x[0]);
#pragma unroll
    for (int r = 1; r < CPT; ++r) mx = fmaxf(mx, chunk_max<Fmt>(x[r]));
    mx = wave_max_u(mx);
    if (lane == 0) s_mx[wid] = mx;
    __syncthreads();
    mx = s_mx[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) mx = fmaxf(mx, s_mx[w]);
    empty = !(mx > kNegInf);
    k = shift_of_max(mx, c2);
#pragma unroll
    for (int r = 0; r < CPT; ++r) {
        m[r][0] = exp2_fast(__builtin_fmaf(Fmt::get(x[r], 0), c2, -k));
        float sm = m[r][0];
#pragma unroll
        for (int e = 1; e < EPC; ++e) {
            m[r][e] = exp2_fast(__builtin_fmaf(Fmt::get(x[r], e), c2, -k));
            sm = sm + m[r][e];
        }
        f[r] = fixed40(sm);
        const double t = wave_scan_add(f[r]);
        off[r] = t - f[r];
        if (lane == kWave - 1) s_cell[r * NW + wid] = t;
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    if (wid == 0) {
        const double cv = lane < CELLS ? s_cell[lane] : 0.0;
        const double ci = wave_scan_add(cv);
        if (lane < CELLS) s_excl[lane] = ci - cv;
        if (lane == kWave - 1) *s_tot = ci;
    }
    __syncthreads();
    T = *s_tot;
}

template <typename Fmt, int CPT>
__global__ __launch_bounds__(kSegSampleW) void sample_split_kernel(SplitSampleArgs a) {
    constexpr int W = kSegSampleW, NW = W / kWave, EPC = Fmt::kPerChunk, SEG = CPT * W, CELLS = CPT * NW;
    static_assert(CELLS <= kWave, "one wave scans the cells");
    __shared__ float s_mx[NW];
    __shared__ double s_cell[CELLS];
    __shared__ double s_excl[CELLS];
    __shared__ double s_tot;
    __shared__ float s_k[kMaxSampleSegments];
    __shared__ double s_T[kMaxSampleSegments];
    __shared__ int s_ok;
    __shared__ int s_tok;

    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const int S = a.S, n = blockIdx.x / S, s = blockIdx.x - n * S;
    const char* row = a.row + int64_t(n) * a.stride;
    uint64_t* rec = a.rec + int64_t(n) * kMaxSampleSegments * 2;
    const float c2 = a.c2;

    // The row's uniform is read with the chunks (a load after the exchange
    // would wait for the exchange's own memory operations).
    const float un = a.u[n];
    const RowCut<Fmt> cut(a.V);
    chunk_t x[CPT];
#pragma unroll
    for (int r = 0; r < CPT; ++r) x[r] = load_off(row, cut.off(s * SEG + r * W + tid));
    pad_row_tail<Fmt, W, CPT>(x, cut, s * CPT);
    if (tid == 0) s_tok = -1;  // ordered before the walk by the statistics' barriers
    float k;
    double T;
    bool empty;
    float mass[CPT][EPC];
    double fx[CPT], off[CPT];
    segment_stats<Fmt, CPT>(x, c2, s_mx, s_cell, s_excl, &s_tot, k, T, empty, mass, fx, off);
    if (tid == 0) {
        s_k[s] = empty ? kNegInf : k;
        s_T[s] = T;
        // Both words issued before either completion is waited for.
        const uint64_t o0 = __hip_atomic_exchange(&rec[2 * s], (1ull << 63) | __float_as_uint(empty ? kNegInf : k),
                                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t o1 = __hip_atomic_exchange(&rec[2 * s + 1], ~uint64_t(__double_as_longlong(T)),
                                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("" ::"v"(o0), "v"(o1));
    }
    // The siblings' records: wave 0, lane j reads segment j's two words.
    if (wid == 0) {
        const bool mine = lane < S && lane != s;
        bool ok = false;
        uint64_t w0 = 0, w1 = 0;
        for (int p = 0; p < a.polls; ++p) {
            if (p > 0) __builtin_amdgcn_s_sleep(4);
            bool ready = true;
            if (mine) {
                w0 = poll_u64(&rec[2 * lane]);
                w1 = poll_u64(&rec[2 * lane + 1]);
                ready = w0 != 0 && w1 != 0;
            }
            if (__ballot(!ready) == 0) {
                ok = true;
                break;
            }
        }
        if (ok && mine) {
            s_k[lane] = __uint_as_float(uint32_t(w0));
            s_T[lane] = __longlong_as_double(~w1);
        }
        if (lane == 0) s_ok = ok;
    }
    __syncthreads();
    if (!s_ok) {
        // Out of polls: every other segment's record from the row itself.
        __shared__ double s_cellx[CELLS], s_exclx[CELLS];
        for (int j = 0; j < S; ++j) {
            if (j == s) continue;
            chunk_t y[CPT];
#pragma unroll
            for (int r = 0; r < CPT; ++r) y[r] = stream_chunk<Fmt, W>(row, j * CPT + r, cut);
            float kj;
            double Tj;
            bool ej;
            float mj[CPT][EPC];
            double fj[CPT], oj[CPT];
            segment_stats<Fmt, CPT>(y, c2, s_mx, s_cellx, s_exclx, &s_tot, kj, Tj, ej, mj, fj, oj);
            if (tid == 0) {
                s_k[j] = ej ? kNegInf : kj;
                s_T[j] = Tj;
            }
        }
        __syncthreads();
    }
    // Arrival at the row's counter, once this workgroup holds every record:
    // issued here, its count awaited only at the end (s* walks meanwhile);
    // the last to arrive leaves the row's words zero.  (This workgroup's
    // records went out before its polls, whose waits covered them.)
    uint32_t prev = 0;
    if (tid == 0) prev = __hip_atomic_fetch_add(&a.cnt[int64_t(n) * 4], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    auto arrive_row = [&]() {
        if (tid == 0 && prev == uint32_t(S - 1)) {
            for (int j = 0; j < S; ++j) {
                take_u64(&rec[2 * j]);
                take_u64(&rec[2 * j + 1]);
            }
            take_u32(&a.cnt[int64_t(n) * 4]);
        }
    };
    // The combine, identical in every segment and every wave (no barrier):
    // lane j holds segment j's record; the shift K is their maximum, the
    // weights are scanned in segment order, and s* is the lane whose weight
    // interval holds c.
    const bool have = lane < S;
    const float kj = have ? s_k[lane] : kNegInf;
    const double Tj = have ? s_T[lane] : 0.0;
    const bool bad = __ballot(have && !(Tj >= 0.0 && Tj < 0x1p60)) != 0;
    const float K = wave_max_u(kj);
    uint64_t wj = 0;
    if (have && kj > kNegInf && !bad) wj = uint64_t(floor(__builtin_ldexp(Tj, int(fmaxf(kj - K, -2048.0f)))));
    const uint64_t incl = wave_scan_add(wj);
    const uint64_t Z = readlane_u64(incl, kWave - 1);
    if (bad || Z == 0) {
        if (s == 0 && tid == 0) a.out[n] = -1;
        arrive_row();
        return;
    }
    uint64_t c = uint64_t(double(un) * double(Z));
    if (c >= Z) c = Z - 1;
    const uint64_t hit = __ballot(wj > 0 && incl - wj <= c && c < incl);
    const int sstar = hit ? __builtin_ctzll(hit) : -1;
    if (s != sstar) {
        arrive_row();
        return;
    }
    const uint64_t lo = readlane_u64(incl - wj, sstar);
    // This segment holds the point: its offset in the segment's own units.
    // The cell (round r of this wave) and the lane that hold it, from the
    // prefixes prepared before the exchange; that lane walks its chunk with
    // the same fp32 sums of the same masses.
    const double target = __builtin_ldexp(double(c - lo), int(K - k));
#pragma unroll
    for (int r = 0; r < CPT; ++r) {
        const double cl = s_excl[r * NW + wid];
        if (cl <= target && target < cl + s_cell[r * NW + wid]) {
            const double mylo = cl + off[r];
            if (fx[r] > 0.0 && mylo <= target && target < mylo + fx[r]) {
                const double want = target - mylo;
                float racc = mass[r][0];
                int pick = fixed40(racc) > want ? 0 : -1, last_pos = mass[r][0] > 0.0f ? 0 : -1;
#pragma unroll
                for (int e = 1; e < EPC; ++e) {
                    racc = racc + mass[r][e];
                    if (mass[r][e] > 0.0f) last_pos = e;
                    if (pick < 0 && fixed40(racc) > want) pick = e;
                }
                if (pick < 0) pick = last_pos >= 0 ? last_pos : 0;
                s_tok = cut.token(((s * SEG + r * W + tid) * EPC) + pick);
            }
        }
    }
    __syncthreads();
    if (tid == 0) a.out[n] = s_tok;
    arrive_row();
}

// kSamplePolls, or the value of OSD_SAMPLE_POLLS (read once; 0 makes every
// workgroup compute its siblings' records itself).
int sample_polls() {
    static const int v = [] {
        const char* e = getenv("OSD_SAMPLE_POLLS");
        if (e == nullptr || *e == 0) return kSamplePolls;
        const int k = atoi(e);
        return k < 0 ? kSamplePolls : (k > 65536 ? 65536 : k);
    }();
    return v;
}

template <typename Fmt, int CPT>
hipError_t launch_split(const SampleLaunch& L, const SampleArgs& a, int S) {
    SplitSampleArgs sa{};
    sa.row = a.p;
    sa.stride = a.p_stride;
    sa.N = a.N;
    sa.V = a.V;
    sa.S = S;
    sa.polls = sample_polls();
    sa.c2 = a.c2;
    sa.u = a.u;
    sa.out = a.out;
    char* w = static_cast<char*>(L.workspace);
    sa.rec = reinterpret_cast<uint64_t*>(w);
    sa.cnt = reinterpret_cast<uint32_t*>(w + size_t(L.N) * kMaxSampleSegments * 16);
    return launch_kernel(&sample_split_kernel<Fmt, CPT>, dim3(unsigned(L.N) * unsigned(S)), dim3(kSegSampleW), 0,
                         L.stream, sa);
}

// The split applies to one-row sampling (T > 0, beta 0 or 1) when one
// workgroup per row would leave most CUs idle.
template <typename Fmt>
bool try_split(const SampleLaunch& L, const SampleArgs& a, hipError_t* e) {
    if (!L.workspace || !(L.temperature > 0.0f) || (L.beta > 0.0f && L.beta < 1.0f)) return false;
    if (L.N >= 2 * L.cus) return false;
    const int nchunks = (L.V + Fmt::kPerChunk - 1) / Fmt::kPerChunk;
    const int s2 = (nchunks + 2 * kSegSampleW - 1) / (2 * kSegSampleW);
    const int s4 = (nchunks + 4 * kSegSampleW - 1) / (4 * kSegSampleW);
    if (s2 >= 2 && s2 <= kMaxSampleSegments && int64_t(L.N) * s2 <= 4 * int64_t(L.cus)) {
        *e = launch_split<Fmt, 2>(L, a, s2);
        return true;
    }
    if (s4 >= 2 && s4 <= kMaxSampleSegments && int64_t(L.N) * s4 <= 4 * int64_t(L.cus)) {
        *e = launch_split<Fmt, 4>(L, a, s4);
        return true;
    }
    return false;
}

template <typename Fmt, int W, int CPT, bool VEC>
hipError_t launch_tile(const SampleLaunch& L, const SampleArgs& a) {
    if (L.temperature == 0.0f) return launch_mode<Fmt, W, CPT, VEC, kModeGreedy>(L, a);
    if (L.beta > 0.0f && L.beta < 1.0f) return launch_mode<Fmt, W, CPT, VEC, kModeMix>(L, a);
    return launch_mode<Fmt, W, CPT, VEC, kModeOne>(L, a);
}

// Rows that fill the chip: streamed where the chunks and sums of the row (pair)
// would take more than the 64 VGPRs that leave room for eight waves per SIMD
// (4 chunks per thread of a pair, 8 of one row); shorter rows keep their chunks
// (4096 rows of V = 2000 bf16 10.6 us, streamed 12.1).
template <typename Fmt, int W, int CPT>
hipError_t launch_rows(const SampleLaunch& L, const SampleArgs& a) {
    if (L.temperature == 0.0f) return launch_mode<Fmt, W, CPT, true, kModeGreedy>(L, a);
    const dim3 grid(unsigned(L.N)), block(W);
    if (L.beta > 0.0f && L.beta < 1.0f) {
        if constexpr (CPT < 4)
            return launch_mode<Fmt, W, CPT, true, kModeMix>(L, a);
        else
            return launch_kernel(&sample_stream_kernel<Fmt, W, CPT, kStreamUnroll, true>, grid, block, 0, L.stream, a);
    }
    if constexpr (CPT < 8)
        return launch_mode<Fmt, W, CPT, true, kModeOne>(L, a);
    else
        return launch_kernel(&sample_stream_kernel<Fmt, W, CPT, kStreamUnroll, false>, grid, block, 0, L.stream, a);
}

template <typename Fmt>
hipError_t launch_fmt(const SampleLaunch& L, const SampleArgs& a) {
    if (L.V < Fmt::kPerChunk) return launch_tile<Fmt, 256, 1, false>(L, a);  // shorter than one chunk
    hipError_t se;
    if (try_split<Fmt>(L, a, &se)) return se;
    RowTile t;
    if (!pick_tile(L.V, Fmt::kPerChunk, &t)) return launch_rows<Fmt, 1024, 16>(L, a);
    // Fewer rows than two per CU: the rows' latency is the cost, so each row
    // gets the widest workgroup (half the elements per thread), and keeps its
    // chunks while they fit.
    if (L.N < 2 * L.cus) {
        const int per = 1024 * Fmt::kPerChunk;
        if (L.V <= 2 * per) return launch_tile<Fmt, 1024, 2, true>(L, a);
        if (L.V <= 4 * per) return launch_tile<Fmt, 1024, 4, true>(L, a);
        return launch_rows<Fmt, 1024, 8>(L, a);
    }
    switch (t.W * 100 + t.CPT) {
        case 25601: return launch_rows<Fmt, 256, 1>(L, a);
        case 25602: return launch_rows<Fmt, 256, 2>(L, a);
        case 25604: return launch_rows<Fmt, 256, 4>(L, a);
        case 51204: return launch_rows<Fmt, 512, 4>(L, a);
        case 51208: return launch_rows<Fmt, 512, 8>(L, a);
        case 102408: return launch_rows<Fmt, 1024, 8>(L, a);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_sample(const SampleLaunch& L) {
    SampleArgs a{};
    // One-row modes sample the row with weight 1: p when beta == 1, q when
    // beta == 0 (the row with weight 0 is never read).
    const bool q_only = L.beta == 0.0f;
    a.p = static_cast<const char*>(q_only ? L.q : L.p);
    a.q = static_cast<const char*>(L.q);
    const int64_t elem = L.dtype == 1 ? 2 : 4;
    a.p_stride = (q_only ? L.q_stride : L.p_stride) * elem;
    a.q_stride = L.q_stride * elem;
    a.N = L.N;
    a.V = L.V;
    a.c2 = L.temperature > 0.0f ? float(1.4426950408889634 / double(L.temperature)) : 0.0f;
    a.beta = L.beta;
    a.u = L.u;
    a.out = L.out;
    return L.dtype == 1 ? launch_fmt<BF16>(L, a) : launch_fmt<F32>(L, a);
}

}  // namespace osd
