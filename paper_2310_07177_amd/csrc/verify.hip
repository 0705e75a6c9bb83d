// verify.hip -- speculative-sampling verification on gfx950.
//
// Method (Appendix A.1 and Eq. 5 of arXiv:2310.07177; Algorithm 1, the step
// that determines the accepted count and samples one more token): proposals
// y_1..y_k are tested in order, y_i is accepted when u_i < p(y_i)/q(y_i), the
// first rejection at position a ends the test, and one extra token is drawn
// from norm(max(0, p - q)) at row a, or from p at the bonus row when all k
// were accepted.  p and q are temperature softmaxes of the logits.
//
// Work layout (rows of up to 8 chunks per thread of 512 threads; the other
// lengths and few rows below).  One workgroup per (sequence b, proposal row i),
// numbered position-major, then one workgroup per bonus row.  A proposal workgroup
// reads its target and draft rows from HBM exactly once into registers,
// reduces the row maxima and sums of exponentials, and takes the acceptance
// test.  A rejecting workgroup announces the rejection at once, then learns
// (by polling the records of the earlier positions of its sequence, with a
// bounded number of polls) whether it is the first rejection; only the first
// draws the correction token, from the rows it already holds.  If the polls
// run out it draws anyway, which is always correct.  A bonus workgroup first
// checks whether an earlier position has already rejected and, if so, skips
// its row entirely.  Every workgroup publishes a one-word record; the last of
// the k_b + 1 workgroups of a sequence to arrive selects the first rejection,
// writes the outputs, and clears the records and the counter.
#include <stdlib.h>

#include "osd_device.hpp"
#include "osd_internal.hpp"
#include "row_draw.hpp"
#include "stream_device.hpp"

namespace osd {
namespace {

// Record word: state in bits 31..28, token in bits 27..0.
enum : uint32_t {
    kRecEmpty = 0,
    kRecAccept = 1,
    kRecReject = 2,          // rejected, correction token attached
    kRecRejectSkipped = 3,   // rejected after an earlier rejection was seen
    kRecBadRow = 4,          // no finite logit in a row that was read
    kRecBadToken = 5,        // proposal outside [0, V)
    kRecBonus = 6,           // bonus token attached
    kRecBonusSkipped = 7,    // an earlier rejection was seen
    kRecRejectPending = 8,   // rejected, correction not yet decided
};

__device__ inline uint32_t make_rec(uint32_t state, uint32_t tok) {
    return (state << 28) | (tok & 0x0FFFFFFFu);
}
__device__ inline uint32_t rec_state(uint32_t r) { return r >> 28; }
__device__ inline int rec_token(uint32_t r) { return int(r & 0x0FFFFFFFu); }
__device__ inline bool rejects(uint32_t s) {
    return s == kRecReject || s == kRecRejectSkipped || s == kRecRejectPending || s == kRecBadToken;
}

// Residual masses are handled in units of S_t (the target row's sum of
// exponentials), where every element is at most about 1: chunk sums stay
// below 16 and row totals below 2^17, so a 2^-44 fixed point never overflows.
constexpr int kFixedShift = 44;
// Looks at the earlier positions' records before a rejecting workgroup draws
// speculatively (a speculative draw is always correct: the finalizer takes
// the first rejection's token).  Each look is one device-coherent round trip.
// The row-resident kernel looks once: its draw works on registers it already
// holds, and waiting for a late earlier row costs more than drawing (a
// measured 0.4 us at B = 64, k = 8).  The streamed kernel, whose draw reads
// the row pair again, waits longer (24 looks with a short sleep).
constexpr int kMaxPolls = 1;

struct VerifyArgs {
    const void* target;
    const void* draft;
    int B, K, V;
    const int32_t* tokens;
    const int32_t* draft_len;
    const float* u_accept;
    const float* u_resample;
    float c2;        // log2(e) / T, the scale of every exponent
    double c2d;      // the same value in fp64
    int32_t* accepted_len;
    int32_t* out_tokens;
    uint8_t* reject_mask;
    VerifyRow* rows;
};

__device__ void write_invalid(const VerifyArgs& a, int b) {
    const int K = a.K;
    for (int j = threadIdx.x; j <= K; j += blockDim.x) {
        a.out_tokens[int64_t(b) * (K + 1) + j] = -1;
        if (a.reject_mask && j < K) a.reject_mask[int64_t(b) * K + j] = 0;
    }
    if (threadIdx.x == 0) a.accepted_len[b] = -1;
}

// Executed by all 64 lanes of one wave with the same `record`: publish this
// row's final record, and if it is the last of the k_b + 1 rows of sequence b
// to arrive, emit the outputs.  Lane j handles position j (K < 64).  The record is
// in place before the arrival is issued, so the last arriver finds every record
// final.  (The wait between the two costs 0.2 to 0.4 us a call: B = 8, K = 5, V =
// 32000 bf16 11.8 -> 12.1, B = 64, K = 8, V = 32128 19.5 -> 19.8.  One word for states
// and arrivals, so that only tokens are waited for, took 12.2 and 19.6.)
__device__ void publish(const VerifyArgs& a, int b, int i, int kb, uint32_t record) {
    const int K = a.K;
    const int lane = threadIdx.x & (kWave - 1);
    VerifyRow* rows = a.rows + int64_t(b) * (K + 1);
    uint32_t prev = 0;
    if (lane == 0) {
        publish_u32(&rows[i].record, record);
        prev = arrive(&rows[0].arrivals);
    }
    prev = __shfl(prev, 0, kWave);
    if (prev != uint32_t(kb)) return;

    // The last arriver reads every record and clears it.
    uint32_t r = 0u;
    if (lane <= kb) r = take_u32(&rows[lane].record);

    // First rejection (Appendix A.1: the test stops there).  A proposal
    // outside the vocabulary invalidates the sequence wherever it sits; a row
    // without finite logits only if the test reaches it.
    const uint32_t s = rec_state(r);
    const bool bad_token = __ballot(lane < kb && s == kRecBadToken) != 0;
    const uint64_t stop = __ballot(lane < kb && s != kRecAccept);
    int acc = kb;
    if (stop) acc = __builtin_ctzll(stop);
    const uint32_t ra = __shfl(r, acc, kWave);
    bool bad = bad_token;
    int extra = -1;
    if (!bad) {
        const uint32_t sa = rec_state(ra);
        if (acc < kb ? sa == kRecReject : sa == kRecBonus)
            extra = rec_token(ra);
        else
            bad = true;  // a row without finite logits
    }
    const int32_t* y = a.tokens + int64_t(b) * K;
    if (lane <= K) {
        int32_t o = -1;
        if (!bad) o = lane < acc ? y[lane] : (lane == acc ? extra : -1);
        a.out_tokens[int64_t(b) * (K + 1) + lane] = o;
        if (a.reject_mask && lane < K)
            a.reject_mask[int64_t(b) * K + lane] = (!bad && lane == acc && acc < kb) ? 1 : 0;
    }
    if (lane == 0) {
        a.accepted_len[b] = bad ? -1 : acc;
        __hip_atomic_store(&rows[0].arrivals, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Called by all lanes of a wave.  Looks at the records of positions 0..i-1:
// returns 2 if one of them rejected (or proposed an invalid token), 1 if all
// accepted, 0 if still undecided after `polls` looks.
__device__ int poll_earlier(const VerifyArgs& a, int b, int i, int polls) {
    const int lane = threadIdx.x & (kWave - 1);
    const VerifyRow* rows = a.rows + int64_t(b) * (a.K + 1);
    for (int p = 0;; ++p) {
        const uint32_t s = lane < i ? rec_state(load_relaxed(&rows[lane].record)) : uint32_t(kRecAccept);
        if (__ballot(rejects(s)) != 0) return 2;
        if (__ballot(s != kRecAccept) == 0) return 1;
        if (p + 1 >= polls) return 0;
        __builtin_amdgcn_s_sleep(8);
    }
}

// Announce row i's rejection before its token is drawn, without waiting for the word:
// the row's final record goes to the same word after it.  (Waiting took B = 64, K = 8,
// V = 32128 bf16 24.0 us a call instead of 23.8.)
__device__ inline void announce_reject(const VerifyArgs& a, int b, int i) {
    __hip_atomic_exchange(&a.rows[int64_t(b) * (a.K + 1) + i].record, make_rec(kRecRejectPending, 0), __ATOMIC_RELAXED,
                          __HIP_MEMORY_SCOPE_AGENT);
}

// p(y)/q(y) = 2^e S_d / S_t with e = (t_y c2 - K_t) - (d_y c2 - K_d) in fp64; 2^e is
// split into an exact power of two and 2^frac (v_exp_f32, 1 ulp).
__device__ inline double acceptance_ratio(float ty, float dy, float Kt, double St, float Kd, double Sd, double c2d) {
    const double e = (double(ty) * c2d - double(Kt)) - (double(dy) * c2d - double(Kd));
    if (!(e > -2000.0)) return 0.0;  // p(y) = 0 (or both probabilities 0)
    if (e > 2000.0) return __builtin_huge_val();
    const double n = floor(e);
    return __builtin_ldexp(double(exp2_fast(float(e - n))), int(n)) * (Sd / St);
}

template <typename Fmt, int W, int CPT, bool VEC, bool GREEDY>
__global__ __launch_bounds__(W, min_waves_per_simd(W, CPT)) void verify_kernel(VerifyArgs a) {
    constexpr int NW = W / kWave;
    constexpr int EPC = Fmt::kPerChunk;
    __shared__ float s_max[2][NW];
    __shared__ double s_sum[2][NW];
    __shared__ int s_idx[NW];
    __shared__ int s_flag;
    __shared__ int s_tok;
    __shared__ unsigned long long s_tot[CPT * NW];
    __shared__ DrawShared s_draw;
    __shared__ chunk_t s_stage[GREEDY ? 1 : 2 * CPT * kWave];

    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const int B = a.B, K = a.K, V = a.V;
    const bool bonus = int(blockIdx.x) >= B * K;
    int b, i;
    if (!bonus) {
        i = blockIdx.x / B;
        b = blockIdx.x - i * B;
    } else {
        b = blockIdx.x - B * K;
        i = -1;
    }
    const int kb = a.draft_len ? a.draft_len[b] : K;
    if (kb < 1 || kb > K) {
        if (bonus) write_invalid(a, b);
        return;
    }
    if (bonus) {
        i = kb;
    } else if (i >= kb) {
        return;  // padding row of a short proposal
    }
    const int y = bonus ? 0 : a.tokens[int64_t(b) * K + i];
    if (!bonus && (y < 0 || y >= V)) {
        if (wid == 0) publish(a, b, i, kb, make_rec(kRecBadToken, 0));
        return;
    }
    if (bonus) {
        // The bonus row matters only if every proposal is accepted: skip it
        // when a rejection is already visible.
        if (wid == 0) {
            const int st = poll_earlier(a, b, i, 1);
            if (lane == 0) s_flag = st;
            if (st == 2) publish(a, b, i, kb, make_rec(kRecBonusSkipped, 0));
        }
        __syncthreads();
        if (s_flag == 2) return;
    }

    const char* trow = static_cast<const char*>(a.target) +
                       (int64_t(b) * (K + 1) + i) * int64_t(V) * Fmt::kBytes;
    // A bonus row has no draft row: its draft loads re-read the target row
    // (ignored), so that every workgroup issues the same loads without a
    // branch and the compiler can wait for each chunk exactly.
    const char* drow = GREEDY || bonus
                           ? trow
                           : static_cast<const char*>(a.draft) + (int64_t(b) * K + i) * int64_t(V) * Fmt::kBytes;
    // The logits of the proposal itself, for the acceptance test, requested
    // before the rows and converted only after the statistics: loads complete
    // in issue order, so a value used early that was loaded after the rows
    // would make the sweeps wait for the whole row pair.
    uint32_t ty_raw = 0u, dy_raw = 0u;
    if constexpr (!GREEDY) {
        ty_raw = Fmt::load_raw(trow, bonus ? 0 : y);
        dy_raw = Fmt::load_raw(drow, bonus ? 0 : y);
    }
    __builtin_amdgcn_sched_barrier(0);
    // The rows are loaded without padding and the statistics pad each chunk
    // as they take it, so they fold in as the loads land.
    const RowCut<Fmt> cut(V);
    chunk_t tv[CPT];

    if constexpr (GREEDY) {
        static_assert(!VEC, "rows of a chunk or more take the segmented greedy kernels");
        load_row<Fmt, W, CPT, VEC>(tv, trow, cut, V);
        // Target argmax, lowest index on ties: within a thread indices grow
        // with (n, e), so a strict ">" keeps the first maximum.
        float best = kNegInf;
        int bi = 0x7FFFFFFF;
#pragma unroll
        for (int n = 0; n < CPT; ++n)
#pragma unroll
            for (int e = 0; e < EPC; ++e) {
                const float x = Fmt::get(tv[n], e);
                if (x > best) {
                    best = x;
                    bi = (n * W + tid) * EPC + e;
                }
            }
        wave_argmax(best, bi);
        if (lane == 0) {
            s_max[0][wid] = best;
            s_idx[wid] = bi;
        }
        __syncthreads();
        if (wid == 0) {
            float bv = s_max[0][0];
            int g = s_idx[0];
            for (int w = 1; w < NW; ++w)
                if (s_max[0][w] > bv || (s_max[0][w] == bv && s_idx[w] < g)) {
                    bv = s_max[0][w];
                    g = s_idx[w];
                }
            uint32_t r;
            if (!(bv > kNegInf) || bv == -kNegInf)
                r = make_rec(kRecBadRow, 0);
            else if (bonus)
                r = make_rec(kRecBonus, uint32_t(g));
            else
                r = make_rec(y == g ? kRecAccept : kRecReject, uint32_t(g));
            publish(a, b, i, kb, r);
        }
        return;
    } else {
        const float c2 = a.c2;
        // The draft row is read only for proposal rows.
        chunk_t dv[CPT];
        if constexpr (VEC) {
            load_rows_interleaved<Fmt, W, CPT>(tv, dv, trow, drow, cut);
        } else {
            load_row<Fmt, W, CPT, VEC>(tv, trow, cut, V);
            load_row<Fmt, W, CPT, VEC>(dv, drow, cut, V);
        }

        // Row statistics (K, S), folded in chunk by chunk as the loads land.
        float Kt = kNegInf, Kd = kNegInf;
        {
            float st = 0.0f, sd = 0.0f;
            if constexpr (VEC) {
                row_stats2<Fmt, W, CPT>(tv, dv, cut, c2, !bonus, Kt, st, Kd, sd);
            } else {
                row_stats<Fmt, W, CPT, false>(tv, cut, c2, Kt, st);
                if (!bonus) row_stats<Fmt, W, CPT, false>(dv, cut, c2, Kd, sd);
            }
            double dt = st, dd = sd;
            wave_merge_stats(Kt, dt);
            wave_merge_stats(Kd, dd);
            if (lane == 0) {
                s_max[0][wid] = Kt;
                s_max[1][wid] = Kd;
                s_sum[0][wid] = dt;
                s_sum[1][wid] = dd;
            }
        }
        if (tid == 0) s_tok = -1;
        __syncthreads();
        Kt = s_max[0][0];
        Kd = s_max[1][0];
#pragma unroll
        for (int w = 1; w < NW; ++w) {
            Kt = fmaxf(Kt, s_max[0][w]);
            Kd = fmaxf(Kd, s_max[1][w]);
        }
        double St = 0.0, Sd = 0.0;
        for (int w = 0; w < NW; ++w) {
            St += rescale(s_sum[0][w], s_max[0][w], Kt);
            Sd += rescale(s_sum[1][w], s_max[1][w], Kd);
        }
        // A row without finite logits, or with a NaN logit (its sum is NaN),
        // cannot be tested or drawn from.
        const bool bad = !(Kt > kNegInf && Kt < -kNegInf) || !usable_sum(St) ||
                         (!bonus && (!(Kd > kNegInf && Kd < -kNegInf) || !usable_sum(Sd)));
        if (bad) {
            if (wid == 0) publish(a, b, i, kb, make_rec(kRecBadRow, 0));
            return;
        }

        // Wave 0 decides whether this workgroup draws a token.
        if (wid == 0) {
            int flag = 1;
            if (!bonus) {
                asm volatile("" : "+v"(ty_raw), "+v"(dy_raw));  // converted here, not at the load
                const double ratio =
                    acceptance_ratio(Fmt::from_raw(ty_raw), Fmt::from_raw(dy_raw), Kt, St, Kd, Sd, a.c2d);
                const double u = a.u_accept[int64_t(b) * K + i];
                if (u < ratio) {
                    flag = 0;
                    publish(a, b, i, kb, make_rec(kRecAccept, 0));
                } else {
                    // Announce the rejection, then find out whether it is the
                    // first one of the sequence.
                    if (lane == 0) announce_reject(a, b, i);
                    if (i > 0 && poll_earlier(a, b, i, kMaxPolls) == 2) {
                        flag = 0;
                        publish(a, b, i, kb, make_rec(kRecRejectSkipped, 0));
                    }
                }
            } else if (poll_earlier(a, b, i, kMaxPolls) == 2) {
                flag = 0;
                publish(a, b, i, kb, make_rec(kRecBonusSkipped, 0));
            }
            if (lane == 0) s_flag = flag;
        }
        __syncthreads();
        if (s_flag == 0) return;

        // Draw the extra token: from max(0, p - q) after a rejection, from p
        // at the bonus row (and, should max(0, p - q) have no mass after
        // rounding, from p as well).  Masses are in units of S_t:
        //   p_j S_t = 2^(t_j c2 - K_t),  q_j S_t = 2^(d_j c2 - K_d) (S_t / S_d).
        const float rho = bonus ? 0.0f : float(St / Sd);
        const float u = a.u_resample[b];
        bool use_p = bonus;
        for (int attempt = 0; attempt < 2; ++attempt) {
            // Opaque copies of the shifts, fresh in each attempt: without them
            // the compiler may keep exponentials alive across passes (to reuse
            // them) and spill.
            float mtc_d = Kt, mdc_d = Kd;
            asm volatile("" : "+v"(mtc_d), "+v"(mdc_d));
            opaque(tv);
            if (!use_p) opaque(dv);
            const bool p_only = use_p;
            auto mass = [=](const chunk_t& tc, const chunk_t& dc, int e) -> float {
                const float pt = exp2_fast(__builtin_fmaf(Fmt::get(tc, e), c2, -mtc_d));
                if (p_only) return pt;
                const float qt = exp2_fast(__builtin_fmaf(Fmt::get(dc, e), c2, -mdc_d));
                return fmaxf(__builtin_fmaf(-qt, rho, pt), 0.0f);
            };
            bool z_zero = false;
            const int at = draw_inverse_cdf<kFixedShift, W, CPT, EPC>(tv, dv, mass, u, s_tot, &s_draw, s_stage, &z_zero);
            if (at >= 0) s_tok = VEC ? cut.token(at) : at;
            if (!z_zero || use_p) break;
            use_p = true;
        }
        __syncthreads();
        if (wid == 0) {
            const int tok = s_tok;
            uint32_t r;
            if (tok >= 0)
                r = make_rec(bonus ? kRecBonus : kRecReject, uint32_t(tok));
            else
                r = make_rec(kRecBadRow, 0);  // no mass anywhere
            publish(a, b, i, kb, r);
        }
    }
}

// Rows too long to hold, and more of them than one per CU (verify_stream_kernel):
// the same per-row protocol as verify_kernel, with the rows streamed.  The
// statistics take one pass over the row pair, kUnroll rounds of loads in flight
// per thread; the workgroup that draws streams the row pair again (pass A of
// draw_inverse_cdf_streamed) and its winning wave reloads one round (pass B).
// Nothing but (K, S) is held across passes, so eight waves per SIMD hide the
// loads: 2304 rows of V = 50304 bf16 118.7 -> 95.6 us (held, 1024 threads x 8 chunks,
// 124 VGPRs, before); 256 sequences of V = 128256, ragged, 159 -> 152 us.
constexpr int kUnroll = 4;
constexpr int kStreamW = 512;
// Looks at the earlier positions before a draw that reads the rows again.
constexpr int kMaxStreamPolls = 24;

template <typename Fmt, int W>
__global__ __launch_bounds__(W, 1) void verify_stream_kernel(VerifyArgs a) {
    constexpr int NW = W / kWave, EPC = Fmt::kPerChunk, U = kUnroll;
    __shared__ float s_max[2][NW];
    __shared__ double s_sum[2][NW];
    __shared__ int s_flag;
    __shared__ int s_tok;
    __shared__ unsigned long long s_tot[kMaxStreamCells];
    __shared__ DrawShared s_draw;

    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const int B = a.B, K = a.K, V = a.V;
    const bool bonus = int(blockIdx.x) >= B * K;
    int b, i;
    if (!bonus) {
        i = blockIdx.x / B;
        b = blockIdx.x - i * B;
    } else {
        b = blockIdx.x - B * K;
        i = -1;
    }
    const int kb = a.draft_len ? a.draft_len[b] : K;
    if (kb < 1 || kb > K) {
        if (bonus) write_invalid(a, b);
        return;
    }
    if (bonus) {
        i = kb;
    } else if (i >= kb) {
        return;
    }
    const int y = bonus ? 0 : a.tokens[int64_t(b) * K + i];
    if (!bonus && (y < 0 || y >= V)) {
        if (wid == 0) publish(a, b, i, kb, make_rec(kRecBadToken, 0));
        return;
    }
    if (bonus) {
        if (wid == 0) {
            const int st = poll_earlier(a, b, i, 1);
            if (lane == 0) s_flag = st;
            if (st == 2) publish(a, b, i, kb, make_rec(kRecBonusSkipped, 0));
        }
        __syncthreads();
        if (s_flag == 2) return;
    }
    const char* trow = static_cast<const char*>(a.target) + (int64_t(b) * (K + 1) + i) * int64_t(V) * Fmt::kBytes;
    const char* drow =
        bonus ? trow : static_cast<const char*>(a.draft) + (int64_t(b) * K + i) * int64_t(V) * Fmt::kBytes;
    uint32_t ty_raw = 0u, dy_raw = 0u;
    if (!bonus) {
        ty_raw = Fmt::load_raw(trow, y);
        dy_raw = Fmt::load_raw(drow, y);
    }
    const float c2 = a.c2;
    const RowCut<Fmt> cut(V);
    const int R = (cut.nchunks + W - 1) / W;

    // Statistics, U rounds of loads at a time.
    float Kt = kNegInf, Kd = kNegInf, st = 0.0f, sd = 0.0f;
    for (int r0 = 0; r0 < R; r0 += U) {
        chunk_t xt[U], xd[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int off = cut.off((r0 + u) * W + tid);
            xt[u] = load_off(trow, off);
            if (!bonus) xd[u] = load_off(drow, off);
        }
        pad_shared_head<Fmt, W, U>(xt, cut, r0);
        if (!bonus) pad_shared_head<Fmt, W, U>(xd, cut, r0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            fold_chunk<Fmt>(chunk_or_pad<Fmt, W>(xt[u], r0 + u, cut), c2, Kt, st);
            if (!bonus) fold_chunk<Fmt>(chunk_or_pad<Fmt, W>(xd[u], r0 + u, cut), c2, Kd, sd);
        }
    }
    {
        double dt = st, dd = sd;
        wave_merge_stats(Kt, dt);
        wave_merge_stats(Kd, dd);
        if (lane == 0) {
            s_max[0][wid] = Kt;
            s_max[1][wid] = Kd;
            s_sum[0][wid] = dt;
            s_sum[1][wid] = dd;
        }
    }
    if (tid == 0) s_tok = -1;
    __syncthreads();
    Kt = s_max[0][0];
    Kd = s_max[1][0];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
        Kt = fmaxf(Kt, s_max[0][w]);
        Kd = fmaxf(Kd, s_max[1][w]);
    }
    double St = 0.0, Sd = 0.0;
    for (int w = 0; w < NW; ++w) {
        St += rescale(s_sum[0][w], s_max[0][w], Kt);
        Sd += rescale(s_sum[1][w], s_max[1][w], Kd);
    }
    const bool bad = !(Kt > kNegInf && Kt < -kNegInf) || !usable_sum(St) ||
                     (!bonus && (!(Kd > kNegInf && Kd < -kNegInf) || !usable_sum(Sd)));
    if (bad) {
        if (wid == 0) publish(a, b, i, kb, make_rec(kRecBadRow, 0));
        return;
    }
    // Wave 0 decides whether this workgroup draws (as verify_kernel).
    if (wid == 0) {
        int flag = 1;
        if (!bonus) {
            const double ratio =
                acceptance_ratio(Fmt::from_raw(ty_raw), Fmt::from_raw(dy_raw), Kt, St, Kd, Sd, a.c2d);
            const double u = a.u_accept[int64_t(b) * K + i];
            if (u < ratio) {
                flag = 0;
                publish(a, b, i, kb, make_rec(kRecAccept, 0));
            } else {
                if (lane == 0) announce_reject(a, b, i);
                if (i > 0 && poll_earlier(a, b, i, kMaxStreamPolls) == 2) {
                    flag = 0;
                    publish(a, b, i, kb, make_rec(kRecRejectSkipped, 0));
                }
            }
        } else if (poll_earlier(a, b, i, kMaxStreamPolls) == 2) {
            flag = 0;
            publish(a, b, i, kb, make_rec(kRecBonusSkipped, 0));
        }
        if (lane == 0) s_flag = flag;
    }
    __syncthreads();
    if (s_flag == 0) return;

    // The draw, the masses of verify_kernel on the streamed chunks.
    const float rho = bonus ? 0.0f : float(St / Sd);
    const float u = a.u_resample[b];
    bool use_p = bonus;
    for (int attempt = 0; attempt < 2; ++attempt) {
        const bool p_only = use_p;
        const float kt = Kt, kd = Kd;
        const auto mass = [=](const chunk_t& tc, const chunk_t& dc, int e) -> float {
            const float pt = exp2_fast(__builtin_fmaf(Fmt::get(tc, e), c2, -kt));
            if (p_only) return pt;
            const float qt = exp2_fast(__builtin_fmaf(Fmt::get(dc, e), c2, -kd));
            return fmaxf(__builtin_fmaf(-qt, rho, pt), 0.0f);
        };
        bool z_zero = false;
        const int at = draw_inverse_cdf_streamed<kFixedShift, Fmt, W, U>(trow, drow, !p_only, cut, mass, u, s_tot, &s_draw,
                                                                        &z_zero);
        if (at >= 0) s_tok = cut.token(at);
        if (!z_zero || use_p) break;
        use_p = true;
        __syncthreads();  // s_tot and s_draw are reused
    }
    __syncthreads();
    if (wid == 0) {
        const int tok = s_tok;
        publish(a, b, i, kb, tok >= 0 ? make_rec(bonus ? kRecBonus : kRecReject, uint32_t(tok)) : make_rec(kRecBadRow, 0));
    }
}

// ---------------------------------------------------------------------------
// Rows split over workgroups (verify_split_kernel): rows longer than the
// resident tiles, and few rows, where one workgroup per row would leave most of
// the chip idle.  Each row (pair) is cut into at most kMaxSplit segments of
// W * CPT chunks; the workgroup of a segment holds it in registers.
//   1. It folds its (K, S) pairs and publishes them, reads its siblings' and
//      merges all in segment order, so every segment has the same normalisers,
//      bit for bit, and takes the same decision.
//   2. An accepted row is reported by segment 0.  A rejected one (or a bonus
//      row) draws: each segment publishes the fixed-point mass of its part,
//      reads its siblings', and the one whose part holds the point walks to the
//      token and reports the row.  A row without residual mass after rounding
//      repeats this with the masses of p.
// A rejecting row does not ask whether an earlier position rejected as well: its
// segments would have to agree on what they saw, which costs as much as the
// draw from registers.  The finalizer takes the first rejection's token.  A
// bonus row is skipped if an earlier rejection is on record when its first
// segment looks (the segments agree through one compare-and-swap).
// Published words are never zero, so a reader polls the words themselves; a wait
// is bounded (kSplitPolls polls, or the value of OSD_VERIFY_POLLS), and a
// workgroup that runs out computes the missing records itself from the rows in
// memory, bit for bit as their owners do.  Each segment arrives at its row's
// counter once it has read all it needs; the last one clears the row's words.
//
// One workgroup per row before: B = 1, K = 4, V = 32000 bf16 13.5 -> 10.4 us (a chain
// of memory latencies and barriers, not bandwidth, bounds these calls), B = 8,
// K = 5 14.5 -> 11.8; B = 1, V = 128256 46.1 -> 13.0, B = 16 49.2 -> 20.6.
// ---------------------------------------------------------------------------
constexpr int kMaxSplit = 8;
constexpr int kSplitPolls = 256;

// A row's words in the workspace (VerifyRow::words).
struct SplitRow {
    uint64_t stats[kMaxSplit][3];  // ~S_t, ~S_d, ~(K_t | K_d << 32) (bits)
    uint64_t mass[2][kMaxSplit];   // 2^63 | mass: of the residual, of p
    uint32_t arrivals;
    uint32_t bonus;                // a bonus row: 1 read it, 2 skip it
};
static_assert(sizeof(SplitRow) == sizeof(VerifyRow::words), "the row's words");

struct SplitVerifyArgs {
    VerifyArgs v;
    int nseg;
    int polls;
};

template <int NW, int CPT>
struct SplitShared {
    float k[2 * NW];
    double s[2 * NW];
    float rk[kMaxSplit][2];    // the row's records, by segment
    double rs[kMaxSplit][2];
    float kt, kd;              // merged
    double st, sd;
    uint64_t rz[kMaxSplit];    // the row's masses, by segment
    unsigned long long tot[CPT * NW];
    DrawShared draw;
    // One flag per use: a wave may still be reading one when wave 0 writes the next.
    int skip, stats_ok, mass_ok, decision, tok;
};

// The segment's (K, S) pairs of both rows into slot `slot` (by thread 0).
template <typename Fmt, int W, int CPT, int NW>
__device__ inline void split_stats(chunk_t (&tv)[CPT], chunk_t (&dv)[CPT], float c2, bool second,
                                   SplitShared<NW, CPT>& sh, int slot) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    float Kt = kNegInf, Kd = kNegInf, ft = 0.0f, fd = 0.0f;
#pragma unroll
    for (int n = 0; n < CPT; ++n) {
        fold_chunk<Fmt>(tv[n], c2, Kt, ft);
        if (second) fold_chunk<Fmt>(dv[n], c2, Kd, fd);
        __builtin_amdgcn_sched_barrier(0);
    }
    double st = ft, sd = fd;
    wave_merge_stats_u(Kt, st);
    wave_merge_stats_u(Kd, sd);
    __syncthreads();  // sh.k and sh.s are reused
    if (lane == 0) {
        sh.k[wid] = Kt;
        sh.k[NW + wid] = Kd;
        sh.s[wid] = st;
        sh.s[NW + wid] = sd;
    }
    __syncthreads();
    if (wid == 0) {
        const bool in = lane < NW;
        float k0 = in ? sh.k[lane] : kNegInf, k1 = in ? sh.k[NW + lane] : kNegInf;
        double s0 = in ? sh.s[lane] : 0.0, s1 = in ? sh.s[NW + lane] : 0.0;
        row0_merge_stats_u(k0, s0);
        row0_merge_stats_u(k1, s1);
        if (lane == 0) {
            sh.rk[slot][0] = k0;
            sh.rk[slot][1] = k1;
            sh.rs[slot][0] = s0;
            sh.rs[slot][1] = s1;
        }
    }
}

// The segment's cell masses into sh.tot and their sum into sh.rz[slot] (wave 0).
template <typename Fmt, int W, int CPT, int NW, typename MassFn>
__device__ inline void split_mass(const chunk_t (&tv)[CPT], const chunk_t (&dv)[CPT], MassFn mass,
                                  SplitShared<NW, CPT>& sh, int slot) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    __syncthreads();  // sh.tot is reused
#pragma unroll
    for (int n = 0; n < CPT; ++n) {
        float s = 0.0f;
#pragma unroll
        for (int e = 0; e < Fmt::kPerChunk; ++e) s = s + mass(tv[n], dv[n], e);
        const double t = wave_sum(fixed_f64<kFixedShift>(s));
        if (lane == 0) sh.tot[n * NW + wid] = uint64_t(t);
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    if (wid == 0) {
        const uint64_t z = wave_sum(lane < CPT * NW ? uint64_t(sh.tot[lane]) : uint64_t(0));
        if (lane == 0) sh.rz[slot] = z;
    }
}

// Wave 0: lane j < nseg, j != s, reads words[j * WORDS ..] until every one is
// there or the polls run out; true if they are.
template <int WORDS>
__device__ inline bool poll_siblings(const uint64_t* words, int nseg, int s, int polls, uint64_t (&w)[WORDS]) {
    const int lane = threadIdx.x & (kWave - 1);
    const bool mine = lane < nseg && lane != s;
    for (int p = 0; p < polls; ++p) {
        if (p > 0) __builtin_amdgcn_s_sleep(2);
        bool ready = true;
        if (mine) {
#pragma unroll
            for (int k = 0; k < WORDS; ++k) {
                w[k] = poll_u64(words + lane * WORDS + k);
                ready = ready && w[k] != 0;
            }
        }
        if (__ballot(!ready) == 0) return true;
    }
    return false;
}

__device__ inline void store_word(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename Fmt, int W, int CPT>
__device__ inline void split_load(chunk_t (&tv)[CPT], chunk_t (&dv)[CPT], const char* trow, const char* drow, bool second,
                                  int s, int V) {
    asm volatile("" : "+s"(V), "+s"(s));  // nothing derived from them is hoisted out of a loop over segments
    const RowCut<Fmt> cut(V);
    const int tid = opaque_tid();
#pragma unroll
    for (int n = 0; n < CPT; ++n) {
        const int off = cut.off((s * CPT + n) * W + tid);
        tv[n] = load_off(trow, off);
        if (second) dv[n] = load_off(drow, off);
    }
}
template <typename Fmt, int W, int CPT>
__device__ inline void split_pad(chunk_t (&tv)[CPT], chunk_t (&dv)[CPT], bool second, int s, int V) {
    asm volatile("" : "+s"(V), "+s"(s));
    const RowCut<Fmt> cut(V);
    pad_row_tail<Fmt, W, CPT>(tv, cut, s * CPT);
    if (second) pad_row_tail<Fmt, W, CPT>(dv, cut, s * CPT);
}

template <typename Fmt, int W, int CPT>
__global__ __launch_bounds__(W, Fmt::kPerChunk == 8 ? 6 : 5) void verify_split_kernel(SplitVerifyArgs sa) {
    constexpr int NW = W / kWave, EPC = Fmt::kPerChunk;
    static_assert(CPT * NW <= kWave, "one wave sums the cells");
    __shared__ SplitShared<NW, CPT> sh;
    const VerifyArgs& a = sa.v;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const int B = a.B, K = a.K, V = a.V, nseg = sa.nseg;
    const int r = blockIdx.x / nseg, s = blockIdx.x - r * nseg;
    const bool bonus = r >= B * K;
    int i = bonus ? -1 : r / B;
    const int b = bonus ? r - B * K : r - i * B;
    const int kb = a.draft_len ? a.draft_len[b] : K;
    if (kb < 1 || kb > K) {
        if (bonus && s == 0) write_invalid(a, b);
        return;
    }
    if (bonus)
        i = kb;
    else if (i >= kb)
        return;  // padding row of a short proposal
    const int y = bonus ? 0 : a.tokens[int64_t(b) * K + i];
    if (!bonus && (y < 0 || y >= V)) {
        if (s == 0 && wid == 0) publish(a, b, i, kb, make_rec(kRecBadToken, 0));
        return;
    }
    SplitRow* const row = reinterpret_cast<SplitRow*>(a.rows[int64_t(b) * (K + 1) + i].words);
    if (bonus) {
        // The first segment to look decides for all of them.
        if (wid == 0) {
            const uint32_t want = poll_earlier(a, b, i, 1) == 2 ? 2u : 1u;
            uint32_t seen = 0u;
            if (lane == 0) {
                __hip_atomic_compare_exchange_strong(&row->bonus, &seen, want, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
                sh.skip = (seen != 0u ? seen : want) == 2u;
            }
        }
        __syncthreads();
        if (sh.skip) {
            if (wid == 0) {
                uint32_t prev = 0;
                if (lane == 0)
                    prev = __hip_atomic_fetch_add(&row->arrivals, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (lane == 0 && prev == uint32_t(nseg - 1)) {  // every segment has taken the decision
                    __hip_atomic_store(&row->bonus, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(&row->arrivals, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                if (s == 0) publish(a, b, i, kb, make_rec(kRecBonusSkipped, 0));
            }
            return;
        }
    }
    const bool pair = !bonus;
    const char* trow = static_cast<const char*>(a.target) + (int64_t(b) * (K + 1) + i) * int64_t(V) * Fmt::kBytes;
    const char* drow =
        bonus ? trow : static_cast<const char*>(a.draft) + (int64_t(b) * K + i) * int64_t(V) * Fmt::kBytes;
    const float c2 = a.c2;
    // The test's and the draw's scalars, requested before the rows.
    const uint32_t ty_raw = Fmt::load_raw(trow, y), dy_raw = Fmt::load_raw(drow, y);
    const float u_acc = bonus ? 0.0f : a.u_accept[int64_t(b) * K + i], u_res = a.u_resample[b];
    chunk_t tv[CPT], dv[CPT];
    split_load<Fmt, W, CPT>(tv, dv, trow, drow, pair, s, V);
    split_pad<Fmt, W, CPT>(tv, dv, pair, s, V);

    // 1. statistics
    split_stats<Fmt, W, CPT, NW>(tv, dv, c2, pair, sh, s);
    if (wid == 0) {
        if (lane == 0) {
            store_word(&row->stats[s][0], ~uint64_t(__double_as_longlong(sh.rs[s][0])));
            store_word(&row->stats[s][1], ~uint64_t(__double_as_longlong(sh.rs[s][1])));
            store_word(&row->stats[s][2], ~(uint64_t(__float_as_uint(sh.rk[s][0])) |
                                            (uint64_t(__float_as_uint(sh.rk[s][1])) << 32)));
        }
        uint64_t w[3] = {0, 0, 0};
        const bool ok = poll_siblings<3>(&row->stats[0][0], nseg, s, sa.polls, w);
        if (ok && lane < nseg && lane != s) {
            sh.rs[lane][0] = __longlong_as_double(~w[0]);
            sh.rs[lane][1] = __longlong_as_double(~w[1]);
            sh.rk[lane][0] = __uint_as_float(uint32_t(~w[2]));
            sh.rk[lane][1] = __uint_as_float(uint32_t(~w[2] >> 32));
        }
        if (lane == 0) sh.stats_ok = ok;
    }
    __syncthreads();
    if (!sh.stats_ok) {  // out of polls: every other segment's record from memory, then this segment again
#pragma unroll 1
        for (int j = 0; j < nseg; ++j) {
            if (j == s) continue;
            split_load<Fmt, W, CPT>(tv, dv, trow, drow, pair, j, V);
            split_pad<Fmt, W, CPT>(tv, dv, pair, j, V);
            split_stats<Fmt, W, CPT, NW>(tv, dv, c2, pair, sh, j);
        }
        split_load<Fmt, W, CPT>(tv, dv, trow, drow, pair, s, V);
        split_pad<Fmt, W, CPT>(tv, dv, pair, s, V);
    }
    // The decision, the same in every segment.
    if (wid == 0) {
        const bool in = lane < nseg;
        float Kt = in ? sh.rk[lane][0] : kNegInf, Kd = in ? sh.rk[lane][1] : kNegInf;
        double St = in ? sh.rs[lane][0] : 0.0, Sd = in ? sh.rs[lane][1] : 0.0;
        row0_merge_stats_u(Kt, St);
        row0_merge_stats_u(Kd, Sd);
        const bool bad = !(Kt > kNegInf && Kt < -kNegInf) || !usable_sum(St) ||
                         (pair && (!(Kd > kNegInf && Kd < -kNegInf) || !usable_sum(Sd)));
        const bool accept = !bad && pair &&
                            double(u_acc) < acceptance_ratio(Fmt::from_raw(ty_raw), Fmt::from_raw(dy_raw), Kt, St, Kd, Sd, a.c2d);
        if (lane == 0) {
            sh.kt = Kt;
            sh.kd = Kd;
            sh.st = St;
            sh.sd = Sd;
            sh.decision = bad ? 0 : (accept ? 1 : 2);
            sh.tok = -1;
        }
        if (s == 0 && (bad || accept)) publish(a, b, i, kb, make_rec(bad ? kRecBadRow : kRecAccept, 0));
    }
    __syncthreads();
    const bool draws = sh.decision == 2;
    const float Kt = sh.kt, Kd = sh.kd;
    const float rho = bonus ? 0.0f : float(sh.st / sh.sd);

    // 2. the extra token: masses in units of S_t, as verify_kernel's.
    int attempt = bonus ? 1 : 0;  // 0: max(0, p - q), 1: p
    bool mine = false;
    uint32_t rec = 0u;
    while (draws) {
        float mtc = Kt, mdc = Kd;
        asm volatile("" : "+v"(mtc), "+v"(mdc));  // the exponentials are taken afresh (bounded VGPRs)
        opaque(tv);
        const bool p_only = attempt == 1;
        if (!p_only) opaque(dv);
        const auto mass = [=](const chunk_t& tc, const chunk_t& dc, int e) -> float {
            const float pt = exp2_fast(__builtin_fmaf(Fmt::get(tc, e), c2, -mtc));
            if (p_only) return pt;
            const float qt = exp2_fast(__builtin_fmaf(Fmt::get(dc, e), c2, -mdc));
            return fmaxf(__builtin_fmaf(-qt, rho, pt), 0.0f);
        };
        split_mass<Fmt, W, CPT, NW>(tv, dv, mass, sh, s);
        if (wid == 0) {
            if (lane == 0) store_word(&row->mass[attempt][s], (1ull << 63) | sh.rz[s]);
            uint64_t w[1] = {0};
            const bool ok = poll_siblings<1>(row->mass[attempt], nseg, s, sa.polls, w);
            if (ok && lane < nseg && lane != s) sh.rz[lane] = w[0] & ~(1ull << 63);
            if (lane == 0) sh.mass_ok = ok;
        }
        __syncthreads();
        if (!sh.mass_ok) {
#pragma unroll 1
            for (int j = 0; j < nseg; ++j) {
                if (j == s) continue;
                split_load<Fmt, W, CPT>(tv, dv, trow, drow, pair, j, V);
                split_pad<Fmt, W, CPT>(tv, dv, pair, j, V);
                split_mass<Fmt, W, CPT, NW>(tv, dv, mass, sh, j);
            }
            split_load<Fmt, W, CPT>(tv, dv, trow, drow, pair, s, V);
            split_pad<Fmt, W, CPT>(tv, dv, pair, s, V);
            split_mass<Fmt, W, CPT, NW>(tv, dv, mass, sh, s);
            __syncthreads();
        }
        // The point in the whole row's CDF, exact, the same in every segment.
        uint64_t Z = 0, lo = 0;
        for (int j = 0; j < nseg; ++j) {
            const uint64_t z = sh.rz[j];
            if (j < s) lo += z;
            Z += z;
        }
        if (Z == 0) {
            if (!p_only) {  // no residual mass after rounding: from p
                attempt = 1;
                continue;
            }
            mine = s == 0;
            rec = make_rec(kRecBadRow, 0);
            break;
        }
        uint64_t c = static_cast<uint64_t>(double(u_res) * double(Z));
        if (c >= Z) c = Z - 1;
        if (c < lo || c - lo >= sh.rz[s]) break;  // another segment holds it
        mine = true;
        locate_cell<NW>(CPT * NW, sh.tot, 0.0f, static_cast<long long>(c - lo), &sh.draw);
        const int nstar = sh.draw.cell_round;
        if (wid == sh.draw.cell_wave) {
            chunk_t tc = tv[0], dc = dv[0];
#pragma unroll
            for (int n = 1; n < CPT; ++n)
                if (n == nstar) {
                    tc = tv[n];
                    dc = dv[n];
                }
            float m[EPC], sum = 0.0f;
#pragma unroll
            for (int e = 0; e < EPC; ++e) {
                m[e] = mass(tc, dc, e);
                sum = sum + m[e];
            }
            const int at = walk_chunk<kFixedShift, W, EPC>(m, sum, sh.draw.target, s * CPT + nstar);
            if (at >= 0) sh.tok = RowCut<Fmt>(V).token(at);
        }
        __syncthreads();
        rec = sh.tok >= 0 ? make_rec(bonus ? kRecBonus : kRecReject, uint32_t(sh.tok)) : make_rec(kRecBadRow, 0);
        break;
    }
    // This segment has read all it needs; the last one clears the row's words.
    if (wid == 0) {
        uint32_t prev = 0;
        if (lane == 0) {
            wait_memory();  // its own words are in place before they may be cleared
            prev = __hip_atomic_fetch_add(&row->arrivals, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (mine) publish(a, b, i, kb, rec);
        if (__builtin_amdgcn_readfirstlane(int(prev)) == nseg - 1) {
            uint64_t* words = reinterpret_cast<uint64_t*>(row);
            if (lane < int(sizeof(SplitRow) / 8)) store_word(words + lane, 0ull);
        }
    }
}

template <typename Fmt, int W, int CPT>
hipError_t launch_tile(const VerifyLaunch& L, const VerifyArgs& a) {
    const dim3 grid(unsigned(L.B) * unsigned(L.K + 1)), block(W);
    return launch_kernel(&verify_kernel<Fmt, W, CPT, true, false>, grid, block, 0, L.stream, a);
}

// kSplitPolls, or the value of OSD_VERIFY_POLLS (read once; 0 makes every
// workgroup compute its siblings' records itself).
int verify_polls() {
    static const int v = [] {
        const char* e = getenv("OSD_VERIFY_POLLS");
        if (e == nullptr || *e == 0) return kSplitPolls;
        const int k = atoi(e);
        return k < 0 ? kSplitPolls : (k > 65536 ? 65536 : k);
    }();
    return v;
}

template <typename Fmt, int W, int CPT>
hipError_t launch_split(const VerifyLaunch& L, const VerifyArgs& a, int nchunks) {
    SplitVerifyArgs sa;
    sa.v = a;
    sa.nseg = (nchunks + W * CPT - 1) / (W * CPT);
    sa.polls = verify_polls();
    const int64_t grid = int64_t(L.B) * (L.K + 1) * sa.nseg;
    if (grid > 0x7FFFFFFFll) return hipErrorInvalidValue;
    return launch_kernel(&verify_split_kernel<Fmt, W, CPT>, dim3(unsigned(grid)), dim3(W), 0, L.stream, sa);
}

template <typename Fmt>
hipError_t launch_fmt(const VerifyLaunch& L, const VerifyArgs& a) {
    const dim3 grid(unsigned(L.B) * unsigned(L.K + 1));
    if (L.V < Fmt::kPerChunk) {  // rows shorter than one chunk, element by element
        return L.temperature == 0.0f
                   ? launch_kernel(&verify_kernel<Fmt, 256, 1, false, true>, grid, dim3(256), 0, L.stream, a)
                   : launch_kernel(&verify_kernel<Fmt, 256, 1, false, false>, grid, dim3(256), 0, L.stream, a);
    }
    if (!(L.temperature > 0.0f)) return hipErrorInvalidValue;  // the segmented greedy kernels take these
    if (L.V > max_vocab_for(Fmt::kPerChunk)) return hipErrorInvalidValue;
    const int nchunks = (L.V + Fmt::kPerChunk - 1) / Fmt::kPerChunk;
    const int64_t rows = int64_t(L.B) * (L.K + 1);
    const bool resident = nchunks <= 512 * 8;
    // Few rows are split: up to one per CU beyond the resident tiles (split and whole: 224
    // rows of V = 50257 bf16 22.7 and 30.1 us, 576 rows of V = 50304 38.8 and 37.4, 100 rows
    // of V = 128256 23.1 and 48.3).  In bf16, one per two CUs where 4 to 8 chunks per thread
    // would be held (128 rows of V = 32000 14.5 and 14.9, 216 rows 18.5 and 15.5), one per
    // eight CUs for 2 to 4 (30 rows of V = 9000 9.9 and 10.4, 125 rows 11.6 and 10.6).  A
    // chunk of fp32 is half the work, so less is gained: one per four CUs for 4 to 8 (60
    // rows of V = 16000 11.2 and 12.0, 125 rows 13.4 and 12.1), none for fewer (5 rows of
    // V = 5000 9.0 and 8.2).
    constexpr bool wide = Fmt::kPerChunk == 8;
    const int most = !resident ? L.cus : nchunks > 2048 ? L.cus / (wide ? 2 : 4) : wide && nchunks > 1024 ? L.cus / 8 : 0;
    if (rows <= most) {
        if constexpr (wide)
            if (nchunks <= kMaxSplit * 256) return launch_split<Fmt, 256, 1>(L, a, nchunks);
        if (nchunks <= kMaxSplit * 512) return launch_split<Fmt, 256, 2>(L, a, nchunks);
        if (nchunks <= kMaxSplit * 1024) return launch_split<Fmt, 256, 4>(L, a, nchunks);
        return launch_split<Fmt, 512, 4>(L, a, nchunks);
    }
    if (!resident) return launch_kernel(&verify_stream_kernel<Fmt, kStreamW>, grid, dim3(kStreamW), 0, L.stream, a);
    RowTile t;
    if (!pick_tile(L.V, Fmt::kPerChunk, &t)) return hipErrorInvalidValue;
    switch (t.W * 100 + t.CPT) {
        case 25601: return launch_tile<Fmt, 256, 1>(L, a);
        case 25602: return launch_tile<Fmt, 256, 2>(L, a);
        case 25604: return launch_tile<Fmt, 256, 4>(L, a);
        case 51204: return launch_tile<Fmt, 512, 4>(L, a);
        case 51208: return launch_tile<Fmt, 512, 8>(L, a);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

// The largest row every entry point takes: 16 rounds of 1024 threads
// (131072 bf16 or 65536 fp32 logits); the streamed kernels' cell tables are
// sized for it.
int max_vocab_for(int per_chunk) { return 1024 * kMaxStreamRounds * per_chunk; }

// Register-resident tiles (a row pair in registers, at most 8 chunks per
// thread); longer rows are streamed.
bool pick_tile(int V, int per_chunk, RowTile* t) {
    static const RowTile tiles[] = {{256, 1}, {256, 2}, {256, 4}, {512, 4},
                                    {512, 8}, {1024, 8}};
    for (const RowTile& c : tiles)
        if (int64_t(V) <= int64_t(c.W) * c.CPT * per_chunk) {
            *t = c;
            return true;
        }
    return false;
}

hipError_t launch_verify(const VerifyLaunch& L) {
    VerifyArgs a{};
    a.target = L.target;
    a.draft = L.draft;
    a.B = L.B;
    a.K = L.K;
    a.V = L.V;
    a.tokens = L.tokens;
    a.draft_len = L.draft_len;
    a.u_accept = L.u_accept;
    a.u_resample = L.u_resample;
    a.c2 = L.temperature > 0.0f ? float(1.4426950408889634 / double(L.temperature)) : 0.0f;
    a.c2d = double(a.c2);
    a.accepted_len = L.accepted_len;
    a.out_tokens = L.out_tokens;
    a.reject_mask = L.reject_mask;
    a.rows = L.rows;
    return L.dtype == 1 ? launch_fmt<BF16>(L, a) : launch_fmt<F32>(L, a);
}

}  // namespace osd
