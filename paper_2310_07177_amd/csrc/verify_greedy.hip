// verify_greedy.hip -- greedy verification (T = 0) on gfx950.
//
// Method: with T = 0 the target distribution is its argmax (lowest index on
// ties); proposal y_i is accepted while it equals the argmax of target row
// i, the first mismatch at position a ends the test (the exit of the
// acceptance loop in Appendix A.1), and the extra token is the argmax of row
// a, or of the bonus row k_b when every proposal matched.  Only target rows
// are read.
//
// Work layout: one flat grid of small workgroups, one per (target row, vocabulary
// segment of kW*4 chunks), so the hardware dispatcher balances the work over every
// CU whatever B and k are.  Each posts its segment's (max, lowest index) as one
// word and, once the word is in place, arrives at its sequence's counter; the
// last of a sequence to arrive merges the words of rows 0..k_b in segment order,
// finds the first mismatch, writes the outputs and clears words and counter.
// (The wait for the word costs 0.2 to 0.3 us: B = 1, K = 4, V = 32000 bf16 5.1 -> 5.4, B = 64,
// K = 8, V = 32128 9.6 -> 9.9.  The decision in a kernel of its own took the first of the
// two 0.5 us longer than the variant without the wait.  With the counters of all
// sequences side by side the larger batch took 22.1 us: see VerifyRow.)
#include "osd.h"
#include "osd_device.hpp"
#include "osd_internal.hpp"
#include "stream_device.hpp"

namespace osd {
namespace {

constexpr int kW = 256;          // threads per workgroup
constexpr int kNW = kW / kWave;  // waves per workgroup
// Workgroups per launch (grid sizes stay far below the 2^32 work-item limit).
constexpr int64_t kMaxGrid = int64_t(1) << 22;

struct SegArgs {
    const void* target;        // [B, K+1, V]
    int B, K, V;
    const int32_t* tokens;     // [B, K]
    const int32_t* draft_len;  // [B] or null
    int nseg;                  // segments per row
    int64_t first;             // first work unit of this launch
    VerifyRow* rows;           // [B*(K+1)], zero between calls
    int32_t* accepted_len;
    int32_t* out_tokens;
    uint8_t* reject_mask;
};

__device__ inline int seq_k(const SegArgs& a, int b) { return a.draft_len ? scalar_load(a.draft_len + b) : a.K; }

// Every argument word, requested together on entry: each dependent request
// would cost a round trip to the argument buffer (about a microsecond).
__device__ inline void request_args(const SegArgs& a) {
    asm volatile("" ::"s"(a.target), "s"(a.B), "s"(a.K), "s"(a.V), "s"(a.tokens), "s"(a.draft_len), "s"(a.nseg),
                 "s"(a.first), "s"(a.rows));
    asm volatile("" ::"s"(a.accepted_len), "s"(a.out_tokens), "s"(a.reject_mask));
}

// Outputs of sequence b, written by wave 0 (lane j handles position j; K < 64).
__device__ inline void write_outputs(const SegArgs& a, int b, int kb, int acc, bool bad, int extra) {
    const int lane = threadIdx.x & (kWave - 1);
    const int K = a.K;
    if (lane <= K) {
        int32_t o = -1;
        if (!bad) o = lane < acc ? a.tokens[int64_t(b) * K + lane] : (lane == acc ? extra : -1);
        a.out_tokens[int64_t(b) * (K + 1) + lane] = o;
        if (a.reject_mask && lane < K)
            a.reject_mask[int64_t(b) * K + lane] = (!bad && lane == acc && acc < kb) ? 1 : 0;
    }
    if (lane == 0) a.accepted_len[b] = bad ? -1 : acc;
}

// A segment's argmax as one word: larger for a larger value, then for a lower
// index; never zero (a segment without finite logits: -inf).  The keys order
// -0.0 below +0.0, which are equal logits, so either zero gets the key of +0.0.
__device__ inline uint64_t argmax_word(float v, int idx) {
    const uint32_t key = v == 0.0f ? 0x80000000u : float_key(v);
    return (uint64_t(key) << 32) | (0xFFFFFFFFu - uint32_t(idx));
}

template <typename Fmt, int CPT>
__global__ __launch_bounds__(kW) void verify_greedy_kernel(SegArgs a) {
    constexpr int EPC = Fmt::kPerChunk;
    __shared__ float s_k[kNW];
    __shared__ int s_i[kNW];
    __shared__ int s_last;
    __shared__ unsigned long long s_row[OSD_MAX_K + 1][kMaxSeg];

    request_args(a);
    const int tid = threadIdx.x;
    const int64_t unit = a.first + blockIdx.x;
    const int s = int(unit % a.nseg);
    const int64_t pair = unit / a.nseg;  // b*(K+1) + i
    const int b = int(pair / (a.K + 1));
    const int i = int(pair - int64_t(b) * (a.K + 1));
    const int kb = seq_k(a, b);
    if (kb < 1 || kb > a.K) {
        if (i == 0 && s == 0 && tid < kWave) write_outputs(a, b, kb, 0, true, -1);
        return;
    }
    if (i > kb) return;  // a padding row

    const char* trow = static_cast<const char*>(a.target) + pair * int64_t(a.V) * Fmt::kBytes;
    // Segment s holds rounds s*CPT .. s*CPT + CPT - 1 of the row.
    const RowCut<Fmt> cut(a.V);
    chunk_t xt[CPT];
#pragma unroll
    for (int n = 0; n < CPT; ++n) xt[n] = load_off(trow, cut.off((s * CPT + n) * kW + tid));
    pad_row_tail<Fmt, kW, CPT>(xt, cut, s * CPT);
    const int c0 = s * kW * CPT + tid;  // this thread's first chunk in the row
    // Within a thread indices grow with (n, e): a strict ">" keeps the first
    // maximum.
    float best = kNegInf;
    int bi = 0x7FFFFFFF;
#pragma unroll
    for (int n = 0; n < CPT; ++n)
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
            const float v = Fmt::get(xt[n], e);
            if (v > best) {
                best = v;
                bi = (c0 + n * kW) * EPC + e;
            }
        }
    const int lane = tid & (kWave - 1), wid = tid / kWave;
    wave_argmax_u(best, bi);
    if (lane == 0) {
        s_k[wid] = best;
        s_i[wid] = bi;
    }
    __syncthreads();
    if (tid == 0) {
        float bv = s_k[0];
        int bx = s_i[0];
        for (int w = 1; w < kNW; ++w)
            if (s_k[w] > bv || (s_k[w] == bv && s_i[w] < bx)) {
                bv = s_k[w];
                bx = s_i[w];
            }
        const uint64_t word = argmax_word(bv, bx == 0x7FFFFFFF ? bx : cut.token(bx));
        publish_u64(&a.rows[pair].words[s], word);
        const uint32_t prev = arrive(&a.rows[int64_t(b) * (a.K + 1)].arrivals);  // after the word
        s_last = prev == uint32_t((kb + 1) * a.nseg - 1);
    }
    __syncthreads();
    if (!s_last) return;

    // The sequence's last arriver: every word is in place; read and clear them.
    VerifyRow* rows = a.rows + int64_t(b) * (a.K + 1);
    for (int j = tid; j < (kb + 1) * a.nseg; j += kW) {
        const int r = j / a.nseg, q = j - r * a.nseg;
        s_row[r][q] = take_u64(&rows[r].words[q]);
    }
    if (tid == 0) __hip_atomic_store(&rows[0].arrivals, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (tid >= kWave) return;
    // Lane r: row r's argmax (lowest index on ties); accept while y_r equals it,
    // emit the argmax where the test stops.
    uint64_t w = 0;
    if (lane <= kb)
        for (int q = 0; q < a.nseg; ++q) {
            const uint64_t v = s_row[lane][q];
            if (v > w) w = v;
        }
    const float top = key_float(uint32_t(w >> 32));
    const int g = int(0xFFFFFFFFu - uint32_t(w));
    const bool bad_row = !(top > kNegInf && top < -kNegInf);
    const int y = lane < kb ? a.tokens[int64_t(b) * a.K + lane] : 0;
    const uint64_t tok_bad = __ballot(lane < kb && (y < 0 || y >= a.V));
    const uint64_t stop = __ballot(lane < kb && (bad_row || y != g));
    const int acc = stop ? __builtin_ctzll(stop) : kb;
    const uint64_t row_bad = __ballot(lane <= kb && bad_row);
    const bool bad = tok_bad != 0 || ((row_bad >> acc) & 1ull) != 0;
    write_outputs(a, b, kb, acc, bad, __shfl(g, acc, kWave));
}

template <typename Fmt>
hipError_t launch_fmt(const VerifyLaunch& L, SegArgs a) {
    if (!greedy_segments(L.V, Fmt::kPerChunk, &a.nseg)) return hipErrorInvalidValue;
    // Twice the chunks per thread beyond 8 segments (the sequence's arrivals
    // meet at one word).
    const auto kernel = a.nseg > 8 ? &verify_greedy_kernel<Fmt, 8> : &verify_greedy_kernel<Fmt, 4>;
    if (a.nseg > 8) a.nseg = (a.nseg + 1) / 2;
    const int64_t units = int64_t(a.B) * (a.K + 1) * a.nseg;
    for (int64_t f = 0; f < units; f += kMaxGrid) {
        a.first = f;
        const unsigned g = unsigned(units - f < kMaxGrid ? units - f : kMaxGrid);
        const hipError_t e = launch_kernel(kernel, dim3(g), dim3(kW), 0, L.stream, a);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

// Segments of a row of at least one chunk for greedy verification: kW threads
// x 4 chunks each (8192 bf16 or 4096 fp32 logits), at most kMaxSeg of them.
bool greedy_segments(int V, int per_chunk, int* nseg) {
    if (V < per_chunk) return false;
    const int64_t nchunks = (int64_t(V) + per_chunk - 1) / per_chunk;
    const int64_t n = (nchunks + int64_t(kW) * 4 - 1) / (int64_t(kW) * 4);
    if (n > kMaxSeg) return false;
    *nseg = int(n);
    return true;
}

hipError_t launch_verify_greedy(const VerifyLaunch& L) {
    SegArgs a{};
    a.target = L.target;
    a.B = L.B;
    a.K = L.K;
    a.V = L.V;
    a.tokens = L.tokens;
    a.draft_len = L.draft_len;
    a.first = 0;
    a.rows = L.rows;
    a.accepted_len = L.accepted_len;
    a.out_tokens = L.out_tokens;
    a.reject_mask = L.reject_mask;
    return L.dtype == 1 ? launch_fmt<BF16>(L, a) : launch_fmt<F32>(L, a);
}

}  // namespace osd
