// distill_stream.hip -- distillation divergence and its gradient with respect
// to the student logits on gfx950, streaming form (persistent workgroups)
// (Section 4.1, Eq. 2-4 of arXiv:2310.07177).
//
// For each row n = (b, i) with mask 1, with p = softmax(t / tau) (teacher) and
// q = softmax(s / tau) (student):
//   FKL  D = sum p (log p - log q)                  g = (q - p) / tau
//   RKL  D = sum q (log q - log p)                  g = q (log q - log p - D) / tau
//   JSD  D = beta KL(p || m) + (1-beta) KL(q || m)   g = (1-beta) q (log q - log m - KL(q || m)) / tau
//        with m = beta p + (1-beta) q
// and 0 log 0 = 0.  Rows with mask 0 get D = 0 and a zero gradient row.
//
// Work layout.  About one workgroup per CU walks rows g, g+G, ... or (LISTED),
// with a mask and more than two rows each, its equal share of the rows that are on
// (share_rows), each step loading the next of them; the zero gradient rows are
// written between the passes of a step.  (With every row g, g+G, ... whatever its
// mask, a workgroup's share of the rows that are on varied by a third and a row
// that was off left nothing in flight under the row before it: 16384 rows of
// V = 32000 bf16, 40 % on, JSD, took 459 us, now 374.)
// Each thread owns chunks n*W + tid of both rows.  The statistics pass
// consumes the raw chunks of row j while each register chunk is reloaded with
// the same chunk of row j+G; what the later passes need is kept per element in
// a cache of two floats (c0 in LDS, in thread-private float4 slots; c1 in
// registers), so the loss and gradient passes of row j run while row j+G is
// landing.  The statistics pass caches both exponents, (t c2 - K_t,
// s c2 - K_s), for every kind; the loss pass replaces them by
//   JSD  (log2 q - log2 m, 2^(s c2 - K_s))
//   FKL  (p, log2 q)
//   RKL  (log2 p - log2 q, q)
// (c2 = log2(e)/tau, K a whole number per thread and row).  The log-ratio of
// FKL and RKL is the difference of the two cached exponents less the
// difference of the normalisers (taken in fp64), so it carries no rounding
// of the (much larger) normalisers themselves.
//
// Each workgroup adds the D of its rows in fp64 in the order it takes them and posts the
// partial at the device-wide coherence point; the last workgroup to finish
// adds the partials in workgroup order, so the loss is reproducible for a
// given grid.
#include <algorithm>

#include "osd_device.hpp"
#include "osd_internal.hpp"
#include "stream_device.hpp"
#include "distill_common.hpp"

namespace osd {
namespace {

struct StreamDistillArgs {
    const void* teacher;
    int64_t tstride;
    const void* student;
    int64_t sstride;
    int B, K, V;
    const uint8_t* mask;
    float beta;
    float c2;       // log2(e) / tau
    float inv_tau;  // 1 / tau
    float* row_loss_out;
    void* grad_out;
    double* row_ws;     // [grid] per-workgroup loss partials, zero between calls
    uint32_t* done;     // workgroups finished, zero between calls
    float* loss_out;    // {masked mean, masked sum}
    int nrows;
    uint32_t row_bytes;
    int G;          // workgroups in the grid
    int slice, gs;  // rows and workgroups of a slice: shares are made inside a slice
};

struct Row {
    bool on;
    const char* trow;
    const char* srow;
};

// Row n (none if n < 0).
template <typename Fmt>
__device__ inline Row decode_row(const StreamDistillArgs& a, int n) {
    Row r;
    r.on = n >= 0;
    r.trow = nullptr;
    r.srow = nullptr;
    if (n < 0) return r;
    const int b = n / a.K, i = n - b * a.K;
    r.trow = static_cast<const char*>(a.teacher) + (int64_t(b) * a.tstride + int64_t(i) * a.V) * Fmt::kBytes;
    r.srow = static_cast<const char*>(a.student) + (int64_t(b) * a.sstride + int64_t(i) * a.V) * Fmt::kBytes;
    return r;
}

// The place of the n-th set bit.
__device__ inline int nth_bit(uint32_t bits, int n) {
    for (; n > 0; --n) bits &= bits - 1u;
    return __builtin_ctz(bits);
}

// A workgroup's share of its slice: rows that are on, rows that are off.
struct RowShare {
    int on, off;
};
// Rows of a slice per thread: one 16-byte load of mask flags.
constexpr int kFlags = 16;
// Places in a workgroup's list of rows (the launch keeps a share below W * 17 / 16 + 4).
template <int W>
constexpr int kShareMax = W + W / 8 + 8;

// Divides a slice of `rows` rows from row `base` among its G workgroups:
// those that are on round robin, and those that are off, so no two workgroups
// differ by more than one of either.  s_list receives workgroup l's
// rows on from the front and its rows off from the back.  Ends with a barrier.
template <int W>
__device__ inline RowShare share_rows(const uint8_t* mask, int base, int rows, int G, int l, int* s_list,
                                     uint64_t* s_cnt) {
    constexpr int NW = W / kWave;
    const int tid = opaque_tid(), lane = tid & (kWave - 1), wid = tid / kWave;
    const int at = kFlags * tid;
    // The last 16 flags are moved back to end with the slice (in a slice of
    // fewer, to before its start: the launch has more rows than that).
    const int off = at < rows - kFlags ? at : rows - kFlags;
    const chunk_t raw = load_off(mask + base, off);
    uint32_t on = 0;
#pragma unroll
    for (int e = 0; e < kFlags; ++e) on |= ((raw[e / 4] >> (8 * (e % 4))) & 0xFFu) ? 1u << e : 0u;
    on = at - off < kFlags ? on >> (at - off) : 0u;
    const int here = rows - at;  // rows of this thread
    const uint32_t in = here <= 0 ? 0u : (here >= kFlags ? (1u << kFlags) - 1u : (1u << here) - 1u);
    uint32_t bits[2] = {on & in, ~on & in};
    const uint64_t cnt = uint64_t(__popc(bits[0])) | uint64_t(__popc(bits[1])) << 32;
    const uint64_t incl = wave_inclusive_scan(cnt);
    if (lane == kWave - 1) s_cnt[wid] = incl;
    __syncthreads();
    uint64_t before = incl - cnt, all = 0;
#pragma unroll 1
    for (int w = 0; w < NW; ++w) {
        const uint64_t v = s_cnt[w];
        if (w < wid) before += v;
        all += v;
    }
    RowShare share;
#pragma unroll
    for (int z = 0; z < 2; ++z) {
        // This thread's rows of the kind have ranks r0 .. r0 + n - 1; the workgroup
        // takes ranks l, l + G, ...
        const int r0 = int(before >> (32 * z)) & 0x7FFFFFFF, n = __popc(bits[z]);
        const int total = int(all >> (32 * z)) & 0x7FFFFFFF;
        int j = r0 > l ? (r0 - l + G - 1) / G : 0;
#pragma unroll 1
        for (int r = l + j * G; r < r0 + n; r += G, ++j)
            s_list[z == 0 ? j : kShareMax<W> - 1 - j] = base + at + nth_bit(bits[z], r - r0);
        (z == 0 ? share.on : share.off) = __builtin_amdgcn_readfirstlane(total > l ? (total - l - 1) / G + 1 : 0);
    }
    __syncthreads();
    return share;
}

template <typename Fmt, int W, int CPT, int KIND, bool LISTED, int WAVES, bool PART>
__global__ __launch_bounds__(W, WAVES) void distill_stream_kernel(StreamDistillArgs a) {
    constexpr int NW = W / kWave, EPC = Fmt::kPerChunk, NG = EPC / 4;
    // JSD caches exponentials (the others, exponents): see the statistics pass.
    constexpr bool XV = KIND == 2;
    __shared__ float s_k[2 * NW];
    __shared__ double s_s[2 * NW];
    __shared__ RowPair s_rp;
    __shared__ double s_a[2 * NW];
    __shared__ int s_list[LISTED ? kShareMax<W> : 1];
    __shared__ uint64_t s_cnt[NW];
    __shared__ int s_on[2];  // the flags of a workgroup's only rows
    __shared__ double s_part[1];  // sum of this workgroup's row divergences
    __shared__ LossTail s_tail;
    __shared__ f32x4_t s_c0[CPT * NG * W];
    const LdsCache<W, EPC> lc{s_c0};

    // Every argument word, requested together: each dependent request would
    // cost a round trip to the argument buffer (about a microsecond).
    asm volatile("" ::"s"(a.teacher), "s"(a.tstride), "s"(a.student), "s"(a.sstride), "s"(a.B), "s"(a.K), "s"(a.V),
                 "s"(a.mask), "s"(a.beta), "s"(a.c2), "s"(a.inv_tau));
    asm volatile("" ::"s"(a.row_loss_out), "s"(a.grad_out), "s"(a.row_ws), "s"(a.done), "s"(a.loss_out), "s"(a.nrows),
                 "s"(a.row_bytes), "s"(a.G), "s"(a.slice), "s"(a.gs));
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const int G = a.G;
    const float c2 = a.c2;
    const LastChunk<PART> last = last_chunk<Fmt, W, CPT, PART>(a.V);
    const float beta = a.beta;

    chunk_t rt[CPT], rs[CPT];
    float c1[CPT][EPC];

    if (tid == 0) {
        s_part[0] = 0.0;  // read and written by thread 0 only
        s_tail.row_ws = a.row_ws;
        s_tail.done = a.done;
        s_tail.loss_out = a.loss_out;
        s_tail.mask = a.mask;
        s_tail.nrows = a.nrows;
        s_tail.G = a.G;
    }
    uint32_t mine = 1u;
    int more = 0, zeros = 0;  // LISTED: rows after the next; rows off, not yet written
    int next = int(blockIdx.x);
    if constexpr (LISTED) {
        // This workgroup's slice and place in it.  One slice unless the mask has more
        // flags than the workgroup loads at once.
        const int q = a.gs < G ? int(blockIdx.x) / a.gs : 0;
        const int Gq = a.gs, l = int(blockIdx.x) - q * a.gs, base = q * a.slice;
        const int rows = a.nrows - base < a.slice ? a.nrows - base : a.slice;
        next = l < rows ? base + l : -1;
        // A slice of few rows is dealt out as it is: the flags of its workgroups' one or two
        // rows are staged as below.
        const bool listed = rows > 2 * Gq;
        if (!listed && tid < 2 && l + tid * Gq < rows) mine = a.mask[base + l + tid * Gq];
        // More rows: this workgroup's list of them, in LDS, so that nothing in the row
        // loop reads global memory except the rows themselves (a scalar load there
        // would share its wait counter with LDS traffic).
        if (listed) {
            const RowShare share = share_rows<W>(a.mask, base, rows, Gq, l, s_list, s_cnt);
            more = share.on > 0 ? share.on - 1 : 0;
            zeros = share.off;
            next = share.on > 0 ? __builtin_amdgcn_readfirstlane(s_list[0]) : -1;
        } else if (l < rows) {
            more = (rows - l - 1) / Gq;  // at most 1
            if (tid <= more) s_list[tid] = base + l + tid * Gq;
        }
    } else {
        // Rows g, g + G, ...  With a mask (then one or two of them) their flags,
        // loaded before the row so that waiting for them never waits for the row,
        // and staged in LDS by step -1.
        if (a.mask && tid < 2 && tid * G < a.nrows - next) mine = a.mask[next + tid * G];
    }
    const int quota = zeros / (more + 1) + 1;  // rows off written by a step
    // The pipeline starts one step early: step -1 computes nothing; it issues
    // the loads of the workgroup's first row, from the same code as every later
    // step (so the compiler sees one load order throughout).
    int n = -1;  // this step's row (-1: none)
    bool live = false;
    for (int k = -1; k < 0 || n >= 0; ++k) {
        // (The first row is read whatever its flag, which is not known yet.)
        const bool skip = (LISTED || a.mask) && k == 0 && __builtin_amdgcn_readfirstlane(s_on[1]) == 0;
        const Row nxt = decode_row<Fmt>(a, skip ? -1 : next);
        const rsrc_t ntr = make_rsrc(nxt.on ? nxt.trow : a.teacher, nxt.on ? a.row_bytes : 0u);
        const rsrc_t nsr = make_rsrc(nxt.on ? nxt.srow : a.student, nxt.on ? a.row_bytes : 0u);
        // The gradient row of the current row (0 bytes before the first row:
        // nothing is written).
        const bool has_row = n >= 0;
        const rsrc_t gr = make_rsrc(a.grad_out && has_row ? static_cast<char*>(a.grad_out) + int64_t(n) * a.row_bytes
                                                          : static_cast<char*>(nullptr),
                                    a.grad_out && has_row ? a.row_bytes : 0u);
        double D = 0.0;
        // ---- statistics pass: consumes the raw chunks and reloads each
        // with the next row's.  The loads are issued whether or not the row
        // is computed: a branch around them would make the compiler copy
        // registers with loads still in flight, which waits for all of them.
        float kc_t = 0.0f, kc_s = 0.0f;
        double S_t = 0.0, S_s = 0.0;
        if constexpr (XV) {
            // JSD caches each element's 2^(x c2 - k) itself, so the thread's
            // shift k is taken over all its chunks: every cached value is at
            // most 1 and no sum leaves the fp32 range.
            if (live) {
                const float mt = chunks_max<Fmt, CPT>(rt, last);
                const float ms = chunks_max<Fmt, CPT>(rs, last);
                kc_t = shift_of_max(mt, c2);
                kc_s = shift_of_max(ms, c2);
            }
        }
#pragma unroll
        for (int r = 0; r < CPT; ++r) {
            if (live) {
                chunk_t xt = rt[r], xs = rs[r];
                if (r == CPT - 1) pad_last<Fmt>(xt, xs, last);
                if (!XV && r == 0) {
                    kc_t = first_chunk_shift<Fmt>(xt, c2);
                    kc_s = first_chunk_shift<Fmt>(xs, c2);
                }
                float st = 0.0f, ss = 0.0f;
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    float c0v[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int e = 4 * g + j;
                        const float t = Fmt::get(xt, e), s = Fmt::get(xs, e);
                        const float vt = __builtin_fmaf(t, c2, -kc_t);
                        const float vs = __builtin_fmaf(s, c2, -kc_s);
                        const float et = exp2_fast(vt), es = exp2_fast(vs);
                        // (the first term starts the sums: 0 + x would cost an add)
                        st = e == 0 ? et : st + et;
                        ss = e == 0 ? es : ss + es;
                        if constexpr (XV) {
                            c0v[j] = et;
                            c1[r][e] = es;
                        } else {
                            // Both exponents: each side's probability is
                            // rebuilt from its own exponent, so a -inf logit
                            // on either side alone gives that side 0 and the
                            // other its true value.  One floor suffices: with
                            // the target's exponent finite, a draft exponent
                            // of -inf still gives q = 0, and two -inf
                            // exponents give a finite difference.
                            c0v[j] = fmaxf(vt, kLogFloor);
                            c1[r][e] = vs;
                        }
                    }
                    lc.store(r, g, f32x4_t{c0v[0], c0v[1], c0v[2], c0v[3]});
                }
                // Keep each round's sums in the round (without this the
                // compiler may defer one row's exponentials past the loop).
                asm volatile("" : "+v"(st), "+v"(ss));
                S_t = r == 0 ? double(st) : S_t + double(st);
                S_s = r == 0 ? double(ss) : S_s + double(ss);
            }
            rt[r] = load_round<W, CPT>(ntr, r, last);
            rs[r] = load_round<W, CPT>(nsr, r, last);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (k < 0 && (LISTED || a.mask)) {  // step -1: stage the flags
            if (tid < 2) s_on[tid] = int(mine);
            __syncthreads();
        }
        if constexpr (LISTED) {
            // The zero rows, spread over the steps (all by step -1 if there is no other).
#pragma unroll 1
            for (int z = 0; z < quota && zeros > 0; ++z) {
                --zeros;
                const int64_t zr = __builtin_amdgcn_readfirstlane(s_list[kShareMax<W> - 1 - zeros]);
                if (a.grad_out)
                    zero_row<W>(make_rsrc(static_cast<char*>(a.grad_out) + zr * a.row_bytes, a.row_bytes), a.row_bytes,
                                tid);
                if (tid == 0 && a.row_loss_out) a.row_loss_out[zr] = 0.0f;
            }
        }
        if (!live) {
            if (a.grad_out && has_row) {
#pragma unroll
                for (int r = 0; r < CPT; ++r) store_round<Fmt, W, CPT>(gr, r, chunk_t{0u, 0u, 0u, 0u}, last);
            }
        } else {
            // Exponent range exceeded by an element far above the first
            // chunk's maximum: rescale exactly from the cached exponents.
            float ks_t = kc_t, ks_s = kc_s;
            if (!XV && S_t >= 1.0e300) {  // (a NaN sum stays NaN: it marks a NaN logit)
                ks_t = kc_t + rescue_sum<CPT, EPC>(S_t, [&](int r, int e) -> float { return lc.load(r, e / 4)[e % 4]; });
            }
            if (!XV && S_s >= 1.0e300) {
                ks_s = kc_s + rescue_sum<CPT, EPC>(S_s, [&](int r, int e) -> float { return c1[r][e]; });
            }
            const RowPair rp = merge_row_pair<NW>(ks_t, S_t, ks_s, S_s, s_k, s_s, &s_rp);
            // FKL/RKL take log2(p/q) from the same rounded exponents as the sums
            // (so the normalisers and the log-ratios agree: rows with p ~ q keep
            // their small divergence accurate); only the difference of the
            // normalisers is needed in fp64 (from the ratio of the sums).
            const RowScales z = row_scales(rp, kc_t, S_t == 0.0, kc_s, S_s == 0.0, beta);

            // ---- loss pass (from the cache) ----
            float acc0 = 0.0f, acc1 = 0.0f;
#pragma unroll
            for (int r = 0; r < CPT; ++r) {
                float a0 = 0.0f, a1 = 0.0f;
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    const f32x4_t v = lc.load(r, g);
                    float c0v[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int e = 4 * g + j;
                        loss_term<KIND>(c0v[j], c1[r][e], z.k, a0, a1);
                    }
                    lc.store(r, g, f32x4_t{c0v[0], c0v[1], c0v[2], c0v[3]});
                }
                acc0 = acc0 + a0;
                acc1 = acc1 + a1;
                __builtin_amdgcn_sched_barrier(0);
            }
            double A0 = double(acc0), A1 = 0.0;
            if constexpr (KIND == 2) {
                A0 *= double(z.at);
                A1 = double(acc1) * double(z.as);
            }
            block_sum2<NW>(A0, A1, s_a);
            // Terms were accumulated in log2 units.
            if constexpr (KIND == 2)
                D = kLn2 * (double(a.beta) * A0 + (1.0 - double(a.beta)) * A1);
            else if constexpr (KIND == 0)
                D = kLn2 * A0;
            else
                D = -kLn2 * A0;

            // ---- gradient pass (from the cache) ----
            if (a.grad_out) {
                const float ln2 = float(kLn2);
                const float scale = KIND == 0   ? a.inv_tau
                                    : KIND == 2 ? z.as * ((1.0f - beta) * ln2 * a.inv_tau)
                                                : ln2 * a.inv_tau;
                const float shift = KIND == 2 ? float(A1) : float(A0);
#pragma unroll
                for (int r = 0; r < CPT; ++r) {
                    float g[EPC];
#pragma unroll
                    for (int q4 = 0; q4 < NG; ++q4) {
                        const f32x4_t v = lc.load(r, q4);
                        const float c0v[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const int e = 4 * q4 + j;
                            g[e] = grad_term<KIND>(c0v[j], c1[r][e], scale, shift);
                        }
                    }
                    store_round<Fmt, W, CPT>(gr, r, pack_grad<Fmt>(g), last);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        if (tid == 0 && has_row) {
            if (a.row_loss_out) a.row_loss_out[n] = float(D);
            s_part[0] += D;  // this workgroup's rows, in the order taken
        }
        n = next;
        if constexpr (LISTED) {
            live = n >= 0 && (k >= 1 || __builtin_amdgcn_readfirstlane(s_on[k + 1]) != 0);
            next = k + 1 < more ? __builtin_amdgcn_readfirstlane(s_list[k + 2]) : -1;
        } else {
            live = n >= 0 && (!a.mask || __builtin_amdgcn_readfirstlane(s_on[k + 1]) != 0);
            next = n >= 0 && a.nrows - n > G ? n + G : -1;
        }
    }
    finish_loss<W>(s_tail, s_part);
}

template <typename Fmt, int W, int CPT, int KIND, bool LISTED, int WAVES>
int blocks_per_cu() {
    static const int v = [] {
        int nb = 0;
        const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &nb, distill_stream_kernel<Fmt, W, CPT, KIND, LISTED, WAVES, true>, W, 0);
        return (e != hipSuccess || nb < 1) ? 1 : nb;
    }();
    return v;
}

template <typename Fmt, int W, int CPT, int KIND, bool LISTED, int WAVES>
hipError_t launch_rows(const DistillLaunch& L, const StreamDistillArgs& a, int64_t grid) {
    StreamDistillArgs ag = a;
    ag.slice = a.nrows;
    ag.gs = int(grid);
    if (LISTED && a.nrows > W * kFlags) {
        // Slices of equal size, each with an equal number (at least 15) of workgroups.
        const int64_t nq = (int64_t(a.nrows) + W * kFlags - 1) / (W * kFlags);
        ag.slice = int((a.nrows + nq - 1) / nq);
        ag.gs = int(grid / nq);
        grid = ag.gs * nq;
    }
    ag.G = int(grid);
    // Rows of whole chunks have a kernel of their own, without the handling of a row that
    // ends inside one: JSD of 16 rows of V = 5000 bf16 8.9 -> 8.1 us, of 512 rows of V =
    // 32128 28.3 -> 27.5.  (Not the listed rows: 16384 of V = 32000, 40 % on, take 374 us
    // as they are.)
    if constexpr (!LISTED)
        if (L.V % Fmt::kPerChunk == 0)
            return launch_kernel(&distill_stream_kernel<Fmt, W, CPT, KIND, LISTED, WAVES, false>, dim3(unsigned(grid)),
                                 dim3(W), 0, L.stream, ag);
    return launch_kernel(&distill_stream_kernel<Fmt, W, CPT, KIND, LISTED, WAVES, true>, dim3(unsigned(grid)), dim3(W), 0,
                         L.stream, ag);
}

template <typename Fmt, int W, int CPT, int KIND>
hipError_t launch_kind(const DistillLaunch& L, const StreamDistillArgs& a) {
    // Two workgroups of 1024 threads on a CU (8 waves per SIMD) while a thread has at
    // most 8 elements, where there are rows for both: 5000 rows of V = 5000 bf16, FKL,
    // 78.5 -> 68.3 us, but 16 rows 8.2 -> 8.8.  (At 512 threads 5000 rows of V = 3000,
    // JSD, took 46.7 us without the bound on registers and 48.3 with it.)
    constexpr int kMany = W == 1024 && CPT * Fmt::kPerChunk <= 8 ? 8 : 1;
    const bool many = a.nrows > L.cus;
    // At most 7 workgroups on a CU: their arrivals at one counter are served one after
    // another (5000 rows of V = 1000 fp32, JSD: 36.8 us with 8, 33.5 with 7).
    int64_t grid = int64_t(L.cus) * (many ? std::min(blocks_per_cu<Fmt, W, CPT, KIND, true, kMany>(), 7) : 1);
    // At most W rows per workgroup (its list).
    const int64_t min_grid = (int64_t(a.nrows) + W - 1) / W;
    if (grid < min_grid) grid = min_grid;
    if (grid > a.nrows) grid = a.nrows;
    // Up to two rows per workgroup are not worth the list: finding it keeps the first
    // row's loads waiting for the flags.  (512 rows of V = 32128 bf16, all on: 30.7 us
    // with it and 27.8 without, RKL 27.9 and 25.1; an eighth of them on, behind a
    // verification: 44.7 and 48.9 in all.)  Rows without a mask do not carry its code.
    if (a.mask && a.nrows > 2 * grid) return launch_rows<Fmt, W, CPT, KIND, true, kMany>(L, a, grid);
    return many ? launch_rows<Fmt, W, CPT, KIND, false, kMany>(L, a, grid)
                : launch_rows<Fmt, W, CPT, KIND, false, 1>(L, a, grid);
}

template <typename Fmt, int W, int CPT>
hipError_t launch_tile(const DistillLaunch& L, const StreamDistillArgs& a) {
    switch (L.kind) {
        case 0: return launch_kind<Fmt, W, CPT, 0>(L, a);
        case 1: return launch_kind<Fmt, W, CPT, 1>(L, a);
        default: return launch_kind<Fmt, W, CPT, 2>(L, a);
    }
}

template <typename Fmt>
hipError_t launch_fmt(const DistillLaunch& L, const StreamDistillArgs& a) {
    RowTile t;
    if (!pick_stream_tile(L.V, Fmt::kPerChunk, &t)) return hipErrorInvalidValue;
    switch (t.W * 100 + t.CPT) {
        case 25601: return launch_tile<Fmt, 256, 1>(L, a);
        case 51201: return launch_tile<Fmt, 512, 1>(L, a);
        case 102401: return launch_tile<Fmt, 1024, 1>(L, a);
        case 102402: return launch_tile<Fmt, 1024, 2>(L, a);
        case 102403: return launch_tile<Fmt, 1024, 3>(L, a);
        case 102404: return launch_tile<Fmt, 1024, 4>(L, a);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

// Streaming tiles, smallest first: one chunk to 32768 bf16 or 16384 fp32
// logits per row.  A row of the tile's range fills every round but the last.  Registers hold the raw chunks in flight (and, in the distillation
// kernel, one float per element); the rest of a row's state lives in LDS.
bool pick_stream_tile(int V, int per_chunk, RowTile* t) {
    static const RowTile tiles[] = {{256, 1}, {512, 1}, {1024, 1}, {1024, 2}, {1024, 3}, {1024, 4}};
    if (V < per_chunk) return false;
    for (const RowTile& c : tiles)
        if (int64_t(V) <= int64_t(c.W) * c.CPT * per_chunk) {
            *t = c;
            return true;
        }
    return false;
}

hipError_t launch_distill_stream(const DistillLaunch& L) {
    StreamDistillArgs a{};
    a.teacher = L.teacher;
    a.tstride = L.teacher_stride;
    a.student = L.student;
    a.sstride = L.student_stride;
    a.B = L.B;
    a.K = L.K;
    a.V = L.V;
    a.mask = L.mask;
    a.beta = L.beta;
    a.c2 = float(1.4426950408889634 / double(L.tau));
    a.inv_tau = float(1.0 / double(L.tau));
    a.row_loss_out = L.row_loss_out;
    a.grad_out = L.grad_out;
    a.row_ws = L.row_loss_ws;
    a.done = L.done_counter;
    a.loss_out = L.loss_out;
    a.nrows = L.B * L.K;
    const int eb = L.dtype == 1 ? 2 : 4;
    a.row_bytes = uint32_t(int64_t(L.V) * eb);
    return L.dtype == 1 ? launch_fmt<BF16>(L, a) : launch_fmt<F32>(L, a);
}

}  // namespace osd
