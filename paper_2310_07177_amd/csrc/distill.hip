// distill.hip -- distillation divergence and its gradient with respect to the
// student logits on gfx950 (Section 4.1, Eq. 2-4 of arXiv:2310.07177).
//
// For each row n = (b, i) with mask 1, with p = softmax(t / tau) (teacher) and
// q = softmax(s / tau) (student):
//   FKL  D = sum p (log p - log q)                  g = (q - p) / tau
//   RKL  D = sum q (log q - log p)                  g = q (log q - log p - D) / tau
//   JSD  D = beta KL(p || m) + (1-beta) KL(q || m)   g = (1-beta) q (log q - log m - KL(q || m)) / tau
//        with m = beta p + (1-beta) q
// and 0 log 0 = 0.  Rows with mask 0 get D = 0 and a zero gradient row.
//
// Rows longer than the streaming tiles (distill_stream.hip), split over
// workgroups, and rows shorter than one 16-byte chunk.  The scalar loss is
// reduced without floating-point atomics: each row stores its D, the last row
// of every 64-row slab to arrive sums its slab in a fixed order, and the last
// slab to arrive sums the slabs in a fixed order -- the result is bitwise
// reproducible.
#include <stdlib.h>

#include <type_traits>

#include "osd_device.hpp"
#include "osd_internal.hpp"
#include "stream_device.hpp"
#include "distill_common.hpp"

namespace osd {
namespace {

struct DistillArgs {
    const void* teacher;
    int64_t tstride;
    const void* student;
    int64_t sstride;
    int B, K, V;
    const uint8_t* mask;
    float beta;
    float c2;       // log2(e) / tau
    float inv_tau;  // 1 / tau
    float* loss_out;
    float* row_loss_out;
    void* grad_out;
    double* row_ws;    // [B*K]
    double* slab_ws;   // [2*nslabs]: {sum, count} per slab
    uint32_t* slab_cnt;
    uint32_t* done_cnt;
    int nslabs;
};

// Wave-wide fp64 sum with a fixed butterfly: every lane ends with the same,
// run-to-run reproducible value.
__device__ inline double wave_sum_fixed(double v) { return wave_sum(v); }

// Executed by all lanes of wave 0: record D for row n and fold it into the
// masked sum once every row has arrived.  Up to kOneLevelRows rows, the last
// row to arrive sums them all (each lane a fixed strided subset, then a fixed
// butterfly); beyond that, rows are summed per 64-row slab first and the last
// slab to arrive sums the slabs.  Every order is fixed, so the result is
// reproducible bit for bit.
__device__ void finish_loss(const DistillArgs& a, double sum, double count) {
    const int lane = threadIdx.x & (kWave - 1);
    if (lane == 0) {
        a.loss_out[0] = count > 0.0 ? float(sum / count) : 0.0f;
        a.loss_out[1] = float(sum);
    }
}

__device__ void reduce_loss(const DistillArgs& a, int n, double D) {
    const int lane = threadIdx.x & (kWave - 1);
    const int rows = a.B * a.K;
    uint32_t prev = 0;
    if (rows <= kOneLevelRows) {
        if (lane == 0) {
            publish_f64(&a.row_ws[n], D);
            prev = arrive(a.done_cnt);
        }
        prev = __shfl(prev, 0, kWave);
        if (prev != uint32_t(rows - 1)) return;
        double v[kOneLevelRows / kWave];
#pragma unroll
        for (int k = 0; k < kOneLevelRows / kWave; ++k) {
            const int r = k * kWave + lane;
            v[k] = r < rows ? take_f64(&a.row_ws[r]) : 0.0;  // read and clear
        }
        double s = 0.0, c = 0.0;
#pragma unroll
        for (int k = 0; k < kOneLevelRows / kWave; ++k) {
            const int r = k * kWave + lane;
            s += v[k];
            c += (r < rows && (a.mask == nullptr || a.mask[r] != 0)) ? 1.0 : 0.0;
        }
        s = wave_sum_fixed(s);
        c = wave_sum_fixed(c);
        finish_loss(a, s, c);
        if (lane == 0) take_u32(a.done_cnt);
        return;
    }
    const int slab = n / kSlabRows;
    const int first = slab * kSlabRows;
    const int in_slab = min(kSlabRows, rows - first);
    if (lane == 0) {
        publish_f64(&a.row_ws[n], D);
        prev = arrive(&a.slab_cnt[slab]);
    }
    prev = __shfl(prev, 0, kWave);
    if (prev != uint32_t(in_slab - 1)) return;
    double v = 0.0, c = 0.0;
    if (lane < in_slab) {
        v = take_f64(&a.row_ws[first + lane]);  // read and clear
        c = (a.mask == nullptr || a.mask[first + lane] != 0) ? 1.0 : 0.0;
    }
    const double slab_sum = wave_sum_fixed(v);
    const double slab_cnt = wave_sum_fixed(c);
    if (lane == 0) {
        publish_f64(&a.slab_ws[2 * slab], slab_sum);
        publish_f64(&a.slab_ws[2 * slab + 1], slab_cnt);
        take_u32(&a.slab_cnt[slab]);
        prev = arrive(a.done_cnt);
    }
    prev = __shfl(prev, 0, kWave);
    if (prev != uint32_t(a.nslabs - 1)) return;
    double ts = 0.0, tc = 0.0;
    for (int s = lane; s < a.nslabs; s += kWave) {
        ts += take_f64(&a.slab_ws[2 * s]);
        tc += take_f64(&a.slab_ws[2 * s + 1]);
    }
    ts = wave_sum_fixed(ts);
    tc = wave_sum_fixed(tc);
    finish_loss(a, ts, tc);
    if (lane == 0) take_u32(a.done_cnt);
}

// A row is split into segments of 8192 logits, one 256-thread workgroup
// each, which cooperate through device memory (a row of one segment alone
// needs no exchange):
//   1. each segment turns its chunks of both rows into the cached pairs of
//      distill_common.hpp, held in registers for the rest of the row (two
//      floats per element pair instead of the raw logits: no later pass takes
//      the exponentials again), folds its (K, S) pairs and publishes them;
//      every segment reads all the row's records and merges them in segment
//      order (the same normalisers in every workgroup);
//   2. each segment sums its divergence terms and publishes the partials;
//      FKL's gradient needs only the normalisers and is written here;
//   3. RKL and JSD read all the row's partials, add them in segment order and
//      write their gradient segment.
// Published words go out as plain agent-scope atomic stores that are never
// zero (each value is stored bit-inverted, and no value a segment publishes
// has all bits set), so a reader polls the words themselves: a zero word is
// not yet published.  Once a segment has read everything it needs it
// arrives at the row's counter; the last arriver adds the partials in
// segment order, writes the row's divergence, enters the masked-loss
// reduction and clears the row's words and counter (the workspace is left
// zero).  Rows with mask 0 write their zero gradient segments and take no
// part in the exchange.
//
// A wait is bounded (kSplitPolls polls, or the value of OSD_SPLIT_POLLS).  A
// workgroup whose siblings have not all published in time computes the
// missing records (or partials) itself, re-reading every segment of the row
// with the same thread layout and reduction order, so that the result is the
// same bit for bit; it still publishes and arrives, so the row completes as
// usual.
//
// Instruction issue bounds the kernel (a transcendental takes 8 cycles of a
// SIMD, any other vector instruction 4): JSD takes 5 transcendentals per
// element pair from the cache against 9 from the raw logits, RKL 3 against 4,
// FKL 4 against 5.  512 rows of V = 128256 bf16: JSD 145.9 -> 118.9 us, FKL
// 113.9 -> 95.4; 4000 rows of V = 50304: RKL 359.6 -> 319.2, FKL 357.0 -> 274.1;
// 18 rows of V = 54016, JSD: 28.0 -> 11.9 (one 1024-thread workgroup per row
// before, which was no faster at any number of rows).
constexpr int kSegW = 256;
// Chunks per thread of a segment: 32 elements of each row either way, 8192 bf16
// or fp32 logits per segment.  (Segments of 4096 fp32 logits took 28.2 us for
// 256 rows of V = 32000, against 23.2: their 2048 workgroups just missed
// fitting the chip at once.)
template <typename Fmt>
constexpr int kSegCPT = 32 / Fmt::kPerChunk;
constexpr int kSplitPolls = 256;
constexpr int kSegNW = kSegW / kWave;

struct SplitArgs {
    DistillArgs d;
    uint64_t* rec;   // [rows, kMaxSplitSegments, 3]: ~S_t, ~S_s, ~(K_t | K_s << 32) (bits)
    uint64_t* part;  // [rows, kMaxSplitSegments, 2]: ~A0, ~A1 (bits)
    uint32_t* cnt;   // [rows, 4]: arrivals (word 0)
    int nseg;
    int polls;
};

struct SegShared {
    float k[2][kSegNW];
    double s[2][kSegNW];
    float rk[kMaxSplitSegments][2];   // records merged by this workgroup
    double rs[kMaxSplitSegments][2];
    double pa[kMaxSplitSegments][2];  // partials
    RowPair row;
    double total[2];                  // the row's partials, added
    int flag;                         // the polls brought every record
    int last;                         // this workgroup is the row's last arriver
};

__device__ inline bool row_on(const DistillArgs& a, int n) { return a.mask == nullptr || a.mask[n] != 0; }

template <typename Fmt>
__device__ inline const char* row_ptr(const void* base, int64_t stride, int n, int K, int V) {
    const int b = n / K, i = n - b * K;
    return static_cast<const char*>(base) + (int64_t(b) * stride + int64_t(i) * V) * Fmt::kBytes;
}

// Chunk r of this thread in segment s, and its round when the whole row is
// cut into rounds of kSegW chunks.
template <typename Fmt>
__device__ inline int seg_round(int s, int r) { return s * kSegCPT<Fmt> + r; }
template <typename Fmt>
__device__ inline int seg_chunk(int s, int r) { return seg_round<Fmt>(s, r) * kSegW + opaque_tid(); }

// The cached pairs of a thread's elements in one segment, their shifts and
// sums.  Every kind takes the shift over all the thread's chunks, so no
// exponent exceeds 0 and no sum leaves the fp32 range.
template <typename Fmt>
struct SegCache {
    static constexpr int EPC = Fmt::kPerChunk;
    float c0[kSegCPT<Fmt>][EPC], c1[kSegCPT<Fmt>][EPC];
    float kt, ks;
    double St, Ss;
};

template <typename Fmt, int KIND>
__device__ inline void seg_build(SegCache<Fmt>& c, const char* trow, const char* srow, int s, int V, float c2) {
    constexpr int EPC = Fmt::kPerChunk;
    asm volatile("" : "+s"(V), "+s"(s));  // nothing derived from them is hoisted out of a loop over segments
    const RowCut<Fmt> cut(V);
    chunk_t xt[kSegCPT<Fmt>], xs[kSegCPT<Fmt>];
    if (V >= EPC) {
#pragma unroll
        for (int r = 0; r < kSegCPT<Fmt>; ++r) {
            const int off = cut.off(seg_chunk<Fmt>(s, r));
            xt[r] = load_off(trow, off);
            xs[r] = load_off(srow, off);
        }
        if (cut.template ragged<kSegW>(seg_round<Fmt>(s, kSegCPT<Fmt> - 1))) {  // the row's last segment
#pragma unroll
            for (int r = 0; r < kSegCPT<Fmt>; ++r) {
                const int lead = cut.lead(seg_chunk<Fmt>(s, r));
                xt[r] = pad_lead<Fmt>(xt[r], lead);
                xs[r] = pad_lead<Fmt>(xs[r], lead);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    } else {  // a row shorter than one chunk: its elements end thread 0's chunk
#pragma unroll
        for (int r = 0; r < kSegCPT<Fmt>; ++r) xt[r] = xs[r] = pad_chunk<Fmt>();
        if (opaque_tid() == 0) {
            xt[0] = load_short<Fmt>(trow, V);
            xs[0] = load_short<Fmt>(srow, V);
        }
    }
    const LastChunk<false> whole{0, 0, false};  // the padding is in place
    c.kt = shift_of_max(chunks_max<Fmt, kSegCPT<Fmt>>(xt, whole), c2);
    c.ks = shift_of_max(chunks_max<Fmt, kSegCPT<Fmt>>(xs, whole), c2);
#pragma unroll
    for (int r = 0; r < kSegCPT<Fmt>; ++r) {
        // JSD is not first-order sensitive to the normalisers (the mixture
        // absorbs a common scale error): fp32 within a chunk.  FKL and RKL
        // are (an error in S shifts every log-ratio): every term in fp64.
        // (Two running sums per row: half the dependent additions.)
        typedef typename std::conditional<KIND == 2, float, double>::type acc_t;
        acc_t st[2], ss[2];
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
            const float vt = __builtin_fmaf(Fmt::get(xt[r], e), c2, -c.kt);
            const float vs = __builtin_fmaf(Fmt::get(xs[r], e), c2, -c.ks);
            const float et = exp2_fast(vt), es = exp2_fast(vs);
            st[e & 1] = e < 2 ? acc_t(et) : st[e & 1] + acc_t(et);
            ss[e & 1] = e < 2 ? acc_t(es) : ss[e & 1] + acc_t(es);
            if constexpr (KIND == 2) {
                c.c0[r][e] = et;
                c.c1[r][e] = es;
            } else {
                // Both exponents: each side's probability is rebuilt from its
                // own exponent (one floor suffices: two -inf exponents give a
                // finite difference, and a draft exponent of -inf still q = 0).
                c.c0[r][e] = fmaxf(vt, kLogFloor);
                c.c1[r][e] = vs;
            }
        }
        const double ct = double(st[0] + st[1]), cs = double(ss[0] + ss[1]);
        c.St = r == 0 ? ct : c.St + ct;
        c.Ss = r == 0 ? cs : c.Ss + cs;
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The segment's (K, S) pairs, reduced over the workgroup into slot `slot` of
// sh.rk / sh.rs (written by thread 0).  Opens with a barrier (sh.k, sh.s reuse).
template <typename Fmt>
__device__ inline void seg_stats(const SegCache<Fmt>& c, SegShared& sh, int slot) {
    const int tid = opaque_tid(), lane = tid & (kWave - 1), wid = tid / kWave;
    // (A thread without mass has no say in the row's shift.)
    float Kt = c.St == 0.0 ? kNegInf : c.kt, Ks = c.Ss == 0.0 ? kNegInf : c.ks;
    double dt = c.St, ds = c.Ss;
    wave_merge_stats_u(Kt, dt);
    wave_merge_stats_u(Ks, ds);
    __syncthreads();
    if (lane == 0) {
        sh.k[0][wid] = Kt;
        sh.k[1][wid] = Ks;
        sh.s[0][wid] = dt;
        sh.s[1][wid] = ds;
    }
    __syncthreads();
    if (wid == 0) {
        float k0 = lane < kSegNW ? sh.k[0][lane] : kNegInf, k1 = lane < kSegNW ? sh.k[1][lane] : kNegInf;
        double t0 = lane < kSegNW ? sh.s[0][lane] : 0.0, t1 = lane < kSegNW ? sh.s[1][lane] : 0.0;
        row0_merge_stats_u(k0, t0);
        row0_merge_stats_u(k1, t1);
        if (lane == 0) {
            sh.rk[slot][0] = k0;
            sh.rk[slot][1] = k1;
            sh.rs[slot][0] = t0;
            sh.rs[slot][1] = t1;
        }
    }
}

// The segment's divergence partials from its cache (which it turns into the
// gradient's terms), reduced over the workgroup into slot `slot` of sh.pa.
template <typename Fmt, int KIND>
__device__ inline void seg_partial(SegCache<Fmt>& c, const RowScales& z, SegShared& sh, int slot) {
    constexpr int EPC = Fmt::kPerChunk;
    const int tid = opaque_tid(), lane = tid & (kWave - 1), wid = tid / kWave;
    float acc0 = 0.0f, acc1 = 0.0f;
#pragma unroll
    for (int r = 0; r < kSegCPT<Fmt>; ++r) {
        float a0 = 0.0f, a1 = 0.0f;
#pragma unroll
        for (int e = 0; e < EPC; ++e) loss_term<KIND>(c.c0[r][e], c.c1[r][e], z.k, a0, a1);
        acc0 = acc0 + a0;
        acc1 = acc1 + a1;
        __builtin_amdgcn_sched_barrier(0);
    }
    double A0 = double(acc0), A1 = 0.0;
    if constexpr (KIND == 2) {
        A0 *= double(z.at);
        A1 = double(acc1) * double(z.as);
    }
    A0 = wave_sum_u(A0);
    if constexpr (KIND == 2) A1 = wave_sum_u(A1);
    __syncthreads();
    if (lane == 0) {
        sh.s[0][wid] = A0;
        sh.s[1][wid] = A1;
    }
    __syncthreads();
    if (wid == 0) {
        A0 = row0_sum_u(lane < kSegNW ? sh.s[0][lane] : 0.0);
        A1 = row0_sum_u(lane < kSegNW ? sh.s[1][lane] : 0.0);
        if (lane == 0) {
            sh.pa[slot][0] = A0;
            sh.pa[slot][1] = A1;
        }
    }
}

// Wave 0: the row's normalisers from the records in sh, merged in segment
// order by one scan (lane j: segment j), into sh.row.
__device__ inline void merge_records(SegShared& sh, int nseg) {
    const int lane = opaque_tid() & (kWave - 1);
    const bool mine = lane < nseg;
    store_row_pair(mine ? sh.rk[lane][0] : kNegInf, mine ? sh.rs[lane][0] : 0.0, mine ? sh.rk[lane][1] : kNegInf,
                   mine ? sh.rs[lane][1] : 0.0, lane, &sh.row);
}

// Wave 0: the row's partials in sh, added in segment order, into sh.total.
__device__ inline void merge_partials(SegShared& sh, int nseg) {
    const int lane = opaque_tid() & (kWave - 1);
    const double A0 = row0_sum_u(lane < nseg ? sh.pa[lane][0] : 0.0);
    const double A1 = row0_sum_u(lane < nseg ? sh.pa[lane][1] : 0.0);
    if (lane == 0) {
        sh.total[0] = A0;
        sh.total[1] = A1;
    }
}

// The row's divergence from its added partials.
template <int KIND>
__device__ inline double row_divergence(const SegShared& sh, float beta) {
    if constexpr (KIND == 2)
        return kLn2 * (double(beta) * sh.total[0] + (1.0 - double(beta)) * sh.total[1]);
    else
        return (KIND == 0 ? kLn2 : -kLn2) * sh.total[0];
}

template <typename Fmt, int KIND>
__device__ inline void seg_grad(const SegCache<Fmt>& c, const RowScales& z, const DistillArgs& a, float shift, void* grow,
                                int s, const RowCut<Fmt>& cut) {
    constexpr int EPC = Fmt::kPerChunk;
    const float ln2 = float(kLn2);
    const float scale = KIND == 0 ? a.inv_tau : (KIND == 2 ? z.as * (z.k.omb * ln2 * a.inv_tau) : ln2 * a.inv_tau);
    RowWriter<Fmt> out(grow, cut);
#pragma unroll
    for (int r = 0; r < kSegCPT<Fmt>; ++r) {
        float g[EPC];
#pragma unroll
        for (int e = 0; e < EPC; ++e) g[e] = grad_term<KIND>(c.c0[r][e], c.c1[r][e], scale, shift);
        out.put(seg_chunk<Fmt>(s, r), pack_grad<Fmt>(g));
        __builtin_amdgcn_sched_barrier(0);
    }
    out.finish();
}

__device__ inline uint64_t load_u64(const uint64_t* p) {
    return __hip_atomic_load(const_cast<uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void store_u64(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline uint64_t pack_k(float kt, float ks) {
    return uint64_t(__float_as_uint(kt)) | (uint64_t(__float_as_uint(ks)) << 32);
}

// Wave 0 polls the published words of the row's other segments: lane j < nseg
// (j != s) reads the `words` words of segment j until every one is non-zero
// or the polls run out.  On success, lane j leaves them (un-inverted) in
// w[0..words).
template <int WORDS>
__device__ inline bool poll_words(const uint64_t* base, int nseg, int s, int polls, uint64_t (&w)[WORDS]) {
    const int lane = opaque_tid() & (kWave - 1);
    const bool mine = lane < nseg && lane != s;
    bool ok = false;
    for (int p = 0; p < polls; ++p) {
        if (p > 0) __builtin_amdgcn_s_sleep(4);
        bool ready = true;
        if (mine) {
#pragma unroll
            for (int k = 0; k < WORDS; ++k) {
                w[k] = load_u64(base + int64_t(lane) * WORDS + k);
                ready = ready && w[k] != 0;
            }
        }
        if (__ballot(!ready) == 0) {
            ok = true;
            break;
        }
    }
#pragma unroll
    for (int k = 0; k < WORDS; ++k) w[k] = ~w[k];
    return ok;
}

// Arrival at the row's counter once this workgroup's published words are
// complete; the returned count is awaited only where it is used.
__device__ inline uint32_t arrive_row(uint32_t* counter) {
    wait_memory();
    return __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename Fmt, int KIND>
__global__ __launch_bounds__(kSegW, 4) void split_row_kernel(SplitArgs sa) {
    __shared__ SegShared sh;
    const DistillArgs& a = sa.d;
    const int nseg = sa.nseg, V = a.V;
    const RowCut<Fmt> cut(V);
    const int n = blockIdx.x / nseg, s = blockIdx.x - n * nseg;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    void* grow = a.grad_out ? static_cast<char*>(a.grad_out) + int64_t(n) * V * Fmt::kBytes : nullptr;
    if (!row_on(a, n)) {
        if (grow) {
            RowWriter<Fmt> out(grow, cut);
#pragma unroll
            for (int r = 0; r < kSegCPT<Fmt>; ++r) out.put(seg_chunk<Fmt>(s, r), chunk_t{0u, 0u, 0u, 0u});
            out.finish();
        }
        if (s == 0 && wid == 0) {
            if (a.row_loss_out && lane == 0) a.row_loss_out[n] = 0.0f;
            reduce_loss(a, n, 0.0);
        }
        return;
    }
    const char* trow = row_ptr<Fmt>(a.teacher, a.tstride, n, a.K, V);
    const char* srow = row_ptr<Fmt>(a.student, a.sstride, n, a.K, V);
    uint64_t* rec = sa.rec + int64_t(n) * kMaxSplitSegments * 3;
    uint64_t* part = sa.part + int64_t(n) * kMaxSplitSegments * 2;
    uint32_t* cnt = sa.cnt + int64_t(n) * 4;
    const float c2 = a.c2;

    // 1. statistics
    SegCache<Fmt> c;
    seg_build<Fmt, KIND>(c, trow, srow, s, V, c2);
    seg_stats<Fmt>(c, sh, s);
    if (wid == 0) {
        bool ok = true;
        if (nseg > 1) {
            if (lane == 0) {
                store_u64(&rec[3 * s], ~uint64_t(__double_as_longlong(sh.rs[s][0])));
                store_u64(&rec[3 * s + 1], ~uint64_t(__double_as_longlong(sh.rs[s][1])));
                store_u64(&rec[3 * s + 2], ~pack_k(sh.rk[s][0], sh.rk[s][1]));
            }
            uint64_t w[3];
            ok = poll_words<3>(rec, nseg, s, sa.polls, w);
            if (ok && lane < nseg && lane != s) {
                sh.rs[lane][0] = __longlong_as_double(w[0]);
                sh.rs[lane][1] = __longlong_as_double(w[1]);
                sh.rk[lane][0] = __uint_as_float(uint32_t(w[2]));
                sh.rk[lane][1] = __uint_as_float(uint32_t(w[2] >> 32));
            }
        }
        if (lane == 0) sh.flag = ok;
        if (ok) merge_records(sh, nseg);
    }
    __syncthreads();
    if (!sh.flag) {
#pragma unroll 1
        for (int j = 0; j < nseg; ++j) {
            if (j == s) continue;
            seg_build<Fmt, KIND>(c, trow, srow, j, V, c2);
            seg_stats<Fmt>(c, sh, j);
        }
        seg_build<Fmt, KIND>(c, trow, srow, s, V, c2);
        if (wid == 0) merge_records(sh, nseg);
        __syncthreads();
    }
    const RowPair rp = sh.row;

    // 2. divergence
    RowScales z = row_scales(rp, c.kt, c.St == 0.0, c.ks, c.Ss == 0.0, a.beta);
    seg_partial<Fmt, KIND>(c, z, sh, s);
    uint32_t prev = 0;
    if constexpr (KIND == 0) {
        if (tid == 0) {
            if (nseg > 1) {
                store_u64(&part[2 * s], ~uint64_t(__double_as_longlong(sh.pa[s][0])));
                store_u64(&part[2 * s + 1], ~uint64_t(__double_as_longlong(sh.pa[s][1])));
                prev = arrive_row(&cnt[0]);
            }
        }
        if (grow) seg_grad<Fmt, KIND>(c, z, a, 0.0f, grow, s, cut);
    } else {
        // 3. gradient
        if (wid == 0) {
            bool ok = true;
            if (nseg > 1) {
                if (lane == 0) {
                    store_u64(&part[2 * s], ~uint64_t(__double_as_longlong(sh.pa[s][0])));
                    store_u64(&part[2 * s + 1], ~uint64_t(__double_as_longlong(sh.pa[s][1])));
                }
                uint64_t w[2];
                ok = poll_words<2>(part, nseg, s, sa.polls, w);
                if (ok && lane < nseg && lane != s) {
                    sh.pa[lane][0] = __longlong_as_double(w[0]);
                    sh.pa[lane][1] = __longlong_as_double(w[1]);
                }
            }
            if (lane == 0) sh.flag = ok;
            if (ok) merge_partials(sh, nseg);
        }
        __syncthreads();
        if (!sh.flag) {
#pragma unroll 1
            for (int j = 0; j < nseg; ++j) {
                if (j == s) continue;
                seg_build<Fmt, KIND>(c, trow, srow, j, V, c2);
                z = row_scales(rp, c.kt, c.St == 0.0, c.ks, c.Ss == 0.0, a.beta);
                seg_partial<Fmt, KIND>(c, z, sh, j);
            }
            seg_build<Fmt, KIND>(c, trow, srow, s, V, c2);
            z = row_scales(rp, c.kt, c.St == 0.0, c.ks, c.Ss == 0.0, a.beta);
            seg_partial<Fmt, KIND>(c, z, sh, s);
            if (wid == 0) merge_partials(sh, nseg);
            __syncthreads();
        }
        if (tid == 0 && nseg > 1) prev = arrive_row(&cnt[0]);
        if (grow) seg_grad<Fmt, KIND>(c, z, a, float(sh.total[KIND == 2 ? 1 : 0]), grow, s, cut);
    }
    if (nseg > 1) {
        if (tid == 0) sh.last = prev == uint32_t(nseg - 1);
        __syncthreads();
        if (sh.last == 0) return;
    }
    // The row's last arriver: every segment has read what it needed.
    if (wid != 0) return;
    if constexpr (KIND == 0) {
        if (lane < nseg && lane != s) {
            sh.pa[lane][0] = __longlong_as_double(~load_u64(&part[2 * lane]));
            sh.pa[lane][1] = __longlong_as_double(~load_u64(&part[2 * lane + 1]));
        }
        merge_partials(sh, nseg);
    }
    if (nseg > 1) {
        if (lane < nseg) {
            store_u64(&rec[3 * lane], 0ull);
            store_u64(&rec[3 * lane + 1], 0ull);
            store_u64(&rec[3 * lane + 2], 0ull);
            store_u64(&part[2 * lane], 0ull);
            store_u64(&part[2 * lane + 1], 0ull);
        }
        if (lane == 0) __hip_atomic_store(&cnt[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const double D = row_divergence<KIND>(sh, a.beta);
    if (a.row_loss_out && lane == 0) a.row_loss_out[n] = float(D);
    reduce_loss(a, n, D);
}

template <typename Fmt, int KIND>
hipError_t launch_split_kind(const DistillLaunch& L, const SplitArgs& sa) {
    const unsigned rows = unsigned(L.B) * unsigned(L.K);
    return launch_kernel(&split_row_kernel<Fmt, KIND>, dim3(rows * unsigned(sa.nseg)), dim3(kSegW), 0, L.stream, sa);
}

// kSplitPolls, or the value of OSD_SPLIT_POLLS (read once; 0 makes every
// workgroup compute its row's records and partials itself).
int split_polls() {
    static const int v = [] {
        const char* e = getenv("OSD_SPLIT_POLLS");
        if (e == nullptr || *e == 0) return kSplitPolls;
        const int k = atoi(e);
        return k < 0 ? kSplitPolls : (k > 65536 ? 65536 : k);
    }();
    return v;
}

template <typename Fmt>
hipError_t launch_split(const DistillLaunch& L, const DistillArgs& a) {
    SplitArgs sa;
    sa.d = a;
    const int nchunks = (L.V + Fmt::kPerChunk - 1) / Fmt::kPerChunk;
    const int seg_chunks = kSegW * kSegCPT<Fmt>;
    sa.nseg = (nchunks + seg_chunks - 1) / seg_chunks;
    if (sa.nseg > kMaxSplitSegments) return hipErrorInvalidValue;
    const size_t rows = size_t(L.B) * size_t(L.K);
    char* w = static_cast<char*>(L.split_ws);
    sa.rec = reinterpret_cast<uint64_t*>(w);
    sa.part = reinterpret_cast<uint64_t*>(w + rows * kMaxSplitSegments * 24);
    sa.cnt = reinterpret_cast<uint32_t*>(w + rows * kMaxSplitSegments * 40);
    sa.polls = split_polls();
    if (rows * size_t(sa.nseg) > size_t(0x7FFFFFFF)) return hipErrorInvalidValue;
    switch (L.kind) {
        case 0: return launch_split_kind<Fmt, 0>(L, sa);
        case 1: return launch_split_kind<Fmt, 1>(L, sa);
        default: return launch_split_kind<Fmt, 2>(L, sa);
    }
}

}  // namespace

hipError_t launch_distill(const DistillLaunch& L) {
    DistillArgs a{};
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
    a.loss_out = L.loss_out;
    a.row_loss_out = L.row_loss_out;
    a.grad_out = L.grad_out;
    a.row_ws = L.row_loss_ws;
    a.slab_ws = L.slab_ws;
    a.slab_cnt = L.slab_counters;
    a.done_cnt = L.done_counter;
    a.nslabs = (L.B * L.K + kSlabRows - 1) / kSlabRows;
    return L.dtype == 1 ? launch_split<BF16>(L, a) : launch_split<F32>(L, a);
}

}  // namespace osd
