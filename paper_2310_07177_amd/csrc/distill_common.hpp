// distill_common.hpp -- pieces shared by the streaming distillation kernel
// and the fused verification + distillation kernel (gfx950): numerical
// floors, the bf16 gradient packer, the exponent-range rescue, the LDS half of
// the per-element cache, and the last-workgroup loss reduction.
#pragma once

#include "osd_device.hpp"
#include "stream_device.hpp"

namespace osd {

// Largest finite fp32 magnitude used to stand in for log2(0) = -inf, so that
// p * log2(p) stays 0 * finite = 0 for logits of -inf.
constexpr float kLogFloor = -1.0e30f;

template <typename Fmt>
__device__ inline chunk_t pack_grad(const float (&g)[Fmt::kPerChunk]) {
    if constexpr (Fmt::kPerChunk == 8) {
        return chunk_t{pack_bf16x2(g[0], g[1]), pack_bf16x2(g[2], g[3]),
                       pack_bf16x2(g[4], g[5]), pack_bf16x2(g[6], g[7])};
    } else {
        return chunk_t{__float_as_uint(g[0]), __float_as_uint(g[1]),
                       __float_as_uint(g[2]), __float_as_uint(g[3])};
    }
}

// Rescale a thread's sum of 2^v over its cached exponents when the first
// chunk's shift left the fp32 range: returns the extra whole-number shift o
// and replaces S by sum 2^(v - o).  v(r, e) reads the exponent of element e
// of round r; rounds are processed one at a time (a scheduling barrier after
// each) so that the rarely taken branch adds few live registers.
template <int CPT, int EPC, typename VFn>
__device__ inline float rescue_sum(double& S, VFn v) {
    float m = kNegInf;
#pragma unroll
    for (int r = 0; r < CPT; ++r) {
#pragma unroll
        for (int e = 0; e < EPC; ++e) m = fmaxf(m, v(r, e));
        __builtin_amdgcn_sched_barrier(0);
    }
    const float o = (m > -3.0e38f && m < 3.0e38f) ? ceilf(m) : 0.0f;
    S = 0.0;
#pragma unroll
    for (int r = 0; r < CPT; ++r) {
        float t = 0.0f;
#pragma unroll
        for (int e = 0; e < EPC; ++e) t = t + exp2_fast(v(r, e) - o);
        S += double(t);
        __builtin_amdgcn_sched_barrier(0);
    }
    return o;
}

// One element of the divergence (in log2 units) and of the gradient, from its
// cached pair of floats (c0, c1) and the thread's scales.
//   JSD      c0 = 2^(t c2 - k_t), c1 = 2^(s c2 - k_s); p = c0 at, q = c1 as;
//            the loss term leaves (log2(q/m), c1)
//   FKL/RKL  c0 = t c2 - k_t, c1 = s c2 - k_s; log2 p = c0 - ct, log2 q = c1 - cs;
//            the loss term leaves (p, log2 q) and (log2(p/q), q)
struct PairScales {
    float ratio;       // JSD: as / at
    float beta, omb;   // JSD: beta, 1 - beta
    float ct, cs, dTk; // FKL/RKL: log2(p/q) = (c0 - c1) - dTk
};
// a0, a1 collect, per thread: JSD the sums of -c0 L and c1 x (times at and as:
// the sums of p log2(p/m) and q log2(q/m)); FKL and RKL (in a0) the sums of
// p log2(p/q) and q log2(p/q).
template <int KIND>
__device__ inline void loss_term(float& c0, float& c1, const PairScales& k, float& a0, float& a1) {
    if constexpr (KIND == 2) {
        // rho = q/p, clamped to 2^+-126 (both limits stay exact enough: the
        // vanishing side carries no weight; 0/0 and inf*0 take the lower one).
        // log2 m = log2 p + L, L = log2(beta + (1 - beta) rho): the mixture's
        // log relative to p, a number near 0 when p ~ q, so the rounding of a
        // log does not bias every term of a small divergence.  At beta = 0, L
        // is d itself (the same log of the same value): x = 0.
        const float rho = __builtin_amdgcn_fmed3f((c1 * k.ratio) * __builtin_amdgcn_rcpf(c0), 0x1p-126f, 0x1p126f);
        const float d = log2_fast(rho);
        const float L = log2_fast(__builtin_fmaf(k.omb, rho, k.beta));
        const float x = d - L;  // log2(q/m)
        a0 = __builtin_fmaf(c0, -L, a0);
        a1 = __builtin_fmaf(c1, x, a1);
        c0 = x;
    } else {
        // log2(p/q) from the difference of the two exponents, clamped so that
        // a zero probability times an infinite log-ratio stays 0.
        const float lr = fmaxf(fminf((c0 - c1) - k.dTk, -kLogFloor), kLogFloor);
        if constexpr (KIND == 0) {
            const float p = exp2_fast(c0 - k.ct);
            a0 = __builtin_fmaf(p, lr, a0);
            c0 = p;
            c1 = c1 - k.cs;  // log2 q
        } else {
            const float q = exp2_fast(c1 - k.cs);
            a0 = __builtin_fmaf(q, lr, a0);
            c0 = lr;
            c1 = q;
        }
    }
}
// The gradient of one element from what loss_term left: scale and shift are
//   JSD  as (1-beta) ln2/tau and KL2 = KL(q || m) in log2 units: q (x - KL2)
//   RKL  ln2/tau and the sum of q log2(p/q): q (shift - log2(p/q))
//   FKL  1/tau: q - p
template <int KIND>
__device__ inline float grad_term(float c0, float c1, float scale, float shift) {
    if constexpr (KIND == 0)
        return (exp2_fast(c1) - c0) * scale;
    else if constexpr (KIND == 2)
        return (c1 * scale) * (c0 - shift);
    else
        return (c1 * scale) * (shift - c0);
}

// A row pair's merged softmax statistics and the row-uniform values derived
// from them (fp64), computed once per row pair by wave 0 and read from LDS by
// every thread: K, S of each row, T_t - T_s (T = K + log2 S, the log2
// normalisers), 1/S and log2 S.
struct RowPair {
    float kt, ks;
    double st, ss, dtd, ist, iss, lt, ls;
};

// A thread's scales for a row pair, from its shifts kt, ks in the rows and whether
// its sums are empty: at, as are 2^(k - K) / S, what an exponential of the thread
// times is its probability.
struct RowScales {
    PairScales k;
    float at, as;
};
__device__ inline RowScales row_scales(const RowPair& rp, float kt, bool none_t, float ks, bool none_s, float beta) {
    RowScales z;
    const float ct = float(double(rp.kt - kt) + rp.lt), cs = float(double(rp.ks - ks) + rp.ls);
    const int nt = int(fmaxf(kt - rp.kt, -2048.0f)), ns = int(fmaxf(ks - rp.ks, -2048.0f));
    // A thread without mass in a row has scale 0 there (its own shift may lie
    // far above the row's), and any positive ratio serves its zeros.
    z.at = none_t ? 0.0f : float(__builtin_ldexp(rp.ist, nt));
    z.as = none_s ? 0.0f : float(__builtin_ldexp(rp.iss, ns));
    z.k = PairScales{none_t || none_s ? 1.0f : float(__builtin_ldexp(rp.st * rp.iss, ns - nt)), beta, 1.0f - beta, ct, cs,
                     float(rp.dtd - double(kt - ks))};
    return z;
}

// Wave 0: merge the (K, S) pairs that lanes 0..15 hold (identity elsewhere) of
// both rows and store the row values.
__device__ inline void store_row_pair(float k0, double t0, float k1, double t1, int lane, RowPair* s_r) {
    row0_merge_stats_u(k0, t0);
    row0_merge_stats_u(k1, t1);
    // The three quotients and the three logarithms are taken side by side in
    // lanes 0-2 (one division and one log2_pos in sequence instead of three and
    // three): lane 0 t0/t1, lane 1 1/t0, lane 2 1/t1, then the log2 of t0/t1, t0
    // and t1.  Each value is the one the scalar formula gives.
    const double qv = (lane == 0 ? t0 : 1.0) / (lane == 1 ? t0 : t1);
    const double lv = log2_pos(lane == 0 ? qv : (lane == 1 ? t0 : t1));
    const double l_q = readlane_f64(lv, 0), l_t = readlane_f64(lv, 1), l_s = readlane_f64(lv, 2);
    const double i_t = readlane_f64(qv, 1), i_s = readlane_f64(qv, 2);
    if (lane == 0) {
        RowPair r;
        r.kt = k0;
        r.ks = k1;
        r.st = t0;
        r.ss = t1;
        r.dtd = double(k0 - k1) + (t0 == t1 ? 0.0 : l_q);
        r.ist = i_t;
        r.iss = i_s;
        r.lt = l_t;
        r.ls = l_s;
        *s_r = r;
    }
}

// Every wave merges its lanes' (K, S) pairs and posts them; after one
// barrier wave 0 merges the waves' pairs and derives the row values; after a
// second, every thread reads them.  The values are those of block_merge2
// followed by the same formulas, bit for bit.
template <int NW>
__device__ inline RowPair merge_row_pair(float Kt, double St, float Ks, double Ss, float* s_k, double* s_s,
                                         RowPair* s_r) {
    static_assert(NW <= 16, "the posted pairs fit one DPP row");
    const int t = opaque_tid(), lane = t & (kWave - 1), wid = t / kWave;
    wave_merge_stats_u(Kt, St);
    wave_merge_stats_u(Ks, Ss);
    if (lane == 0) {
        s_k[wid] = Kt;
        s_k[NW + wid] = Ks;
        s_s[wid] = St;
        s_s[NW + wid] = Ss;
    }
    __syncthreads();
    if (wid == 0) {
        float k0 = kNegInf, k1 = kNegInf;
        double t0 = 0.0, t1 = 0.0;
        if (lane < NW) {
            k0 = s_k[lane];
            k1 = s_k[NW + lane];
            t0 = s_s[lane];
            t1 = s_s[NW + lane];
        }
        store_row_pair(k0, t0, k1, t1, lane, s_r);
    }
    __syncthreads();
    return *s_r;
}
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// The LDS half of the cache: element e of chunk r of this thread, in float4
// slots laid out [r][e/4][tid] so that a wave's accesses are contiguous.
template <int W, int EPC>
struct LdsCache {
    f32x4_t* base;
    __device__ f32x4_t load(int r, int g) const { return base[(r * (EPC / 4) + g) * W + threadIdx.x]; }
    __device__ void store(int r, int g, const f32x4_t& v) const { base[(r * (EPC / 4) + g) * W + threadIdx.x] = v; }
};

// Masked sum and mean of the row divergences.  Each workgroup adds its rows
// in row order (D = 0 for masked-out rows) and posts the partial at the
// device-wide coherence point; the last workgroup to finish adds the
// partials in workgroup order, counts the mask, writes the loss and zeroes
// what it read.  The result depends only on the grid size.
// What the tail needs, staged in LDS at kernel start so that none of it stays
// in registers across the row loop.
struct LossTail {
    double* row_ws;
    uint32_t* done;
    float* loss_out;
    const uint8_t* mask;
    int nrows;
    int G;  // workgroups in the grid
};

template <int W>
__device__ inline void finish_loss(const LossTail& a, const double* s_part) {
    __shared__ int s_last;
    __shared__ double s_sum[W / kWave], s_cnt[W / kWave];
    // Thread indices recomputed from an opaque copy: values derived from them
    // before the row loop are then not kept alive across it.
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & (kWave - 1), wid = tid / kWave;
    const int G = a.G;
    __syncthreads();
    if (tid == 0) {
        __hip_atomic_exchange(&a.row_ws[blockIdx.x], s_part[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = int(arrive(a.done)) == G - 1;  // after the post completed
    }
    __syncthreads();
    if (!s_last) return;
    // Thread t adds partials t, t+W, ... (one each when G <= W).
    double sm = 0.0, cn = 0.0;
    for (int g = tid; g < G; g += W) sm += take_f64(&a.row_ws[g]);
    for (int r = tid; r < a.nrows; r += W) cn += (a.mask == nullptr || a.mask[r] != 0) ? 1.0 : 0.0;
    sm = wave_sum(sm);
    cn = wave_sum(cn);
    if (lane == 0) {
        s_sum[wid] = sm;
        s_cnt[wid] = cn;
    }
    __syncthreads();
    if (tid == 0) {
        double ts = 0.0, tc = 0.0;
        for (int w = 0; w < W / kWave; ++w) {
            ts += s_sum[w];
            tc += s_cnt[w];
        }
        a.loss_out[0] = tc > 0.0 ? float(ts / tc) : 0.0f;
        a.loss_out[1] = float(ts);
        take_u32(a.done);
    }
}

}  // namespace osd
