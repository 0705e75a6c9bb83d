// row_draw.hpp -- inverse-CDF draw over a register-resident row (pair), the
// sampling rule of the verification's extra token (Eq. 5 of
// arXiv:2310.07177, Appendix A.1) and of token sampling.
//
// Element masses are fp32; each thread's chunk sums are converted exactly to
// 2^-SH fixed point, so every partial sum of the CDF is an exact integer and
// the cells partition [0, Z) without gaps or overlaps whatever the reduction
// order.  The token is the first element (ascending id) whose running sum
// exceeds u*Z.
#pragma once

#include "osd_device.hpp"

namespace osd {

// x 2^SH as a whole number held in fp64, equal to the fixed-point value (an
// integer conversion takes more instructions).  Exact while every wave sum stays
// below 2^53: SH = 44 for masses of at most 1 per element (chunk sums at most
// 8, wave sums at most 2^53), SH = 52 for probabilities (a row's total 1).
template <int SH>
__device__ inline double fixed_f64(float x) {
    static_assert(SH <= 52, "a row's total must stay below 2^53");
    return floor(double(x) * double(1ull << SH));
}

struct DrawShared {
    int cell_round, cell_wave;
    unsigned long long target;  // offset of u*Z inside the winning cell
};

// The winning wave's last step (both draws): this lane's chunk of round
// nstar has masses m[] (sum s, added left to right from 0); target is the
// point's offset inside the wave's cell.  The lanes' fixed-point chunk sums
// are scanned to find the lane holding the target, which walks its elements
// with the same left-to-right fp32 sums.  Returns the element's place (chunk *
// EPC + e; RowCut::token gives its id) on that lane and -1 on the others.
template <int SH, int W, int EPC>
__device__ inline int walk_chunk(const float (&m)[EPC], float s, uint64_t target, int nstar) {
    const int tid = threadIdx.x;
    int pick = -1, last_pos = -1;
    const double v = fixed_f64<SH>(s);
    const double incl = wave_scan_add(v);
    const double lo = incl - v, t = double(target);
    if (!(v > 0.0 && lo <= t && t < incl)) return -1;
    const double want = t - lo;
    float run = 0.0f;
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        run = run + m[e];
        if (m[e] > 0.0f) last_pos = e;
        if (pick < 0 && fixed_f64<SH>(run) > want) pick = e;
    }
    if (pick < 0) pick = last_pos >= 0 ? last_pos : 0;
    return (nstar * W + tid) * EPC + pick;
}

// The cell that holds the point, from the totals of all cells (round n, wave w;
// n*NW + w < cells) in s_tot: s_draw receives its round (-1 if there is no mass),
// its wave and the point's offset inside it.  The point is floor(u * Z), or
// c_given when >= 0 (a point already chosen in a larger CDF of which this row is
// one part); either is clamped to Z - 1.  All threads call it; it opens and ends
// with a barrier.
template <int NW>
__device__ inline void locate_cell(int cells, const unsigned long long* s_tot, float u, long long c_given,
                                   DrawShared* s_draw) {
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    __syncthreads();
    if (wid == 0) {
        uint64_t z = 0;
        for (int c0 = lane; c0 < cells; c0 += kWave) z += s_tot[c0];
        z = wave_sum(z);
        if (lane == 0) s_draw->cell_round = -1;
        if (z > 0) {
            uint64_t c = c_given >= 0 ? static_cast<uint64_t>(c_given) : static_cast<uint64_t>(double(u) * double(z));
            if (c >= z) c = z - 1;
            uint64_t carry = 0;
            for (int base = 0; base < cells; base += kWave) {
                const int idx = base + lane;
                const uint64_t v = idx < cells ? uint64_t(s_tot[idx]) : 0;
                const uint64_t incl = wave_inclusive_scan(v) + carry;
                const uint64_t lo = incl - v;
                if (v > 0 && lo <= c && c < incl) {
                    s_draw->cell_round = idx / NW;
                    s_draw->cell_wave = idx % NW;
                    s_draw->target = c - lo;
                }
                carry = static_cast<uint64_t>(__shfl(static_cast<unsigned long long>(incl), kWave - 1, kWave));
            }
        }
    }
    __syncthreads();
}

// Inverse-CDF draw over a register-resident row pair.  mass(t, d, e) returns
// the non-negative fp32 mass of element e of the chunks t, d (0 for padding).
// Returns the drawn element's place (chunk * EPC + e) on exactly one thread and
// -1 on every other thread; *z_zero is set (uniformly) when the total mass is zero.  The point drawn is
// locate_cell's.
//
// Token order is (round n, wave w, lane, element e).  Chunk masses are summed
// left to right in fp32 and converted exactly to fixed point, so every partial
// sum below is an exact integer and the CDF cells (n, w) partition [0, Z)
// without gaps or overlaps whatever the reduction order.  The winning wave
// stages its chunks through LDS (s_stage, 2*CPT*64 chunks) so that the
// winning round is selected by address, never by register index.
template <int SH, int W, int CPT, int EPC, typename MassFn>
__device__ int draw_inverse_cdf(const chunk_t (&tv)[CPT], const chunk_t (&dv)[CPT], MassFn mass,
                                float u, unsigned long long* s_tot, DrawShared* s_draw,
                                chunk_t* s_stage, bool* z_zero, long long c_given = -1) {
    constexpr int NW = W / kWave;
    constexpr int CELLS = CPT * NW;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;

#pragma unroll
    for (int n = 0; n < CPT; ++n) {
        float s = 0.0f;
#pragma unroll
        for (int e = 0; e < EPC; ++e) s = s + mass(tv[n], dv[n], e);
        const double t = wave_sum(fixed_f64<SH>(s));
        if (lane == 0) s_tot[n * NW + wid] = uint64_t(t);
        __builtin_amdgcn_sched_barrier(0);
    }
    locate_cell<NW>(CELLS, s_tot, u, c_given, s_draw);
    const int nstar = s_draw->cell_round;
    *z_zero = nstar < 0;
    if (nstar < 0 || wid != s_draw->cell_wave) return -1;

    // Winning wave: stage every round through LDS, pick round nstar by address.
#pragma unroll
    for (int n = 0; n < CPT; ++n) {
        s_stage[n * kWave + lane] = tv[n];
        s_stage[(CPT + n) * kWave + lane] = dv[n];
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const chunk_t tc = s_stage[nstar * kWave + lane];
    const chunk_t dc = s_stage[(CPT + nstar) * kWave + lane];
    float m[EPC];
    float s = 0.0f;
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        m[e] = mass(tc, dc, e);
        s = s + m[e];
    }
    return walk_chunk<SH, W, EPC>(m, s, s_draw->target, nstar);
}

}  // namespace osd

namespace osd {

// Rounds of the longest row in a workgroup of 1024 threads (131072 bf16 or 65536
// fp32 logits per row).
constexpr int kMaxStreamRounds = 16;
// Cells (round, wave) of the longest row, whatever the workgroup's width.
constexpr int kMaxStreamCells = kMaxStreamRounds * (1024 / kWave);

// Inverse-CDF draw over a row whose chunk masses are already known: chunk[n] is
// the mass of this thread's chunk of round n (the left-to-right fp32 sum of its
// elements' masses up to rounding), element(n, m) fills m with the masses of the
// elements of the chunk of round n (a run-time, uniform n; called by one wave).
// Cells and result as draw_inverse_cdf.
template <int SH, int W, int CPT, int EPC, typename ElementFn>
__device__ int draw_from_sums(const float (&chunk)[CPT], ElementFn element, float u, unsigned long long* s_tot,
                              DrawShared* s_draw) {
    constexpr int NW = W / kWave;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
#pragma unroll
    for (int n = 0; n < CPT; ++n) {
        const double t = wave_sum(fixed_f64<SH>(chunk[n]));
        if (lane == 0) s_tot[n * NW + wid] = uint64_t(t);
    }
    locate_cell<NW>(CPT * NW, s_tot, u, -1, s_draw);
    const int nstar = s_draw->cell_round;
    if (nstar < 0 || wid != s_draw->cell_wave) return -1;
    float s = 0.0f;
#pragma unroll
    for (int n = 0; n < CPT; ++n)
        if (n == nstar) s = chunk[n];
    float m[EPC];
    element(nstar, m);
    return walk_chunk<SH, W, EPC>(m, s, s_draw->target, nstar);
}

// Inverse-CDF draw over a row (pair) that is streamed from memory instead of
// held in registers: U rounds of loads in flight per thread (one at a time, each
// round cost a memory latency).  mass(t, d, e) as in draw_inverse_cdf; use_d: whether the second
// row is read.  Pass A sums every chunk; pass B, by the winning wave, reads its
// round again.  Returns the element's place on one thread and -1 on the others;
// *z_zero is set (uniformly) when the total mass is zero.  s_tot holds R * (W / 64)
// cells.  All threads call it.
template <int SH, typename Fmt, int W, int U, typename MassFn>
__device__ int draw_inverse_cdf_streamed(const void* trow, const void* drow, bool use_d, const RowCut<Fmt>& cut,
                                         MassFn mass, float u, unsigned long long* s_tot, DrawShared* s_draw,
                                         bool* z_zero) {
    constexpr int NW = W / kWave, EPC = Fmt::kPerChunk;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const int R = (cut.nchunks + W - 1) / W;
    for (int r0 = 0; r0 < R; r0 += U) {
        chunk_t xt[U], xd[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int off = cut.off((r0 + k) * W + tid);
            xt[k] = load_off(trow, off);
            if (use_d) xd[k] = load_off(drow, off);
        }
        pad_row_tail<Fmt, W, U>(xt, cut, r0);
        if (use_d) pad_row_tail<Fmt, W, U>(xd, cut, r0);
#pragma unroll
        for (int k = 0; k < U; ++k) {
            float s = 0.0f;
#pragma unroll
            for (int e = 0; e < EPC; ++e) s = s + mass(xt[k], xd[k], e);
            const double t = wave_sum(fixed_f64<SH>(s));
            if (lane == 0 && r0 + k < R) s_tot[(r0 + k) * NW + wid] = uint64_t(t);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    locate_cell<NW>(R * NW, s_tot, u, -1, s_draw);
    const int nstar = s_draw->cell_round;
    *z_zero = nstar < 0;
    if (nstar < 0 || wid != s_draw->cell_wave) return -1;
    const chunk_t tc = stream_chunk<Fmt, W>(trow, nstar, cut);
    const chunk_t dc = use_d ? stream_chunk<Fmt, W>(drow, nstar, cut) : tc;
    float m[EPC];
    float s = 0.0f;
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        m[e] = mass(tc, dc, e);
        s = s + m[e];
    }
    return walk_chunk<SH, W, EPC>(m, s, s_draw->target, nstar);
}

}  // namespace osd
