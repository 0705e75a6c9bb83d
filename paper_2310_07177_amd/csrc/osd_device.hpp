// osd_device.hpp -- device-side building blocks shared by the verification and
// distillation kernels (gfx950, wave64).
//
// Rows are read as 16-byte chunks (8 bf16 or 4 fp32 logits).  A workgroup of W
// threads holds a row in registers as CPT chunks per thread: chunk n*W + tid
// for round n, so each round is one fully coalesced sweep over W*16 bytes and
// token ids grow with (round, thread, element).
//
// A row may start at any element and have any length of at least one chunk
// (RowCut): 16-byte loads from addresses that are not 16-byte multiples are
// part of the gfx950 memory model.  A read of 8192 rows of V = 32003 bf16 logits
// that way runs at 5.0 TB/s (rows on 4-byte boundaries 6.3, on 16-byte ones
// 6.7).  Element by element, verification of B = 32, K = 8, V = 32003 took
// 38.6 us and takes 18.9, verification and distillation of B = 32, K = 6,
// V = 50257 89.5 and 51.5.  Only rows shorter than one chunk are read element
// by element (VEC = false).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace osd {

constexpr int kWave = 64;

// One 16-byte chunk of a row (a native vector so that loads stay dwordx4).
typedef uint32_t chunk_t __attribute__((ext_vector_type(4)));
constexpr float kNegInf = -__builtin_huge_valf();
constexpr float kLog2e = 1.4426950408889634f;
constexpr double kLn2 = 0.69314718055994530942;

// ---------------------------------------------------------------------------
// Exponentials.  v_exp_f32 computes 2^x; scaled logits are formed as
// (x - max) * log2(e)/T so that the term carrying the mass is exact-ish.
// ---------------------------------------------------------------------------
__device__ inline float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ inline float log2_fast(float x) { return __builtin_amdgcn_logf(x); }

// ---------------------------------------------------------------------------
// Logit formats
// ---------------------------------------------------------------------------
struct BF16 {
    static constexpr int kPerChunk = 8;
    static constexpr int kBytes = 2;
    // One padding element: -inf has zero probability and never wins a max.
    static constexpr uint16_t kPad = 0xFF80u;
    __device__ static inline float get(const chunk_t& c, int e) {
        const uint32_t w = (e >> 1) == 0 ? c.x : (e >> 1) == 1 ? c.y : (e >> 1) == 2 ? c.z : c.w;
        return (e & 1) ? __uint_as_float(w & 0xFFFF0000u) : __uint_as_float(w << 16);
    }
    __device__ static inline float load_one(const void* row, int j) {
        return __uint_as_float(uint32_t(static_cast<const uint16_t*>(row)[j]) << 16);
    }
    // The bits of element j, and their value (a load kept apart from its use).
    __device__ static inline uint32_t load_raw(const void* row, int j) { return static_cast<const uint16_t*>(row)[j]; }
    __device__ static inline float from_raw(uint32_t r) { return __uint_as_float(r << 16); }
    __device__ static inline chunk_t load_scalar(const void* row, int64_t first, int V) {
        const uint16_t* p = static_cast<const uint16_t*>(row);
        uint16_t v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (first + e < V) ? p[first + e] : kPad;
        chunk_t c;
        c.x = v[0] | (uint32_t(v[1]) << 16);
        c.y = v[2] | (uint32_t(v[3]) << 16);
        c.z = v[4] | (uint32_t(v[5]) << 16);
        c.w = v[6] | (uint32_t(v[7]) << 16);
        return c;
    }
};

struct F32 {
    static constexpr int kPerChunk = 4;
    static constexpr int kBytes = 4;
    __device__ static inline float get(const chunk_t& c, int e) {
        const uint32_t w = e == 0 ? c.x : e == 1 ? c.y : e == 2 ? c.z : c.w;
        return __uint_as_float(w);
    }
    __device__ static inline float load_one(const void* row, int j) {
        return static_cast<const float*>(row)[j];
    }
    __device__ static inline uint32_t load_raw(const void* row, int j) { return static_cast<const uint32_t*>(row)[j]; }
    __device__ static inline float from_raw(uint32_t r) { return __uint_as_float(r); }
    __device__ static inline chunk_t load_scalar(const void* row, int64_t first, int V) {
        const float* p = static_cast<const float*>(row);
        uint32_t v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            v[e] = (first + e < V) ? __float_as_uint(p[first + e]) : 0xFF800000u;
        return chunk_t{v[0], v[1], v[2], v[3]};
    }
};

// Whole chunk of padding (past the end of the row).
template <typename Fmt>
__device__ inline chunk_t pad_chunk() {
    if constexpr (Fmt::kPerChunk == 8)
        return chunk_t{0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u};
    else
        return chunk_t{0xFF800000u, 0xFF800000u, 0xFF800000u, 0xFF800000u};
}

// How a row of V elements (at least one chunk) is cut into chunks.  Chunk ch
// starts at element ch*kPerChunk, except that the last chunk of a row whose
// length is not a whole number of chunks is moved back to end with the row:
// its first `dup` elements belong to the chunk before it and count as
// padding.  Chunks past the row re-read the last one and are all padding.  (In
// a row shorter than one chunk the only chunk starts before the row: its
// elements are loaded one by one, load_short.)
template <typename Fmt>
struct RowCut {
    int nchunks;   // chunks that hold elements of the row
    int nfull;     // chunks before the first one with any padding
    int dup;       // padding elements at the head of the last chunk
    int last_off;  // byte offset of the last chunk
    __device__ explicit RowCut(int V) {
        constexpr int EPC = Fmt::kPerChunk;
        nchunks = (V + EPC - 1) / EPC;
        dup = nchunks * EPC - V;
        nfull = dup ? nchunks - 1 : nchunks;
        last_off = (V - EPC) * Fmt::kBytes;
    }
    __device__ int off(int ch) const { return min(ch * 16, last_off); }
    // Leading elements of chunk ch that are padding.
    __device__ int lead(int ch) const { return ch < nfull ? 0 : (ch < nchunks ? dup : Fmt::kPerChunk); }
    // The token id of element e of chunk ch, given as ch*kPerChunk + e.
    __device__ int token(int t) const { return t >= nfull * Fmt::kPerChunk ? t - dup : t; }
    // Whether round n of a workgroup of W threads holds any padding (uniform).
    template <int W>
    __device__ bool ragged(int n) const { return (n + 1) * W > nfull; }
};

// A 16-byte load from any element of a row.
typedef chunk_t chunk_any_t __attribute__((aligned(2)));
__device__ inline chunk_t load_off(const void* row, int off) {
    return __builtin_nontemporal_load(reinterpret_cast<const chunk_any_t*>(static_cast<const char*>(row) + off));
}

// The chunk with its first `lead` elements replaced by padding.  (An opaque
// copy of lead: its comparisons, needed by one wave per row, would otherwise be
// hoisted out of a row loop and held in scalar registers.)
template <typename Fmt>
__device__ inline chunk_t pad_lead(const chunk_t& c, int lead) {
    asm volatile("" : "+v"(lead));
    const chunk_t pad = pad_chunk<Fmt>();
    if constexpr (Fmt::kPerChunk == 8) {
        const auto w = [lead](uint32_t x, int e) {
            const uint32_t p = 0xFF80u;
            return lead > e + 1 ? (p | (p << 16)) : (lead > e ? (x & 0xFFFF0000u) | p : x);
        };
        return chunk_t{w(c.x, 0), w(c.y, 2), w(c.z, 4), w(c.w, 6)};
    } else {
        return chunk_t{lead > 0 ? pad.x : c.x, lead > 1 ? pad.y : c.y, lead > 2 ? pad.z : c.z, lead > 3 ? pad.w : c.w};
    }
}

// The only chunk of a row of V < kPerChunk elements (they end the chunk).
template <typename Fmt>
__device__ inline chunk_t load_short(const void* row, int V) {
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int e = 0; e < Fmt::kPerChunk; ++e) {
        const int j = e - (Fmt::kPerChunk - V);
        if constexpr (Fmt::kPerChunk == 8)
            w[e >> 1] |= (j >= 0 ? Fmt::load_raw(row, j) : uint32_t(Fmt::kPad)) << (16 * (e & 1));
        else
            w[e] = j >= 0 ? Fmt::load_raw(row, j) : 0xFF800000u;
    }
    return chunk_t{w[0], w[1], w[2], w[3]};
}

// Writes a thread's chunks of a row back: 16-byte stores, except that the last
// chunk, when it shares elements with the chunk before it, is kept until
// finish() stores its own elements one by one (one copy of that code, outside
// the unrolled rounds).
template <typename Fmt>
struct RowWriter {
    char* row;
    const RowCut<Fmt>& cut;
    chunk_t tail = chunk_t{0u, 0u, 0u, 0u};
    bool has_tail = false;
    __device__ RowWriter(void* r, const RowCut<Fmt>& c) : row(static_cast<char*>(r)), cut(c) {}
    __device__ void put(int ch, const chunk_t& c) {
        if (ch < cut.nfull) {
            __builtin_nontemporal_store(c, reinterpret_cast<chunk_any_t*>(row + ch * 16));
        } else if (ch < cut.nchunks) {
            tail = c;
            has_tail = true;
        }
    }
    __device__ void finish() {
        if (!has_tail) return;
        const uint32_t w[4] = {tail.x, tail.y, tail.z, tail.w};
#pragma unroll
        for (int e = 0; e < Fmt::kPerChunk; ++e) {
            if (e < cut.dup) continue;
            if constexpr (Fmt::kPerChunk == 8)
                reinterpret_cast<uint16_t*>(row + cut.last_off)[e] = uint16_t(w[e >> 1] >> (16 * (e & 1)));
            else
                reinterpret_cast<uint32_t*>(row + cut.last_off)[e] = w[e];
        }
    }
};

// Load the CPT chunks of one row owned by this thread, as loaded: the
// padding is applied where a chunk is first used (row_stats, pad_row_tail), so
// no instruction right after the loads needs their data and each sweep waits
// only for the chunk it takes next.  VEC = false: a row shorter than one
// chunk, element by element, padded.
template <typename Fmt, int W, int CPT, bool VEC>
__device__ inline void load_row(chunk_t (&c)[CPT], const void* row, const RowCut<Fmt>& cut, int V) {
#pragma unroll
    for (int n = 0; n < CPT; ++n) {
        const int ch = n * W + static_cast<int>(threadIdx.x);
        if constexpr (VEC)
            c[n] = load_off(row, cut.off(ch));
        else
            c[n] = ch == 0 ? Fmt::load_scalar(row, 0, V) : pad_chunk<Fmt>();
    }
}

// Two rows loaded as load_row loads each, chunk by chunk in turn (a0, b0,
// a1, b1, ...), the order in which row_stats2 takes them.
template <typename Fmt, int W, int CPT>
__device__ inline void load_rows_interleaved(chunk_t (&a)[CPT], chunk_t (&b)[CPT], const void* ra, const void* rb,
                                             const RowCut<Fmt>& cut) {
#pragma unroll
    for (int n = 0; n < CPT; ++n) {
        const int off = cut.off(n * W + static_cast<int>(threadIdx.x));
        a[n] = load_off(ra, off);
        b[n] = load_off(rb, off);
    }
}

// Chunk n of this thread as loaded by load_row<VEC>, padding if it lies past
// the row.  Rounds before the row's end take no instruction for it.
template <typename Fmt, int W>
__device__ inline chunk_t chunk_or_pad(const chunk_t& c, int n, const RowCut<Fmt>& cut) {
    if (!cut.template ragged<W>(n)) return c;
    const bool in = n * W + static_cast<int>(threadIdx.x) < cut.nchunks;
    const chunk_t pad = pad_chunk<Fmt>();
    return chunk_t{in ? c.x : pad.x, in ? c.y : pad.y, in ? c.z : pad.z, in ? c.w : pad.w};
}

// Pad the shared head of the row's last chunk in the wave that holds it (among
// rounds first .. first + CPT - 1), as soon as its load has landed.  Kept apart
// from the per-chunk code so that the other waves skip it on one branch: in a
// kernel of a few microseconds the instruction fetch past sixteen inline copies
// cost 0.5 us.
template <typename Fmt, int W, int CPT>
__device__ inline void pad_shared_head(chunk_t (&c)[CPT], const RowCut<Fmt>& cut, int first = 0) {
    const int n = (cut.nchunks - 1) / W - first, t = (cut.nchunks - 1) % W;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
    if (cut.dup == 0 || n < 0 || n >= CPT || t / kWave != wave) return;
    const int lead = static_cast<int>(threadIdx.x) == t ? cut.dup : 0;
#pragma unroll
    for (int r = 0; r < CPT; ++r)
        if (r == n) c[r] = pad_lead<Fmt>(c[r], lead);
}

// Apply the padding to every chunk of load_row<VEC>.
template <typename Fmt, int W, int CPT>
__device__ inline void pad_row_tail(chunk_t (&c)[CPT], const RowCut<Fmt>& cut, int first = 0) {
    pad_shared_head<Fmt, W, CPT>(c, cut, first);
#pragma unroll
    for (int n = 0; n < CPT; ++n) c[n] = chunk_or_pad<Fmt, W>(c[n], first + n, cut);
}

// Make register-resident chunks opaque to the optimiser at the start of a
// sweep.  Unpacking a bf16 pair costs one instruction; without this the
// compiler keeps every unpacked value of an earlier sweep alive to reuse it,
// which doubles the register footprint of a row and spills.
template <int CPT>
__device__ inline void opaque(chunk_t (&c)[CPT]) {
#pragma unroll
    for (int n = 0; n < CPT; ++n) asm volatile("" : "+v"(c[n]));
}

// ---------------------------------------------------------------------------
// Wave64 reductions and scans on DPP (data-parallel primitives: operand lane
// permutations inside the vector ALU).  Lane shuffles compile to LDS permute
// round trips; these do not.  Steps: row_shr 1, 2, 4, 8 form inclusive
// prefixes inside each row of 16 lanes, then row_bcast 15 and 31 carry the row
// totals into the later rows.  Lanes whose source is outside the row (or a
// disabled row) take the identity.  The order of operations is fixed, so
// results are reproducible.  The total ends in lane 63; readlane broadcasts it.
// ---------------------------------------------------------------------------
enum : int { kDppRowShr1 = 0x111, kDppRowShr2 = 0x112, kDppRowShr4 = 0x114, kDppRowShr8 = 0x118,
             kDppRowBcast15 = 0x142, kDppRowBcast31 = 0x143 };

template <int CTRL, int ROWS>
__device__ inline uint32_t dpp(uint32_t identity, uint32_t v) {
    return uint32_t(__builtin_amdgcn_update_dpp(int(identity), int(v), CTRL, ROWS, 0xF, false));
}
__device__ inline uint32_t readlane_u32(uint32_t v, int lane) {
    return uint32_t(__builtin_amdgcn_readlane(int(v), lane));
}
__device__ inline float readlane_f32(float v, int lane) {
    return __uint_as_float(readlane_u32(__float_as_uint(v), lane));
}
__device__ inline uint64_t readlane_u64(uint64_t v, int lane) {
    return uint64_t(readlane_u32(uint32_t(v), lane)) | (uint64_t(readlane_u32(uint32_t(v >> 32), lane)) << 32);
}
__device__ inline double readlane_f64(double v, int lane) {
    return __builtin_bit_cast(double, readlane_u64(__builtin_bit_cast(uint64_t, v), lane));
}

// Floats as unsigned keys in the same order (no NaN): a float maximum over
// lanes becomes an unsigned one, which the DPP move folds into (identity 0)
// and which needs no NaN quieting of each operand.
__device__ inline uint32_t float_key(float f) {
    const uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ inline float key_float(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}
template <int CTRL, int ROWS>
__device__ inline uint32_t dpp_umax_step(uint32_t k) {
    const uint32_t o = dpp<CTRL, ROWS>(0u, k);
    return k > o ? k : o;
}
// A 32-bit lane permutation for a sum (identity 0).  Every row enabled
// (the row shifts): lanes whose source is outside the row read 0 through
// the bound control, and no register has to be preset to the identity.
template <int CTRL, int ROWS>
__device__ inline uint32_t dpp_sum_src(uint32_t v) {
    if constexpr (ROWS == 0xF)
        return uint32_t(__builtin_amdgcn_mov_dpp(int(v), CTRL, 0xF, 0xF, true));
    else
        return dpp<CTRL, ROWS>(0u, v);
}
template <int CTRL, int ROWS>
__device__ inline double dpp_add_step(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint64_t o = uint64_t(dpp_sum_src<CTRL, ROWS>(uint32_t(b))) |
                       (uint64_t(dpp_sum_src<CTRL, ROWS>(uint32_t(b >> 32))) << 32);
    return v + __builtin_bit_cast(double, o);
}
template <int CTRL, int ROWS>
__device__ inline uint64_t dpp_add_step(uint64_t v) {
    const uint64_t o = uint64_t(dpp_sum_src<CTRL, ROWS>(uint32_t(v))) |
                       (uint64_t(dpp_sum_src<CTRL, ROWS>(uint32_t(v >> 32))) << 32);
    return v + o;
}

// Inclusive scans over the wave (lane 63 holds the total).
template <typename T>
__device__ inline T wave_scan_add(T v) {
    v = dpp_add_step<kDppRowShr1, 0xF>(v);
    v = dpp_add_step<kDppRowShr2, 0xF>(v);
    v = dpp_add_step<kDppRowShr4, 0xF>(v);
    v = dpp_add_step<kDppRowShr8, 0xF>(v);
    v = dpp_add_step<kDppRowBcast15, 0xA>(v);
    v = dpp_add_step<kDppRowBcast31, 0xC>(v);
    return v;
}


// Wave totals and scans on the primitives above; every lane gets the total.
__device__ inline float wave_max(float v) {  // values without NaN
    uint32_t k = float_key(v);
    k = dpp_umax_step<kDppRowShr1, 0xF>(k);
    k = dpp_umax_step<kDppRowShr2, 0xF>(k);
    k = dpp_umax_step<kDppRowShr4, 0xF>(k);
    k = dpp_umax_step<kDppRowShr8, 0xF>(k);
    k = dpp_umax_step<kDppRowBcast15, 0xA>(k);
    k = dpp_umax_step<kDppRowBcast31, 0xC>(k);
    return key_float(readlane_u32(k, kWave - 1));
}
__device__ inline double wave_sum(double v) { return readlane_f64(wave_scan_add(v), kWave - 1); }
__device__ inline uint64_t wave_sum(uint64_t v) { return readlane_u64(wave_scan_add(v), kWave - 1); }
__device__ inline uint64_t wave_inclusive_scan(uint64_t v) { return wave_scan_add(v); }

// Max value, lowest index among equal maxima.
__device__ inline void wave_argmax(float& v, int& idx) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ov = __shfl_xor(v, o, kWave);
        const int oi = __shfl_xor(idx, o, kWave);
        if (ov > v || (ov == v && oi < idx)) {
            v = ov;
            idx = oi;
        }
    }
}

// ---------------------------------------------------------------------------
// Streaming softmax statistics of a register-resident row.
//
// Each thread keeps S = sum_j 2^(x_j c2 - K) over its elements, where c2 =
// log2(e)/T and the shift K is a whole number at least ceil(max_j x_j c2).
// Chunks are folded in as their loads land (no barrier between the maximum
// and the sum); raising K rescales S by an exact power of two (ldexp), so
// the statistics carry no rounding from the shift.  Lanes and waves merge
// the same way.  A row without finite logits ends with K = -inf, S = 0.
// ---------------------------------------------------------------------------
template <typename Fmt>
__device__ inline float chunk_max(const chunk_t& c) {
    float m = Fmt::get(c, 0);
#pragma unroll
    for (int e = 1; e < Fmt::kPerChunk; ++e) m = fmaxf(m, Fmt::get(c, e));
    return m;
}

// 2^(from - to) * S for whole numbers from <= to (exact; -inf/NaN -> 0).
__device__ inline float rescale(float S, float from, float to) {
    return __builtin_ldexpf(S, int(fmaxf(from - to, -256.0f)));
}
__device__ inline double rescale(double S, float from, float to) {
    return __builtin_ldexp(S, int(fmaxf(from - to, -2048.0f)));
}

// Fold one chunk into a thread's (K, S): fp32 accumulation, pairwise within
// the chunk.
template <typename Fmt>
__device__ inline void fold_chunk(const chunk_t& x, float c2, float& K, float& S) {
    constexpr int EPC = Fmt::kPerChunk;
    const float kn = fmaxf(K, ceilf(chunk_max<Fmt>(x) * c2));
    S = rescale(S, K, kn);
    K = kn;
    // While K is still -inf every element seen is -inf: a finite stand-in
    // keeps 2^(x c2 - K) at 2^-inf = 0 instead of -inf + inf = NaN.
    const float kx = fmaxf(K, -3.0e38f);
    float e8[EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) e8[e] = exp2_fast(__builtin_fmaf(Fmt::get(x, e), c2, -kx));
#pragma unroll
    for (int w = 1; w < EPC; w <<= 1)
#pragma unroll
        for (int e = 0; e < EPC; e += 2 * w) e8[e] = e8[e] + e8[e + w];
    S = S + e8[0];
}

// The same with every term accumulated in fp64 (for quantities first-order
// sensitive to the normaliser).
template <typename Fmt>
__device__ inline void fold_chunk(const chunk_t& x, float c2, float& K, double& S) {
    constexpr int EPC = Fmt::kPerChunk;
    const float kn = fmaxf(K, ceilf(chunk_max<Fmt>(x) * c2));
    S = rescale(S, K, kn);
    K = kn;
    const float kx = fmaxf(K, -3.0e38f);
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int e = 0; e < EPC; e += 2) {
        s0 += double(exp2_fast(__builtin_fmaf(Fmt::get(x, e), c2, -kx)));
        s1 += double(exp2_fast(__builtin_fmaf(Fmt::get(x, e + 1), c2, -kx)));
    }
    S += s0 + s1;
}

// A row's statistics over chunks from load_row, in its precision Acc.  VEC:
// each chunk is padded, in place, as the sweep takes it (after its load has
// landed).
template <typename Fmt, int W, int CPT, bool VEC, typename Acc>
__device__ inline void row_stats(chunk_t (&c)[CPT], const RowCut<Fmt>& cut, float c2, float& K, Acc& S) {
    if constexpr (VEC) pad_shared_head<Fmt, W, CPT>(c, cut);
#pragma unroll
    for (int n = 0; n < CPT; ++n) {
        if constexpr (VEC) c[n] = chunk_or_pad<Fmt, W>(c[n], n, cut);
        fold_chunk<Fmt>(c[n], c2, K, S);
        __builtin_amdgcn_sched_barrier(0);  // one chunk in flight: bounded VGPRs
    }
}

// Two rows from load_rows_interleaved swept together: chunk n of both rows
// in iteration n, in the order the loads were issued, each row folded exactly
// as row_stats folds it.  With second == false only the first row is folded
// (its partner's loads are ignored).
template <typename Fmt, int W, int CPT>
__device__ inline void row_stats2(chunk_t (&a)[CPT], chunk_t (&b)[CPT], const RowCut<Fmt>& cut, float c2, bool second,
                                  float& Ka, float& Sa, float& Kb, float& Sb) {
    pad_shared_head<Fmt, W, CPT>(a, cut);
    if (second) pad_shared_head<Fmt, W, CPT>(b, cut);
#pragma unroll
    for (int n = 0; n < CPT; ++n) {
        a[n] = chunk_or_pad<Fmt, W>(a[n], n, cut);
        fold_chunk<Fmt>(a[n], c2, Ka, Sa);
        if (second) {
            b[n] = chunk_or_pad<Fmt, W>(b[n], n, cut);
            fold_chunk<Fmt>(b[n], c2, Kb, Sb);
        }
        __builtin_amdgcn_sched_barrier(0);  // one chunk pair in flight: bounded VGPRs
    }
}

// Chunk n*W + tid of a row streamed from memory, padded.
template <typename Fmt, int W>
__device__ inline chunk_t stream_chunk(const void* row, int n, const RowCut<Fmt>& cut) {
    const int ch = n * W + static_cast<int>(threadIdx.x);
    const chunk_t c = load_off(row, cut.off(ch));
    return cut.template ragged<W>(n) ? pad_lead<Fmt>(c, cut.lead(ch)) : c;
}

// Merge (K, S) across the wave; every lane returns the wave's pair.
template <typename Acc>
__device__ inline void wave_merge_stats(float& K, Acc& S) {
    const float kw = wave_max(K);
    S = wave_sum(rescale(S, K, kw));
    K = kw;
}

// ---------------------------------------------------------------------------
// Fixed-point probability mass.  A non-negative fp32 value x < 2^(63-SH) maps
// to floor(x * 2^SH); the conversion is exact for x >= 2^(23-SH) (the
// mantissa is shifted, not rounded).  Integer sums of such values are
// associative, so every reduction order partitions a CDF identically.
// Values outside the domain never shift by 64 or more: negatives and
// subnormals give 0, and anything at or above 2^(63-SH) -- infinities and
// NaN included -- saturates at 2^39 * (2^24 - 1) < 2^63.  (Callers reject
// rows whose sums are not finite before they draw, so none reaches a draw.)
// ---------------------------------------------------------------------------
template <int SH>
__device__ inline uint64_t mass_to_fixed(float x) {
    const uint32_t b = __float_as_uint(x);
    const int e = int((b >> 23) & 0xFF) - 127;
    if (e < -126 || (b >> 31)) return 0;  // zero, subnormal or negative
    const uint64_t m = uint64_t((b & 0x7FFFFFu) | 0x800000u);
    int sh = e + SH - 23;  // x * 2^SH = m * 2^(e - 23 + SH)
    if (sh > 39) sh = 39;  // beyond the domain: saturate below 2^63
    if (sh >= 0) return m << sh;
    if (sh <= -64) return 0;
    return m >> (-sh);
}

// A row's sum of exponentials that a draw or a test can use: positive and
// finite (a NaN logit makes it NaN, an overflow makes it infinite).
__device__ inline bool usable_sum(double s) { return s > 0.0 && s < 1.0e300; }

// Two fp32 values to a packed pair of bf16, round to nearest even, with the
// native v_cvt_pk_bf16_f32 of gfx950.
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ inline uint32_t pack_bf16x2(float lo, float hi) {
    const f32x2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// ---------------------------------------------------------------------------
// Cross-workgroup hand-off through device memory, without cache flushes.
//
// Every word that crosses workgroups is written and read with agent-scope
// atomic operations, which the hardware performs at the device-wide coherence
// point (not in an XCD's private L2).  A publisher waits for its payload to be in
// place (s_waitcnt) before it bumps the arrival counter; the last arriver reads
// (and clears) the payloads after its counter RMW returned.  Where workgroups
// exchange words without a counter (the split rows), no word is ever zero and
// readers poll the words themselves, a bounded number of times; the counter that
// decides who clears them is still bumped after the words.  Release/acquire fences
// would instead write back and invalidate the whole L2 of the XCD on every arrival.
// ---------------------------------------------------------------------------
__device__ inline void wait_memory() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The publishing RMWs return their old value (consumed by an empty asm) so
// that the hardware reports their completion to the waiting s_waitcnt.
__device__ inline void publish_u32(uint32_t* p, uint32_t v) {
    uint32_t old = __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" ::"v"(old));
}
__device__ inline uint32_t take_u32(uint32_t* p) {  // read and clear
    return __hip_atomic_exchange(p, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void publish_f64(double* p, double v) {
    double old = __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" ::"v"(old));
}
__device__ inline double take_f64(double* p) {
    return __hip_atomic_exchange(p, 0.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void publish_u64(uint64_t* p, uint64_t v) {
    uint64_t old = __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" ::"v"(old));
}
__device__ inline uint64_t take_u64(uint64_t* p) {  // read and clear
    return __hip_atomic_exchange(p, uint64_t(0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline uint64_t poll_u64(const uint64_t* p) {
    return __hip_atomic_load(const_cast<uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline uint32_t load_relaxed(const uint32_t* p) {
    return __hip_atomic_load(const_cast<uint32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Arrive at a counter; returns the number of earlier arrivals.  The caller's
// payload RMWs have completed before the add is issued.
__device__ inline uint32_t arrive(uint32_t* counter) {
    wait_memory();
    const uint32_t prev = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    wait_memory();
    return prev;
}

}  // namespace osd
