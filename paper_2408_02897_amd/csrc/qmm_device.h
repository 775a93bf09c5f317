// Device-side helpers shared by the HIP kernels of libqmm: number formats of the
// paper (INT8, E4M3, E5M2; Methodology, Eq. 1 and the implementation bullets),
// their round-to-nearest-even and stochastic encoders, the Philox4x32-10 counter
// generator, and wavefront (64-lane) reductions.  gfx950 only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qmm.h"

namespace qmm {

#define QMM_DEV __device__ __forceinline__

constexpr int kWave = 64;

QMM_DEV float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

// ---------------------------------------------------------------------------
// Format constants.  E4M3: 1-4-3, bias 7, max 448 (0x7E), min normal 2^-6,
// min subnormal 2^-9, one NaN pattern, no inf.  E5M2: 1-5-2, bias 15, max
// 57344 (0x7B), min normal 2^-14, min subnormal 2^-16.
// ---------------------------------------------------------------------------
template <int FMT> struct Fp8;
template <> struct Fp8<QMM_FMT_E4M3> {
    static constexpr int M = 3, BIAS = 7;
    static constexpr uint32_t MAX_BITS = 0x43E00000u;      // 448.0f
    static constexpr uint32_t MINNORM_BITS = 0x3C800000u;  // 2^-6
    static constexpr float TO_SUBNORMAL_UNITS = 512.0f;    // 1 / min subnormal
};
template <> struct Fp8<QMM_FMT_E5M2> {
    static constexpr int M = 2, BIAS = 15;
    static constexpr uint32_t MAX_BITS = 0x47600000u;      // 57344.0f
    static constexpr uint32_t MINNORM_BITS = 0x38800000u;  // 2^-14
    static constexpr float TO_SUBNORMAL_UNITS = 65536.0f;
};

// Nearest finite FP8 value, ties to the even mantissa, saturating, sign kept, NaN -> 0x7F, for two values at once through the
// hardware converter: v_cvt_pk_fp8_f32 / v_cvt_pk_bf8_f32 round to nearest even onto the OCP grids including subnormals and
// keep the sign of zero; clamping to +-max first gives the saturation rule, NaN is handled here.  Equal to the oracle's integer
// arithmetic for every bfloat16 and for binary32 values of every upper half with the lower half at and around the ties.
// Returns code(t0) | code(t1) << 8.
template <int FMT> QMM_DEV uint32_t encode_fp8_rtne_pair(float t0, float t1)
{
    const float mx = FMT == QMM_FMT_E4M3 ? 448.0f : 57344.0f;
    const float c0 = __builtin_amdgcn_fmed3f(t0, -mx, mx), c1 = __builtin_amdgcn_fmed3f(t1, -mx, mx);
    uint32_t r;
    if constexpr (FMT == QMM_FMT_E4M3) r = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(c0, c1, 0, false);
    else r = (uint32_t)__builtin_amdgcn_cvt_pk_bf8_f32(c0, c1, 0, false);
    r &= 0xFFFFu;
    if (t0 != t0) r = (r & 0xFF00u) | 0x7Fu;
    if (t1 != t1) r = (r & 0x00FFu) | 0x7F00u;
    return r;
}

// Eq. 1 for INT8: round half to even, keep the symmetric range [-127, 127].
QMM_DEV uint32_t encode_int8_rtne(float t)
{
    const float c = fminf(fmaxf(t, -127.0f), 127.0f);
    const int q = (int)__builtin_rintf(c);
    return (t != t) ? 0u : ((uint32_t)q & 0xFFu);
}

// 16 bfloat16 values (two 16-byte vectors) times rho -> 16 RTNE codes (one 16-byte vector).
typedef unsigned int qmm_u32x4 __attribute__((ext_vector_type(4)));
template <int FMT> QMM_DEV qmm_u32x4 encode16_bf16_rtne(qmm_u32x4 w0, qmm_u32x4 w1, float rho)
{
    qmm_u32x4 out;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t wa = q < 2 ? w0[2 * q] : w1[2 * q - 4], wb = q < 2 ? w0[2 * q + 1] : w1[2 * q - 3];
        const float t0 = __uint_as_float(wa << 16) * rho, t1 = __uint_as_float(wa & 0xFFFF0000u) * rho;
        const float t2 = __uint_as_float(wb << 16) * rho, t3 = __uint_as_float(wb & 0xFFFF0000u) * rho;
        if constexpr (FMT == QMM_FMT_INT8)
            out[q] = encode_int8_rtne(t0) | (encode_int8_rtne(t1) << 8) | (encode_int8_rtne(t2) << 16) | (encode_int8_rtne(t3) << 24);
        else
            out[q] = encode_fp8_rtne_pair<FMT>(t0, t1) | (encode_fp8_rtne_pair<FMT>(t2, t3) << 16);
    }
    return out;
}

// Stochastic rounding: up iff u24 / 2^24 < (|t| - lo) / (hi - lo), u24 the top 24 bits of a random word.  With Y the
// magnitude in units of the grid step there, times 2^24 and rounded up to an integer, that is a carry into bit 24 of
// Y + (2^24 - 1 - u24): u24 < frac holds iff u24 < ceil(frac).  2^24 - 1 - u24 is the top of the word's complement.  In a
// format's normal range the magnitude's own bit pattern is Y (23 - M fraction bits, so the complement is shifted by
// M + 1 more); below it, and for INT8, Y comes from an exact multiplication by a power of two.
// Four elements -> four codes in a dword.  What is rare in a scaled tensor -- magnitudes below the normal range, NaN -- is
// looked for once for the four, and a wavefront without any goes past it.  (E4M3, 16384 x 4096 normal values, rows
// contracting: 51.8 us; with both ranges computed for every element and selected 66.7, with a branch per element 59.5.)
template <int FMT> QMM_DEV uint32_t encode_sr4(const float* t, const uint32_t* word)
{
    uint32_t code[4];
    if constexpr (FMT == QMM_FMT_INT8) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float y = __builtin_ceilf(fminf(fabsf(t[i]), 127.0f) * 16777216.0f);     // exact product; at most 127 * 2^24
            const int r = (int)(((uint32_t)y + (~word[i] >> 8)) >> 24);
            code[i] = (uint32_t)((__float_as_uint(t[i]) >> 31) ? -r : r) & 0xFFu;
        }
    } else {
        using F = Fp8<FMT>;
        uint32_t a[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a[i] = min(__float_as_uint(t[i]) & 0x7FFFFFFFu, F::MAX_BITS);              // the maximum itself has no fraction: never up
            code[i] = ((a[i] + (~word[i] >> (9 + F::M))) >> (23 - F::M)) - ((127u - F::BIAS) << F::M);
        }
        if (__any(min(min(a[0], a[1]), min(a[2], a[3])) < F::MINNORM_BITS)) {
            asm volatile("; below the normal range");
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float y = __builtin_ceilf(__uint_as_float(a[i]) * (F::TO_SUBNORMAL_UNITS * 16777216.0f));   // exact product
                const uint32_t sub = ((uint32_t)fminf(y, 268435456.0f) + (~word[i] >> 8)) >> 24;   // (the cap: not used above 2^27)
                code[i] = a[i] >= F::MINNORM_BITS ? code[i] : sub;
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) code[i] |= (__float_as_uint(t[i]) >> 24) & 0x80u;
    }
    if (__any(__builtin_isunordered(t[0], t[1]) || __builtin_isunordered(t[2], t[3]))) {
        asm volatile("; NaN");
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (t[i] != t[i]) code[i] = FMT == QMM_FMT_INT8 ? 0u : 0x7Fu;
    }
    return code[0] | (code[1] << 8) | (code[2] << 16) | (code[3] << 24);
}

// Philox4x32-10 (Salmon et al., SC'11): ten rounds of two 32x32->64 multiplies
// with the Weyl key schedule.
struct Philox4 { uint32_t v[4]; };
QMM_DEV Philox4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        if (round > 0) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
        // one 32 x 32 -> 64 multiply per product (v_mad_u64_u32) instead of separate high and low halves: integer
        // multiplies issue at a quarter of the plain rate and are what bounds stochastic rounding
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
        const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
        const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
    }
    return Philox4{{c0, c1, c2, c3}};
}

// Step size from the magnitude bits of a group's absmax (Eq. 1): one IEEE
// division; zero group -> 1; quotient below 2^-126 raised to 2^-126.
QMM_DEV float delta_from_absmax_bits(uint32_t bits, float qmax)
{
    const float a = __uint_as_float(bits);
    float d = a / qmax;
    if (d < 0x1p-126f) d = 0x1p-126f;
    return bits == 0u ? 1.0f : d;
}

// ---------------------------------------------------------------------------
// A store that goes through the XCD's L2 to memory at once (4, 8 or 16 bytes at any element boundary).  An ordinary store's
// line stays dirty in the L2 -- up to 32 MB over the XCDs -- until the kernel ends, and the end of the kernel waits for the
// write-back: 3 us for 16 MB of codes written in a kernel's last phase (16384 x 1024 bfloat16, scale + quantize 17.0 -> 14.9 us).
// A streaming (nontemporal) store leaves as early but is not kept by the memory-side cache: the same codes made the
// product that reads them several times slower (16384 x 4096 x 1024: 60 -> 75 us).
// For lines that leave whole, or nearly: one that leaves in pieces (a product's ragged rows, a tile's part of a row) is a write to memory
// per piece.  64 matrices of 1000 x 1000 transposed: quantize_cols 40 us by the L2, 54 past it; quantize_rows, 300000 x 20 per row,
// 16.7 / 28.2.  Where a wavefront's 16-byte stores follow one another through memory, rows off a line's boundary do no harm: the
// one-launch kernels' codes (see resident_cols), dequantized rows up to 48 MB (dequantize_lines).
// ---------------------------------------------------------------------------
template <typename V> QMM_DEV void store_through(void* p, V v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(sizeof(V) == 4 || sizeof(V) == 8 || sizeof(V) == 16, "one store");
    // (the wait states: the compiler does not see that a 16-byte store still reads its registers)
    if constexpr (sizeof(V) == 16) asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" :: "v"(p), "v"(v) : "memory");
    else if constexpr (sizeof(V) == 8) asm volatile("global_store_dwordx2 %0, %1, off sc1\n\ts_nop 1" :: "v"(p), "v"(v) : "memory");
    else asm volatile("global_store_dword %0, %1, off sc1" :: "v"(p), "v"(v) : "memory");
#endif
}

// ---------------------------------------------------------------------------
// Wavefront reductions (64 lanes).
// ---------------------------------------------------------------------------
QMM_DEV uint32_t wave_max_u32(uint32_t v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, off, kWave));
    return v;
}
// Butterflies on the vector unit alone: rotations within the rows of sixteen lanes, then the gfx950 swaps of neighbouring
// rows and of wavefront halves (of two copies of a value the swap leaves one lane set in the first and the other in the
// second, so first op second is the pair's result in every lane).  A shuffle goes through the LDS crossbar and back, and
// the fourteen sums of the metric pass were 132 of them, one behind the other (qmm_metric.hip).
template <int N> QMM_DEV double row_rotate(double v)
{
    constexpr int ROW_ROR = 0x120;
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, ROW_ROR + N, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), ROW_ROR + N, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <int WIDTH> QMM_DEV void swap_copies(double v, double& first, double& second)
{
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
    u2 l, h;
    if constexpr (WIDTH == 16) {
        l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    } else {
        l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    }
    first = __builtin_bit_cast(double, ((uint64_t)h[0] << 32) | l[0]);
    second = __builtin_bit_cast(double, ((uint64_t)h[1] << 32) | l[1]);
}
QMM_DEV double wave_sum_f64(double v)
{
    v += row_rotate<8>(v); v += row_rotate<4>(v); v += row_rotate<2>(v); v += row_rotate<1>(v);
    double a, b;
    swap_copies<16>(v, a, b); v = a + b;
    swap_copies<32>(v, a, b); return a + b;
}
QMM_DEV double wave_max_f64(double v)
{
    v = fmax(v, row_rotate<8>(v)); v = fmax(v, row_rotate<4>(v)); v = fmax(v, row_rotate<2>(v)); v = fmax(v, row_rotate<1>(v));
    double a, b;
    swap_copies<16>(v, a, b); v = fmax(a, b);
    swap_copies<32>(v, a, b); return fmax(a, b);
}

// ---------------------------------------------------------------------------
// Maxima of magnitude bits over 16-byte vectors of elements.
// ---------------------------------------------------------------------------
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// 8 bfloat16 magnitudes packed in a 16-byte vector -> running packed maxima.
QMM_DEV void fold_bf16x8(qmm_u32x4 w, u16x2 (&m)[4])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t a = w[i] & 0x7FFF7FFFu;
        m[i] = __builtin_elementwise_max(m[i], __builtin_bit_cast(u16x2, a));
    }
}
QMM_DEV uint32_t finish_bf16(const u16x2 (&m)[4])
{
    uint32_t r = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) r = max(r, max((uint32_t)m[i][0], (uint32_t)m[i][1]));
    return r << 16;   // bfloat16 magnitude -> binary32 magnitude bits
}

template <typename T> QMM_DEV uint32_t mag_bits(T v);
template <> QMM_DEV uint32_t mag_bits<uint16_t>(uint16_t v) { return ((uint32_t)v & 0x7FFFu) << 16; }
template <> QMM_DEV uint32_t mag_bits<float>(float v) { return __float_as_uint(v) & 0x7FFFFFFFu; }

// Running maxima over 16-byte vectors (8 bfloat16 or 4 binary32 elements), kept per position.
template <typename T> struct VecMax;
template <> struct VecMax<uint16_t> {
    static constexpr int V = 8;
    u16x2 m[4] = {};
    QMM_DEV void fold(qmm_u32x4 w) { fold_bf16x8(w, m); }
    QMM_DEV uint32_t finish() const { return finish_bf16(m); }
    QMM_DEV void words(uint32_t (&out)[4]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] = __builtin_bit_cast(uint32_t, m[i]);
    }
    QMM_DEV void fold_words(const uint32_t (&in)[4])
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) m[i] = __builtin_elementwise_max(m[i], __builtin_bit_cast(u16x2, in[i]));
    }
    QMM_DEV uint32_t at(int e) const { return (uint32_t)m[e >> 1][e & 1] << 16; }
};
template <> struct VecMax<float> {
    static constexpr int V = 4;
    uint32_t m[4] = {};
    QMM_DEV void fold(qmm_u32x4 w)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) m[i] = max(m[i], w[i] & 0x7FFFFFFFu);
    }
    QMM_DEV uint32_t finish() const { return max(max(m[0], m[1]), max(m[2], m[3])); }
    QMM_DEV void words(uint32_t (&out)[4]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] = m[i];
    }
    QMM_DEV void fold_words(const uint32_t (&in)[4])
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) m[i] = max(m[i], in[i]);
    }
    QMM_DEV uint32_t at(int e) const { return m[e]; }
};

// ---------------------------------------------------------------------------
// "The workgroup that arrives last folds the partial results": one launch per reduction instead of two.
// For calls being recorded into a graph; the others use a board (below), which saves the chain of counting.
// A call takes one slot (per reduced tensor) of a ring of arrival counters that live in the library's device
// image and are zero between calls; every workgroup publishes its partial result, counts itself in, and the one
// that completes the count folds all partials in a fixed order (so results do not depend on which one it is),
// then puts the counters back to zero.  Counting is in two levels -- workgroups of one residue class of
// blockIdx mod 8 (the XCD a workgroup runs on under round-robin dispatch) share a counter, the last of each class
// counts into the slot's first word -- so that no counter takes more than an eighth of the grid's arrivals, each in
// a cache line of its own.  The ring has kArrivalSlots slots handed out round robin: two calls can only meet on
// one slot if that many calls are issued while the first is still running.
// ---------------------------------------------------------------------------
constexpr int kArrivalSlots = 8192;
constexpr int kArrivalStride = 32;                       // words between the counters of a slot: 128 bytes
constexpr int kArrivalWords = 9 * kArrivalStride;        // per slot: the slot's counter + eight class counters
qmm_status arrival_slots(int count, uint32_t** first);   // host: `count` consecutive slots (qmm_api.hip)

// Partial results cross from one workgroup to another through device-coherent accesses (they bypass the per-XCD
// caches), not through fences: a release fence writes back the whole L2 of the XCD, and a thousand workgroups doing
// that cost more than the reduction itself.  publish_* stores and waits until the store has left the CU; the
// arrival is counted afterwards in program order; the last workgroup reads with coherent_load.
QMM_DEV void publish_u32(uint32_t* p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}
QMM_DEV void publish_f64(double* p, double v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}
QMM_DEV uint32_t coherent_load(const uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
QMM_DEV double coherent_load(const double* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Called by all threads of a workgroup after its partial results have been published; true, for every thread, in
// the one workgroup of the `total` that arrives last.
QMM_DEV bool arrive_last(uint32_t* slot, unsigned id, unsigned total)
{
    __shared__ int s_last;
    __syncthreads();                 // every publishing thread of the workgroup has waited for its store
    if (threadIdx.x == 0) {
        int last = 0;
        const unsigned cls = id & 7u, in_cls = (total - cls + 7u) >> 3, classes = total < 8u ? total : 8u;
        uint32_t* c = slot + (1 + cls) * kArrivalStride;
        if (__hip_atomic_fetch_add(c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == in_cls - 1u) {
            __hip_atomic_store(c, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (__hip_atomic_fetch_add(slot, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == classes - 1u) {
                __hip_atomic_store(slot, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                last = 1;
            }
        }
        s_last = last;
    }
    __syncthreads();
    return s_last != 0;
}

// ---------------------------------------------------------------------------
// A board of posted values: how the workgroups of ONE launch hand partial results to one another while it runs.
// A word is 64 bits, the call's tag above a 32-bit value, written and read whole by device-coherent accesses: a word with
// the call's tag holds that call's value, any other word has not been posted yet.  Nothing is cleared or counted, there are no
// atomics, and no ordering between words is needed.  Tags are handed out by the host, one per launch (take_board), so a
// call that is being recorded into a graph, whose replays would repeat the tag, does not use a board.
// Boards are cut from rings in the library's device image, each call as many words as it needs (calls whose readers wait long,
// the error sums and the step sizes alone, have a ring of their own: what they share words with is a call of their own kind at least
// sixteen, mostly a thousand calls before).  A reader's wait is bounded
// (`patience`, in ticks of the 100 MHz clock): a value that has not come by then -- its workgroup may not be resident, other
// work holding the CUs, or a call a whole ring before may still be running on the same words -- the reader's workgroup forms
// itself and posts, the same value.  So every workgroup ends whatever the others do, and what the words hold decides about
// time, never about results.
// ---------------------------------------------------------------------------
enum Ring { RING_SHORT = 0, RING_LONG = 1, kRings = 2 };
constexpr uint32_t kRingWords = 1u << 20, kBoardMax = 1u << 17;      // 8 MB a ring
constexpr uint32_t kPatience = 1200;                                 // 12 us: then a workgroup looks closer (collect in qmm_resident.hip)
// Where only the workgroups that fold wait and the others never do, so that every word comes whatever else the GPU does: 10 ms, for
// the workgroups of a long pass end far apart (16 GB read for a step size, 2.9 ms: with 50 us the folder began to read others' slices
// again, alone, 3.6 ms; 4 GB 0.71 / 0.87).
constexpr uint32_t kFolderPatience = 1000000;
struct Board { uint64_t* words; uint32_t tag, patience; };
bool take_board(hipStream_t s, Ring ring, uint32_t words, Board* b); // host (qmm_api.hip), words <= kBoardMax; false: do without one
int cu_count();                                                      // host: CUs of the current device, 0 if unknown

QMM_DEV void board_post(const Board& b, uint32_t i, uint32_t v)
{
    __hip_atomic_store(b.words + i, ((uint64_t)b.tag << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
QMM_DEV bool board_read(const Board& b, uint32_t i, uint32_t& v)
{
    const uint64_t w = __hip_atomic_load(b.words + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    v = (uint32_t)w;
    return (uint32_t)(w >> 32) == b.tag;
}
QMM_DEV uint64_t ticks() { return __builtin_amdgcn_s_memrealtime(); }
// Waits for word i until `patience` ticks after `start`; false: it did not come.
QMM_DEV bool board_wait(const Board& b, uint32_t i, uint64_t start, uint32_t& v)
{
    while (!board_read(b, i, v)) {
        if (ticks() - start >= b.patience) return false;
        __builtin_amdgcn_s_sleep(2);
    }
    return true;
}

// The scale group of a matrix: its matrices are ((k / inner) * G + g) * inner + k % inner for k = 0 .. count - 1.  A group's
// words stand together on the board, slot(k) for its k-th matrix (a matrix apart, its readers' requests would be to many times
// the lines: 512 matrices in 16 groups 17.4 us, this way 15.9).
struct Group {
    uint32_t g, G, inner, count, k_of_b, slots;
    QMM_DEV uint32_t matrix(uint32_t k) const
    {
        const uint32_t q = inner > 1 ? k / inner : k;
        return (q * G + g) * inner + (k - q * inner);
    }
    QMM_DEV uint32_t slot(uint32_t k) const { return g * slots + k; }
};

QMM_DEV Group group_at(uint32_t batch, uint32_t G, uint32_t inner, uint32_t b)      // (inner <= batch)
{
    const uint32_t run = inner > 1 ? b / inner : b, runs = inner > 1 ? (batch + inner - 1) / inner : batch;
    const uint32_t g = G > 1 ? run % G : 0, mine = G > 1 ? (runs - g + G - 1) / G : runs;
    const uint32_t last_run = (mine - 1) * G + g, last = min(inner, batch - last_run * inner);
    return Group{g, G, inner, (mine - 1) * inner + last, (G > 1 ? run / G : run) * inner + (b - run * inner), (runs + G - 1) / G * inner};
}

// The scale pass in two halves (qmm_scale.hip), for the call that hands the partial maxima to the quantize pass.
constexpr int kFoldSlabs = 32;       // row slabs per matrix in the column maxima: what the quantize pass can fold on its way, at most
struct ScalePartials {
    int64_t batch, P, C;       // layout of the partial maxima: [batch][P][C] (C = channels of a step size each, else 1)
    bool done;                 // the step sizes have been written already
};
qmm_status scale_arguments(const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g, const float* delta_out,
                           const void* workspace, size_t workspace_bytes, bool fold);
size_t scale_partials_size(const qmm_tensor* x, const qmm_granularity* g, bool fold);    // bytes of partial maxima
qmm_status scale_partials(const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g, float* delta_out, uint32_t* partial,
                          bool fold_here, ScalePartials* out, hipStream_t s, uint32_t patience = kFolderPatience);
qmm_status scale_fold(const ScalePartials& pp, const uint32_t* partial, qmm_format fmt, const qmm_granularity* g,
                      float* delta_out, hipStream_t s);
// Both steps in one launch (qmm_resident.hip), for the calls it is for.
qmm_status scale_quantize_resident(const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g, qmm_round mode, uint64_t seed,
                                   uint64_t offset, float* delta, uint8_t* codes, uint32_t patience, hipStream_t s, bool* taken);
// Runs of contiguous output that are whole lines: `p` starts one, and `bytes` from one run's start to the next are a multiple (0: one run).
inline bool in_lines(const void* p, int64_t bytes) { return ((reinterpret_cast<uintptr_t>(p) | (uint64_t)bytes) & 127u) == 0; }
inline float host_qmax(qmm_format fmt) { return fmt == QMM_FMT_INT8 ? 127.0f : (fmt == QMM_FMT_E4M3 ? 448.0f : 57344.0f); }

inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }
inline qmm_status launch_status() { return hipGetLastError() == hipSuccess ? QMM_OK : QMM_ERR_LAUNCH; }
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace qmm
