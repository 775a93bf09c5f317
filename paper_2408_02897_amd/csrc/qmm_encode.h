// Device code of the quantize pass shared by its translation units: vectors of a tensor's elements, their codes in either
// rounding mode, and the arguments of its kernels.
#pragma once
#include "qmm_device.h"

namespace qmm {
namespace {

constexpr int kThreads = 256;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
// global memory takes vector accesses at any element boundary: rows of odd length need no path of their own
typedef unsigned int u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
typedef unsigned int u32x4_byte __attribute__((ext_vector_type(4), aligned(1)));
typedef unsigned int u32x2_byte __attribute__((ext_vector_type(2), aligned(1)));
typedef unsigned int u32_byte __attribute__((aligned(1)));

struct QArgs {
    const void* x;
    float* delta;          // step sizes: read, or (FOLD, one-pass kernel) formed and written
    uint8_t* codes;
    int64_t batch, rows, cols, batch_stride, row_stride;
    int64_t groups;        // batch groups
    int64_t inner;         // consecutive matrices sharing a group: group = (b / inner) % groups
    int64_t channels;      // step sizes per group (1 when not per-channel)
    uint64_t seed, offset;
    const uint32_t* partial;   // FOLD: partial maxima [batch][P][channels]; one scale group: fold_total of them
    int64_t P;
    int fold_total;
    float qmax;
    int streaming;         // quantize_rows_bf16x16: streaming stores of the codes (host: allowed, the scale pass has just read the tensor)
    int through;           // quantize_rows_bf16x16: the codes go past the L2 (store_through)
};

// A 16-byte vector of a tensor: 8 bfloat16 or 4 binary32 elements.
template <typename T> struct Vec;
template <> struct Vec<uint16_t> {
    static constexpr int V = 8;
    static QMM_DEV float at(const u32x4& w, int e) { return __uint_as_float((e & 1) ? (w[e >> 1] & 0xFFFF0000u) : (w[e >> 1] << 16)); }
    static QMM_DEV uint32_t max_bits(const u32x4& w)
    {
        uint32_t m = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) m = max(m, max((w[i] << 16) & 0x7FFFFFFFu, w[i] & 0x7FFF0000u));
        return m;
    }
    static QMM_DEV u32x4 partial_load(const uint16_t* p, int left)       // the first `left` elements, zeros behind them
    {
        u32x4 w = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int e = 0; e < V; ++e)
            if (e < left) w[e >> 1] |= (uint32_t)p[e] << (16 * (e & 1));
        return w;
    }
};
template <> struct Vec<float> {
    static constexpr int V = 4;
    static QMM_DEV float at(const u32x4& w, int e) { return __uint_as_float(w[e]); }
    static QMM_DEV uint32_t max_bits(const u32x4& w)
    {
        return max(max(w[0] & 0x7FFFFFFFu, w[1] & 0x7FFFFFFFu), max(w[2] & 0x7FFFFFFFu, w[3] & 0x7FFFFFFFu));
    }
    static QMM_DEV u32x4 partial_load(const float* p, int left)
    {
        u32x4 w = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int e = 0; e < V; ++e)
            if (e < left) w[e] = __float_as_uint(p[e]);
        return w;
    }
};

// Codes of 4 Q consecutive output elements, the first of them number g of the random stream, four to a dword.
// `whole`: g is known to be a multiple of 4.
template <int FMT, int MODE, int Q> QMM_DEV void encode_quads(const float (&t)[4 * Q], uint64_t g, uint64_t seed, bool whole, uint32_t (&out)[Q])
{
    if constexpr (MODE == QMM_ROUND_RTNE) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if constexpr (FMT == QMM_FMT_INT8)
                out[q] = encode_int8_rtne(t[4 * q]) | (encode_int8_rtne(t[4 * q + 1]) << 8) | (encode_int8_rtne(t[4 * q + 2]) << 16) |
                         (encode_int8_rtne(t[4 * q + 3]) << 24);
            else out[q] = encode_fp8_rtne_pair<FMT>(t[4 * q], t[4 * q + 1]) | (encode_fp8_rtne_pair<FMT>(t[4 * q + 2], t[4 * q + 3]) << 16);
        }
    } else {
        // The elements are Q whole blocks of the generator when the first of them starts one (always, unless the caller's
        // offset or the row length is not a multiple of 4), else parts of Q + 1.
        const uint64_t c = g >> 2;
        const uint32_t j = (uint32_t)g & 3u, k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
        auto block = [&](int q) { return philox4x32_10((uint32_t)(c + q), (uint32_t)((c + q) >> 32), 0u, 0u, k0, k1); };
        uint32_t w[4 * Q + 4];
        auto take = [&](int q) {
            const Philox4 p = block(q);
#pragma unroll
            for (int e = 0; e < 4; ++e) w[4 * q + e] = p.v[e];
        };
#pragma unroll
        for (int q = 0; q < Q; ++q) take(q);
        if (!whole) {
            asm volatile("; parts of blocks");       // (keeps the compiler from computing this for every call and selecting)
            take(Q);
#pragma unroll
            for (int e = 0; e < 4 * Q; ++e)          // word j + e, by compares (an indexed array would live in memory)
                w[e] = j == 0 ? w[e] : j == 1 ? w[e + 1] : j == 2 ? w[e + 2] : w[e + 3];
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) out[q] = encode_sr4<FMT>(t + 4 * q, w + 4 * q);
    }
}

// The V codes of a vector, from `rho` and the number of its first element.
template <typename T, int FMT, int MODE> QMM_DEV u32x2 encode_vec(const u32x4& w, float rho, uint64_t g, uint64_t seed)
{
    constexpr int Q = Vec<T>::V / 4;
    float t[4 * Q];
#pragma unroll
    for (int e = 0; e < 4 * Q; ++e) t[e] = Vec<T>::at(w, e) * rho;
    uint32_t c[Q];
    // One test for a vector and a wavefront: with one per block the blocks -- chains of ten dependent multiplies -- run one
    // behind the other.
    encode_quads<FMT, MODE, Q>(t, g, seed, MODE == QMM_ROUND_STOCHASTIC && !__any((g & 3u) != 0u), c);
    return u32x2{c[0], Q > 1 ? c[Q - 1] : 0u};
}
template <typename T> QMM_DEV void store_codes(uint8_t* dst, u32x2 c, int64_t left)
{
    if (left >= Vec<T>::V) {
        if constexpr (Vec<T>::V == 8) *reinterpret_cast<u32x2_byte*>(dst) = c;
        else *reinterpret_cast<u32_byte*>(dst) = c[0];
    } else {
#pragma unroll
        for (int e = 0; e < Vec<T>::V; ++e)
            if (e < left) dst[e] = (uint8_t)(c[e >> 2] >> (8 * (e & 3)));
    }
}

// Scale group of matrix b < 65536 (host), in 32-bit divisions and only those the grouping needs.
QMM_DEV int64_t group_of(const QArgs& a, int64_t b)
{
    if (a.groups == 1) return 0;
    uint32_t q = (uint32_t)b;
    if (a.inner > 1) q = a.inner > 65535 ? 0u : q / (uint32_t)a.inner;
    return a.groups > 65535 ? q : q % (uint32_t)a.groups;
}

// V neighbouring elements of a row, the first `left` of them inside the matrix (zeros for the others).
template <typename T, int V> QMM_DEV u32x4 load_columns(const T* p, int left)
{
    u32x4 w = {0u, 0u, 0u, 0u};
    if constexpr (V == Vec<T>::V) {
        if (left == V) w = *reinterpret_cast<const u32x4_any*>(p);
        else if (left > 0) w = Vec<T>::partial_load(p, left);
    } else {
        static_assert(V == 2, "two elements, or a vector");
        typedef unsigned int pair_any __attribute__((ext_vector_type(sizeof(T) == 2 ? 1 : 2), aligned(sizeof(T))));
        if (left == 2) {
            const pair_any q = *reinterpret_cast<const pair_any*>(p);
            w[0] = q[0];
            if constexpr (sizeof(T) == 4) w[1] = q[1];
        } else if (left == 1) {
            if constexpr (sizeof(T) == 2) w[0] = *p; else w[0] = __float_as_uint(*p);
        }
    }
    return w;
}
// The first `left` of B bytes (B = 8, 16; left < B).
template <int B> QMM_DEV void store_bytes(uint8_t* dst, u32x4 w, int left)
{
    typedef unsigned short u16_byte __attribute__((aligned(1)));
    if (B > 8 && (left & 8)) { *reinterpret_cast<u32x2_byte*>(dst) = u32x2{w[0], w[1]}; dst += 8; w[0] = w[2]; w[1] = w[3]; }
    if (left & 4) { *reinterpret_cast<u32_byte*>(dst) = w[0]; dst += 4; w[0] = w[1]; }
    if (left & 2) { *reinterpret_cast<u16_byte*>(dst) = (unsigned short)w[0]; dst += 2; w[0] >>= 16; }
    if (left & 1) *dst = (uint8_t)w[0];
}

// Every column's codes start a block of the random generator.
__host__ QMM_DEV bool whole_blocks(const QArgs& a) { return ((a.rows | (int64_t)a.offset) & 3) == 0; }

}  // namespace
}  // namespace qmm
