// qmm_dequantize: the reduced-precision value of every quantized element (the v-tilde of Eq. 2): value of the
// code times the step size of its scale group, one binary32 multiply.  HBM-bound: 1 B read, 2 or 4 B written per
// element.  Codes [batch][rows][K] as qmm_quantize writes them; delta indexed the same way.
#include <algorithm>
#include "qmm_device.h"

namespace qmm {
namespace {

constexpr int kThreads = 256;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Four codes of a dword -> their values.  FP8 through the hardware converter (exact: every code's value is a binary32
// number; its NaN becomes the one quiet pattern).
template <int FMT> QMM_DEV void decode4(uint32_t w, float (&v)[4])
{
    if constexpr (FMT == QMM_FMT_INT8) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = (float)(int8_t)(uint8_t)(w >> (8 * i));
    } else {
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        f32x2 lo, hi;
        if constexpr (FMT == QMM_FMT_E4M3) { lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, false); hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, true); }
        else { lo = __builtin_amdgcn_cvt_pk_f32_bf8((int)w, false); hi = __builtin_amdgcn_cvt_pk_f32_bf8((int)w, true); }
        v[0] = lo[0]; v[1] = lo[1]; v[2] = hi[0]; v[3] = hi[1];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = v[i] != v[i] ? __uint_as_float(0x7FC00000u) : v[i];
    }
}

struct DArgs {
    const uint8_t* codes; const float* delta; void* out;
    int64_t lines, K;                 // lines of K codes that share a step size: rows, whole matrices, or the whole tensor
    int64_t lines_per_matrix, matrices;
    int64_t groups; int64_t inner;    // matrix -> scale group (neither above the number of matrices)
    int64_t units;                    // pieces of work for one wavefront
    int64_t pieces;                   // long lines: units per line
    int through;                      // the values go past the L2 (store_through)
    int lane_shift, half_shift;       // short lines: 1 << lane_shift lanes a line, in 1 << half_shift halves
};

// A wavefront takes four vectors a lane, each vector 16 bytes of output: either one piece of a long line, so that a store
// instruction covers 1 KB of it without gaps, whatever the type; or (SHORT: lines of at most 128 vectors) several lines,
// each on as many lanes as it has vectors, so that here too nearly every lane works and neighbouring lanes write
// neighbouring memory.  All four loads are in flight before the first value is formed.  Any K and alignment.
// Coordinates are of type I: 32-bit divisions, four to six times cheaper than 64-bit ones, where the counts allow it, and
// none that the form does not need.  (Launches back to back, E4M3.  One thread per 16 codes wrote four 16-byte pieces 64
// bytes apart from its neighbours': 67 million codes with one step size to binary32 108 us; this way 61, 5.5 TB/s.  A
// wavefront per line whatever its length took 131 us for 262144 rows of 64 with a step size each to bfloat16; lines side
// by side take 9.1, one thread per 16 codes 12.4.)
// PIECE: four vectors a lane, or one for small tensors, where what counts is how soon the last wavefront is through its
// own arithmetic (5000 rows of 33 to bfloat16 3.1 -> 2.1 us).
template <int FMT, bool OUT_BF16, bool SHORT, typename I, int PIECE> __global__ void __launch_bounds__(kThreads)
dequantize_lines(DArgs a)
{
    constexpr int V = OUT_BF16 ? 8 : 4;
    typedef unsigned int u32_any __attribute__((aligned(1)));
    typedef unsigned int u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
    const int lane = threadIdx.x & (kWave - 1);
    const I lines = (I)a.lines, lines_per_matrix = (I)a.lines_per_matrix, inner = (I)a.inner, groups = (I)a.groups;
    auto step_size = [&](I line) -> float {
        I b = 0, r = line;
        if (a.matrices > 1) { b = line / lines_per_matrix; r = line - b * lines_per_matrix; }
        if (a.inner > 1) b /= inner;
        if (a.groups == 1) b = 0; else if (a.groups < a.matrices) b %= groups;
        return a.delta[(int64_t)b * a.lines_per_matrix + r];
    };
    const I step = (I)gridDim.x * (kThreads / kWave), units = (I)a.units;
    for (I u = (I)blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave; u < units; u += step) {
        int64_t at[PIECE], left[PIECE];            // first code of each vector, and codes from there to the end of its line
        float d[PIECE];
        if constexpr (SHORT) {
#pragma unroll
            for (int i = 0; i < PIECE; ++i) {
                const I slot = u * PIECE + i;
                const I line = ((slot >> a.half_shift) << (6 - a.lane_shift)) + (lane >> a.lane_shift);
                const int c = (((int)(slot & ((1 << a.half_shift) - 1)) << 6) + (lane & ((1 << a.lane_shift) - 1))) * V;
                at[i] = (int64_t)line * a.K + c;
                left[i] = line < lines ? a.K - c : 0;
                d[i] = left[i] > 0 ? step_size(line) : 0.0f;
            }
        } else {
            const I line = a.lines == 1 ? 0 : u / (I)a.pieces, piece = u - line * (I)a.pieces;
            d[0] = step_size(line);
#pragma unroll
            for (int i = 0; i < PIECE; ++i) {
                const int64_t c = ((int64_t)piece * PIECE + i) * (kWave * V) + lane * V;
                at[i] = (int64_t)line * a.K + c;
                left[i] = a.K - c;
                d[i] = d[0];
            }
        }
        // the last, partial vector of a line is taken back by what it lacks: the codes it shares with the one before it get the
        // same values twice
        if (a.K >= V) {
#pragma unroll
            for (int i = 0; i < PIECE; ++i)
                if (left[i] > 0 && left[i] < V) { at[i] -= V - left[i]; left[i] = V; }
        }
        uint32_t w[PIECE][V / 4];
#pragma unroll
        for (int i = 0; i < PIECE; ++i) {
            const uint8_t* src = a.codes + at[i];
#pragma unroll
            for (int q = 0; q < V / 4; ++q) {
                w[i][q] = 0u;
                if (left[i] >= V) w[i][q] = *reinterpret_cast<const u32_any*>(src + 4 * q);
                else if (left[i] > 0) {
                    for (int e = 0; e < 4; ++e)
                        if (4 * q + e < left[i]) w[i][q] |= (uint32_t)src[4 * q + e] << (8 * e);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < PIECE; ++i) {
            float y[V];
#pragma unroll
            for (int q = 0; q < V / 4; ++q) {
                float v[4];
                decode4<FMT>(w[i][q], v);
#pragma unroll
                for (int e = 0; e < 4; ++e) y[4 * q + e] = v[e] * d[i];
            }
            u32x4 o;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if constexpr (OUT_BF16) {
                    typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
                    typedef float f2 __attribute__((ext_vector_type(2)));
                    o[q] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{y[2 * q], y[2 * q + 1]}, bf2));
                } else o[q] = __float_as_uint(y[q]);
            }
            if (left[i] >= V) {
                void* dst = static_cast<uint8_t*>(a.out) + at[i] * (16 / V);
                if (a.through) store_through(dst, o); else *static_cast<u32x4_any*>(dst) = o;
            } else if (left[i] > 0) {
#pragma unroll
                for (int e = 0; e < V; ++e)
                    if (e < left[i]) {
                        if constexpr (OUT_BF16) static_cast<__bf16*>(a.out)[at[i] + e] = (__bf16)y[e];
                        else static_cast<float*>(a.out)[at[i] + e] = y[e];
                    }
            }
        }
    }
}

template <int FMT, bool BF16> qmm_status launch(DArgs a, hipStream_t s)
{
    constexpr int V = BF16 ? 8 : 4;
    const int64_t nvec = (a.K + V - 1) / V;
    // Past the L2 where the lines are whole (by the L2 / past it: 65536 x 1024 a step size per row, bfloat16 36.1 / 35.2 us, binary32
    // 57.8 / 55.4), and up to 48 MB where they are not (16384 x 1031
    // bfloat16 10.7 / 9.9, 300000 x 20 binary32 8.2 / 6.5, 100000 x 129 14.1 / 12.6; at 48 MB 13.7 / 13.7 to 15.1 / 15.2, 57 MB 18.5 / 19.8);
    // beyond, memory takes a line's parts one by one (65536 x 1031 38.6 / 43.0 and 63.7 / 74.6, 300000 x 129 binary32 42.4 / 54.1).
    a.through = in_lines(a.out, a.lines > 1 ? a.K * (16 / V) : 0) || a.lines * a.K * (16 / V) <= (int64_t)48 << 20;
    const bool is_short = nvec <= 2 * kWave && a.lines > 1;
    int64_t slots, slots_per_line = (nvec + kWave - 1) / kWave;                     // wavefront-wide rows of vectors
    if (is_short) {
        while (a.lane_shift < 6 && (1 << a.lane_shift) < nvec) ++a.lane_shift;
        a.half_shift = nvec > kWave ? 1 : 0;
        const int64_t at_once = kWave >> a.lane_shift;
        slots = ((a.lines + at_once - 1) / at_once) << a.half_shift;
    } else {
        slots = a.lines * slots_per_line;
    }
    const bool small = slots <= 4096;                // one vector a lane: sixteen wavefronts per CU and fewer
    const int piece = small ? 1 : 4;
    if (is_short) a.units = (slots + piece - 1) / piece;
    else { a.pieces = (slots_per_line + piece - 1) / piece; a.units = a.lines * a.pieces; }
    const unsigned grid = (unsigned)std::min<int64_t>((a.units + kThreads / kWave - 1) / (kThreads / kWave), 1 << 20);
    // lines, units and slots (and one grid stride beyond) below 2^32
    const bool narrow = a.lines < (int64_t(1) << 31) && a.units < (int64_t(1) << 28);
    if (is_short) {
        if (small) dequantize_lines<FMT, BF16, true, uint32_t, 1><<<grid, kThreads, 0, s>>>(a);
        else if (narrow) dequantize_lines<FMT, BF16, true, uint32_t, 4><<<grid, kThreads, 0, s>>>(a);
        else dequantize_lines<FMT, BF16, true, uint64_t, 4><<<grid, kThreads, 0, s>>>(a);
    } else {
        if (small) dequantize_lines<FMT, BF16, false, uint32_t, 1><<<grid, kThreads, 0, s>>>(a);
        else if (narrow) dequantize_lines<FMT, BF16, false, uint32_t, 4><<<grid, kThreads, 0, s>>>(a);
        else dequantize_lines<FMT, BF16, false, uint64_t, 4><<<grid, kThreads, 0, s>>>(a);
    }
    return launch_status();
}
template <int FMT> qmm_status launch_type(const DArgs& a, bool bf16, hipStream_t s)
{
    return bf16 ? launch<FMT, true>(a, s) : launch<FMT, false>(a, s);
}

}  // namespace
}  // namespace qmm

using namespace qmm;

extern "C" qmm_status qmm_dequantize(const uint8_t* codes, int64_t batch, int64_t rows, int64_t K, qmm_format fmt,
                                     const qmm_granularity* g, const float* delta, void* out, qmm_dtype out_dtype,
                                     void* stream)
{
    if (!g) return QMM_ERR_NULL;
    if (fmt != QMM_FMT_INT8 && fmt != QMM_FMT_E4M3 && fmt != QMM_FMT_E5M2) return QMM_ERR_ENUM;
    if (out_dtype != QMM_DT_BF16 && out_dtype != QMM_DT_F32) return QMM_ERR_ENUM;
    if (g->batch_groups < 1 || g->batch_inner < 0 || (g->per_channel != 0 && g->per_channel != 1)) return QMM_ERR_ENUM;
    if (batch < 0 || rows < 0 || K < 0) return QMM_ERR_SHAPE;
    if (batch * rows * K == 0) return QMM_OK;
    if (!codes || !delta || !out) return QMM_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(out) & (out_dtype == QMM_DT_BF16 ? 1u : 3u)) return QMM_ERR_ALIGN;
    const bool bf16 = out_dtype == QMM_DT_BF16;
    DArgs a{};
    a.codes = codes; a.delta = delta; a.out = out;
    // (groups and runs beyond the batch: the same mapping with the batch's own extent)
    a.groups = std::min(g->batch_groups, batch); a.inner = std::min<int64_t>(g->batch_inner > 0 ? g->batch_inner : 1, batch);
    // the longest runs with one step size: rows, matrices, or all of the tensor
    if (g->per_channel) { a.lines = batch * rows; a.K = K; a.lines_per_matrix = rows; a.matrices = batch; }
    else if (a.groups > 1) { a.lines = batch; a.K = rows * K; a.lines_per_matrix = 1; a.matrices = batch; }
    else { a.lines = 1; a.K = batch * rows * K; a.lines_per_matrix = 1; a.matrices = 1; }
    hipStream_t s = as_stream(stream);
    if (fmt == QMM_FMT_INT8) return launch_type<QMM_FMT_INT8>(a, bf16, s);
    if (fmt == QMM_FMT_E4M3) return launch_type<QMM_FMT_E4M3>(a, bf16, s);
    return launch_type<QMM_FMT_E5M2>(a, bf16, s);
}
