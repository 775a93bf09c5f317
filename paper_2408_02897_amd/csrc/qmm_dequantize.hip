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
    int64_t lines_per_matrix;
    int64_t groups; int64_t inner;    // matrix -> scale group
    int64_t pieces;                   // pieces of kPiece vectors a lane that a line is cut into
};

// A wavefront takes one piece of a line: four vectors a lane, each vector 16 bytes of output, so that a store instruction
// covers 1 KB of it without gaps, whatever the type; all four loads are in flight before the first value is formed.  Any K
// and alignment.  (One thread per 16 codes wrote four 16-byte pieces 64 bytes apart from its neighbours': 67 million codes
// to binary32 81 us; this way 58, 5.8 TB/s.)
constexpr int kPiece = 4;
template <int FMT, bool OUT_BF16> __global__ void __launch_bounds__(kThreads)
dequantize_lines(DArgs a)
{
    constexpr int V = OUT_BF16 ? 8 : 4;
    typedef unsigned int u32_any __attribute__((aligned(1)));
    typedef unsigned int u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t step = (int64_t)gridDim.x * (kThreads / kWave), units = a.lines * a.pieces;
    for (int64_t u = (int64_t)blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave; u < units; u += step) {
        const int64_t line = a.lines == 1 ? 0 : u / a.pieces, piece = u - line * a.pieces;
        const int64_t b = line / a.lines_per_matrix, r = line - b * a.lines_per_matrix;
        const float d = a.delta[((b / a.inner) % a.groups) * a.lines_per_matrix + r];
        const uint8_t* src = a.codes + line * a.K;
        const int64_t c0 = piece * (kPiece * kWave * V) + lane * V;
        uint32_t w[kPiece][V / 4];
#pragma unroll
        for (int i = 0; i < kPiece; ++i) {
            const int64_t c = c0 + i * (kWave * V), left = a.K - c;
#pragma unroll
            for (int q = 0; q < V / 4; ++q) {
                w[i][q] = 0u;
                if (left >= V) w[i][q] = *reinterpret_cast<const u32_any*>(src + c + 4 * q);
                else {
                    for (int e = 0; e < 4; ++e)
                        if (4 * q + e < left) w[i][q] |= (uint32_t)src[c + 4 * q + e] << (8 * e);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < kPiece; ++i) {
            const int64_t c = c0 + i * (kWave * V), left = a.K - c;
            float y[V];
#pragma unroll
            for (int q = 0; q < V / 4; ++q) {
                float v[4];
                decode4<FMT>(w[i][q], v);
#pragma unroll
                for (int e = 0; e < 4; ++e) y[4 * q + e] = v[e] * d;
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
            if (left >= V) {
                if constexpr (OUT_BF16) *reinterpret_cast<u32x4_any*>(static_cast<uint16_t*>(a.out) + line * a.K + c) = o;
                else *reinterpret_cast<u32x4_any*>(static_cast<float*>(a.out) + line * a.K + c) = o;
            } else {
#pragma unroll
                for (int e = 0; e < V; ++e)
                    if (e < left) {
                        if constexpr (OUT_BF16) static_cast<__bf16*>(a.out)[line * a.K + c + e] = (__bf16)y[e];
                        else static_cast<float*>(a.out)[line * a.K + c + e] = y[e];
                    }
            }
        }
    }
}

template <int FMT> qmm_status launch(const DArgs& a, bool bf16, hipStream_t s)
{
    const int64_t blocks = std::min<int64_t>((a.lines * a.pieces + kThreads / kWave - 1) / (kThreads / kWave), 1 << 20);
    if (bf16) dequantize_lines<FMT, true><<<(unsigned)blocks, kThreads, 0, s>>>(a);
    else dequantize_lines<FMT, false><<<(unsigned)blocks, kThreads, 0, s>>>(a);
    return launch_status();
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
    a.groups = g->batch_groups; a.inner = g->batch_inner > 0 ? g->batch_inner : 1;
    // the longest runs with one step size: rows, matrices, or all of the tensor
    if (g->per_channel) { a.lines = batch * rows; a.K = K; a.lines_per_matrix = rows; }
    else if (a.groups > 1) { a.lines = batch; a.K = rows * K; a.lines_per_matrix = 1; }
    else { a.lines = 1; a.K = batch * rows * K; a.lines_per_matrix = 1; }
    const int64_t span = (int64_t)kPiece * kWave * (bf16 ? 8 : 4);
    a.pieces = (a.K + span - 1) / span;
    hipStream_t s = as_stream(stream);
    if (fmt == QMM_FMT_INT8) return launch<QMM_FMT_INT8>(a, bf16, s);
    if (fmt == QMM_FMT_E4M3) return launch<QMM_FMT_E4M3>(a, bf16, s);
    return launch<QMM_FMT_E5M2>(a, bf16, s);
}
