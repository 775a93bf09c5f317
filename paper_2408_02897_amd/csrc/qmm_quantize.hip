// qmm_quantize: codes = round(X / delta) onto INT8 / E4M3 / E5M2 (Eq. 1, left
// half; Methodology bullets on saturation, underflow and the two rounding
// modes).  HBM-bound: 2 B read + 1 B written per bfloat16 element.  The quotient
// is x * (1/delta) with one IEEE reciprocal per thread-row and one product per
// element.  Codes are written with the contracting axis contiguous; when the
// input contracts over its rows the tile is transposed through LDS.
// qmm_scale_quantize: both steps.  The step size is formed where it is used:
// with one per row in a single pass that keeps the row in registers, otherwise
// in one launch that keeps the tensor in registers (qmm_resident.hip), or --
// larger tensors, calls being recorded -- by the quantize pass, which folds the
// partial maxima of its scale group while its first elements are on their way.
#include <algorithm>
#include <type_traits>
#include "qmm_encode.h"

namespace qmm {
namespace {

QMM_DEV uint32_t block_max_u32(uint32_t v)
{
    __shared__ uint32_t s[kThreads / kWave];
    v = wave_max_u32(v);
    if ((threadIdx.x & (kWave - 1)) == 0) s[threadIdx.x / kWave] = v;
    __syncthreads();
    uint32_t r = s[0];
#pragma unroll
    for (int i = 1; i < kThreads / kWave; ++i) r = max(r, s[i]);
    return r;
}

// Step size of matrix b (one per batch group), folded by the whole workgroup from the group's partial maxima (at most
// kFoldMax of them: host).  `writer`: this workgroup also writes it out.
constexpr int kFoldMax = 1024;
QMM_DEV float fold_delta(const QArgs& a, int64_t b, bool writer)
{
    const int64_t g = group_of(a, b);
    uint32_t m = 0;
    if (a.groups == 1) {
#pragma unroll
        for (int k = 0; k < kFoldMax / kThreads; ++k) {
            const int i = threadIdx.x + k * kThreads;
            if (i < a.fold_total) m = max(m, a.partial[i]);
        }
    } else {
        // the k-th matrix of group g is ((k / inner) * G + g) * inner + k % inner, increasing with k (32 bits: batch < 65536)
        const uint32_t P = (uint32_t)a.P, G = (uint32_t)a.groups, inner = (uint32_t)a.inner, batch = (uint32_t)a.batch;
        for (uint32_t it = threadIdx.x;; it += kThreads) {
            const uint32_t k = P > 1 ? it / P : it, p = it - k * P;
            uint32_t mb = k * G + (uint32_t)g;
            if (inner > 1) { const uint32_t q = k / inner; mb = (q * G + (uint32_t)g) * inner + (k - q * inner); }
            if (mb >= batch) break;
            m = max(m, a.partial[mb * P + p]);
        }
    }
    const float d = delta_from_absmax_bits(block_max_u32(m), a.qmax);
    if (writer && threadIdx.x == 0) a.delta[g] = d;
    return d;
}
// the workgroup of a grid that writes a group's step size: the first of its first matrix
QMM_DEV bool writes_group(const QArgs& a, int64_t b) { return b % a.inner == 0 && b / a.inner < a.groups; }

// Row-contracting fast path: bfloat16, cols % 16 == 0, 16-byte aligned rows.  One thread = 16 consecutive
// elements of a row: two 16-byte loads, one 16-byte store.  grid (ceil(rows*cols/16 / 256), batch).
template <int FMT, int MODE, bool FOLD> __global__ void __launch_bounds__(kThreads)
quantize_rows_bf16x16(QArgs a)
{
    const int64_t vpr = a.cols >> 4;
    const int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t b = blockIdx.y;
    const bool live = v < vpr * a.rows;
    if (!FOLD && !live) return;
    // (a matrix with one step size comes in as one row: host; otherwise 32-bit arithmetic where it reaches)
    int64_t r = 0;
    if (a.rows > 1) r = vpr * a.rows <= 0xFFFFFFFFll ? (int64_t)((uint32_t)v / (uint32_t)vpr) : v / vpr;
    const int64_t cv = v - r * vpr;
    const u32x4* src = reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(a.x) + b * a.batch_stride +
                                                      r * a.row_stride + cv * 16);
    // The step size is requested in front of the elements: behind them its reciprocal starts when they have arrived
    // (16384 x 1024 with one step size 9.7 against 10.4 us).
    float d = 0.0f;
    if constexpr (!FOLD) d = a.delta[group_of(a, b) * a.channels + (a.channels > 1 ? r : 0)];
    u32x4 w0 = {0u, 0u, 0u, 0u}, w1 = {0u, 0u, 0u, 0u};
    if (live) { w0 = src[0]; w1 = src[1]; }
    if constexpr (FOLD) {
        d = fold_delta(a, b, blockIdx.x == 0 && writes_group(a, b));
        if (!live) return;
    }
    const float rho = 1.0f / d;
    const int64_t p0 = (b * a.rows + r) * a.cols + cv * 16;
    u32x4 out;
    if constexpr (MODE == QMM_ROUND_RTNE) {
        out = encode16_bf16_rtne<FMT>(w0, w1, rho);
    } else {
        float t[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) t[e] = Vec<uint16_t>::at(e < 8 ? w0 : w1, e & 7) * rho;
        uint32_t c[4];
        encode_quads<FMT, MODE, 4>(t, (uint64_t)p0 + a.offset, a.seed, !__any((((uint64_t)p0 + a.offset) & 3u) != 0u), c);
        out = u32x4{c[0], c[1], c[2], c[3]};
    }
    if (a.streaming) __builtin_nontemporal_store(out, reinterpret_cast<u32x4*>(a.codes + p0));
    else if (a.through) store_through(a.codes + p0, out);
    else *reinterpret_cast<u32x4*>(a.codes + p0) = out;
}

// Row-contracting, any type, extent, stride and alignment.  A wavefront takes PIECE 16-byte vectors a lane: a piece of a
// long row, or (SHORT: rows of at most 128 vectors) several rows, each on as many lanes as it has vectors.  Dense tensors
// with one step size come in as one long row per matrix.  Two vectors a lane, or one for small tensors, which need the
// wavefronts.  (One thread per code / a wavefront a row, whatever its length / this way, a step size per row: 262144 x 64
// binary32 45 / 70 / 14.4 us, 300000 x 20 bfloat16 16 / 125 / 6.0, 100 x 20000 binary32 6.8 / 28 / 3.2.  Four vectors a lane:
// 19, 6.4 and 3.6 us.)
struct RowPlan {
    int64_t units;                 // pieces of work for one wavefront, per matrix
    int64_t pieces;                // long rows: units per row (0: short rows)
    int lane_shift, half_shift;    // short rows: 1 << lane_shift lanes a row, in 1 << half_shift halves
};
template <typename T, int FMT, int MODE, bool FOLD, int PIECE, bool SHORT> __global__ void __launch_bounds__(kThreads)
quantize_rows(QArgs a, RowPlan plan)
{
    constexpr int V = Vec<T>::V;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t b = blockIdx.y;
    const T* base = static_cast<const T*>(a.x) + b * a.batch_stride;
    const float* delta = a.delta + group_of(a, b) * a.channels;
    float rho_matrix = 1.0f;
    if constexpr (FOLD) rho_matrix = 1.0f / fold_delta(a, b, blockIdx.x == 0 && writes_group(a, b));
    else if (a.channels == 1) rho_matrix = 1.0f / delta[0];
    const bool per_row = !FOLD && a.channels > 1, whole = a.cols >= V;
    const int64_t step = (int64_t)gridDim.x * (kThreads / kWave);
    const int64_t first = (int64_t)blockIdx.x * (kThreads / kWave) + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    for (int64_t u = first; u < plan.units; u += step) {
        // vector i: `left` elements (at most V) at row_at + at[i], their codes at code_at + at[i] (SHORT: + code_row[i] instead)
        const T* row_at = base;
        int64_t code_at = b * a.rows * a.cols;
        typename std::conditional<SHORT, int64_t, int>::type at[PIECE];
        int64_t code_row[SHORT ? PIECE : 1];
        int left[PIECE];
        float rho[PIECE];
        if constexpr (!SHORT) {
            int64_t r = 0;
            if (a.rows > 1) r = plan.units <= 0xFFFFFFFFll ? (int64_t)((uint32_t)u / (uint32_t)plan.pieces) : u / plan.pieces;
            const int64_t c0 = (u - r * plan.pieces) * (PIECE * kWave * V);
            const int rest = (int)min(a.cols - c0, (int64_t)(PIECE * kWave * V));
            const float rho_row = per_row ? 1.0f / delta[r] : rho_matrix;
            row_at += r * a.row_stride + c0;
            code_at += r * a.cols + c0;
            if (rest == PIECE * kWave * V) {         // no vector to mask: most pieces
                const T* src = row_at + lane * V;
                uint8_t* dst = a.codes + code_at + lane * V;
                u32x4 w[PIECE];
#pragma unroll
                for (int i = 0; i < PIECE; ++i) w[i] = *reinterpret_cast<const u32x4_any*>(src + i * kWave * V);
#pragma unroll
                for (int i = 0; i < PIECE; ++i)
                    store_codes<T>(dst + i * kWave * V,
                                   encode_vec<T, FMT, MODE>(w[i], rho_row, (uint64_t)(code_at + (i * kWave + lane) * V) + a.offset, a.seed), V);
                continue;
            }
#pragma unroll
            for (int i = 0; i < PIECE; ++i) {
                at[i] = (i * kWave + lane) * V;
                left[i] = min(rest - at[i], V);
                rho[i] = rho_row;
            }
        } else {
#pragma unroll
            for (int i = 0; i < PIECE; ++i) {
                const int64_t slot = u * PIECE + i;
                const int64_t r = ((slot >> plan.half_shift) << (6 - plan.lane_shift)) + (lane >> plan.lane_shift);
                const int c = (int)(((slot & ((1 << plan.half_shift) - 1)) << 6) + (lane & ((1 << plan.lane_shift) - 1))) * V;
                left[i] = r < a.rows ? min((int)a.cols - c, V) : 0;
                at[i] = r * a.row_stride + c;
                code_row[i] = r * a.cols + c;
                rho[i] = rho_matrix;
                if (per_row && left[i] > 0) rho[i] = delta[r];
            }
            if (per_row) {
#pragma unroll
                for (int i = 0; i < PIECE; ++i) rho[i] = 1.0f / rho[i];
            }
        }
        u32x4 w[PIECE];
#pragma unroll
        for (int i = 0; i < PIECE; ++i) w[i] = u32x4{0u, 0u, 0u, 0u};
        if (whole) {
            // a partial last vector is taken back by what it lacks: the elements it shares with the one before it give the
            // same codes twice
#pragma unroll
            for (int i = 0; i < PIECE; ++i) {
                if (left[i] > 0) {
                    at[i] -= V - left[i];
                    if constexpr (SHORT) code_row[i] -= V - left[i];
                    left[i] = V;
                    w[i] = *reinterpret_cast<const u32x4_any*>(row_at + at[i]);
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < PIECE; ++i)
                if (left[i] > 0) w[i] = Vec<T>::partial_load(row_at + at[i], left[i]);
        }
#pragma unroll
        for (int i = 0; i < PIECE; ++i) {
            if (left[i] > 0) {
                const int64_t p = code_at + (SHORT ? code_row[SHORT ? i : 0] : (int64_t)at[i]);
                store_codes<T>(a.codes + p, encode_vec<T, FMT, MODE>(w[i], rho[i], (uint64_t)p + a.offset, a.seed), left[i]);
            }
        }
    }
}

// Both steps in one pass, one step size per row: LPR lanes (a part of a wavefront, a wavefront, or the four of a
// workgroup) take a row, hold it in registers (NV vectors a lane), form its step size and write it and the codes.  The row
// is read once (2 B + 1 B per bfloat16 element) where the two passes read it twice, in one launch instead of two.  Any
// type, stride and alignment, cols <= LPR * NV * V (host).
template <typename T, int FMT, int MODE, int LPR, int NV> __global__ void __launch_bounds__(kThreads)
scale_quantize_rows(QArgs a)
{
    constexpr int V = Vec<T>::V, RPB = kThreads / LPR;       // rows per workgroup
    __shared__ uint32_t s_max[kThreads / kWave];
    const int64_t total = a.batch * a.rows;
    const int c0 = (int)(threadIdx.x % LPR) * V;
    for (int64_t blk = blockIdx.x; blk * RPB < total; blk += gridDim.x) {
        const int64_t row_id = blk * RPB + threadIdx.x / LPR;
        const bool live = row_id < total;
        const int64_t b = live && a.batch > 1 ? row_id / a.rows : 0, r = live ? row_id - b * a.rows : 0;
        const T* row = static_cast<const T*>(a.x) + b * a.batch_stride + r * a.row_stride;
        const int cols = live ? (int)a.cols : 0;
        u32x4 w[NV];
        uint32_t m = 0;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int c = c0 + i * LPR * V, left = cols - c;
            w[i] = u32x4{0u, 0u, 0u, 0u};
            if (left >= V) w[i] = *reinterpret_cast<const u32x4_any*>(row + c);
            else if (left > 0) w[i] = Vec<T>::partial_load(row + c, left);
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) m = max(m, Vec<T>::max_bits(w[i]));
#pragma unroll
        for (int off = (LPR < kWave ? LPR : kWave) / 2; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, kWave));
        if constexpr (LPR > kWave) {
            static_assert(LPR <= kWave || LPR == kThreads, "a row of several wavefronts takes the whole workgroup");
            if ((threadIdx.x & (kWave - 1)) == 0) s_max[threadIdx.x / kWave] = m;
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kThreads / kWave; ++k) m = max(m, s_max[k]);
            __syncthreads();                                 // reused by the next row
        }
        if (!live) continue;                                 // (LPR > 64: never, a workgroup's only row is live)
        const float d = delta_from_absmax_bits(m, a.qmax);
        if (threadIdx.x % LPR == 0) a.delta[row_id] = d;
        const float rho = 1.0f / d;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int c = c0 + i * LPR * V, left = cols - c;
            if (left > 0) {
                const int64_t p = row_id * a.cols + c;
                store_codes<T>(a.codes + p, encode_vec<T, FMT, MODE>(w[i], rho, (uint64_t)p + a.offset, a.seed), left);
            }
        }
    }
}

// Several dense bfloat16 tensors with one step size each, RTNE, rows contracting, in one launch
// (qmm_quantize_multi): blockIdx.y picks the tensor; the arithmetic is quantize_rows_bf16x16's.
constexpr int kMaxMulti = 8;
struct MultiQ {
    const uint16_t* x[kMaxMulti];
    uint8_t* codes[kMaxMulti];
    const float* delta[kMaxMulti];
    int64_t nvec16[kMaxMulti];
};
template <int FMT> __global__ void __launch_bounds__(kThreads)
quantize_flat_multi(MultiQ a)
{
    const int t = blockIdx.y;
    const int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (v >= a.nvec16[t]) return;
    const float rho = 1.0f / a.delta[t][0];
    const u32x4* src = reinterpret_cast<const u32x4*>(a.x[t]) + 2 * v;
    const u32x4 w0 = src[0], w1 = src[1];
    store_through(a.codes[t] + 16 * v, encode16_bf16_rtne<FMT>(w0, w1, rho));
}

// Column-contracting (the input is [K][N], codes are [N][K]): any type, extent, stride and alignment.  Workgroup tile =
// 128 k x kTileN n.  A thread loads RT rows (k) x V elements (n), packs the codes of each column along k into dwords and
// parks them in an LDS tile [n][k]; then every thread writes 16-byte (kTileN = 16: 8-byte) pieces of finished code rows.
// kTileN = 64, 16 bytes a thread and row; 128 for large bfloat16 tensors: from 2048 wide tiles on 256 contiguous bytes per
// input row count for more than twice the workgroups (bfloat16 16384 x 3072: 29.7 against 32.8 us; 16384 x 1024, 1024 wide
// tiles: 12.1 against 11.5 us; 512 matrices of 512 x 64: 14.9 against 11.2 us).  16, two elements a thread and row, where
// the chip would be idle otherwise, up to 192 tiles of 64 (256 with stochastic rounding): a thread's 32 codes, with
// stochastic rounding eight generator blocks one behind the other, are what such a tensor takes (tiles of 64 / 16: 768 x 768
// bfloat16 3.3 / 2.9 us, stochastic 5.5 / 3.6; 16384 x 128, 256 tiles, 3.4 / 3.8, stochastic 5.7 / 5.2).
// grid (tiles, batch), tiles numbered along n first; workgroups loop where the grid would be too large to launch.
constexpr int kTileK = 128;
constexpr int kTileRowBytes = kTileK + 16;   // padded row of the LDS code tile

template <typename T, int FMT, int MODE, bool FOLD, int kTileN> __global__ void __launch_bounds__(kThreads)
quantize_cols(QArgs a, int64_t tiles_n, int64_t tiles)
{
    constexpr int V = kTileN == 16 ? 2 : Vec<T>::V;
    constexpr int TN = kTileN / V, TK = kThreads / TN, RT = kTileK / TK;       // 8 x 32 threads of 4 rows, or 16 x 16 of 8
    constexpr int Q = kThreads / kTileN;                                       // threads per column in the fold
    constexpr int PB = kTileN * kTileK / kThreads < 16 ? 8 : 16;               // bytes of a finished piece
    static_assert(RT % 4 == 0, "codes are packed four rows at a time");
    __shared__ __attribute__((aligned(16))) uint8_t tile[kTileN * kTileRowBytes];
    __shared__ uint32_t s_max[Q][kTileN];
    __shared__ float s_rho[kTileN];
    const int tn = threadIdx.x % TN, tk = threadIdx.x / TN;
    const int64_t b = blockIdx.y;
    const int64_t K = a.rows, N = a.cols;
    // 16-byte chunk c of code row n lies at chunk position c ^ ((n >> 3) & 7): the eight column vectors of a wavefront's
    // dword stores would otherwise meet in the same banks
    auto place = [](int n, int k) { return n * kTileRowBytes + ((((k >> 4) ^ (n >> 3)) & 7) << 4) + (k & 15); };
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int64_t tile_k = tiles <= 0xFFFFFFFFll ? (int64_t)((uint32_t)t / (uint32_t)tiles_n) : t / tiles_n;
        const int64_t tile_n = t - tile_k * tiles_n;
        const int64_t n0 = tile_n * kTileN, k0 = tile_k * kTileK;
        const int64_t n = n0 + tn * V, k_first = k0 + tk * RT;
        const int n_left = (int)max((int64_t)0, min((int64_t)V, N - n));          // columns of this thread inside the matrix
        const bool live = k_first < K && n_left > 0;
        u32x4 w[RT];
#pragma unroll
        for (int i = 0; i < RT; ++i) w[i] = u32x4{0u, 0u, 0u, 0u};
        if (live) {
            // (rows past the last one are the last one again, without a test for each: their codes are not stored)
            const T* base = static_cast<const T*>(a.x) + b * a.batch_stride + k_first * a.row_stride + n;
            const int last = (int)min(K - 1 - k_first, (int64_t)(RT - 1));
            if (n_left == V) {
#pragma unroll
                for (int i = 0; i < RT; ++i) w[i] = load_columns<T, V>(base + min(i, last) * a.row_stride, V);
            } else {
#pragma unroll
                for (int i = 0; i < RT; ++i) w[i] = load_columns<T, V>(base + min(i, last) * a.row_stride, n_left);
            }
        }
        // step sizes of the tile's columns, while the elements are on their way
        const int c = threadIdx.x & (kTileN - 1), q4 = threadIdx.x / kTileN;
        const int64_t col = n0 + c;
        if (FOLD && a.channels > 1) {
            // one scale group per matrix (host): fold the column's P partial maxima, Q threads a column
            uint32_t m = 0;
            if (col < N) {
                const uint32_t* p = a.partial + b * a.P * N + col;
#pragma unroll
                for (int i = 0; i < kFoldSlabs / Q; ++i) {
                    const int64_t s = q4 + Q * i;
                    if (s < a.P) m = max(m, p[s * N]);
                }
            }
            s_max[q4][c] = m;
            __syncthreads();
            if (q4 == 0) {
#pragma unroll
                for (int i = 1; i < Q; ++i) m = max(m, s_max[i][c]);
                const float d = delta_from_absmax_bits(m, a.qmax);
                s_rho[c] = 1.0f / d;
                if (tile_k == 0 && col < N) a.delta[group_of(a, b) * N + col] = d;
            }
        } else if (FOLD) {
            const float d = fold_delta(a, b, t == 0 && writes_group(a, b));
            if (q4 == 0) s_rho[c] = 1.0f / d;
        } else if (q4 == 0) {
            s_rho[c] = 1.0f / a.delta[group_of(a, b) * a.channels + (a.channels > 1 ? min(col, N - 1) : 0)];
        }
        __syncthreads();
        // Column by column: RT codes of consecutive output elements, in one run of code for columns that start generator blocks
        // and one for others, which share the blocks among a column's codes (not in the wide tile: host).  One part at a time:
        // interleaved, the generator blocks of a thread need up to 240 registers.
        auto columns = [&](auto at_block, auto quads) {
            constexpr int B = decltype(quads)::value;
            uint64_t g = (uint64_t)((b * N + n) * K + k_first) + a.offset;        // number of the column's first code
#pragma unroll
            for (int j = 0; j < V; ++j, g += (uint64_t)K) {
                const float rho = s_rho[tn * V + j];
#pragma unroll
                for (int q = 0; q < RT / 4; q += B) {
                    float v[4 * B];
#pragma unroll
                    for (int e = 0; e < 4 * B; ++e) v[e] = Vec<T>::at(w[4 * q + e], j) * rho;
                    uint32_t code[B];
                    encode_quads<FMT, MODE, B>(v, g + 4 * q, a.seed, at_block.value, code);
#pragma unroll
                    for (int e = 0; e < B; ++e) *reinterpret_cast<uint32_t*>(&tile[place(tn * V + j, tk * RT + 4 * (q + e))]) = code[e];
                    if constexpr (MODE == QMM_ROUND_STOCHASTIC && kTileN > 16) __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        if (live) {
            if constexpr (MODE == QMM_ROUND_RTNE || kTileN == 128) columns(std::true_type{}, std::integral_constant<int, 1>{});
            else if (whole_blocks(a)) columns(std::true_type{}, std::integral_constant<int, 1>{});
            else columns(std::false_type{}, std::integral_constant<int, RT / 4>{});
        }
        __syncthreads();
        // finished pieces, 1, 2 or 4 per thread
#pragma unroll
        for (int it = 0; it < kTileN * kTileK / PB / kThreads; ++it) {
            const int piece = it * kThreads + threadIdx.x;
            const int row = piece / (kTileK / PB), at = piece % (kTileK / PB) * PB;
            const int64_t nn = n0 + row, kk = k0 + at;
            if (nn >= N || kk >= K) continue;
            uint8_t* dst = a.codes + (b * N + nn) * K + kk;
            const uint8_t* srcp = &tile[place(row, at)];
            u32x4 codes;
            if constexpr (PB == 16) codes = *reinterpret_cast<const u32x4*>(srcp);
            else { const u32x2 h = *reinterpret_cast<const u32x2*>(srcp); codes = u32x4{h[0], h[1], 0u, 0u}; }
            if (kk + PB <= K) {
                if constexpr (PB == 16) *reinterpret_cast<u32x4_byte*>(dst) = codes;
                else *reinterpret_cast<u32x2_byte*>(dst) = u32x2{codes[0], codes[1]};
            } else {
                store_bytes<PB>(dst, codes, (int)(K - kk));
            }
        }
        if (t + gridDim.x < tiles) __syncthreads();          // the tile and the step sizes are reused
    }
}

// One thread per code, for tensors so small that nothing but the length of a thread's own work counts, and for contractions
// over so few rows that a tile of 128 would be idle but for a strip (8 x 200000 bfloat16 4.0 against 7.6 us, stochastic 6.6
// against 12.4; 3000 matrices of 16 x 64 7.8 against 7.3, stochastic 11.3 against 11.8).  Small tensors, contracting over
// rows 33 x 70 1.8 us against 2.6 in tiles of 16, stochastic 1.9 against 3.8; 256 x 768 2.5 against 2.6.  Contracting over
// columns the vectors of the row kernels are as fast, but for stochastic rounding of rows that are not whole generator
// blocks (301 x 202: 2.0 against 2.8 us).
constexpr int64_t kEachMax = 1 << 18;
template <typename T, int FMT, int MODE> __global__ void __launch_bounds__(kThreads)
quantize_each(QArgs a, int contract_axis)
{
    const uint32_t NC = (uint32_t)(contract_axis == 1 ? a.rows : a.cols), KC = (uint32_t)(contract_axis == 1 ? a.cols : a.rows);
    const uint32_t i = blockIdx.x * kThreads + threadIdx.x, n = i / KC, k = i - n * KC;
    if (n >= NC) return;
    const int64_t b = blockIdx.y;
    const float d = a.delta[group_of(a, b) * a.channels + (a.channels > 1 ? n : 0u)];
    const int64_t r = contract_axis == 1 ? n : k, c = contract_axis == 1 ? k : n;
    const u32x4 x = Vec<T>::partial_load(static_cast<const T*>(a.x) + b * a.batch_stride + r * a.row_stride + c, 1);
    const float t = Vec<T>::at(x, 0) * (1.0f / d);
    const int64_t p = (b * NC + n) * KC + k;
    if constexpr (MODE == QMM_ROUND_RTNE) {
        const float v[4] = {t, t, t, t};
        uint32_t code[1];
        encode_quads<FMT, MODE, 1>(v, 0, 0, true, code);
        a.codes[p] = (uint8_t)code[0];
    } else {
        const uint64_t g = (uint64_t)p + a.offset, blk = g >> 2;
        const Philox4 q = philox4x32_10((uint32_t)blk, (uint32_t)(blk >> 32), 0u, 0u, (uint32_t)a.seed, (uint32_t)(a.seed >> 32));
        const uint32_t j = (uint32_t)g & 3u, word = j == 0 ? q.v[0] : j == 1 ? q.v[1] : j == 2 ? q.v[2] : q.v[3];
        const float v[4] = {t, t, t, t};
        const uint32_t words[4] = {word, word, word, word};
        a.codes[p] = (uint8_t)encode_sr4<FMT>(v, words);
    }
}

template <typename T, int FMT, int MODE, bool FOLD> void launch_rows(const QArgs& q, hipStream_t s)
{
    RowPlan plan{};
    const int64_t nvec = (q.cols + Vec<T>::V - 1) / Vec<T>::V, slots_per_row = (nvec + kWave - 1) / kWave;
    const bool is_short = nvec <= 2 * kWave && q.rows > 1;
    int64_t slots = q.rows * slots_per_row;                                  // wavefront-wide rows of vectors, per matrix
    if (is_short) {
        while (plan.lane_shift < 6 && (1 << plan.lane_shift) < nvec) ++plan.lane_shift;
        plan.half_shift = nvec > kWave ? 1 : 0;
        const int64_t at_once = kWave >> plan.lane_shift;
        slots = ((q.rows + at_once - 1) / at_once) << plan.half_shift;
    }
    const bool small = slots * q.batch <= 4096;                              // sixteen wavefronts per CU and fewer
    const int piece = small ? 1 : 2;
    if (is_short) plan.units = (slots + piece - 1) / piece;
    else { plan.pieces = (slots_per_row + piece - 1) / piece; plan.units = q.rows * plan.pieces; }
    constexpr int kWaves = kThreads / kWave;
    // (FOLD: every workgroup fetches its group's partial maxima, so no more of them than the chip holds at a time)
    const dim3 grid((unsigned)std::min<int64_t>((plan.units + kWaves - 1) / kWaves, FOLD ? std::max<int64_t>(2048 / q.batch, 1) : 65536), (unsigned)q.batch);
    if (is_short) {
        if (small) quantize_rows<T, FMT, MODE, FOLD, 1, true><<<grid, kThreads, 0, s>>>(q, plan);
        else quantize_rows<T, FMT, MODE, FOLD, 2, true><<<grid, kThreads, 0, s>>>(q, plan);
    } else {
        if (small) quantize_rows<T, FMT, MODE, FOLD, 1, false><<<grid, kThreads, 0, s>>>(q, plan);
        else quantize_rows<T, FMT, MODE, FOLD, 2, false><<<grid, kThreads, 0, s>>>(q, plan);
    }
}

// fold: the step sizes are formed by this pass from a.partial, else read from a.delta.
template <int FMT, int MODE, bool FOLD> qmm_status launch(const qmm_tensor* x, const QArgs& a, hipStream_t s)
{
    const bool bf16 = x->dtype == QMM_DT_BF16;
    if constexpr (!FOLD) {
        const int64_t n = x->rows * x->cols;
        const bool few_rows = x->contract_axis == 0 && x->rows <= (MODE == QMM_ROUND_RTNE ? 12 : 16) && n < (int64_t(1) << 31);
        const bool tiny = n * x->batch <= kEachMax && (x->contract_axis == 0 || (MODE == QMM_ROUND_STOCHASTIC && x->cols % 4 != 0));
        if (few_rows || tiny) {
            const dim3 grid((unsigned)((n + kThreads - 1) / kThreads), (unsigned)x->batch);
            if (bf16) quantize_each<uint16_t, FMT, MODE><<<grid, kThreads, 0, s>>>(a, x->contract_axis);
            else quantize_each<float, FMT, MODE><<<grid, kThreads, 0, s>>>(a, x->contract_axis);
            return launch_status();
        }
    }
    if (x->contract_axis == 0) {
        const int64_t tiles_k = (x->rows + kTileK - 1) / kTileK;
        const bool wide = bf16 && tiles_k * (x->cols / 128) * x->batch >= 2048 && (MODE == QMM_ROUND_RTNE || whole_blocks(a));
        const bool narrow = tiles_k * ((x->cols + 63) / 64) * x->batch <= (MODE == QMM_ROUND_RTNE ? 192 : 256);
        const int tile_n = wide ? 128 : narrow ? 16 : 64;
        const int64_t tiles_n = (x->cols + tile_n - 1) / tile_n, tiles = tiles_n * tiles_k;
        const dim3 grid((unsigned)std::min<int64_t>(tiles, 1 << 23), (unsigned)x->batch);
        if (wide) quantize_cols<uint16_t, FMT, MODE, FOLD, 128><<<grid, kThreads, 0, s>>>(a, tiles_n, tiles);
        else if (narrow && bf16) quantize_cols<uint16_t, FMT, MODE, FOLD, 16><<<grid, kThreads, 0, s>>>(a, tiles_n, tiles);
        else if (narrow) quantize_cols<float, FMT, MODE, FOLD, 16><<<grid, kThreads, 0, s>>>(a, tiles_n, tiles);
        else if (bf16) quantize_cols<uint16_t, FMT, MODE, FOLD, 64><<<grid, kThreads, 0, s>>>(a, tiles_n, tiles);
        else quantize_cols<float, FMT, MODE, FOLD, 64><<<grid, kThreads, 0, s>>>(a, tiles_n, tiles);
        return launch_status();
    }
    // a matrix that is dense with one step size is one long row
    QArgs q = a;
    if (q.channels == 1 && q.row_stride == q.cols) {
        q.cols *= q.rows;
        q.row_stride = q.cols;
        q.rows = 1;
    }
    const bool aligned = aligned16(x->data) && (q.row_stride % 8 == 0 || q.rows == 1) && (x->batch_stride % 8 == 0 || x->batch == 1);
    if (bf16 && aligned && (q.cols % 16 == 0) && aligned16(a.codes)) {
        const int64_t nv = q.rows * (q.cols / 16);
        // Codes of many matrices that an XCD's L2 holds, half the memory-side cache and more in all, behind the scale pass (a.streaming): that
        // pass has filled the cache with the tensor, and codes that are kept push out what is being read.  Kept / streaming, both
        // steps and the product that reads the codes, E4M3, matrices of 1024 x 1024, codes on the left of 64 columns and on the right of
        // 64, 256 and 1024 rows: 64 matrices 72 / 75 us, 76 / 80, 82 / 86, 132 / 132; 96 of them 116 / 115, 125 / 124, 130 / 128, 201 / 195;
        // 128 150 / 143, 155 / 149, 165 / 156, 268 / 255; 256 297 / 286, 305 / 297, 324 / 310, 505 / 501.  Of 512 x 512: 256 71 / 76 to
        // 152 / 158; 384 118 / 120, 126 / 126, 135 / 131, 232 / 228; 512 155 / 151, 161 / 155, 180 / 171, 311 / 305; 2048 of 256 x 256 174 / 168,
        // 175 / 170, 223 / 215, 477 / 470.  With step sizes that were there already the codes are better kept: quantize and product, 128
        // of 1024 x 1024 94 / 103, 105 / 109, 113 / 116, 223 / 220.  One matrix of 67 MB of codes: the pass the same, the product 51 / 55.
        const int64_t matrix = q.rows * q.cols;
        q.streaming = a.streaming && q.batch > 1 && matrix <= (int64_t(1) << 20) && q.batch * matrix >= (int64_t(1) << 27);
        // Past the L2, matrices off a line's boundary in calls of up to 32 MB only (by the L2 / past it: 300 matrices of 100016 codes 16.5 / 16.0
        // us, 40 of 1000016 23.1 / 23.2, 64 of them 35.8 / 36.8, 128 68.5 / 74.0; of whole lines, 64 of 1048576, 36.3 / 35.5).
        q.through = in_lines(q.codes, q.batch > 1 ? matrix : 0) || q.batch * matrix <= (int64_t)32 << 20;
        quantize_rows_bf16x16<FMT, MODE, FOLD><<<dim3((unsigned)((nv + kThreads - 1) / kThreads), (unsigned)x->batch), kThreads, 0, s>>>(q);
        return launch_status();
    }
    if (bf16) launch_rows<uint16_t, FMT, MODE, FOLD>(q, s);
    else launch_rows<float, FMT, MODE, FOLD>(q, s);
    return launch_status();
}

template <int FMT> qmm_status launch_mode(const qmm_tensor* x, const QArgs& a, qmm_round mode, hipStream_t s)
{
    return mode == QMM_ROUND_RTNE ? launch<FMT, QMM_ROUND_RTNE, false>(x, a, s) : launch<FMT, QMM_ROUND_STOCHASTIC, false>(x, a, s);
}

// One step size per row, every matrix a scale group of its own, rows that fit the registers of one wavefront (8 vectors a
// lane: 4096 bfloat16 / 2048 binary32 elements) or of the four of a workgroup (4 vectors a lane: 8192 / 4096).
bool one_pass(const qmm_tensor* x, const qmm_granularity* g)
{
    return g->per_channel && x->contract_axis == 1 && x->batch == g->batch_groups && g->batch_inner <= 1 &&
           x->cols <= (x->dtype == QMM_DT_BF16 ? 8192 : 4096);
}
template <typename T, int FMT, int MODE> qmm_status launch_one_pass(const QArgs& a, hipStream_t s)
{
    constexpr int V = Vec<T>::V;
    const int64_t rows = a.batch * a.rows;
    const int64_t nvec = (a.cols + V - 1) / V;
    auto blocks = [&](int lpr) { return (unsigned)std::min<int64_t>((rows + kThreads / lpr - 1) / (kThreads / lpr), 1 << 23); };
    // lanes x vectors with little idle: 96 and 384 vectors (768 and 3072 bfloat16 columns) in three and six rather than four
    // and eight (stochastic rounding is bound by the generator's multiplies, and idle lanes wait for them)
    auto run = [&](auto lpr, auto nv) { scale_quantize_rows<T, FMT, MODE, lpr.value, nv.value><<<blocks(lpr.value), kThreads, 0, s>>>(a); };
    if (nvec <= 8) run(std::integral_constant<int, 8>{}, std::integral_constant<int, 1>{});
    else if (nvec <= 16) run(std::integral_constant<int, 16>{}, std::integral_constant<int, 1>{});
    else if (nvec <= 32) run(std::integral_constant<int, 32>{}, std::integral_constant<int, 1>{});
    else if (nvec <= 64) run(std::integral_constant<int, 64>{}, std::integral_constant<int, 1>{});
    else if (nvec <= 96) run(std::integral_constant<int, 32>{}, std::integral_constant<int, 3>{});
    else if (nvec <= 128) run(std::integral_constant<int, 64>{}, std::integral_constant<int, 2>{});
    else if (nvec <= 192) run(std::integral_constant<int, 64>{}, std::integral_constant<int, 3>{});
    else if (nvec <= 256) run(std::integral_constant<int, 64>{}, std::integral_constant<int, 4>{});
    else if (nvec <= 384) run(std::integral_constant<int, 64>{}, std::integral_constant<int, 6>{});
    else if (nvec <= 512) run(std::integral_constant<int, 64>{}, std::integral_constant<int, 8>{});
    else run(std::integral_constant<int, 256>{}, std::integral_constant<int, 4>{});
    return launch_status();
}
template <int FMT> qmm_status launch_one_pass_mode(const qmm_tensor* x, const QArgs& a, qmm_round mode, hipStream_t s)
{
    if (x->dtype == QMM_DT_BF16)
        return mode == QMM_ROUND_RTNE ? launch_one_pass<uint16_t, FMT, QMM_ROUND_RTNE>(a, s) : launch_one_pass<uint16_t, FMT, QMM_ROUND_STOCHASTIC>(a, s);
    return mode == QMM_ROUND_RTNE ? launch_one_pass<float, FMT, QMM_ROUND_RTNE>(a, s) : launch_one_pass<float, FMT, QMM_ROUND_STOCHASTIC>(a, s);
}
template <int FMT> qmm_status launch_fold_mode(const qmm_tensor* x, const QArgs& a, qmm_round mode, hipStream_t s)
{
    return mode == QMM_ROUND_RTNE ? launch<FMT, QMM_ROUND_RTNE, true>(x, a, s) : launch<FMT, QMM_ROUND_STOCHASTIC, true>(x, a, s);
}

}  // namespace
}  // namespace qmm

using namespace qmm;

namespace {
// Everything qmm_quantize can refuse, checked without launching: QMM_OK means the call will enqueue (or has nothing to do).
qmm_status quantize_check(const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g, const float* delta,
                          qmm_round mode, const uint8_t* codes_out)
{
    if (!x || !g) return QMM_ERR_NULL;
    if (x->dtype != QMM_DT_BF16 && x->dtype != QMM_DT_F32) return QMM_ERR_ENUM;
    if (x->contract_axis != 0 && x->contract_axis != 1) return QMM_ERR_ENUM;
    if (fmt != QMM_FMT_INT8 && fmt != QMM_FMT_E4M3 && fmt != QMM_FMT_E5M2) return QMM_ERR_ENUM;
    if (mode != QMM_ROUND_RTNE && mode != QMM_ROUND_STOCHASTIC) return QMM_ERR_ENUM;
    if (g->batch_groups < 1 || g->batch_inner < 0 || (g->per_channel != 0 && g->per_channel != 1)) return QMM_ERR_ENUM;
    if (x->batch < 0 || x->rows < 0 || x->cols < 0 || x->row_stride < x->cols) return QMM_ERR_SHAPE;
    if (x->batch > 1 && x->rows > 0 && x->batch_stride < (x->rows - 1) * x->row_stride + x->cols) return QMM_ERR_SHAPE;
    if (x->batch > 65535) return QMM_ERR_UNSUPPORTED;
    if (x->batch * x->rows * x->cols == 0) return QMM_OK;
    if (!x->data || !delta || !codes_out) return QMM_ERR_NULL;
    return QMM_OK;
}

QArgs quantize_args(const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g, float* delta, uint64_t seed, uint64_t offset,
                    uint8_t* codes_out)
{
    QArgs a{};
    a.x = x->data; a.delta = delta; a.codes = codes_out;
    a.batch = x->batch; a.rows = x->rows; a.cols = x->cols;
    a.batch_stride = x->batch_stride; a.row_stride = x->row_stride;
    a.groups = g->batch_groups;
    a.inner = g->batch_inner > 0 ? g->batch_inner : 1;
    a.channels = g->per_channel ? (x->contract_axis == 1 ? x->rows : x->cols) : 1;
    a.seed = seed; a.offset = offset;
    a.qmax = host_qmax(fmt);
    return a;
}
}  // namespace

extern "C" qmm_status qmm_quantize(const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g, const float* delta,
                                   qmm_round mode, uint64_t seed, uint64_t offset, uint8_t* codes_out, void* stream)
{
    const qmm_status chk = quantize_check(x, fmt, g, delta, mode, codes_out);
    if (chk != QMM_OK) return chk;
    if (x->batch * x->rows * x->cols == 0) return QMM_OK;

    const QArgs a = quantize_args(x, fmt, g, const_cast<float*>(delta), seed, offset, codes_out);
    hipStream_t s = as_stream(stream);
    switch (fmt) {
    case QMM_FMT_INT8: return launch_mode<QMM_FMT_INT8>(x, a, mode, s);
    case QMM_FMT_E4M3: return launch_mode<QMM_FMT_E4M3>(x, a, mode, s);
    default: return launch_mode<QMM_FMT_E5M2>(x, a, mode, s);
    }
}

namespace {
// The quantize pass folds the partial maxima when every group has a matrix (its first workgroup writes the step size), a
// group's partial maxima are few -- each workgroup fetches them -- and the tensor is not large: per workgroup the fold costs
// about what it fetches, against one small kernel and its launch.  One step size per column: one matrix per group, up to
// 2^24 elements (bfloat16, fold / small kernel apart from its launch: 4096 x 3072 +1.7 / 3.8 us, 16384 x 3072 +11 / 3.8; both
// steps, tall, 65536 x 128 20.5 / 18.1, binary32 262144 x 64 75 / 33).  One
// step size per group: up to 2^23 elements, or 2^24 where a group has at most 256 (both steps, bfloat16, fold / not: one group of
// 1024, 8192 x 1024 9.9 / 10.7 us, 16384 x 1024 19.4 / 17.8; sixteen groups of 64, 512 matrices of 512 x 64 18.1 / 18.6, with
// their rows contracting 18.0 / 19.4).
bool folds(const qmm_tensor* x, const qmm_granularity* g)
{
    if (!(x->batch > 0 && x->rows > 0 && x->cols > 0) || g->batch_groups < 1) return false;
    const int64_t inner = g->batch_inner > 0 ? g->batch_inner : 1, n = x->batch * x->rows * x->cols;
    const bool many_channels = g->per_channel && (x->contract_axis == 1 ? x->rows : x->cols) > 1;
    if (many_channels) {
        // (a tall, narrow tensor: the few slabs that can be folded leave the chip idle)
        const int64_t column_blocks = (x->cols + 127) / 128 * x->batch;
        const bool tall = x->rows > 1024 * kFoldSlabs && column_blocks * kFoldSlabs < 256;
        return n <= (int64_t(1) << 24) && x->contract_axis == 0 && g->batch_groups == x->batch && inner == 1 && !tall;
    }
    if (n > (int64_t(1) << 24) || g->batch_groups > x->batch || (g->batch_groups - 1) * inner >= x->batch) return false;
    const int64_t words = (int64_t)(scale_partials_size(x, g, true) / sizeof(uint32_t));
    // (many small matrices in few groups: a workgroup would fetch more than it quantizes; 4096 of 32 x 64 in 8, 512 partial maxima
    // each: 13.3 against 12.4 us, with their rows contracting 24.8 against 16.8)
    if (g->batch_groups > 1 && words > std::max<int64_t>(n / x->batch / 8, 32) * g->batch_groups) return false;
    return words <= (n > (int64_t(1) << 23) ? kFoldMax / 4 : kFoldMax) * g->batch_groups;
}
}  // namespace

extern "C" size_t qmm_scale_quantize_workspace_size(const qmm_tensor* x, const qmm_granularity* g)
{
    if (!x || !g || one_pass(x, g)) return 0;
    return scale_partials_size(x, g, folds(x, g));
}

extern "C" qmm_status qmm_scale_quantize(const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g, qmm_round mode,
                                         uint64_t seed, uint64_t offset, float* delta_out, uint8_t* codes_out,
                                         void* workspace, size_t workspace_bytes, void* stream)
{
    // the arguments of both steps first; a call that needs no workspace is checked against one of full size
    if (!x || !g) return QMM_ERR_NULL;
    const bool single = one_pass(x, g), fold = !single && folds(x, g);
    qmm_status st = scale_arguments(x, fmt, g, delta_out, single ? reinterpret_cast<const void*>(uintptr_t(256)) : workspace,
                                    single ? ~size_t(0) : workspace_bytes, fold);
    if (st != QMM_OK) return st;
    st = quantize_check(x, fmt, g, delta_out, mode, codes_out);
    if (st != QMM_OK) return st;
    if (x->batch * x->rows * x->cols == 0) {       // no codes; the groups of an empty tensor still get their step size
        if (qmm_num_scales(x, g) == 0) return QMM_OK;
        const ScalePartials none{0, 0, g->per_channel ? (x->contract_axis == 1 ? x->rows : x->cols) : 1, false};
        return scale_fold(none, nullptr, fmt, g, delta_out, as_stream(stream));
    }
    hipStream_t s = as_stream(stream);
    QArgs a = quantize_args(x, fmt, g, delta_out, seed, offset, codes_out);
    if (single) {
        switch (fmt) {
        case QMM_FMT_INT8: return launch_one_pass_mode<QMM_FMT_INT8>(x, a, mode, s);
        case QMM_FMT_E4M3: return launch_one_pass_mode<QMM_FMT_E4M3>(x, a, mode, s);
        default: return launch_one_pass_mode<QMM_FMT_E5M2>(x, a, mode, s);
        }
    }
    bool taken = false;
    st = scale_quantize_resident(x, fmt, g, mode, seed, offset, delta_out, codes_out, kPatience, s, &taken);
    if (taken || st != QMM_OK) return st;
    uint32_t* partial = static_cast<uint32_t*>(workspace);
    ScalePartials pp;
    st = scale_partials(x, fmt, g, delta_out, partial, fold, &pp, s);
    if (st != QMM_OK) return st;
    if (!pp.done && !fold) { st = scale_fold(pp, partial, fmt, g, delta_out, s); if (st != QMM_OK) return st; }
    a.streaming = 1;
    if (fold && !pp.done) {
        a.partial = partial; a.P = pp.P; a.fold_total = (int)(pp.batch * pp.P);
        switch (fmt) {
        case QMM_FMT_INT8: return launch_fold_mode<QMM_FMT_INT8>(x, a, mode, s);
        case QMM_FMT_E4M3: return launch_fold_mode<QMM_FMT_E4M3>(x, a, mode, s);
        default: return launch_fold_mode<QMM_FMT_E5M2>(x, a, mode, s);
        }
    }
    switch (fmt) {
    case QMM_FMT_INT8: return launch_mode<QMM_FMT_INT8>(x, a, mode, s);
    case QMM_FMT_E4M3: return launch_mode<QMM_FMT_E4M3>(x, a, mode, s);
    default: return launch_mode<QMM_FMT_E5M2>(x, a, mode, s);
    }
}

extern "C" qmm_status qmm_quantize_multi(int32_t count, const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g,
                                         const float* const* delta, qmm_round mode, uint64_t seed, const uint64_t* offsets,
                                         uint8_t* const* codes_out, void* stream)
{
    if (count < 0) return QMM_ERR_SHAPE;
    if (count == 0) return QMM_OK;
    if (!x || !g || !delta || !codes_out) return QMM_ERR_NULL;
    if (fmt != QMM_FMT_INT8 && fmt != QMM_FMT_E4M3 && fmt != QMM_FMT_E5M2) return QMM_ERR_ENUM;
    if (mode != QMM_ROUND_RTNE && mode != QMM_ROUND_STOCHASTIC) return QMM_ERR_ENUM;
    bool one_launch = count <= kMaxMulti && mode == QMM_ROUND_RTNE;
    for (int32_t t = 0; t < count && one_launch; ++t) {
        const qmm_tensor& q = x[t];
        one_launch = q.data && delta[t] && codes_out[t] && q.dtype == QMM_DT_BF16 && q.contract_axis == 1 && q.batch == 1 &&
                     !g[t].per_channel && g[t].batch_groups == 1 && g[t].batch_inner >= 0 && q.rows >= 1 && q.cols >= 16 &&
                     q.cols % 16 == 0 && q.row_stride == q.cols && aligned16(q.data) && aligned16(codes_out[t]);
    }
    if (!one_launch) {
        for (int32_t t = 0; t < count; ++t) {      // every tensor's arguments before the first launch
            const qmm_status st = quantize_check(x + t, fmt, g + t, delta[t], mode, codes_out[t]);
            if (st != QMM_OK) return st;
        }
        for (int32_t t = 0; t < count; ++t) {
            const qmm_status st = qmm_quantize(x + t, fmt, g + t, delta[t], mode, seed, offsets ? offsets[t] : 0, codes_out[t], stream);
            if (st != QMM_OK) return st;
        }
        return QMM_OK;
    }
    MultiQ a{};
    int64_t max_vec = 1;
    for (int32_t t = 0; t < count; ++t) {
        a.x[t] = static_cast<const uint16_t*>(x[t].data);
        a.codes[t] = codes_out[t];
        a.delta[t] = delta[t];
        a.nvec16[t] = x[t].rows * x[t].cols / 16;
        max_vec = std::max(max_vec, a.nvec16[t]);
    }
    const int64_t blocks = (max_vec + kThreads - 1) / kThreads;
    if (blocks > 0x7FFFFFFF) return QMM_ERR_UNSUPPORTED;
    hipStream_t s = as_stream(stream);
    const dim3 grid((unsigned)blocks, (unsigned)count);
    if (fmt == QMM_FMT_INT8) quantize_flat_multi<QMM_FMT_INT8><<<grid, kThreads, 0, s>>>(a);
    else if (fmt == QMM_FMT_E4M3) quantize_flat_multi<QMM_FMT_E4M3><<<grid, kThreads, 0, s>>>(a);
    else quantize_flat_multi<QMM_FMT_E5M2><<<grid, kThreads, 0, s>>>(a);
    return launch_status();
}
