// qmm_scale: step size delta = max|X| / qmax per scale group (Eq. 1, right half;
// Methodology bullets on scale granularity and on aligning the absmax with the
// format maximum).  HBM-bound: every element is read once (2 B for bfloat16),
// the maximum is taken on magnitude bit patterns (exact, order-free), partial
// maxima are folded per group, followed by the one division.  One step size per
// matrix or group of matrices and the several-tensors call: one launch, the
// maxima crossing through a board.  Calls being recorded into a graph, which a
// board's tags do not fit, leave them in the workspace, for a second small kernel
// or, from 2^24 elements, the workgroup that finishes last.  Step sizes per row
// or column: a second kernel, or the quantize pass of qmm_scale_quantize.  The
// maximum is order-free, so the result does not depend on launch geometry or on
// which workgroup folds.
#include <algorithm>
#include <atomic>
#include <type_traits>
#include "qmm_device.h"

namespace qmm {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxFlatBlocks = 1024;   // 4 workgroups per CU on 256 CUs; 4 partials per thread in the fold
constexpr int kColSlabRows = 128;      // rows folded by one workgroup in the column-group kernel, at least
constexpr int kMaxColSlabs = 512;      // and slabs of them, at most

typedef qmm_u32x4 u32x4;
typedef unsigned int u32x4_any __attribute__((ext_vector_type(4), aligned(2)));   // global memory takes vector loads at any element boundary

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

// The fold of a tensor's partial maxima by the workgroup that arrived last: all of them are one scale group.
QMM_DEV void fold_all_partials(const uint32_t* partial, int64_t count, float qmax, float* delta)
{
    uint32_t v[4] = {0u, 0u, 0u, 0u}, m = 0;
    int64_t i = threadIdx.x;
    for (; i + 3 * kThreads < count; i += 4 * kThreads) {         // four requests in flight
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = coherent_load(partial + i + k * kThreads);
        m = max(max(m, max(v[0], v[1])), max(v[2], v[3]));
    }
    for (; i < count; i += kThreads) m = max(m, coherent_load(partial + i));
    m = block_max_u32(m);
    if (threadIdx.x == 0) delta[0] = delta_from_absmax_bits(m, qmax);
}
// The same by way of a board: the workgroups of a scale group post their maxima, and one of them, the last to start, waits for the
// words, folds them and writes the step size.  word(i): the i-th of the group's `total` words; slice(w): this thread's part of the
// maximum of the workgroup of word w, for words that do not come in time (looked for kThreads at a time).  A post and a read where publishing, counting in two
// levels and reading are a chain of four, and a launch less where a second kernel folded.  Kernel time, before / this: one step size,
// bfloat16, 131072 elements 4.4 / 3.8 us, 8 million 9.4 / 7.6, 16.8 million 10.4 / 9.3, 50 million 18.9 / 18.5; the several-tensors call
// on 16384 x 1024 and 4096 x 1024 10.8 / 9.6, 2048 x 768 and 768 x 768 5.2 / 4.4.
template <class Word, class Slice> QMM_DEV void fold_board(const Board& bd, uint32_t mine_at, uint32_t mine, bool folder, uint32_t total, float qmax, float* delta,
                                                           Word word, Slice slice)
{
    __shared__ uint32_t s_word;
    if (threadIdx.x == 0) board_post(bd, mine_at, mine);
    if (!folder) return;
    const uint64_t start = ticks();
    uint32_t m = 0;
    bool missing = false;
    for (uint32_t i = threadIdx.x; i < total; i += kThreads) {
        uint32_t v;
        if (board_wait(bd, word(i), start, v)) m = max(m, v); else missing = true;
    }
    if (__syncthreads_or(missing)) {
        __shared__ uint64_t s_missing[kThreads / kWave];
        for (uint32_t base = 0; base < total; base += kThreads) {
            const uint32_t i = base + threadIdx.x;
            uint32_t v;
            const bool none = i < total && !board_read(bd, word(i), v);
            if (i < total && !none) m = max(m, v);
            const uint64_t bits = __ballot(none);
            if ((threadIdx.x & (kWave - 1)) == 0) s_missing[threadIdx.x / kWave] = bits;
            __syncthreads();
            for (int k = 0; k < kThreads / kWave; ++k) {
                for (uint64_t left = s_missing[k]; left; left &= left - 1) {
                    const uint32_t w = word(base + k * kWave + (uint32_t)__ffsll((unsigned long long)left) - 1);
                    if (threadIdx.x == 0) { uint32_t late; s_word = board_read(bd, w, late) ? late : ~0u; }      // (others go on meanwhile)
                    __syncthreads();
                    const uint32_t late = s_word;
                    __syncthreads();
                    m = max(m, late != ~0u ? late : slice(w));             // (a posted value is below 2^31)
                }
            }
            __syncthreads();
        }
    }
    __syncthreads();                                         // block_max_u32's shared words are used a second time
    m = block_max_u32(m);
    if (threadIdx.x == 0) *delta = delta_from_absmax_bits(m, qmax);
}

// Dense matrix (row_stride == cols) from a 16-byte boundary on, n elements: grid (nblk, batch).  With a board one workgroup
// of each of the `groups` scale groups folds its partial maxima and writes the step size; with `slot` (one scale group) the one that arrives last.
template <typename T> __global__ void __launch_bounds__(kThreads)
absmax_flat(const T* __restrict__ x, int64_t batch_stride, int64_t n, uint32_t* __restrict__ partial,
            uint32_t* __restrict__ slot, Board bd, uint32_t groups, uint32_t inner, float qmax, float* __restrict__ delta)
{
    constexpr int V = VecMax<T>::V;
    const int64_t nvec = n / V;
    // A workgroup takes four consecutive 4 KB pieces per trip and the grid sweeps the tensor front to back: the
    // four loads a thread has in flight are then neighbours in memory.  (With the loads a whole grid stride apart
    // the same kernel reads a large tensor up to 25 % slower: four distant streams per thread.)  Ordinary loads on
    // purpose: streaming loads make this pass 7 % faster on a 134 MB tensor (23.0 against 24.6 us), but the quantize
    // pass that follows then finds less of the tensor in the memory-side cache and loses twice that.
    auto slice = [&](uint32_t bx, uint32_t by) -> uint32_t {
        const T* base = x + (int64_t)by * batch_stride;
        const u32x4* p = reinterpret_cast<const u32x4*>(base);
        VecMax<T> m;
        const int64_t stride = (int64_t)gridDim.x * kThreads * 4;
        int64_t i = (int64_t)bx * kThreads * 4 + threadIdx.x;
        for (; i + 3 * kThreads < nvec; i += stride) {
            const u32x4 a = p[i], b = p[i + kThreads];
            const u32x4 c = p[i + 2 * kThreads], d = p[i + 3 * kThreads];
            m.fold(a); m.fold(b); m.fold(c); m.fold(d);
        }
        // the ragged end: at most three pieces of one workgroup, and the elements past the last whole vector
        if (i < nvec) {
            for (int u = 0; u < 4; ++u)
                if (i + u * kThreads < nvec) m.fold(p[i + u * kThreads]);
        }
        uint32_t r = m.finish();
        if (bx == 0 && threadIdx.x < (unsigned)(n % V)) r = max(r, mag_bits<T>(base[nvec * V + threadIdx.x]));
        return r;
    };
    const uint32_t r = block_max_u32(slice(blockIdx.x, blockIdx.y));
    const unsigned id = blockIdx.y * gridDim.x + blockIdx.x, total = gridDim.x * gridDim.y;
    if (bd.words) {
        const uint32_t P = gridDim.x;
        const Group grp = group_at(gridDim.y, groups, inner, blockIdx.y);
        const bool folder = blockIdx.x == P - 1 && grp.k_of_b == grp.count - 1;
        fold_board(bd, id, r, folder, grp.count * P, qmax, delta + grp.g,
                   [&](uint32_t i) { const uint32_t k = i / P; return grp.matrix(k) * P + (i - k * P); },
                   [&](uint32_t w) { const uint32_t by = w / P; return slice(w - by * P, by); });
        return;
    }
    if (threadIdx.x == 0) {
        if (slot) publish_u32(partial + id, r); else partial[id] = r;
    }
    if (slot && arrive_last(slot, id, total)) {
        __syncthreads();                         // block_max_u32's shared words are reused by the fold
        fold_all_partials(partial, total, qmax, delta);
    }
}

// Several dense bfloat16 tensors, one step size each, in one launch (qmm_scale_multi): blockIdx.y picks the tensor,
// workgroups past a tensor's own count leave at once.  The 2-8 MB weight matrices of a layer are latency-bound on
// their own; launched beside the activations they cost next to nothing.
constexpr int kMaxMulti = 8;
struct MultiFlat {
    const uint16_t* x[kMaxMulti];
    int64_t nvec[kMaxMulti];        // 16-byte vectors
    uint32_t* partial[kMaxMulti];
    float* delta[kMaxMulti];
    int nblk[kMaxMulti];
    uint32_t* slots;                // kMaxMulti consecutive slots of arrival counters, one per tensor
    Board board;                    // kMaxFlatBlocks words per tensor, or none
    float qmax;
};
__global__ void __launch_bounds__(kThreads)
absmax_flat_multi(MultiFlat a)
{
    const int t = blockIdx.y;
    const int nblk = a.nblk[t];
    if ((int)blockIdx.x >= nblk) return;
    const u32x4* p = reinterpret_cast<const u32x4*>(a.x[t]);
    const int64_t nvec = a.nvec[t];
    auto slice = [&](uint32_t bx) -> uint32_t {
        u16x2 m[4] = {};
        const int64_t stride = (int64_t)nblk * kThreads * 4;
        int64_t i = (int64_t)bx * kThreads * 4 + threadIdx.x;
        for (; i + 3 * kThreads < nvec; i += stride) {
            const u32x4 v0 = p[i], v1 = p[i + kThreads];
            const u32x4 v2 = p[i + 2 * kThreads], v3 = p[i + 3 * kThreads];
            fold_bf16x8(v0, m); fold_bf16x8(v1, m); fold_bf16x8(v2, m); fold_bf16x8(v3, m);
        }
        if (i < nvec) {
            for (int u = 0; u < 4; ++u)
                if (i + u * kThreads < nvec) fold_bf16x8(p[i + u * kThreads], m);
        }
        return finish_bf16(m);
    };
    const uint32_t r = block_max_u32(slice(blockIdx.x));
    if (a.board.words) {
        fold_board(Board{a.board.words + t * kMaxFlatBlocks, a.board.tag, a.board.patience}, blockIdx.x, r, (int)blockIdx.x == nblk - 1, (uint32_t)nblk, a.qmax,
                   a.delta[t], [](uint32_t i) { return i; }, slice);
        return;
    }
    if (threadIdx.x == 0) publish_u32(a.partial[t] + blockIdx.x, r);
    // the tensor's last workgroup folds its partial maxima (at most kMaxFlatBlocks) and writes its step size
    if (arrive_last(a.slots + (size_t)t * kArrivalWords, blockIdx.x, (unsigned)nblk)) {
        __syncthreads();
        fold_all_partials(a.partial[t], nblk, a.qmax, a.delta[t]);
    }
}

// One wavefront per (matrix, row): partial[b*rows + r] = absmax of the row.  Any stride, any dtype.
template <typename T> __global__ void __launch_bounds__(kThreads)
absmax_rows(const T* __restrict__ x, int64_t batch_stride, int64_t row_stride, int64_t rows, int64_t cols,
            int64_t total_rows, uint32_t* __restrict__ partial, float qmax, float* __restrict__ delta)
{
    const int64_t wr = (int64_t)blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave;
    if (wr >= total_rows) return;
    const int64_t b = wr / rows, r = wr % rows;
    const T* p = x + b * batch_stride + r * row_stride;
    const int lane = threadIdx.x & (kWave - 1);
    constexpr int V = VecMax<T>::V;
    VecMax<T> mm;
    const int64_t nvec = cols / V;
    for (int64_t i = lane; i < nvec; i += kWave) mm.fold(*reinterpret_cast<const u32x4_any*>(p + i * V));
    uint32_t m = mm.finish();
    if (lane < (int)(cols - nvec * V)) m = max(m, mag_bits<T>(p[nvec * V + lane]));
    m = wave_max_u32(m);
    // delta != NULL: every row is a scale group of its own (one step size per row, one matrix per batch group), so
    // the row's maximum is final and the step size is written here, without the second kernel
    if (lane == 0) { if (delta) delta[wr] = delta_from_absmax_bits(m, qmax); else partial[wr] = m; }
}

// Short rows (at most 32 vectors), any alignment: LPR lanes per row, one 16-byte vector each, so a wavefront takes 64 / LPR
// rows at once instead of one (with the rows dense in memory it reads 1 KB contiguous).  A partial last vector is taken
// back to the end of its row: the maximum does not mind the elements it sees twice.
template <typename T, int LPR> __global__ void __launch_bounds__(kThreads)
absmax_rows_short(const T* __restrict__ x, int64_t batch_stride, int64_t row_stride, int64_t rows, int64_t cols,
                  int64_t total_rows, uint32_t* __restrict__ partial, float qmax, float* __restrict__ delta)
{
    constexpr int RPW = kWave / LPR, V = VecMax<T>::V;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t w = (int64_t)blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave;
    const int64_t row = w * RPW + lane / LPR;
    const int c = (lane % LPR) * V;
    uint32_t m = 0;
    if (row < total_rows && c < cols) {
        int64_t b = 0, r = row;
        if (rows < total_rows) { b = total_rows <= 0xFFFFFFFFll ? (int64_t)((uint32_t)row / (uint32_t)rows) : row / rows; r = row - b * rows; }
        const T* p = x + b * batch_stride + r * row_stride;
        if (cols >= V) {
            VecMax<T> mm;
            mm.fold(*reinterpret_cast<const u32x4_any*>(p + min((int64_t)c, cols - V)));
            m = mm.finish();
        } else {
            for (int e = 0; e < (int)cols; ++e) m = max(m, mag_bits<T>(p[e]));
        }
    }
#pragma unroll
    for (int off = LPR / 2; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, kWave));
    if (c == 0 && row < total_rows) { if (delta) delta[row] = delta_from_absmax_bits(m, qmax); else partial[row] = m; }
}

// Column groups: workgroup = CV column vectors (16: 128 bfloat16 or 64 binary32 columns, 256 contiguous bytes of every row; 8
// and 4 for tensors that narrow; 32 for wide ones, whose rows may start off the cache lines) x 256 / CV row lanes over a slab of rows.  partial[(b*nslab + slab)*cols + c].  Any extent,
// stride and alignment: a vector that straddles the last column is read element by element.  Four rows of a lane are on their
// way together; past the slab's end the last row is read again, which the maximum does not mind.
template <typename T, int CV> __global__ void __launch_bounds__(kThreads)
absmax_cols(const T* __restrict__ x, int64_t batch_stride, int64_t row_stride, int64_t rows, int64_t cols, int64_t slab_rows,
            uint32_t* __restrict__ partial)
{
    constexpr int V = VecMax<T>::V, RL = kThreads / CV;
    __shared__ uint32_t s[kThreads / kWave][CV][4];
    const int cv = threadIdx.x % CV, rl = threadIdx.x / CV, lane = threadIdx.x & (kWave - 1);
    const int64_t c0 = ((int64_t)blockIdx.x * CV + cv) * V;
    const int64_t r0 = (int64_t)blockIdx.y * slab_rows;
    const int64_t r1 = min(rows, r0 + slab_rows);
    VecMax<T> m;
    const T* base = x + (int64_t)blockIdx.z * batch_stride + c0;
    if (c0 + V <= cols) {
        auto row = [&](int64_t r) { return *reinterpret_cast<const u32x4_any*>(base + r * row_stride); };
        int64_t r = r0 + rl;
        for (; r + 3 * RL < r1; r += 4 * RL) {
            const u32x4 a = row(r), b = row(r + RL), c = row(r + 2 * RL), d = row(r + 3 * RL);
            m.fold(a); m.fold(b); m.fold(c); m.fold(d);
        }
        if (r < r1) {
            const int64_t end = r1 - 1;
            const u32x4 a = row(r), b = row(min(r + RL, end)), c = row(min(r + 2 * RL, end)), d = row(min(r + 3 * RL, end));
            m.fold(a); m.fold(b); m.fold(c); m.fold(d);
        }
    } else if (c0 < cols) {
        const int left = (int)(cols - c0);
        for (int64_t r = r0 + rl; r < r1; r += RL) {
            u32x4 w = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int e = 0; e < V; ++e)
                if (e < left) {
                    if constexpr (sizeof(T) == 2) w[e >> 1] |= (uint32_t)base[r * row_stride + e] << (16 * (e & 1));
                    else w[e] = __float_as_uint(base[r * row_stride + e]);
                }
            m.fold(w);
        }
    }
    // the row lanes of a wavefront, then its four wavefronts
    uint32_t w[4];
#pragma unroll
    for (int off = CV; off < kWave; off <<= 1) {
        m.words(w);
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = (uint32_t)__shfl_xor((int)w[i], off, kWave);
        m.fold_words(w);
    }
    m.words(w);
    if (lane < CV) {
#pragma unroll
        for (int i = 0; i < 4; ++i) s[threadIdx.x / kWave][cv][i] = w[i];
    }
    __syncthreads();
    if (threadIdx.x < CV && c0 < cols) {
        for (int k = 1; k < kThreads / kWave; ++k) {
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = s[k][cv][i];
            m.fold_words(w);
        }
        uint32_t* out = partial + ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * cols + c0;
#pragma unroll
        for (int e = 0; e < V; ++e)
            if (c0 + e < cols) out[e] = m.at(e);
    }
}

// Fold partial[b][P][C] over the matrices b of group g, (b / inner) % G == g, and over p; then delta = absmax / qmax.
// The matrices of a group: b = q * inner + i for q = g, g + G, ... and i = 0 .. inner - 1.
// C == 1: one workgroup per group.  C > 1: one thread per (g, c).
__global__ void __launch_bounds__(kThreads)
finalize_single(const uint32_t* __restrict__ partial, int64_t batch, int64_t P, int64_t G, int64_t inner, float qmax,
                float* __restrict__ delta)
{
    const int64_t g = blockIdx.x;
    uint32_t m = 0;
    if (inner == 1 && batch <= G && P <= 4 * kThreads) {
        // one matrix per group and few partials: request them all before folding
        uint32_t v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t p = threadIdx.x + k * kThreads;
            v[k] = (g < batch && p < P) ? partial[g * P + p] : 0u;
        }
        m = max(max(v[0], v[1]), max(v[2], v[3]));
    } else {
        // the (matrix, partial) pairs of the group, spread over the threads: the k-th matrix of group g is
        // b = ((k / inner) * G + g) * inner + k % inner, increasing with k
        for (int64_t it = threadIdx.x;; it += kThreads) {
            const int64_t k = it / P, p = it - k * P;
            const int64_t b = ((k / inner) * G + g) * inner + k % inner;
            if (b >= batch) break;
            m = max(m, partial[b * P + p]);
        }
    }
    m = block_max_u32(m);
    if (threadIdx.x == 0) delta[g] = delta_from_absmax_bits(m, qmax);
}
// Workgroup = CL channels x 256 / CL lanes over the (matrix, partial) pairs of the group; max is order-free.
template <int CL> __global__ void __launch_bounds__(kThreads)
finalize_channels(const uint32_t* __restrict__ partial, int64_t batch, int64_t P, int64_t C, int64_t G, int64_t inner,
                  float qmax, float* __restrict__ delta)
{
    constexpr int L = kThreads / CL;
    __shared__ uint32_t s[L][CL];
    const int cl = threadIdx.x % CL, pl = threadIdx.x / CL;
    const int64_t c = (int64_t)blockIdx.x * CL + cl;
    const int64_t g = blockIdx.y;
    uint32_t m = 0;
    if (c < C) {
        // the (matrix, partial) pairs of the group over the lanes of a channel (k-th matrix of group g:
        // b = ((k / inner) * G + g) * inner + k % inner, increasing with k), four loads in flight
        auto item = [&](int64_t it) -> uint32_t {
            const int64_t k = it / P, p = it - k * P;
            const int64_t b = ((k / inner) * G + g) * inner + k % inner;
            return b < batch ? partial[(b * P + p) * C + c] : 0u;
        };
        const int64_t groups_of_inner = (batch + inner - 1) / inner;                     // q = 0 .. groups_of_inner - 1
        const int64_t nq = groups_of_inner > g ? (groups_of_inner - g + G - 1) / G : 0;  // those with q % G == g
        const int64_t nitems = nq * inner * P;                                           // (items past the batch read as 0)
        int64_t it = pl;
        for (; it + 3 * L < nitems; it += 4 * L) {
            const uint32_t v0 = item(it), v1 = item(it + L), v2 = item(it + 2 * L), v3 = item(it + 3 * L);
            m = max(m, max(max(v0, v1), max(v2, v3)));
        }
        for (; it < nitems; it += L) m = max(m, item(it));
    }
    s[pl][cl] = m;
    __syncthreads();
    if (pl == 0 && c < C) {
#pragma unroll
        for (int k = 1; k < L; ++k) m = max(m, s[k][cl]);
        delta[g * C + c] = delta_from_absmax_bits(m, qmax);
    }
}

struct Plan {
    enum Kind { FLAT, ROWS, COLS } kind;
    int64_t P;        // partials per matrix (per channel for the column kind)
    int64_t C;        // channels
    int flat_blocks;
    int64_t slab_rows;
    int cv;           // column vectors per workgroup of the column kind
};

bool valid_tensor(const qmm_tensor* x, qmm_status* st)
{
    if (!x) { *st = QMM_ERR_NULL; return false; }
    if (x->dtype != QMM_DT_BF16 && x->dtype != QMM_DT_F32) { *st = QMM_ERR_ENUM; return false; }
    if (x->contract_axis != 0 && x->contract_axis != 1) { *st = QMM_ERR_ENUM; return false; }
    if (x->batch < 0 || x->rows < 0 || x->cols < 0) { *st = QMM_ERR_SHAPE; return false; }
    if (x->row_stride < x->cols) { *st = QMM_ERR_SHAPE; return false; }
    if (x->batch > 1 && x->rows > 0 && x->batch_stride < (x->rows - 1) * x->row_stride + x->cols) {
        *st = QMM_ERR_SHAPE; return false;
    }
    return true;
}

// A batch whose matrices lie back to back and share one step size is one matrix.
qmm_tensor one_matrix(const qmm_tensor* x, const qmm_granularity* g)
{
    qmm_tensor t = *x;
    if (!g->per_channel && g->batch_groups == 1 && t.batch > 1 && t.row_stride == t.cols && t.batch_stride == t.rows * t.cols) {
        t.rows *= t.batch;
        t.batch = 1;
    }
    return t;
}

// fold: the quantize pass folds the partial maxima.
Plan make_plan(const qmm_tensor* x, const qmm_granularity* g, bool fold = false)
{
    Plan p{};
    const bool bf16 = x->dtype == QMM_DT_BF16;
    const int64_t es = bf16 ? 2 : 4;
    const bool base_ok = aligned16(x->data) && (x->batch <= 1 || x->batch_stride * es % 16 == 0);
    if (!g->per_channel) {
        p.C = 1;
        const int64_t n = x->rows * x->cols;
        if (base_ok && (x->row_stride == x->cols || x->rows == 1) && n > 0) {
            p.kind = Plan::FLAT;
            const int64_t trips = (n * es + kThreads * 64 - 1) / (kThreads * 64);       // pieces of 16 KB
            const int64_t cap = x->batch > 1 ? (kMaxFlatBlocks + x->batch - 1) / x->batch : kMaxFlatBlocks;
            p.flat_blocks = (int)std::min(trips, cap);
            p.P = p.flat_blocks;
        } else {
            p.kind = Plan::ROWS;
            p.P = x->rows;
        }
    } else if (x->contract_axis == 1) {
        p.kind = Plan::ROWS;
        p.P = 1;
        p.C = x->rows;
    } else {
        p.kind = Plan::COLS;
        // Slabs of whole trips.  Where the quantize pass folds, as many as it takes; else enough for two workgroups per CU, but
        // not more than the second kernel folds in a few trips.  (Slabs of 128 rows / at most 32 slabs, for every call / this way:
        // bfloat16 1048576 x 64 372 / 181 / 29 us, 300000 x 20 116 / 306 / 14.6, 65536 x 128 26.6 / 11.5 / 10.6, 16384 x 1024 11.8 /
        // 8.4 / 7.4, where four workgroups per CU took 9.4; 5000 x 8200 19.8 / 22.1 / 19.2.)
        const int64_t nvec = (x->cols + (bf16 ? 7 : 3)) / (bf16 ? 8 : 4);
        p.cv = nvec <= 4 ? 4 : nvec <= 8 ? 8 : nvec < 512 || x->rows < 1024 ? 16 : 32;
        const int64_t trip = 4 * (kThreads / p.cv), blocks = ((nvec + p.cv - 1) / p.cv) * std::max<int64_t>(x->batch, 1);
        const int64_t want = fold ? kFoldSlabs : std::min<int64_t>(std::max<int64_t>((512 + blocks - 1) / blocks, 1), kMaxColSlabs);
        p.slab_rows = std::max<int64_t>(kColSlabRows, ((x->rows + want - 1) / want + trip - 1) / trip * trip);
        p.P = (x->rows + p.slab_rows - 1) / p.slab_rows;
        p.C = x->cols;
    }
    return p;
}

}  // namespace
}  // namespace qmm

using namespace qmm;

extern "C" int64_t qmm_num_scales(const qmm_tensor* x, const qmm_granularity* g)
{
    if (!x || !g) return 0;
    const int64_t c = g->per_channel ? (x->contract_axis == 1 ? x->rows : x->cols) : 1;
    return g->batch_groups * c;
}

namespace qmm {
size_t scale_partials_size(const qmm_tensor* x, const qmm_granularity* g, bool fold)
{
    qmm_status st;
    if (!g || !valid_tensor(x, &st)) return 0;
    const qmm_tensor t = one_matrix(x, g);
    const Plan p = make_plan(&t, g, fold);
    const int64_t words = t.batch * p.P * p.C;
    return (size_t)(words > 0 ? words : 1) * sizeof(uint32_t);
}
}  // namespace qmm

extern "C" size_t qmm_scale_workspace_size(const qmm_tensor* x, const qmm_granularity* g) { return scale_partials_size(x, g, false); }

namespace {
// Everything qmm_scale can refuse, checked without launching.
qmm_status scale_check(const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g, const float* delta_out,
                       const void* workspace, size_t workspace_bytes, bool fold = false)
{
    qmm_status st;
    if (!g || !delta_out) return QMM_ERR_NULL;
    if (!valid_tensor(x, &st)) return st;
    if (fmt != QMM_FMT_INT8 && fmt != QMM_FMT_E4M3 && fmt != QMM_FMT_E5M2) return QMM_ERR_ENUM;
    if (g->batch_groups < 1 || g->batch_inner < 0 || (g->per_channel != 0 && g->per_channel != 1)) return QMM_ERR_ENUM;
    if (x->batch > 65535) return QMM_ERR_UNSUPPORTED;          // the batch index is a grid dimension in some plans
    if (qmm_num_scales(x, g) == 0) return QMM_OK;
    if (x->batch * x->rows * x->cols > 0 && !x->data) return QMM_ERR_NULL;
    if (!workspace || workspace_bytes < scale_partials_size(x, g, fold)) return QMM_ERR_WORKSPACE;
    if (!aligned16(workspace)) return QMM_ERR_ALIGN;
    return QMM_OK;
}
}  // namespace

namespace qmm {
// The first half of qmm_scale on checked arguments: partial maxima to `partial`, laid out [batch][P][C] (`out` says how).
// out->done: the step sizes have been written as well.  `fold_here`: the caller folds the partial maxima itself, so a
// large tensor's last workgroup need not.
qmm_status scale_partials(const qmm_tensor* x0, qmm_format fmt, const qmm_granularity* g, float* delta_out, uint32_t* partial,
                          bool fold_here, ScalePartials* out, hipStream_t s, uint32_t patience)
{
    const qmm_tensor t = one_matrix(x0, g);
    const qmm_tensor* x = &t;
    const Plan p = make_plan(x, g, fold_here);
    const float qmax = host_qmax(fmt);
    const bool bf16 = x->dtype == QMM_DT_BF16;
    const int64_t nelem = x->batch * x->rows * x->cols;
    out->batch = nelem > 0 ? x->batch : 0;        // an empty tensor: fold over no matrices, every group gets delta = 1
    out->P = p.P; out->C = p.C;
    out->done = false;
    if (nelem == 0) return QMM_OK;
    switch (p.kind) {
    case Plan::FLAT: {
        // One launch: by way of a board, where every group has a matrix.  Calls being recorded: with one scale group and a large tensor
        // the workgroup that arrives last folds (publishing, counting and the coherent reads of the fold are a chain of
        // device-wide round trips, about 11 us for a tensor of any size up to 32 MB against 9-10 us for two small launches;
        // from 32 MB on the single launch wins, 25 us against 27 us at 134 MB), else a second kernel.
        uint32_t* slot = nullptr;
        Board bd{};
        const int64_t inner = std::max<int64_t>(g->batch_inner, 1), words = p.flat_blocks * x->batch;
        const bool every_group = g->batch_groups <= x->batch && (g->batch_groups - 1) * inner < x->batch;
        if (fold_here || !every_group || words > kBoardMax || !take_board(s, RING_LONG, (uint32_t)words, &bd)) {
            bd.words = nullptr;
            if (!fold_here && g->batch_groups == 1 && nelem >= (int64_t(1) << 24) && arrival_slots(1, &slot) != QMM_OK) slot = nullptr;
        }
        bd.patience = std::min(kFolderPatience, patience);
        const uint32_t groups = every_group ? (uint32_t)g->batch_groups : 1u, run = (uint32_t)std::min(inner, x->batch);
        const dim3 grid(p.flat_blocks, (unsigned)x->batch);
        const int64_t n = x->rows * x->cols;
        if (bf16) absmax_flat<uint16_t><<<grid, kThreads, 0, s>>>(static_cast<const uint16_t*>(x->data), x->batch_stride, n, partial, slot, bd, groups, run, qmax, delta_out);
        else absmax_flat<float><<<grid, kThreads, 0, s>>>(static_cast<const float*>(x->data), x->batch_stride, n, partial, slot, bd, groups, run, qmax, delta_out);
        out->done = slot != nullptr || bd.words != nullptr;
        break;
    }
    case Plan::ROWS: {
        // one step size per row with every matrix a batch group of its own: a row's maximum is its group's maximum
        const bool rows_are_groups = g->per_channel && x->batch == g->batch_groups && g->batch_inner <= 1;
        const int64_t total = x->batch * x->rows;
        float* direct = rows_are_groups ? delta_out : nullptr;
        const unsigned nb = (unsigned)((total + kThreads / kWave - 1) / (kThreads / kWave));
        // matrices that follow one another like their rows are one matrix to a kernel that writes a value per row
        const int64_t rows = x->batch_stride == x->rows * x->row_stride ? total : x->rows;
        const int64_t nvec = (x->cols + (bf16 ? 7 : 3)) / (bf16 ? 8 : 4);
        if (nvec <= 32) {
            auto run = [&](auto lanes) {
                constexpr int L = decltype(lanes)::value;
                const int64_t waves = (total + kWave / L - 1) / (kWave / L);
                const unsigned nbs = (unsigned)((waves + kThreads / kWave - 1) / (kThreads / kWave));
                if (bf16) absmax_rows_short<uint16_t, L><<<nbs, kThreads, 0, s>>>(static_cast<const uint16_t*>(x->data), x->batch_stride, x->row_stride,
                                                                               rows, x->cols, total, partial, qmax, direct);
                else absmax_rows_short<float, L><<<nbs, kThreads, 0, s>>>(static_cast<const float*>(x->data), x->batch_stride, x->row_stride,
                                                                          rows, x->cols, total, partial, qmax, direct);
            };
            if (nvec <= 1) run(std::integral_constant<int, 1>{}); else if (nvec <= 2) run(std::integral_constant<int, 2>{});
            else if (nvec <= 4) run(std::integral_constant<int, 4>{}); else if (nvec <= 8) run(std::integral_constant<int, 8>{});
            else if (nvec <= 16) run(std::integral_constant<int, 16>{}); else run(std::integral_constant<int, 32>{});
        } else if (bf16)
            absmax_rows<uint16_t><<<nb, kThreads, 0, s>>>(static_cast<const uint16_t*>(x->data), x->batch_stride,
                                                           x->row_stride, rows, x->cols, total, partial, qmax, direct);
        else
            absmax_rows<float><<<nb, kThreads, 0, s>>>(static_cast<const float*>(x->data), x->batch_stride,
                                                        x->row_stride, rows, x->cols, total, partial, qmax, direct);
        out->done = rows_are_groups;
        break;
    }
    case Plan::COLS: {
        const int64_t cols_per_block = p.cv * (bf16 ? 8 : 4);
        const dim3 grid((unsigned)((x->cols + cols_per_block - 1) / cols_per_block), (unsigned)p.P, (unsigned)x->batch);
        auto run = [&](auto vectors) {
            constexpr int CV = decltype(vectors)::value;
            if (bf16)
                absmax_cols<uint16_t, CV><<<grid, kThreads, 0, s>>>(static_cast<const uint16_t*>(x->data), x->batch_stride,
                                                                    x->row_stride, x->rows, x->cols, p.slab_rows, partial);
            else
                absmax_cols<float, CV><<<grid, kThreads, 0, s>>>(static_cast<const float*>(x->data), x->batch_stride,
                                                                 x->row_stride, x->rows, x->cols, p.slab_rows, partial);
        };
        if (p.cv == 4) run(std::integral_constant<int, 4>{});
        else if (p.cv == 8) run(std::integral_constant<int, 8>{});
        else if (p.cv == 16) run(std::integral_constant<int, 16>{});
        else run(std::integral_constant<int, 32>{});
        break;
    }
    }
    return launch_status();
}

// The second half: partial maxima -> step sizes.  (An empty tensor has no partial maxima: batch = 0, and P = 1 so that the
// folds' divisions by P are defined; they end before they read, and every group's step size becomes 1.)
qmm_status scale_fold(const ScalePartials& pp, const uint32_t* partial, qmm_format fmt, const qmm_granularity* g,
                      float* delta_out, hipStream_t s)
{
    const int64_t G = g->batch_groups, inner = g->batch_inner > 0 ? g->batch_inner : 1, P = pp.batch > 0 ? pp.P : 1;
    if (pp.C == 1)
        finalize_single<<<(unsigned)G, kThreads, 0, s>>>(partial, pp.batch, P, G, inner, host_qmax(fmt), delta_out);
    else
    {
        // many lanes a channel where the channels alone are few workgroups (tall tensors, hundreds of partial maxima each)
        if ((pp.C + 31) / 32 * G < 128)
            finalize_channels<8><<<dim3((unsigned)((pp.C + 7) / 8), (unsigned)G), kThreads, 0, s>>>(
                partial, pp.batch, P, pp.C, G, inner, host_qmax(fmt), delta_out);
        else
            finalize_channels<32><<<dim3((unsigned)((pp.C + 31) / 32), (unsigned)G), kThreads, 0, s>>>(
                partial, pp.batch, P, pp.C, G, inner, host_qmax(fmt), delta_out);
    }
    return launch_status();
}

qmm_status scale_arguments(const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g, const float* delta_out,
                           const void* workspace, size_t workspace_bytes, bool fold)
{
    return scale_check(x, fmt, g, delta_out, workspace, workspace_bytes, fold);
}
}  // namespace qmm

namespace {
qmm_status scale_call(const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g, float* delta_out, void* workspace, size_t workspace_bytes,
                      uint32_t patience, void* stream)
{
    const qmm_status chk = scale_check(x, fmt, g, delta_out, workspace, workspace_bytes);
    if (chk != QMM_OK) return chk;
    if (qmm_num_scales(x, g) == 0) return QMM_OK;
    hipStream_t s = as_stream(stream);
    uint32_t* partial = static_cast<uint32_t*>(workspace);
    ScalePartials pp;
    const qmm_status st = scale_partials(x, fmt, g, delta_out, partial, false, &pp, s, patience);
    return st != QMM_OK || pp.done ? st : scale_fold(pp, partial, fmt, g, delta_out, s);
}
}  // namespace

extern "C" qmm_status qmm_scale(const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g, float* delta_out,
                                void* workspace, size_t workspace_bytes, void* stream)
{
    return scale_call(x, fmt, g, delta_out, workspace, workspace_bytes, kFolderPatience, stream);
}

// ---- qmm_scale_static: the same kernels with their partial maxima in a scratch array of the device image.
// `scratch` below is the host-side stand-in of the device array; its device address differs per GPU and is looked
// up once per device (kept in scratch_addr), and only that address is ever handed to a kernel.
static __device__ __align__(256) unsigned char scratch[QMM_SCALE_STATIC_BYTES];
namespace {
constexpr int kMaxDevices = 64;
std::atomic<void*> scratch_addr[kMaxDevices];

qmm_status static_scratch(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return QMM_ERR_LAUNCH;
    if (dev < 0 || dev >= kMaxDevices) return QMM_ERR_UNSUPPORTED;
    void* p = scratch_addr[dev].load(std::memory_order_acquire);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return QMM_ERR_LAUNCH;
        scratch_addr[dev].store(p, std::memory_order_release);      // two first callers store the same address
    }
    *out = p;
    return QMM_OK;
}
}  // namespace

extern "C" qmm_status qmm_scale_static(const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g, float* delta_out,
                                       void* stream)
{
    // argument errors first, exactly as qmm_scale reports them (the workspace checks cannot fail with a dummy of full size)
    const qmm_status chk = scale_check(x, fmt, g, delta_out, reinterpret_cast<const void*>(uintptr_t(256)), ~size_t(0));
    if (chk != QMM_OK) return chk;
    if (qmm_scale_workspace_size(x, g) > QMM_SCALE_STATIC_BYTES) return QMM_ERR_LIMIT;
    void* ws = nullptr;
    const qmm_status st = static_scratch(&ws);
    if (st != QMM_OK) return st;
    return qmm_scale(x, fmt, g, delta_out, ws, QMM_SCALE_STATIC_BYTES, stream);
}

namespace {
size_t multi_slice(const qmm_tensor* x, const qmm_granularity* g)
{
    return (qmm_scale_workspace_size(x, g) + 15u) & ~(size_t)15u;
}
// the tensors absmax_flat_multi takes: one matrix, dense, bfloat16 in whole 16-byte vectors, one step size
bool multi_flat_ok(const qmm_tensor* x, const qmm_granularity* g)
{
    qmm_status st;
    if (!valid_tensor(x, &st) || !x->data) return false;
    return x->dtype == QMM_DT_BF16 && x->batch == 1 && !g->per_channel && g->batch_groups == 1 && g->batch_inner >= 0 &&
           x->row_stride == x->cols && x->rows * x->cols >= 8 && (x->cols % 8 == 0) && aligned16(x->data) &&
           make_plan(x, g).kind == Plan::FLAT;
}
}  // namespace

extern "C" size_t qmm_scale_multi_workspace_size(int32_t count, const qmm_tensor* x, const qmm_granularity* g)
{
    if (count <= 0 || !x || !g) return 0;
    size_t total = 0;
    for (int32_t t = 0; t < count; ++t) total += multi_slice(x + t, g + t);
    return total;
}

namespace {
qmm_status scale_multi_call(int32_t count, const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g, float* const* delta_out,
                            void* workspace, size_t workspace_bytes, uint32_t patience, void* stream)
{
    if (count < 0) return QMM_ERR_SHAPE;
    if (count == 0) return QMM_OK;
    if (!x || !g || !delta_out) return QMM_ERR_NULL;
    if (fmt != QMM_FMT_INT8 && fmt != QMM_FMT_E4M3 && fmt != QMM_FMT_E5M2) return QMM_ERR_ENUM;
    if (!workspace || workspace_bytes < qmm_scale_multi_workspace_size(count, x, g)) return QMM_ERR_WORKSPACE;
    if (!aligned16(workspace)) return QMM_ERR_ALIGN;
    bool one_launch = count <= kMaxMulti;
    for (int32_t t = 0; t < count && one_launch; ++t) one_launch = delta_out[t] && multi_flat_ok(x + t, g + t);
    uint8_t* ws = static_cast<uint8_t*>(workspace);
    if (!one_launch) {
        uint8_t* probe = ws;
        for (int32_t t = 0; t < count; ++t) {      // every tensor's arguments before the first launch
            const size_t slice = multi_slice(x + t, g + t);
            const qmm_status st = scale_check(x + t, fmt, g + t, delta_out[t], probe, slice);
            if (st != QMM_OK) return st;
            probe += slice;
        }
        for (int32_t t = 0; t < count; ++t) {
            const size_t slice = multi_slice(x + t, g + t);
            const qmm_status st = scale_call(x + t, fmt, g + t, delta_out[t], ws, slice, patience, stream);
            if (st != QMM_OK) return st;
            ws += slice;
        }
        return QMM_OK;
    }
    MultiFlat a{};
    int max_blk = 1;
    for (int32_t t = 0; t < count; ++t) {
        const Plan p = make_plan(x + t, g + t);          // FLAT for these tensors: the same workgroup count as qmm_scale
        a.x[t] = static_cast<const uint16_t*>(x[t].data);
        a.nvec[t] = x[t].rows * x[t].cols / 8;
        a.partial[t] = reinterpret_cast<uint32_t*>(ws);
        a.delta[t] = delta_out[t];
        a.nblk[t] = p.flat_blocks;
        max_blk = std::max(max_blk, p.flat_blocks);
        ws += multi_slice(x + t, g + t);
    }
    a.qmax = host_qmax(fmt);
    hipStream_t s = as_stream(stream);
    if (!take_board(s, RING_LONG, (uint32_t)count * kMaxFlatBlocks, &a.board)) {
        a.board.words = nullptr;
        const qmm_status sl = arrival_slots(count, &a.slots);
        if (sl != QMM_OK) return sl;
    }
    a.board.patience = std::min(kFolderPatience, patience);
    absmax_flat_multi<<<dim3((unsigned)max_blk, (unsigned)count), kThreads, 0, s>>>(a);
    return launch_status();
}
}  // namespace

extern "C" qmm_status qmm_scale_multi(int32_t count, const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g,
                                      float* const* delta_out, void* workspace, size_t workspace_bytes, void* stream)
{
    return scale_multi_call(count, x, fmt, g, delta_out, workspace, workspace_bytes, kFolderPatience, stream);
}

// For the tests, not part of the ABI: the folding workgroups wait `patience` ticks for the others (0: they form what is not there yet).
extern "C" qmm_status qmm_internal_scale_multi(int32_t count, const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g,
                                               float* const* delta_out, void* workspace, size_t workspace_bytes, uint32_t patience, void* stream)
{
    return scale_multi_call(count, x, fmt, g, delta_out, workspace, workspace_bytes, patience, stream);
}
