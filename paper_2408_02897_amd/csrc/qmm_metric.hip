// qmm_metric: one pass over (y, y_ref[, denom]) accumulating in binary64 the
// sums behind the noise-to-signal ratio, the relative error of Eq. 2 and the
// element-wise backward error of Eq. 3.  HBM-bound: 8 B per element for a
// binary32 y (6 B for bfloat16 y, +4 B with denominators).  Every thread keeps
// private sums, wavefronts fold them by rotations and swaps of lanes, workgroups through LDS, and the
// first sixteen workgroups, one per field, fold the per-workgroup partials when all are there (large tensors and
// calls being recorded: a small second kernel does), in a fixed order: no atomics, the result is reproducible run to run.
#include <algorithm>
#include <type_traits>
#include "qmm_device.h"

namespace qmm {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxBlocks = 1024;   // 4 workgroups per CU (what up to 128 registers keep resident); also 4 partials per thread in the final fold
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Quotients n / d in binary64 for finite n >= 0 and finite d > 0 where d was converted from binary32 (24 significant
// bits) and n is such a value or the difference of two (exponents within +-150 or so).
//
// reciprocals4: the four reciprocals from ONE hardware estimate: p = d0 d1 d2 d3 (within 2^-596 .. 2^512), one Newton
// step on rcp(p) -- whose error of at most 2^29 ulp, 2^-23, it squares --, then multiplied back by the other factors, a few
// roundings of 2^-53 each.  Each x[i] is 1 / d[i] to 2^-45.
// quotient_with: q0 = n x, r = n - d q0 (exact in one fused multiply-add: d q0 has 77 bits of which the top 44 or more
// cancel), q = fl(q0 + r x).  q0 + r x differs from n / d by |r / d| * |x d - 1| <= 2^-90 relative, and a quotient with a 24-bit
// divisor is either representable or at least 2^-78 relative away from the nearest rounding boundary (n - m d is a
// multiple of 2^(e_m + e_d - 76) for a 54-bit midpoint m), so the single rounding of the last operation lands on the
// IEEE quotient: same bits as `/`, for 6.75 instructions per quotient (a quarter of one at quarter rate) instead of 11 with the
// compiler's sequence.  (The divisions are the pass's largest single cost.)
// A zero, infinite or NaN operand anywhere in the four gives NaN or infinity in the affected quotients, never a wrong
// finite value passed as right for them: the caller tests the quotients and takes the general path then.
QMM_DEV void reciprocals4(const double* d, double* x)
{
    const double p01 = d[0] * d[1], p23 = d[2] * d[3];
    const double p = p01 * p23;
    const double x0 = __builtin_amdgcn_rcp(p);
    const double x1 = fma(x0, fma(-p, x0, 1.0), x0);
    const double x01 = x1 * p23, x23 = x1 * p01;
    x[0] = x01 * d[1]; x[1] = x01 * d[0]; x[2] = x23 * d[3]; x[3] = x23 * d[2];
}
// m = max(m, |v|) for values that are not NaN, as the one instruction.  (fmax() first quiets each operand that the
// compiler cannot prove canonical -- a converted, negated or loaded value -- with an instruction of its own, which
// doubled the cost of the running maxima.)
QMM_DEV void max_abs_plain(double& m, double v)
{
    asm("v_max_f64 %0, %0, |%1|" : "+v"(m) : "v"(v));
}
QMM_DEV double quotient_with(double n, double d, double x)
{
    const double q0 = n * x;
    return fma(fma(-d, q0, n), x, q0);
}

// Running sums of one thread.  Branch-free: an element whose error is NaN contributes zeros and bumps nan_cnt.
struct Acc {
    double s_ee = 0, s_rr = 0, s_ae = 0, s_ar = 0, m_e = 0, m_r = 0;
    double re_sum = 0, re_max = 0, be_sum = 0, be_max = 0;
    unsigned re_cnt = 0, be_cnt = 0, n = 0, nan_cnt = 0;     // a thread sees far fewer than 2^32 elements

    // The common case, taken when the whole wavefront's elements are ordinary (no NaN or infinite error, r != 0 and
    // d > 0 everywhere): |e|, |r| and the quotients come in computed.  Same sums as add(), without its selects.
    // re_sum and be_sum are taken by the caller (it adds the quotients itself, to test them), and so is the maximum of |r|.
    // e and r come in signed.
    template <bool HAS_D> QMM_DEV void add_plain(double e, double r, double q, double qb)
    {
        s_ee = fma(e, e, s_ee);
        s_rr = fma(r, r, s_rr);
        s_ae += fabs(e);
        s_ar += fabs(r);
        max_abs_plain(m_e, e);
        max_abs_plain(re_max, q);
        if constexpr (HAS_D) max_abs_plain(be_max, qb);
    }
    // counts of a run of `k` plain elements
    template <bool HAS_D> QMM_DEV void count_plain(unsigned k)
    {
        re_cnt += k; n += k;
        if constexpr (HAS_D) be_cnt += k;
    }
    template <bool HAS_D> QMM_DEV void add(float yf, float rf, float df)
    {
        const double e = (double)yf - (double)rf;
        const bool ok = (e == e);
        const double ae = ok ? fabs(e) : 0.0;
        const double ar = ok ? fabs((double)rf) : 0.0;
        s_ee = fma(ae, ae, s_ee);
        s_rr = fma(ar, ar, s_rr);
        s_ae += ae;
        s_ar += ar;
        m_e = fmax(m_e, ae);
        m_r = fmax(m_r, ar);
        const bool rnz = ar != 0.0;
        const double q = rnz ? ae / ar : 0.0;                 // Eq. 2 with |v| in the denominator
        re_sum += q;
        re_max = fmax(re_max, q);
        re_cnt += rnz ? 1u : 0u;
        if constexpr (HAS_D) {
            const double d = (double)df;
            const bool dpos = ok && d > 0.0;
            const double qb = dpos ? ae / d : 0.0;            // Eq. 3, element-wise
            be_sum += qb;
            be_max = fmax(be_max, qb);
            be_cnt += dpos ? 1u : 0u;
        }
        n += ok ? 1u : 0u;
        nan_cnt += ok ? 0u : 1u;
    }
};

// Workgroup partials are stored field-major: partial[field * nblocks + block].  ONE: for another workgroup of this launch.
template <bool ONE> QMM_DEV void store_partial(const Acc& a, double* partial, int nblocks, int block)
{
    __shared__ double s[kThreads / kWave][16];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    double v[16];
    v[0] = wave_sum_f64(a.s_ee); v[1] = wave_sum_f64(a.s_rr); v[2] = wave_sum_f64(a.s_ae); v[3] = wave_sum_f64(a.s_ar);
    v[4] = wave_max_f64(a.m_e); v[5] = wave_max_f64(a.m_r);
    v[6] = wave_sum_f64(a.re_sum); v[7] = wave_max_f64(a.re_max); v[8] = wave_sum_f64((double)a.re_cnt);
    v[9] = wave_sum_f64(a.be_sum); v[10] = wave_max_f64(a.be_max); v[11] = wave_sum_f64((double)a.be_cnt);
    v[12] = wave_sum_f64((double)a.n); v[13] = wave_sum_f64((double)a.nan_cnt);
    v[14] = 0.0; v[15] = 0.0;
    if (lane == 0) {
#pragma unroll
        for (int i = 0; i < 16; ++i) s[w][i] = v[i];
    }
    __syncthreads();
    if (threadIdx.x < 16) {
        const int i = threadIdx.x;
        const bool is_max = (i == 4 || i == 5 || i == 7 || i == 10);
        double r = s[0][i];
        for (int k = 1; k < kThreads / kWave; ++k) r = is_max ? fmax(r, s[k][i]) : r + s[k][i];
        double* at = partial + (int64_t)i * nblocks + block;
        if constexpr (ONE) publish_f64(at, r); else *at = r;
    }
}

template <bool Y_BF16> QMM_DEV f32x4 load_y4(const void* yv, int64_t i)
{
    if constexpr (Y_BF16) {
        const u32x2 w = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(yv) + i);
        return f32x4{__uint_as_float(w[0] << 16), __uint_as_float(w[0] & 0xFFFF0000u),
                     __uint_as_float(w[1] << 16), __uint_as_float(w[1] & 0xFFFF0000u)};
    } else {
        return __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(yv) + i);
    }
}

// The sums of block `block` of `nblocks`.
template <bool Y_BF16, bool HAS_D> QMM_DEV Acc block_sums(const void* __restrict__ yv, const float* __restrict__ r, const float* __restrict__ d, int64_t n,
                                                           int block, int nblocks)
{
    Acc acc;
    const int64_t nvec = n >> 2;
    const int64_t tid = (int64_t)block * kThreads + threadIdx.x;
    const f32x4* r4 = reinterpret_cast<const f32x4*>(r);
    const f32x4* d4 = reinterpret_cast<const f32x4*>(d);
    // A workgroup takes two consecutive pieces of 256 vectors per trip and the grid sweeps the arrays front to
    // back, so the loads in flight are neighbours in memory (loads a whole grid stride apart read large arrays
    // up to 25 % slower).  Both loads are in flight before the arithmetic of either starts.
    const int64_t stride = (int64_t)nblocks * kThreads * 2;
    int64_t i = (int64_t)block * kThreads * 2 + threadIdx.x;
    // (y and the reference are read once: streaming loads, which leave the caches to the tensors that are read again --
    // the benchmark's step is 3 % shorter for it, the pass itself 4 %)
    // The vector unit is busy for 80 % of the pass's cycles (at the 1.7 GHz the binary64 work leaves): small tensors are bound
    // by it and its latencies, tensors of tens of millions of elements by memory as well.  The loop is kept to what the sums
    // need: the rare path lies outside it -- inside, the running sums were copied around it on every trip, 11 moves for 8
    // elements --, the maximum of |r| is taken in binary32, which holds it exactly, and the reciprocals need one Newton step.
    // 24 instructions an element before, 20 now (launches back to back: 196608 bfloat16 6.9 -> 5.6 us, 3 million 10.9 -> 8.9, 67
    // million 75 -> 69, 5.8 TB/s; binary32 y 88 -> 86, 6.2 TB/s; with denominators 110 -> 104 and 125 -> 127).
    float mr = 0.0f;
    for (;;) {
        bool special = false;
        for (; i + kThreads < nvec; i += stride) {
            const f32x4 y0 = load_y4<Y_BF16>(yv, i), y1 = load_y4<Y_BF16>(yv, i + kThreads);
            const f32x4 r0 = __builtin_nontemporal_load(r4 + i), r1 = __builtin_nontemporal_load(r4 + i + kThreads);
            f32x4 d0 = {0.f, 0.f, 0.f, 0.f}, d1 = {0.f, 0.f, 0.f, 0.f};
            if constexpr (HAS_D) { d0 = d4[i]; d1 = d4[i + kThreads]; }
            // |e|, |r| and the quotients of all eight elements first, four divisions per reciprocal estimate.  An element
            // the plain sums would get wrong (NaN or infinite e, r == 0, d not in (0, inf)) shows as a quotient that is
            // +infinity or NaN, which makes the running sum of quotients (all >= 0, far from overflow) non-finite, or is
            // caught by the sign test on d: then the whole wavefront takes the general path and the sums are not kept.
            double ae[8], ar[8], dd[8], x[8], q[8], qb[8];
            double re_next = acc.re_sum, be_next = acc.be_sum;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float yf = j < 4 ? y0[j & 3] : y1[j & 3], rf = j < 4 ? r0[j & 3] : r1[j & 3];
                ae[j] = (double)yf - (double)rf;       // signed: the magnitudes are operand modifiers where they are used
                ar[j] = (double)rf;
            }
            reciprocals4(ar, x); reciprocals4(ar + 4, x + 4);      // signed reciprocals: the four signs cancel in pairs
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                q[j] = quotient_with(fabs(ae[j]), fabs(ar[j]), fabs(x[j]));
                re_next += q[j];
                qb[j] = 0.0;
            }
            bool sp = !(re_next < (double)__builtin_inff());
            if constexpr (HAS_D) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float df = j < 4 ? d0[j & 3] : d1[j & 3];
                    dd[j] = (double)df;
                    sp = sp || !(df > 0.0f);
                }
                reciprocals4(dd, x); reciprocals4(dd + 4, x + 4);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    qb[j] = quotient_with(fabs(ae[j]), dd[j], x[j]);
                    be_next += qb[j];
                }
                sp = sp || !(be_next < (double)__builtin_inff());
            }
            if (__any(sp)) { special = true; break; }
#pragma unroll
            for (int j = 0; j < 8; ++j) acc.add_plain<HAS_D>(ae[j], ar[j], q[j], qb[j]);
#pragma unroll
            for (int j = 0; j < 4; ++j) mr = fmaxf(fmaxf(mr, fabsf(r0[j])), fabsf(r1[j]));
            acc.re_sum = re_next;
            if constexpr (HAS_D) acc.be_sum = be_next;
            acc.count_plain<HAS_D>(8u);
        }
        if (!special) break;
        // the rare path, kept rolled: unrolled, its eight interleaved IEEE divisions set the kernel's register count
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
            const f32x4 yy = load_y4<Y_BF16>(yv, i + h * kThreads), rr = r4[i + h * kThreads];
            f32x4 dd = {0.f, 0.f, 0.f, 0.f};
            if constexpr (HAS_D) dd = d4[i + h * kThreads];
#pragma unroll 1
            for (int j = 0; j < 4; ++j) {
                const float yf = j == 0 ? yy[0] : j == 1 ? yy[1] : j == 2 ? yy[2] : yy[3];
                const float rf = j == 0 ? rr[0] : j == 1 ? rr[1] : j == 2 ? rr[2] : rr[3];
                const float df = j == 0 ? dd[0] : j == 1 ? dd[1] : j == 2 ? dd[2] : dd[3];
                acc.add<HAS_D>(yf, rf, df);
            }
        }
        i += stride;
    }
    acc.m_r = fmax(acc.m_r, (double)mr);
    if (i < nvec) {      // ragged end: the first piece of a workgroup's last trip
        const f32x4 y0 = load_y4<Y_BF16>(yv, i);
        const f32x4 r0 = r4[i];
        f32x4 d0 = {0.f, 0.f, 0.f, 0.f};
        if constexpr (HAS_D) d0 = d4[i];
#pragma unroll
        for (int j = 0; j < 4; ++j) acc.add<HAS_D>(y0[j], r0[j], d0[j]);
    }
    // tail elements (n % 4), one thread each
    const int64_t t = (nvec << 2) + tid;
    if (t < n) {
        float y;
        if constexpr (Y_BF16) y = bf16_bits_to_f32(static_cast<const uint16_t*>(yv)[t]);
        else y = static_cast<const float*>(yv)[t];
        acc.add<HAS_D>(y, r[t], HAS_D ? d[t] : 0.f);
    }
    return acc;
}

// The fold of a field's partials, in an order that depends on nblocks only: thread t takes blocks t, t + 256, ... in ascending order,
// the 64 lane values are folded by the fixed butterfly and the four wavefront values in wavefront order.  Thread 0's value.
template <bool COHERENT> QMM_DEV double fold_field(const double* partial, int nblocks, int field)
{
    __shared__ double s[kThreads / kWave];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const bool is_max = (field == 4 || field == 5 || field == 7 || field == 10);
    const double* p = partial + (int64_t)field * nblocks;
    // all of a thread's partials are requested before any is used
    double v[kMaxBlocks / kThreads];
#pragma unroll
    for (int k = 0; k < kMaxBlocks / kThreads; ++k) {
        const int b = threadIdx.x + k * kThreads;
        v[k] = 0.0;
        if (b < nblocks) v[k] = COHERENT ? coherent_load(p + b) : p[b];
    }
    double r = 0.0;
#pragma unroll
    for (int k = 0; k < kMaxBlocks / kThreads; ++k) r = is_max ? fmax(r, v[k]) : r + v[k];
    r = is_max ? wave_max_f64(r) : wave_sum_f64(r);
    if (lane == 0) s[w] = r;
    __syncthreads();
    double t = s[0];
    if (threadIdx.x == 0)
        for (int k = 1; k < kThreads / kWave; ++k) t = is_max ? fmax(t, s[k]) : t + s[k];
    __syncthreads();
    return t;
}

// ONE: the fold within the launch.  A workgroup stores its partials past the caches, waits until they have left and posts a word;
// the first sixteen wait for all words and fold a field each (of fewer workgroups, several).  None of the others waits, so the
// words come whatever else the GPU does; should one not (a board shared by calls in flight), the workgroup that misses it forms that
// block's sums itself.  What it saves is the host's second launch, 2.4 us: the paths of small products, whose time is the host's, take
// 23.2 us where they took 26.5 (256 x 768 x 768), 34.8 / 41.9 (512^3 with its references).  On the GPU the second launch is the shorter way:
// it is on its way while the pass still runs, and the exchange adds itself to the pass (calls back to back, bfloat16, two launches / one:
// 200000 elements 5.9 / 6.2 us, 4 million 10.4 / 10.7, 6 million 12.3 / 13.0, 8 million 14.4 / 15.3, 12.6 million 18.7 / 19.1, 67 million 70.4 / 70.9;
// binary32 6 million 13.7 / 14.1, 17 million 26.6 / 26.9).  So two beyond 2^22 elements, where a pass takes longer than the host for both.
// Not kept: four quotients of the sum over one denominator and the maxima looked for in upper words, 14 instructions an element
// instead of 20 (bfloat16 67 million 67.7 against 69.8, 16.8 million 24.3 against 22.9, binary32 67 million 85.4 against 83.4).
constexpr int kFields = 16;
template <bool Y_BF16, bool HAS_D, bool ONE> __global__ void __launch_bounds__(kThreads)
metric_partial(const void* __restrict__ yv, const float* __restrict__ r, const float* __restrict__ d, int64_t n,
               double* __restrict__ partial, double* __restrict__ out, Board bd)
{
    const int nblocks = (int)gridDim.x;
    if constexpr (!ONE) {
        store_partial<false>(block_sums<Y_BF16, HAS_D>(yv, r, d, n, (int)blockIdx.x, nblocks), partial, nblocks, (int)blockIdx.x);
    } else {
        __shared__ int s_missing;
        uint64_t start = 0;
        for (int block = (int)blockIdx.x, from = 0; block < nblocks; from = block + 1) {
            store_partial<true>(block_sums<Y_BF16, HAS_D>(yv, r, d, n, block, nblocks), partial, nblocks, block);
            if (threadIdx.x == 0) board_post(bd, block, 1u);
            if (blockIdx.x >= kFields) return;
            if (start == 0) { start = ticks(); from = 0; }
            // the first block from `from` on whose word does not come
            if (threadIdx.x == 0) s_missing = nblocks;
            __syncthreads();
            for (int b = from + (int)threadIdx.x; b < nblocks; b += kThreads) {
                uint32_t v;
                if (!board_wait(bd, b, start, v)) { atomicMin(&s_missing, b); break; }
            }
            __syncthreads();
            block = s_missing;
            __syncthreads();
            if (block >= nblocks) break;
        }
        if (nblocks > kFields) {
            const double t = fold_field<true>(partial, nblocks, (int)blockIdx.x);
            if (threadIdx.x == 0) out[blockIdx.x] = t;
        } else {
            // few blocks: a wavefront a field, in fold_field's order (its other wavefronts would add zeros)
            const int lane = threadIdx.x & (kWave - 1), step = nblocks * (kThreads / kWave);
            for (int field = (int)blockIdx.x * (kThreads / kWave) + (int)threadIdx.x / kWave; field < kFields; field += step) {
                const bool is_max = (field == 4 || field == 5 || field == 7 || field == 10);
                const double v = lane < nblocks ? coherent_load(partial + field * nblocks + lane) : 0.0;
                const double t = is_max ? wave_max_f64(v) : wave_sum_f64(v);
                if (lane == 0) out[field] = t;
            }
        }
    }
}

// The fold as a launch of its own, sixteen workgroups, for large tensors and calls that are being recorded.
__global__ void __launch_bounds__(kThreads)
metric_finalize(const double* __restrict__ partial, int nblocks, double* __restrict__ out)
{
    const double t = fold_field<false>(partial, nblocks, (int)blockIdx.x);
    if (threadIdx.x == 0) out[blockIdx.x] = t;
}

int plan_blocks(int64_t n)
{
    // two 4-element vectors per thread at least, one trip: a small tensor is bound by the latency of a trip (196608
    // elements: 5.4 -> 4.6 us against two)
    const int64_t per_block = (int64_t)kThreads * 4 * 2;
    int64_t nb = (n + per_block - 1) / per_block;
    if (nb < 1) nb = 1;
    if (nb > kMaxBlocks) nb = kMaxBlocks;
    return (int)nb;
}

}  // namespace
}  // namespace qmm

using namespace qmm;

extern "C" size_t qmm_metric_workspace_size(int64_t n)
{
    return (size_t)plan_blocks(n < 0 ? 0 : n) * 16 * sizeof(double);
}

namespace {
qmm_status metric_call(const void* y, qmm_dtype y_dtype, const float* y_ref, const float* denom, int64_t n, double* out16,
                       void* workspace, size_t workspace_bytes, uint32_t patience, void* stream)
{
    if (!out16) return QMM_ERR_NULL;
    if (y_dtype != QMM_DT_BF16 && y_dtype != QMM_DT_F32) return QMM_ERR_ENUM;
    if (n < 0) return QMM_ERR_SHAPE;
    if (n > 0 && (!y || !y_ref)) return QMM_ERR_NULL;
    if (!workspace || workspace_bytes < qmm_metric_workspace_size(n)) return QMM_ERR_WORKSPACE;
    if (!aligned16(workspace) || (reinterpret_cast<uintptr_t>(out16) & 7u)) return QMM_ERR_ALIGN;
    if (n > 0 && (!aligned16(y_ref) || (denom && !aligned16(denom)) ||
                  (reinterpret_cast<uintptr_t>(y) & (y_dtype == QMM_DT_BF16 ? 7u : 15u))))
        return QMM_ERR_ALIGN;

    hipStream_t s = as_stream(stream);
    double* partial = static_cast<double*>(workspace);
    const int nb = plan_blocks(n);
    Board bd{};
    // (with denominators the fold's registers would leave a CU three workgroups instead of four)
    const bool one = n <= (int64_t(1) << 22) && !(denom && nb == kMaxBlocks) && take_board(s, RING_LONG, (uint32_t)nb, &bd);
    bd.patience = patience;
    auto run = [&](auto bf16, auto denominators) {
        constexpr bool Y = decltype(bf16)::value, D = decltype(denominators)::value;
        if (one) metric_partial<Y, D, true><<<nb, kThreads, 0, s>>>(y, y_ref, denom, n, partial, out16, bd);
        else metric_partial<Y, D, false><<<nb, kThreads, 0, s>>>(y, y_ref, denom, n, partial, nullptr, bd);
    };
    using T = std::true_type; using F = std::false_type;
    if (y_dtype == QMM_DT_BF16) { if (denom) run(T{}, T{}); else run(T{}, F{}); }
    else { if (denom) run(F{}, T{}); else run(F{}, F{}); }
    if (one) return launch_status();
    if (hipGetLastError() != hipSuccess) return QMM_ERR_LAUNCH;
    metric_finalize<<<kFields, kThreads, 0, s>>>(partial, nb, out16);
    return launch_status();
}
}  // namespace

extern "C" qmm_status qmm_metric(const void* y, qmm_dtype y_dtype, const float* y_ref, const float* denom, int64_t n,
                                 double* out16, void* workspace, size_t workspace_bytes, void* stream)
{
    return metric_call(y, y_dtype, y_ref, denom, n, out16, workspace, workspace_bytes, kFolderPatience, stream);
}

// For the tests, not part of the ABI: the folding workgroups wait `patience` ticks for the others (0: they form what is not there yet).
extern "C" qmm_status qmm_internal_metric(const void* y, qmm_dtype y_dtype, const float* y_ref, const float* denom, int64_t n,
                                          double* out16, void* workspace, size_t workspace_bytes, uint32_t patience, void* stream)
{
    return metric_call(y, y_dtype, y_ref, denom, n, out16, workspace, workspace_bytes, patience < kFolderPatience ? patience : kFolderPatience, stream);
}
