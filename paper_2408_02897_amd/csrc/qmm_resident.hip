// qmm_scale_quantize in ONE launch with one read of the tensor: every workgroup loads its slice into registers, posts the
// slice's maximum on a board, waits for the other slices of its scale group, forms the step size and encodes what it
// holds.  Traffic 2 B + 1 B per bfloat16 element where the two passes move 2 + 2 + 1, and one launch instead of two or
// three.  For tensors whose slices are resident together (plan_rows, plan_cols).  The wait is bounded and every workgroup can do
// without the others (see Board in qmm_device.h, and collect below).
// What bounds it: reading at 6 TB/s, 1.5 us from the last maximum to the step size, then writing, which nothing overlaps any
// more.  Kernel time, two passes / this, inputs from memory, E4M3: bfloat16 16384 x 1024 19.0 / 16.9 us, 16384 x 2048 30.1 / 26.2,
// 512 matrices of 512 x 64 in 16 groups 19.6 / 16.5, transposed 19.9 / 17.0, per column 4096 x 3072 18.8 / 16.2 and 16384 x 1024
// 24.5 / 19.2, 1000 x 1000 8.1 / 5.5; binary32 16384 x 1024 27.8 / 21.4; 256 x 768 5.5 / 5.3 and a launch less for the host.
// With the codes stored past the L2 (store_through), 16384 x 1024 16.9 / 14.9, the 512 matrices 16.5 / 14.2.
// Beyond 67 MB, 384 B a thread, it no longer gains: 16384 x 3072 41.5 / 41.7 (transposed 44.3 / 47).
#include <algorithm>
#include <type_traits>
#include "qmm_encode.h"

namespace qmm {
namespace {

// Maximum over the workgroup; may be called again at once.
template <int THREADS> QMM_DEV uint32_t group_max(uint32_t v)
{
    __shared__ uint32_t s[THREADS / kWave];
    v = wave_max_u32(v);
    if ((threadIdx.x & (kWave - 1)) == 0) s[threadIdx.x / kWave] = v;
    __syncthreads();
    uint32_t r = s[0];
#pragma unroll
    for (int i = 1; i < THREADS / kWave; ++i) r = max(r, s[i]);
    __syncthreads();
    return r;
}

// Words that have not come in time: other work holds CUs -- a kernel on another stream, a second call of this kind --, and the
// workgroups that would post them start only when those that wait have ended.  Of the n words (at most kMaxWords) read(left)
// reads those with left[i] set, by all threads, and clears left[i] where it came.  As long as words come the workgroup waits on;
// when none has for `idle` ticks it forms missing ones itself, form(i) by all threads, the `me`-numbered workgroup
// another one than the others.  tell(missing): called by the first wavefront in front of that, missing(c) the bits of words c .. c + 63.
// Ends: an idle period ends with a word less to come or with one formed.
// What such a call takes, time until both streams are done: 40 calls beside 20 products that hold half of the CUs (2048 x 4096 x 8192
// E4M3), separate launches / this: 16384 x 1024 1610 / 1776 us, transposed 1700 / 1900 to 2040, 512 matrices of 512 x 64 1582 / 1860,
// per column 4096 x 3072 1564 / 1490; a quarter of the CUs 1106 / 1160, 1100 / 1280, 1047 / 1238, 992 / 930; 40 calls beside 40 of 16384 x 1024
// 1150 / 1110, 1182 / 1222, 1140 / 1105, 1160 / 1340 to 1420.  (Before, each workgroup waited 50 us and walked the words
// one by one: 1776 was 6500, 1222 was 38600.)  With words late after 5 us instead of 12, calls that have the GPU to themselves lose up to 10 %.
constexpr uint32_t kMaxWords = 1024;                     // words a workgroup waits for: a grid that is resident together has no more
constexpr uint32_t kIdle = 100;                          // 1 us
// The r-th set bit of the 64-bit words bits(0), bits(64) ..., which have more than r; uniform over a wavefront.
template <class Bits> QMM_DEV uint32_t pick(uint32_t r, Bits bits)
{
    for (uint32_t c = 0;; c += kWave) {
        uint64_t w = bits(c);
        const uint32_t here = (uint32_t)__popcll(w);
        if (r < here) {
            for (; r > 0; --r) w &= w - 1;
            return c + (uint32_t)__ffsll((unsigned long long)w) - 1;
        }
        r -= here;
    }
}
// `follows`: the first wavefront asks next() for the word to form as long as that knows one, kAll if nothing is left to do (false is
// returned), kNone if there is nobody to ask; then as above.
constexpr uint32_t kAll = ~0u, kNone = ~0u - 1;
template <int THREADS, class Read, class Form, class Tell, class Next>
QMM_DEV bool collect(uint32_t n, uint32_t me, uint32_t idle, bool follows, Read read, Form form, Tell tell, Next next)
{
    __shared__ uint8_t s_left[kMaxWords];
    __shared__ uint32_t s_at, s_seen;                    // (shared for the registers: what is held across this path is spilled in resident_cols)
    __shared__ uint64_t s_since;
    for (uint32_t i = threadIdx.x; i < n; i += THREADS) s_left[i] = 1;
    if (threadIdx.x == 0) s_seen = ~0u;
    __syncthreads();
    for (;;) {
        if (!follows) { read(s_left); __syncthreads(); }
        if (threadIdx.x < kWave) {
            uint32_t at = kNone;
            if (follows) at = next();
            else {
                auto missing = [&](uint32_t c) -> uint64_t { return __ballot(c + threadIdx.x < n && s_left[c + threadIdx.x] != 0); };
                uint32_t total = 0;
                for (uint32_t c = 0; c < n; c += kWave) total += (uint32_t)__popcll(missing(c));
                const uint64_t now = ticks();
                const bool news = total < s_seen;
                if (total == 0) at = kAll;
                else if ((news ? 0 : now - s_since) >= idle) { tell(missing); at = pick(me % total, missing); if (threadIdx.x == 0) s_seen = total - 1; }
                else if (news && threadIdx.x == 0) { s_seen = total; s_since = now; }
            }
            if (threadIdx.x == 0) s_at = at;
        }
        __syncthreads();
        const uint32_t at = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_at);
        if (at == kAll) return !follows;
        if (at < n) {
            form(at);
            if (threadIdx.x == 0) s_left[at] = 0;
        } else if (!follows) __builtin_amdgcn_s_sleep(8);
        if (at == kNone) follows = false;
        __syncthreads();
    }
}

// Posts the maximum of slice p of the group's matrix grp.k_of_b and returns the maximum over the group's slices, P a matrix.
// slice(matrix, p): this thread's part of the maximum of that slice, for values that have not come in time.
// A line of the board that many workgroups read at once is read slowly (256 workgroups that all read the same 256 words:
// 5 us; a word that one of them waits for comes 0.6 us after it was posted).  So the first eight workgroups of a group of
// many words read them and post what they find, and the others, their followers, read that.  Where words stay away a leader posts which,
// and its followers form them with it, one each, and go back to waiting.
// A leader's area: a line its followers wait on, of the result and the number and length of the last list, and the list.
constexpr uint32_t kDirect = 32, kLeaders = 8, kListAt = 16;
QMM_DEV uint32_t whole_lines(uint32_t words) { return (words + 15u) & ~15u; }
constexpr uint32_t kAlone = 5000;                        // 50 us without a word from the leader: the board is another call's as well
template <int THREADS, class Slice> QMM_DEV uint32_t fold_group(const Board& bd, const Group& grp, uint32_t P, uint32_t p, uint32_t mine, Slice slice)
{
    __shared__ uint32_t s_word;
    const uint32_t n = grp.count * P;
    const uint32_t first = grp.slot(0) * P;
    if (threadIdx.x == 0) board_post(bd, first + grp.k_of_b * P + p, mine);
    const uint64_t start = ticks();
    const uint32_t me = grp.k_of_b * P + p, most = grp.slots * P;
    const bool led = n > kDirect, leader = me < kLeaders, follows = led && !leader;
    const uint32_t area = whole_lines(grp.G * most) + (grp.g * kLeaders + me % kLeaders) * (kListAt + whole_lines(most));
    uint32_t m = 0;
    bool missing = false;
    if (follows) {
        if (threadIdx.x == 0) { uint32_t v; s_word = board_wait(bd, area, start, v) ? v : ~0u; }
        __syncthreads();
        if (s_word != ~0u) return s_word;                // (a posted value is below 2^31)
        missing = true;
    } else {
        for (uint32_t i = threadIdx.x; i < n; i += THREADS) {
            uint32_t v;
            if (board_wait(bd, first + i, start, v)) m = max(m, v); else missing = true;
        }
    }
    if (__builtin_expect(__syncthreads_or(missing), 0)) {
        __shared__ uint32_t s_lists;                     // posted by a leader, seen by a follower
        __shared__ uint64_t s_heard;
        if (threadIdx.x == 0) { s_lists = 0; s_heard = ticks(); }
        const bool all = collect<THREADS>(n, me, min(kIdle, bd.patience), follows,
            [&](uint8_t* left) {
                for (uint32_t i = threadIdx.x; i < n; i += THREADS) {
                    uint32_t v;
                    if (left[i] && board_read(bd, first + i, v)) { m = max(m, v); left[i] = 0; }
                }
            },
            [&](uint32_t at) {
                const uint32_t k = at / P, v = group_max<THREADS>(slice(grp.matrix(k), at - k * P));
                if (threadIdx.x == 0) board_post(bd, first + at, v);
                m = max(m, v);
            },
            [&](auto bits) {
                if (!led || !leader) return;
                uint32_t total = 0;
                for (uint32_t c = 0; c < n; c += kWave) {
                    const uint64_t w = bits(c), lane = uint64_t(1) << threadIdx.x;
                    if (w & lane) board_post(bd, area + kListAt + total + (uint32_t)__popcll(w & (lane - 1)), c + threadIdx.x);
                    total += (uint32_t)__popcll(w);
                }
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the list is there before its number
                if (threadIdx.x == 0) board_post(bd, area + 1, (s_lists += 1u << 16) | total);
            },
            [&]() -> uint32_t {
                while (ticks() - s_heard < (bd.patience ? kAlone : 0)) {
                    uint32_t v = 0;
                    const uint64_t have = __ballot(threadIdx.x < 2 && board_read(bd, area + threadIdx.x, v));
                    if (have & 1) { if (threadIdx.x == 0) s_word = v; return kAll; }
                    const uint32_t number = (uint32_t)__builtin_amdgcn_readlane((int)v, 1);
                    if ((have & 2) && number != s_lists) {
                        if (threadIdx.x == 0) { s_lists = number; s_heard = ticks(); }
                        // (a next list may be on its way over this one: then it is another word of those missing, or none)
                        const bool there = board_read(bd, area + kListAt + me % (number & 0xFFFFu), v);
                        v = (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
                        if (__any(there) && v < n) return v;
                    }
                    __builtin_amdgcn_s_sleep(2);
                }
                return kNone;
            });
        if (!all) return s_word;
    }
    m = group_max<THREADS>(m);
    if (led && leader && threadIdx.x == 0) board_post(bd, area, m);
    return m;
}

// Rows contracting, one step size per scale group, rows of 16 elements at least.  A thread takes units of 16 elements (two or
// four 16-byte loads, one 16-byte store).  A slice is THREADS * NU units of a matrix: THREADS neighbours at a time, these pieces
// one behind the other or (`sweep`: all matrices are one group) a whole grid's pieces apart, so that the grid reads the
// tensor front to back.  A row's partial last unit is taken back to the end of its row (the same codes twice), and units past
// the matrix are its last one again.  DENSE: the matrix is one row.
constexpr int kUnit = 16;
template <typename T, int FMT, int MODE, int THREADS, int NU, int WAVES, bool DENSE> __global__ void __launch_bounds__(THREADS, WAVES)
resident_rows(QArgs a, Board bd, uint32_t upr, uint32_t units, uint32_t P, uint32_t sweep)
{
    constexpr int V = Vec<T>::V, U = kUnit / V;
    const uint32_t b = blockIdx.x / P, p = blockIdx.x - b * P;
    const uint32_t piece = sweep ? P * THREADS : THREADS;
    auto first_of = [&](uint32_t slice) { return (sweep ? slice * THREADS : slice * (THREADS * NU)) + threadIdx.x; };
    // element offsets of unit u in the tensor and in the codes (DENSE: below 2^31, host)
    using Offset = typename std::conditional<DENSE, uint32_t, int64_t>::type;
    auto place = [&](uint32_t u, Offset& src, Offset& dst) {
        if constexpr (DENSE) {
            src = dst = min(u * kUnit, (uint32_t)a.cols - kUnit);
        } else {
            const uint32_t r = u / upr;
            const int64_t c = min((int64_t)(u - r * upr) * kUnit, a.cols - kUnit);
            src = r * a.row_stride + c;
            dst = r * a.cols + c;
        }
    };
    auto load = [&](const T* base, uint32_t u, u32x4 (&w)[U]) {
        Offset src, dst;
        place(min(u, units - 1), src, dst);
#pragma unroll
        for (int k = 0; k < U; ++k) w[k] = *reinterpret_cast<const u32x4_any*>(base + src + k * V);
    };
    const T* x = static_cast<const T*>(a.x);
    const uint32_t first = first_of(p);
    u32x4 w[NU][U];
#pragma unroll
    for (int i = 0; i < NU; ++i) load(x + b * a.batch_stride, first + i * piece, w[i]);
    VecMax<T> mm;
#pragma unroll
    for (int i = 0; i < NU; ++i)
#pragma unroll
        for (int k = 0; k < U; ++k) mm.fold(w[i][k]);
    const uint32_t mine = group_max<THREADS>(mm.finish());
    const Group grp = group_at((uint32_t)a.batch, (uint32_t)a.groups, (uint32_t)min(a.inner, a.batch), b);
    const uint32_t bits = fold_group<THREADS>(bd, grp, P, p, mine, [&](uint32_t mb, uint32_t slice) {
        const uint32_t u0 = first_of(slice);
        VecMax<T> o;
#pragma unroll 1
        for (int i = 0; i < NU; ++i) {
            u32x4 v[U];
            load(x + mb * a.batch_stride, u0 + i * piece, v);
#pragma unroll
            for (int k = 0; k < U; ++k) o.fold(v[k]);
        }
        return o.finish();
    });
    const float d = delta_from_absmax_bits(bits, a.qmax);
    if (threadIdx.x == 0 && p == 0 && b == grp.matrix(0)) a.delta[grp.g] = d;
    const float rho = 1.0f / d;
    const int64_t out = b * (a.rows * a.cols);
#pragma unroll
    for (int i = 0; i < NU; ++i) {
        const uint32_t u = first + i * piece;
        if (u < units) {
            Offset src, dst;
            place(u, src, dst);
            float t[kUnit];
#pragma unroll
            for (int e = 0; e < kUnit; ++e) t[e] = Vec<T>::at(w[i][e / V], e % V) * rho;
            const uint64_t g = (uint64_t)(out + dst) + a.offset;
            uint32_t c[4];
            encode_quads<FMT, MODE, 4>(t, g, a.seed, MODE == QMM_ROUND_STOCHASTIC && !__any((g & 3u) != 0u), c);
            store_through(a.codes + out + dst, u32x4{c[0], c[1], c[2], c[3]});
        }
    }
}

// Words that fold_group uses.
int64_t board_words(const QArgs& q, int64_t P)
{
    const int64_t inner = std::min(q.inner, q.batch), runs = (q.batch + inner - 1) / inner, a_group = (runs + q.groups - 1) / q.groups * inner * P;
    return a_group * q.groups + (a_group > kDirect ? 16 + q.groups * kLeaders * (kListAt + a_group + 15) : 0);
}

struct RowsPlan { int variant; uint32_t upr, units, P; unsigned blocks; uint32_t words; };
struct RowsVariant { int threads, bytes, per_cu; };      // bytes of the tensor a thread holds
// (the first that the tensor fits: many small workgroups for small tensors, which are bound by the length of a thread's own work)
constexpr RowsVariant kRows[] = {{256, 32, 2}, {256, 64, 4}, {1024, 64, 2}, {1024, 128, 1}, {1024, 256, 1}};

template <typename T, int MODE> bool plan_rows(const QArgs& q, RowsPlan* pl)
{
    if (q.cols < kUnit) return false;
    const int64_t upr = (q.cols + kUnit - 1) / kUnit, units = q.rows * upr;
    const int cus = cu_count();
    if (units > (0x7FFFFFFF / kUnit)) return false;
    // Stochastic rounding, bound by the generator, gains nothing from 33 MB on (binary32 16384 x 1024 32.6 / 33.8 us), nor has it the
    // registers; rows that are not dense need theirs for the coordinates.
    const int variants = MODE != QMM_ROUND_RTNE ? 3 : q.rows > 1 ? 4 : 5;
    for (int i = sizeof(T) == 2 ? 0 : 1; i < variants; ++i) {
        const RowsVariant& r = kRows[i];
        const int64_t slice = r.threads * (r.bytes / (int64_t)(kUnit * sizeof(T)));
        const int64_t P = (units + slice - 1) / slice, blocks = P * q.batch;
        const int64_t words = board_words(q, P);
        if (blocks > std::min<int64_t>(r.per_cu * cus, kMaxWords) || words > kBoardMax) continue;
        // Stochastic rounding: where some CUs get two of the large workgroups and others one, the one waits for the two (bfloat16, separate
        // launches / this: 8192 x 1024, 256 workgroups, 16.2 / 14.3 us, 8704 x 1024, 272, 16.0 / 19.8, 12288 x 1024, 384, 19.1 / 20.7, 14336 x 1024, 448,
        // 21.1 / 21.7, 16384 x 1024, 512, 23.1 / 22.5; in 16 groups 300 x [512 x 64] 18.4 / 20.2, 420 23.0 / 21.5; binary32, half the codes, not).
        if (MODE != QMM_ROUND_RTNE && sizeof(T) == 2 && r.threads == 1024 && blocks > cus && blocks < (q.groups > 1 ? 3 * cus / 2 : 15 * cus / 8)) continue;
        *pl = RowsPlan{i, (uint32_t)upr, (uint32_t)units, (uint32_t)P, (unsigned)blocks, (uint32_t)words};
        return true;
    }
    return false;
}

template <typename T, int FMT, int MODE> qmm_status launch_rows(const QArgs& q, const RowsPlan& pl, const Board& bd, hipStream_t s)
{
    const uint32_t sweep = q.batch == 1;
    auto run = [&](auto variant, auto dense) {
        constexpr RowsVariant r = kRows[decltype(variant)::value];
        constexpr int waves = r.threads == 256 ? 4 : r.per_cu * 4;                 // per SIMD
        resident_rows<T, FMT, MODE, r.threads, r.bytes / (kUnit * sizeof(T)), waves, decltype(dense)::value>
            <<<pl.blocks, r.threads, 0, s>>>(q, bd, pl.upr, pl.units, pl.P, sweep);
    };
    auto either = [&](auto variant) { if (q.rows == 1) run(variant, std::true_type{}); else run(variant, std::false_type{}); };
    switch (pl.variant) {
    case 0: if constexpr (sizeof(T) == 2) either(std::integral_constant<int, 0>{}); break;
    case 1: either(std::integral_constant<int, 1>{}); break;
    case 2: either(std::integral_constant<int, 2>{}); break;
    default:
        if constexpr (MODE == QMM_ROUND_RTNE) {
            if (pl.variant == 3) either(std::integral_constant<int, 3>{});
            else run(std::integral_constant<int, 4>{}, std::true_type{});
        }
    }
    return launch_status();
}

// ---- contracting over rows
constexpr int kStrip = 64;                               // columns of a workgroup's slice

// A slice: S tiles of THREADS / 2 rows by 64 columns of a matrix (one step size per scale group: S tiles that follow one
// another strip by strip; per column: of one strip).  The codes of a tile are transposed through LDS, 16 bytes at a time
// as in quantize_cols.
// They leave past the L2 where a code row is a line and more, whatever its alignment (by the L2 / past it: 16400 rows of 1024 20.2 /
// 18.8 us, 512 matrices of 136 x 64 10.0 / 9.2, of 250 x 64 11.4 / 10.5), and where shorter rows have no remainder (1024 matrices of
// 112 x 64 10.5 / 9.6); a remainder is written in bytes, and the lines of short rows would all leave in parts (of 127 x 64 11.2 / 13.2,
// binary32 14.4 / 16.4, of 120 x 64 10.8 / 10.9).
template <typename T, int FMT, int MODE, int THREADS, int S, bool PER_COLUMN, int WAVES> __global__ void __launch_bounds__(THREADS, WAVES)
resident_cols(QArgs a, Board bd, uint32_t strips, uint32_t tiles_k, uint32_t P)
{
    constexpr int V = Vec<T>::V, TN = kStrip / V, RT = 32 / V, TILE_K = THREADS / TN * RT;
    static_assert(RT % 4 == 0 && TILE_K == THREADS / 2, "codes are packed four rows at a time");
    constexpr int ROW = TILE_K + 16, Q = THREADS / kStrip, PIECES = kStrip * TILE_K / 16 / THREADS;
    __shared__ __attribute__((aligned(16))) uint8_t tile[kStrip * ROW];
    __shared__ uint32_t s_col[kStrip], s_fold[Q][kStrip];
    __shared__ float s_rho[kStrip];
    const int tn = threadIdx.x % TN, tk = threadIdx.x / TN;
    const uint32_t b = blockIdx.x / P, p = blockIdx.x - b * P;
    const int64_t K = a.rows, N = a.cols;
    // tile t of slice p of a matrix: (strip, first row); false: past the end of the matrix
    auto tile_at = [&](uint32_t slice, int t, uint32_t& strip, int64_t& k0) -> bool {
        if constexpr (PER_COLUMN) {
            const uint32_t per_strip = P / strips;
            strip = slice / per_strip;
            const uint32_t kt = (slice - strip * per_strip) * S + t;
            k0 = (int64_t)kt * TILE_K;
            return kt < tiles_k;
        } else {
            const uint32_t at = slice * S + t;
            strip = at / tiles_k;
            k0 = (int64_t)(at - strip * tiles_k) * TILE_K;
            return strip < strips;
        }
    };
    // a thread's RT rows of a tile (rows past the last one are the last one again; columns past the last one are zero)
    auto load = [&](uint32_t mb, uint32_t strip, int64_t k0, auto&& each) {
        const int64_t n = (int64_t)strip * kStrip + tn * V, k = min(k0 + tk * RT, K - 1);
        const int left = (int)max((int64_t)0, min((int64_t)V, N - n)), last = (int)min(K - 1 - k, (int64_t)(RT - 1));
        const T* base = static_cast<const T*>(a.x) + mb * a.batch_stride + k * a.row_stride + n;
        if (left == V) {
            each([&](int i) { return load_columns<T, V>(base + min(i, last) * a.row_stride, V); });
        } else if (sizeof(T) == 2 && left > 1 && N >= V) {
            // the last columns: a vector that ends with the row, moved down.  Element by element it is a chain of loads: 64 matrices of
            // 500 x 500 24.5 us, and 28 to 34 as the compiler took the code around it, against 21.9.  (Chains of up to three, for
            // binary32, are the shorter way: 16 matrices of 1001 x 503 13.1 against 14.5.)
            const int s = (V - left) * (int)sizeof(T) * 8;
            each([&](int i) {
                const u32x4 v = load_columns<T, V>(base + min(i, last) * a.row_stride - (V - left), V);
                const uint64_t lo = v[0] | (uint64_t)v[1] << 32, hi = v[2] | (uint64_t)v[3] << 32;
                const uint64_t down = s < 64 ? lo >> s | hi << (64 - s) : hi >> (s - 64), up = s < 64 ? hi >> s : 0;
                return u32x4{(uint32_t)down, (uint32_t)(down >> 32), (uint32_t)up, (uint32_t)(up >> 32)};
            });
        } else {
            each([&](int i) { return load_columns<T, V>(base + min(i, last) * a.row_stride, left); });
        }
    };
    u32x4 w[S][RT];
#pragma unroll
    for (int t = 0; t < S; ++t) {
#pragma unroll
        for (int i = 0; i < RT; ++i) w[t][i] = u32x4{0u, 0u, 0u, 0u};
        uint32_t strip; int64_t k0;
        if (tile_at(p, t, strip, k0)) load(b, strip, k0, [&](auto row) {
#pragma unroll
            for (int i = 0; i < RT; ++i) w[t][i] = row(i);
        });
    }
    VecMax<T> mm;
#pragma unroll
    for (int t = 0; t < S; ++t)
#pragma unroll
        for (int i = 0; i < RT; ++i) mm.fold(w[t][i]);
    auto slice_max = [&](uint32_t mb, uint32_t slice) {
        VecMax<T> o;
#pragma unroll 1
        for (int t = 0; t < S; ++t) {
            uint32_t strip; int64_t k0;
            if (!tile_at(slice, t, strip, k0)) break;
            // (row by row: w stays in registers meanwhile)
            load(mb, strip, k0, [&](auto row) {
#pragma unroll 1
                for (int i = 0; i < RT; ++i) o.fold(row(i));
            });
        }
        return o;
    };
    if constexpr (PER_COLUMN) {
        // the maxima of a slice's columns, in s_col
        static_assert(kStrip == kWave, "a wavefront reads a slice's words");
        auto columns_max = [&](VecMax<T> o) {
            if (threadIdx.x < kStrip) s_col[threadIdx.x] = 0;
            __syncthreads();
            uint32_t x[4];
#pragma unroll
            for (int off = TN; off < kWave; off <<= 1) {
                o.words(x);
#pragma unroll
                for (int i = 0; i < 4; ++i) x[i] = (uint32_t)__shfl_xor((int)x[i], off, kWave);
                o.fold_words(x);
            }
            if ((threadIdx.x & (kWave - 1)) < TN) {
#pragma unroll
                for (int e = 0; e < V; ++e) atomicMax(&s_col[tn * V + e], o.at(e));
            }
            __syncthreads();
        };
        const uint32_t per_strip = P / strips, strip = p / per_strip, kp = p - strip * per_strip;
        const int c = threadIdx.x & (kStrip - 1), q = threadIdx.x / kStrip;
        const int64_t col = (int64_t)strip * kStrip + c;
        auto word = [&](uint32_t k) { return (uint32_t)(((int64_t)b * per_strip + k) * N + col); };
        columns_max(mm);
        if (q == 0 && col < N) board_post(bd, word(kp), s_col[c]);
        const uint64_t start = ticks();
        uint32_t m = 0;
        bool missing = false;
        if (col < N) {
            for (uint32_t k = q; k < per_strip; k += Q) {
                uint32_t v;
                if (board_wait(bd, word(k), start, v)) m = max(m, v); else missing = true;
            }
        }
        if (__builtin_expect(__syncthreads_or(missing), 0)) {
            // (a wavefront reads the words of a slice, one column a lane)
            collect<THREADS>(per_strip, kp, min(kIdle, bd.patience), false,
                [&](uint8_t* left) {
                    for (uint32_t k = q; k < per_strip; k += Q) {
                        if (!left[k]) continue;
                        uint32_t v = 0;
                        const bool there = col >= N || board_read(bd, word(k), v);
                        if (there) m = max(m, v);
                        if (__all(there) && c == 0) left[k] = 0;
                    }
                },
                [&](uint32_t k) {
                    columns_max(slice_max(b, strip * per_strip + k));
                    const uint32_t v = s_col[c];
                    if (q == 0 && col < N) board_post(bd, word(k), v);
                    m = max(m, v);
                },
                [](auto) {}, [] { return kNone; });
        }
        s_fold[q][c] = m;
        __syncthreads();
        if (q == 0) {
#pragma unroll
            for (int i = 1; i < Q; ++i) m = max(m, s_fold[i][c]);
            const float d = delta_from_absmax_bits(m, a.qmax);
            s_rho[c] = 1.0f / d;
            if (kp == 0 && col < N) a.delta[group_of(a, b) * N + col] = d;
        }
    } else {
        const uint32_t mine = group_max<THREADS>(mm.finish());
        const Group grp = group_at((uint32_t)a.batch, (uint32_t)a.groups, (uint32_t)min(a.inner, a.batch), b);
        const uint32_t bits = fold_group<THREADS>(bd, grp, P, p, mine, [&](uint32_t mb, uint32_t slice) { return slice_max(mb, slice).finish(); });
        const float d = delta_from_absmax_bits(bits, a.qmax);
        if (threadIdx.x == 0 && p == 0 && b == grp.matrix(0)) a.delta[grp.g] = d;
        if (threadIdx.x < kStrip) s_rho[threadIdx.x] = 1.0f / d;
    }
    __syncthreads();
    // 16-byte chunk c of code row n lies at chunk position c ^ ((n >> 3) & 7), as in quantize_cols
    auto place = [](int n, int k) { return n * ROW + (((k >> 4) ^ ((n >> 3) & 7)) << 4) + (k & 15); };
#pragma unroll
    for (int t = 0; t < S; ++t) {
        uint32_t strip; int64_t k0;
        if (!tile_at(p, t, strip, k0)) break;
        const int64_t n0 = (int64_t)strip * kStrip, n = n0 + tn * V, k_first = k0 + tk * RT;
        auto columns = [&](auto at_block, auto quads) {
            constexpr int B = decltype(quads)::value;
            uint64_t g = (uint64_t)(((int64_t)b * N + n) * K + k_first) + a.offset;
#pragma unroll
            for (int j = 0; j < V; ++j, g += (uint64_t)K) {
                const float rho = s_rho[tn * V + j];
#pragma unroll
                for (int q = 0; q < RT / 4; q += B) {
                    float v[4 * B];
#pragma unroll
                    for (int e = 0; e < 4 * B; ++e) v[e] = Vec<T>::at(w[t][4 * q + e], j) * rho;
                    uint32_t code[B];
                    encode_quads<FMT, MODE, B>(v, g + 4 * q, a.seed, at_block.value, code);
#pragma unroll
                    for (int e = 0; e < B; ++e) *reinterpret_cast<uint32_t*>(&tile[place(tn * V + j, tk * RT + 4 * (q + e))]) = code[e];
                    if constexpr (MODE == QMM_ROUND_STOCHASTIC) __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        if (n < N && k_first < K) {
            if constexpr (MODE == QMM_ROUND_RTNE) columns(std::true_type{}, std::integral_constant<int, 1>{});
            else if (whole_blocks(a)) columns(std::true_type{}, std::integral_constant<int, 1>{});
            else columns(std::false_type{}, std::integral_constant<int, RT / 4>{});
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < PIECES; ++it) {
            const int piece = it * THREADS + threadIdx.x, row = piece / (TILE_K / 16), at = piece % (TILE_K / 16) * 16;
            const int64_t nn = n0 + row, kk = k0 + at;
            if (nn >= N || kk >= K) continue;
            uint8_t* dst = a.codes + ((int64_t)b * N + nn) * K + kk;
            const u32x4 codes = *reinterpret_cast<const u32x4*>(&tile[place(row, at)]);
            if (kk + 16 <= K) {
                if (K >= 128 || K % 16 == 0) store_through(dst, codes); else *reinterpret_cast<u32x4_byte*>(dst) = codes;
            } else store_bytes<16>(dst, codes, (int)(K - kk));
        }
        if (t + 1 < S) __syncthreads();
    }
}

struct ColsPlan { int variant; uint32_t strips, tiles_k, P; unsigned blocks; uint32_t words; };
struct ColsVariant { int threads, tiles, per_cu; };
constexpr ColsVariant kCols[] = {{256, 1, 4}, {1024, 1, 2}, {1024, 3, 1}};

template <typename T, int MODE> bool plan_cols(const QArgs& q, ColsPlan* pl)
{
    const int64_t strips = (q.cols + kStrip - 1) / kStrip;
    const int cus = cu_count();
    for (int i = 0; i < (int)(sizeof(kCols) / sizeof(kCols[0])); ++i) {
        const ColsVariant& c = kCols[i];
        // Stochastic rounding and binary32, which takes twice the registers a tile, spill with more than one tile (binary32 4096 x 3072
        // per column 24.4 / 24.9 us).
        if (c.tiles > (MODE != QMM_ROUND_RTNE || sizeof(T) == 4 ? 1 : 3)) continue;
        const int per_cu = c.threads == 1024 && c.tiles == 1 && (MODE != QMM_ROUND_RTNE || sizeof(T) == 4) ? 1 : c.per_cu;
        const int64_t tiles_k = (q.rows + c.threads / 2 - 1) / (c.threads / 2);
        const int64_t P = q.channels > 1 ? strips * ((tiles_k + c.tiles - 1) / c.tiles) : (strips * tiles_k + c.tiles - 1) / c.tiles;
        const int64_t blocks = P * q.batch, words = q.channels > 1 ? P / strips * q.cols * q.batch : board_words(q, P);
        if (blocks > std::min<int64_t>(per_cu * cus, kMaxWords) || words > kBoardMax || tiles_k > 0x7FFFFFFF) continue;
        // Per column every workgroup of a strip reads the maxima of all: of the small tiles' no more than 40, and no fewer than 32 workgroups of
        // the large (bfloat16, 64 columns, separate launches / small tiles / large ones: 4096 rows 7.3 / 7.1 / 7.9 us, 8192 7.5 / 9.8 / 7.9, 16384
        // 8.3 / 14.6 / 8.4, 65536 18.7 / 46.5 / 10.5, 128000 24.3 / 92.5 / 15.5; 256 columns, 4096 8.1 / 7.4 / 8.0, 16384 14.2 / 16.9 / 8.8; binary32
        // 128000 x 64 28.6 / 92.5 / 16.4).
        const int64_t waits = q.channels > 1 ? P / strips : 0;
        if (waits > 0 && (i == 0 ? waits > 40 : blocks < 32)) continue;
        // Stochastic rounding: with few workgroups a thread's generator blocks are what counts, twice as many where columns do not start
        // blocks, and a call is bound by the GPU rather than by its launches (9.5 us for the host of the separate ones, 6.4 for this one's).
        // GPU time of calls back to back, separate launches / this, one step size: 1030 x 1024, 144 workgroups, 9.0 / 10.5 us, 1030 x 1536, 216,
        // 10.3 / 10.7, 2046 x 1024, 256, 10.9 / 10.8, 2046 x 1280, 320, 14.2 / 12.8; 1032 x 1024, 144, 7.9 / 8.2, 2048 x 1024, 256, 9.6 / 8.2;
        // per column 4094 x 512, 256, 10.9 / 11.7, 4094 x 640, 320, 15.6 / 13.8, 4096 x 256, 128, 7.4 / 8.8, 4096 x 384, 192, 8.8 / 8.8; large tiles
        // 8192 x 256, 64, 10.2 / 12.2, 8192 x 384, 96, 12.9 / 12.4, 8190 x 512, 128, 16.9 / 17.8, 8190 x 640, 160, 19.9 / 18.0; 300 x [2 x 128] 13.8 / 14.6.
        if constexpr (MODE != QMM_ROUND_RTNE) {
            const bool whole = whole_blocks(q);
            if (q.cols < 24 || (!whole && q.rows < 8)) continue;       // a strip's other threads are idle (18550 x 4 10.2 / 19.6 us, x 16 10.1 / 11.8, x 32 11.1 / 11.6)
            const int least = waits > 0 && i > 0 ? (whole ? 96 : 144) : waits > 16 ? (whole ? 128 : 320) : whole ? 64 : 256;
            if (blocks < least) continue;
        }
        *pl = ColsPlan{i, (uint32_t)strips, (uint32_t)tiles_k, (uint32_t)P, (unsigned)blocks, (uint32_t)words};
        return true;
    }
    return false;
}

template <typename T, int FMT, int MODE, bool PER_COLUMN> qmm_status launch_cols(const QArgs& q, const ColsPlan& pl, const Board& bd, hipStream_t s)
{
    constexpr int W = MODE == QMM_ROUND_RTNE && sizeof(T) == 2 ? 8 : 4;
    if (pl.variant == 0) resident_cols<T, FMT, MODE, 256, 1, PER_COLUMN, 4><<<pl.blocks, 256, 0, s>>>(q, bd, pl.strips, pl.tiles_k, pl.P);
    else if (pl.variant == 1) resident_cols<T, FMT, MODE, 1024, 1, PER_COLUMN, W><<<pl.blocks, 1024, 0, s>>>(q, bd, pl.strips, pl.tiles_k, pl.P);
    else if constexpr (MODE == QMM_ROUND_RTNE && sizeof(T) == 2)
        resident_cols<T, FMT, MODE, 1024, 3, PER_COLUMN, 4><<<pl.blocks, 1024, 0, s>>>(q, bd, pl.strips, pl.tiles_k, pl.P);
    return launch_status();
}

template <typename T, int FMT, int MODE> qmm_status run(const qmm_tensor* x, const QArgs& a, hipStream_t s, uint32_t patience, bool* taken)
{
    Board bd;
    if (x->contract_axis == 1) {
        QArgs q = a;
        if (q.row_stride == q.cols || q.rows == 1) { q.cols *= q.rows; q.row_stride = q.cols; q.rows = 1; }     // dense: one long row
        if (q.rows == 1 && q.groups == 1 && q.batch > 1 && q.batch_stride == q.cols) { q.cols *= q.batch; q.batch = 1; q.batch_stride = q.cols; q.inner = 1; }
        RowsPlan pl;
        if (!plan_rows<T, MODE>(q, &pl) || !take_board(s, RING_SHORT, pl.words, &bd)) return QMM_OK;
        bd.patience = min(bd.patience, patience);
        *taken = true;
        return launch_rows<T, FMT, MODE>(q, pl, bd, s);
    }
    ColsPlan pl;
    if (!plan_cols<T, MODE>(a, &pl) || !take_board(s, RING_SHORT, pl.words, &bd)) return QMM_OK;
    bd.patience = min(bd.patience, patience);
    *taken = true;
    return a.channels > 1 ? launch_cols<T, FMT, MODE, true>(a, pl, bd, s) : launch_cols<T, FMT, MODE, false>(a, pl, bd, s);
}
template <typename T, int FMT> qmm_status run_mode(const qmm_tensor* x, const QArgs& a, qmm_round mode, hipStream_t s, uint32_t patience, bool* taken)
{
    return mode == QMM_ROUND_RTNE ? run<T, FMT, QMM_ROUND_RTNE>(x, a, s, patience, taken) : run<T, FMT, QMM_ROUND_STOCHASTIC>(x, a, s, patience, taken);
}
template <typename T> qmm_status run_type(const qmm_tensor* x, const QArgs& a, qmm_format fmt, qmm_round mode, hipStream_t s, uint32_t patience, bool* taken)
{
    switch (fmt) {
    case QMM_FMT_INT8: return run_mode<T, QMM_FMT_INT8>(x, a, mode, s, patience, taken);
    case QMM_FMT_E4M3: return run_mode<T, QMM_FMT_E4M3>(x, a, mode, s, patience, taken);
    default: return run_mode<T, QMM_FMT_E5M2>(x, a, mode, s, patience, taken);
    }
}

}  // namespace

// On checked arguments of a tensor that has elements.  *taken = false: nothing was launched, the call goes another way.
qmm_status scale_quantize_resident(const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g, qmm_round mode, uint64_t seed,
                                   uint64_t offset, float* delta, uint8_t* codes, uint32_t patience, hipStream_t s, bool* taken)
{
    *taken = false;
    const int64_t inner = g->batch_inner > 0 ? g->batch_inner : 1;
    const bool columns = g->per_channel && (x->contract_axis == 1 ? x->rows : x->cols) > 1;
    if (columns) {
        // one step size per column, each matrix a group of its own (per row: the one-pass kernel, or rows too long for it)
        if (x->contract_axis == 1 || g->batch_groups != x->batch || inner != 1) return QMM_OK;
    } else if (g->batch_groups > x->batch || (g->batch_groups - 1) * inner >= x->batch) {
        return QMM_OK;                                   // a group without a matrix: its step size is written by the fold kernels
    }
    if (g->batch_groups > 65535 || x->rows > (int64_t(1) << 30) || x->cols > (int64_t(1) << 30)) return QMM_OK;
    QArgs a{};
    a.x = x->data; a.delta = delta; a.codes = codes;
    a.batch = x->batch; a.rows = x->rows; a.cols = x->cols;
    a.batch_stride = x->batch_stride; a.row_stride = x->row_stride;
    a.groups = g->batch_groups; a.inner = inner;
    a.channels = columns ? x->cols : 1;
    a.seed = seed; a.offset = offset; a.qmax = host_qmax(fmt);
    return x->dtype == QMM_DT_BF16 ? run_type<uint16_t>(x, a, fmt, mode, s, patience, taken) : run_type<float>(x, a, fmt, mode, s, patience, taken);
}
}  // namespace qmm

// For the tests, not part of the ABI: the one-launch form alone, its workgroups waiting `patience` ticks for one another
// (0: a workgroup forms every value itself that is not there yet).  *taken = 0: the form does not take this call.
extern "C" qmm_status qmm_internal_scale_quantize(const qmm_tensor* x, qmm_format fmt, const qmm_granularity* g, qmm_round mode,
                                                  uint64_t seed, uint64_t offset, float* delta, uint8_t* codes, uint32_t patience,
                                                  int* taken, void* stream)
{
    bool took = false;
    const qmm_status st = qmm::scale_quantize_resident(x, fmt, g, mode, seed, offset, delta, codes, patience, qmm::as_stream(stream), &took);
    *taken = took;
    return st;
}
