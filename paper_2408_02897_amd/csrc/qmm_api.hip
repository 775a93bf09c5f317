// Small host-only entry points of the C ABI.
#include <atomic>
#include "qmm_device.h"

// The ring of arrival counters of the single-launch reductions (qmm_device.h): part of the device image, so zero
// when the image is loaded; every kernel that uses a slot leaves it zero.  `arrival_ring` is the host-side stand-in
// of the device array: its address on a GPU is looked up once per device and only that address goes to kernels.
static __device__ __align__(256) uint32_t arrival_ring[qmm::kArrivalSlots * qmm::kArrivalWords];
namespace qmm {
namespace {
constexpr int kMaxDevices = 64;
std::atomic<uint32_t*> ring_addr[kMaxDevices];
std::atomic<uint32_t> next_slot{0};
}  // namespace
qmm_status arrival_slots(int count, uint32_t** first)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return QMM_ERR_LAUNCH;
    if (dev < 0 || dev >= kMaxDevices || count < 1 || count > 8) return QMM_ERR_UNSUPPORTED;
    uint32_t* p = ring_addr[dev].load(std::memory_order_acquire);
    if (!p) {
        void* q = nullptr;
        if (hipGetSymbolAddress(&q, HIP_SYMBOL(arrival_ring)) != hipSuccess || !q) return QMM_ERR_LAUNCH;
        p = static_cast<uint32_t*>(q);
        ring_addr[dev].store(p, std::memory_order_release);
    }
    // slots are taken in aligned groups of eight so that a call's `count` slots never wrap around the ring
    const uint32_t group = next_slot.fetch_add(1, std::memory_order_relaxed) % (kArrivalSlots / 8);
    *first = p + (size_t)group * 8 * kArrivalWords;
    return QMM_OK;
}

// ---- boards (qmm_device.h).  A device's tags run from 1 to 2^32 - 1 and start over; the call that starts over clears its rings, which
// might hold, in a place that no call has used since, a word with a tag of the round before.
namespace {
constexpr uint64_t kTags = 0xFFFFFFFFull;
std::atomic<uint64_t*> board_addr[kMaxDevices];
std::atomic<uint64_t> next_tag[kMaxDevices], next_word[kRings];
std::atomic<int> cus[kMaxDevices];
__global__ void ring_clear(uint64_t* words)
{
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < kRings * kRingWords; i += gridDim.x * 256) words[i] = 0;
}
}  // namespace
}  // namespace qmm
static __device__ __align__(256) uint64_t board_ring[qmm::kRings * qmm::kRingWords];
namespace qmm {
bool take_board(hipStream_t s, Ring ring, uint32_t words, Board* b)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusActive;
    if (hipStreamIsCapturing(s, &st) != hipSuccess) { (void)hipGetLastError(); return false; }
    int dev = -1;
    if (st != hipStreamCaptureStatusNone || words > kBoardMax || hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return false;
    uint64_t* p = board_addr[dev].load(std::memory_order_acquire);
    if (!p) {
        void* q = nullptr;
        if (hipGetSymbolAddress(&q, HIP_SYMBOL(board_ring)) != hipSuccess || !q) { (void)hipGetLastError(); return false; }
        p = static_cast<uint64_t*>(q);
        board_addr[dev].store(p, std::memory_order_release);
    }
    const uint64_t size = (words + 15u) & ~15u;                       // whole cache lines
    uint64_t at = next_word[ring].fetch_add(size, std::memory_order_relaxed) % kRingWords;
    if (at + size > kRingWords) at = next_word[ring].fetch_add(2 * size, std::memory_order_relaxed) % kRingWords;   // past the end: from its start on
    if (at + size > kRingWords) at = 0;                               // (another thread got there first: shared, see above)
    const uint64_t n = next_tag[dev].fetch_add(1, std::memory_order_relaxed);
    b->words = p + (size_t)ring * kRingWords + at;
    b->tag = (uint32_t)(n % kTags) + 1u;
    b->patience = kPatience;
    if (n >= kTags && n % kTags == 0) ring_clear<<<256, 256, 0, s>>>(p);
    return true;
}
int cu_count()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
    int n = cus[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) { (void)hipGetLastError(); return 0; }
        cus[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}
}  // namespace qmm

extern "C" const char* qmm_status_string(qmm_status s)
{
    switch (s) {
    case QMM_OK: return "ok";
    case QMM_ERR_NULL: return "required pointer is NULL";
    case QMM_ERR_SHAPE: return "invalid shape or stride";
    case QMM_ERR_ENUM: return "invalid enum value";
    case QMM_ERR_ALIGN: return "alignment rule violated";
    case QMM_ERR_UNSUPPORTED: return "not supported by this build";
    case QMM_ERR_WORKSPACE: return "workspace missing or too small";
    case QMM_ERR_LAUNCH: return "kernel launch failed";
    case QMM_ERR_LIMIT: return "input exceeds a fixed capacity of the call";
    }
    return "unknown status";
}

extern "C" int qmm_version(void) { return 100; }
