// Status strings, the thread-local error message and the version query.
#include "common.h"

#include <atomic>
#include <chrono>
#include <mutex>
#include <vector>

namespace e2eg {

namespace {
struct Profile {
    bool active = false;
    int32_t capacity = 0;
    std::vector<hipEvent_t> start, stop;
};
thread_local Profile g_profile;
}  // namespace

void profile_mark(hipStream_t stream, bool after) {
    Profile& p = g_profile;
    if (!p.active) return;
    if (!after) {
        if ((int32_t)p.start.size() >= p.capacity) return;
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) return;
        (void)hipEventRecord(e, stream);
        p.start.push_back(e);
    } else {
        if (p.stop.size() >= p.start.size()) return;
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) return;
        (void)hipEventRecord(e, stream);
        p.stop.push_back(e);
    }
}

namespace {
// A pinned page of slots, allocated at the first use and kept: a call takes one, has a kernel at the end of its
// stream write the values and then the call's number there, polls for that number and gives the slot back.
// (A copy to pageable memory and a stream wait come 14 us later after one kernel, 32 us after a chain of
// eight: measured 22.9 against 8.9 us and 61 against 29 us from the first launch to the answer.)
constexpr int kSlots = 64;
struct alignas(64) HostSlot {
    int32_t number;
    int32_t value[8];
};
HostSlot* g_slots = nullptr;
std::atomic<uint64_t> g_taken{0};
std::atomic<uint32_t> g_calls{0};
std::once_flag g_slots_once;

int take_slot() {   // -1: none (no page, or all 64 in use)
    std::call_once(g_slots_once, [] {
        void* p = nullptr;
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;   // another thread may be capturing
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        if (hipHostMalloc(&p, kSlots * sizeof(HostSlot), hipHostMallocPortable | hipHostMallocMapped) == hipSuccess)
            g_slots = static_cast<HostSlot*>(p);
        else
            (void)hipGetLastError();
        (void)hipThreadExchangeStreamCaptureMode(&mode);
    });
    if (!g_slots) return -1;
    uint64_t taken = g_taken.load(std::memory_order_relaxed);
    while (~taken) {
        const int i = __builtin_ctzll(~taken);
        if (g_taken.compare_exchange_weak(taken, taken | (1ull << i), std::memory_order_acquire)) return i;
    }
    return -1;
}

__global__ void publish(const int32_t* __restrict__ src, int count, HostSlot* slot, int32_t number) {
    if ((int)threadIdx.x < count)
        __hip_atomic_store(&slot->value[threadIdx.x], src[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __threadfence_system();   // one wavefront: the values are out before the number
    if (threadIdx.x == 0) __hip_atomic_store(&slot->number, number, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
}  // namespace

int32_t read_back(const int32_t* d_src, int count, int32_t* host, hipStream_t stream) {
    const int i = take_slot();
    if (i < 0) {
        E2EG_HIP_TRY(hipMemcpyAsync(host, d_src, (size_t)count * sizeof(int32_t), hipMemcpyDeviceToHost, stream));
        E2EG_HIP_TRY(hipStreamSynchronize(stream));
        return E2EG_OK;
    }
    HostSlot* slot = &g_slots[i];
    const int32_t number = (int32_t)(g_calls.fetch_add(1, std::memory_order_relaxed) | 1u << 31);
    __atomic_store_n(&slot->number, 0, __ATOMIC_RELEASE);
    publish<<<1, 64, 0, stream>>>(d_src, count, slot, number);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
        // Poll for as long as a small call takes; a long one is waited for like any other.
        const auto until = std::chrono::steady_clock::now() + std::chrono::milliseconds(1);
        bool there = false;
        while (!(there = __atomic_load_n(&slot->number, __ATOMIC_ACQUIRE) == number)) {
            __builtin_ia32_pause();
            if (std::chrono::steady_clock::now() > until) break;
        }
        if (!there) {
            e = hipStreamSynchronize(stream);
            if (e == hipSuccess && __atomic_load_n(&slot->number, __ATOMIC_ACQUIRE) != number) e = hipErrorUnknown;
        }
    }
    if (e != hipSuccess) return fail(E2EG_ERR_HIP, "read_back: %s", hipGetErrorString(e));   // the slot is not used again
    for (int k = 0; k < count; ++k) host[k] = slot->value[k];
    g_taken.fetch_and(~(1ull << i), std::memory_order_release);
    return E2EG_OK;
}

static thread_local char g_last_error[512] = "";

void set_error(const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_last_error, sizeof(g_last_error), fmt, ap);
    va_end(ap);
}

int32_t fail(int32_t status, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_last_error, sizeof(g_last_error), fmt, ap);
    va_end(ap);
    return status;
}

size_t sched_carve(void* base, int64_t n, int64_t nnz, SchedView* view, bool weighted, const int32_t* row_ptr) {
    Carver c(base);
    SchedView v;
    const bool small = sched_is_small(nnz);
    const int64_t entries = nnz > 0 ? nnz : 1;
    v.max_plain = sched_max_plain(nnz);
    v.max_multi = sched_max_multi(nnz);
    v.max_slot = sched_max_slot(n, nnz);
    v.header = c.take<SchedHeader>(1);
    v.short_rows = c.take<ShortRow>(n > 0 ? n : 1);
    v.multi_row = c.take<int32_t>(v.max_multi);
    v.slot_base = c.take<int32_t>(v.max_multi);
    v.slot_cnt = c.take<int32_t>(v.max_multi);
    v.singles = c.take<Segment>(v.max_plain);
    v.segs = c.take<Segment>(v.max_slot);
    v.znode = c.take<int32_t>(entries);
    v.zs = c.take<float>(entries);
    if (small) {
        v.orig = nullptr;
        v.zrow_ptr = const_cast<int32_t*>(row_ptr);
        v.zcol = v.znode;
    } else {
        v.orig = c.take<int32_t>(n > 0 ? n : 1);
        v.zrow_ptr = c.take<int32_t>(n + 1);
        v.zcol = c.take<int32_t>(entries);
    }
    v.zval = weighted ? c.take<float>(entries) : nullptr;  // last: the rest of the layout is shared
    if (view) *view = v;
    return c.size();
}

}  // namespace e2eg

namespace e2eg {
// Plain streaming copy, 16 bytes per thread: the traffic of known size against which hardware
// byte counters are scaled.
__global__ void copy_bytes16(uint4* __restrict__ dst, const uint4* __restrict__ src, size_t chunks) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < chunks) dst[i] = src[i];
}
}  // namespace e2eg

extern "C" {

const char* e2eg_status_string(int32_t status) {
    switch (status) {
        case E2EG_OK: return "ok";
        case E2EG_ERR_INVALID_ARG: return "invalid argument";
        case E2EG_ERR_NULL_PTR: return "null pointer";
        case E2EG_ERR_BAD_DTYPE: return "unsupported dtype";
        case E2EG_ERR_CAPACITY: return "output capacity too small";
        case E2EG_ERR_OVERFLOW: return "size does not fit in int32";
        case E2EG_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
        case E2EG_ERR_HIP: return "HIP runtime error";
        case E2EG_ERR_BAD_INDEX: return "input id out of range";
        default: return "unknown status";
    }
}

const char* e2eg_last_error(void) { return e2eg::g_last_error; }

int32_t e2eg_version(void) { return 100; }

int32_t e2eg_profile_begin(int32_t capacity) {
    if (capacity < 0) return e2eg::fail(E2EG_ERR_INVALID_ARG, "profile_begin: negative capacity");
    e2eg::Profile& p = e2eg::g_profile;
    for (hipEvent_t e : p.start) (void)hipEventDestroy(e);
    for (hipEvent_t e : p.stop) (void)hipEventDestroy(e);
    p.start.clear();
    p.stop.clear();
    p.capacity = capacity;
    p.active = true;
    return E2EG_OK;
}

int32_t e2eg_profile_end(float* h_ms, int32_t h_capacity, int32_t* h_count) {
    e2eg::Profile& p = e2eg::g_profile;
    p.active = false;
    if (!h_count || (h_capacity > 0 && !h_ms)) return e2eg::fail(E2EG_ERR_NULL_PTR, "profile_end: null pointer");
    const int32_t count = (int32_t)(p.stop.size() < p.start.size() ? p.stop.size() : p.start.size());
    int32_t status = E2EG_OK;
    for (int32_t k = 0; k < count; ++k) {
        hipError_t err = hipEventSynchronize(p.stop[k]);
        float ms = 0.0f;
        if (err == hipSuccess) err = hipEventElapsedTime(&ms, p.start[k], p.stop[k]);
        if (err != hipSuccess) status = e2eg::fail(E2EG_ERR_HIP, "profile_end: %s", hipGetErrorString(err));
        if (k < h_capacity) h_ms[k] = ms;
    }
    *h_count = count;
    for (hipEvent_t e : p.start) (void)hipEventDestroy(e);
    for (hipEvent_t e : p.stop) (void)hipEventDestroy(e);
    p.start.clear();
    p.stop.clear();
    return status;
}

int32_t e2eg_profile_copy(void* d_dst, const void* d_src, size_t nbytes, void* stream) {
    if (!d_dst || !d_src) return e2eg::fail(E2EG_ERR_NULL_PTR, "profile_copy: null pointer");
    if (nbytes % 16 != 0 || !e2eg::aligned_to(d_dst, 16) || !e2eg::aligned_to(d_src, 16))
        return e2eg::fail(E2EG_ERR_INVALID_ARG, "profile_copy: pointers and size must be multiples of 16 bytes");
    if (nbytes == 0) return E2EG_OK;
    const size_t chunks = nbytes / 16;
    e2eg::copy_bytes16<<<dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, static_cast<hipStream_t>(stream)>>>(
        static_cast<uint4*>(d_dst), static_cast<const uint4*>(d_src), chunks);
    E2EG_LAUNCH_CHECK("copy_bytes16");
    return E2EG_OK;
}

}  // extern "C"
