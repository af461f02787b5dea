// Scratch memory per stream (scratch.h).
#include <atomic>
#include <mutex>
#include <hip/hip_ext.h>
#include "../../include/pbk.h"
#include "scratch.h"

namespace pbk {

struct ScratchEntry {
    hipStream_t stream;
    char* base;                     // tickets, then data
    unsigned long long id;          // of the allocation
    hipEvent_t done;                // of the last launch that uses the memory (not for the null stream)
    std::atomic<int> users;         // calls between finding the entry and their launch
    unsigned long long last;        // when it was found last
};

namespace {

constexpr int kDevices = 32;
constexpr size_t kTicketBytes = (size_t)kScratchTickets * sizeof(unsigned);

struct Pool { ScratchEntry entries[kScratchStreams]; int n; unsigned long long uses; };

std::mutex g_mutex;
Pool g_pools[kDevices];

// Allocating, or asking for an event, while some other thread captures a stream would disturb that capture.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    bool ok = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    ~RelaxedCapture() { if (ok) (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

bool ok(hipError_t e) {
    if (e == hipSuccess) return true;
    (void)hipGetLastError();
    return false;
}

unsigned long long allocation_id(char* base) {
    unsigned long long id = 0;
    return ok(hipPointerGetAttribute(&id, HIP_POINTER_ATTRIBUTE_BUFFER_ID, base)) ? id : 0;
}

// An entry for a stream that has none.
ScratchEntry* obtain(Pool& pool, hipStream_t stream) {
    RelaxedCapture relaxed;
    ScratchEntry* e = nullptr;
    if (pool.n == kScratchStreams) {
        // (never one that is at work: this stream would wait for a stranger, which might wait for what this one does next)
        for (ScratchEntry& x : pool.entries)
            if (x.stream && x.users.load() == 0 && (!e || x.last < e->last) && ok(hipEventQuery(x.done))) e = &x;
        if (e) e->stream = stream;
        return e;
    }
    e = &pool.entries[pool.n];
    void* base = nullptr;
    if (!ok(hipMalloc(&base, kTicketBytes + kScratchBytes))) return nullptr;
    e->stream = stream;
    e->base = (char*)base;
    e->id = allocation_id(e->base);
    if (ok(hipEventCreateWithFlags(&e->done, hipEventDisableTiming))) {
        if (ok(hipMemsetAsync(base, 0, kTicketBytes, stream)) && ok(hipEventRecord(e->done, stream))) {
            ++pool.n;
            return e;
        }
        (void)hipEventDestroy(e->done);
    }
    (void)hipFree(base);            // (waits for the clearing)
    return nullptr;
}

}  // namespace

ScratchUse::ScratchUse(int dev, hipStream_t stream) {
    if (dev < 0 || dev >= kDevices || stream == hipStreamPerThread || stream == hipStreamLegacy) return;
    // (the handle of a stream of another device: events and memory would be the wrong ones)
    hipDevice_t of = dev;
    if (stream && (!ok(hipStreamGetDevice(stream, &of)) || of != dev)) return;
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (!ok(hipStreamIsCapturing(stream, &status)) || status != hipStreamCaptureStatusNone) return;
    std::lock_guard<std::mutex> lock(g_mutex);
    Pool& pool = g_pools[dev];
    // hipDeviceReset takes memory and events of all entries away; other memory may lie there afterwards
    if (pool.n && allocation_id(pool.entries[0].base) != pool.entries[0].id) pool.n = 0;
    ScratchEntry* e = nullptr;
    for (int i = 0; i < pool.n && !e; ++i)
        if (pool.entries[i].stream == stream) e = &pool.entries[i];
    if (!e) e = obtain(pool, stream);
    if (!e) return;
    if (stream) {
        RelaxedCapture relaxed;
        idle = ok(hipEventQuery(e->done));
        if (!idle && !ok(hipStreamWaitEvent(stream, e->done, 0))) return;
    }
    e->users.fetch_add(1);
    e->last = ++pool.uses;
    entry = e;
}

ScratchUse::~ScratchUse() { if (entry) entry->users.fetch_sub(1); }

// (no entry, or the null stream's: nothing to record)
hipError_t ScratchUse::launch(const void* kern, dim3 grid, dim3 block, void** args, size_t lds_bytes, hipStream_t stream) const {
    if (!entry || !entry->stream) return hipLaunchKernel(kern, grid, block, args, lds_bytes, stream);
    if (!idle) return hipExtLaunchKernel(kern, grid, block, args, lds_bytes, stream, nullptr, entry->done, 0);
    const hipError_t e = hipLaunchKernel(kern, grid, block, args, lds_bytes, stream);
    return e == hipSuccess ? hipEventRecord(entry->done, stream) : e;
}

Scratch ScratchUse::mem() const { return entry ? Scratch{entry->base + kTicketBytes, (unsigned*)entry->base} : Scratch{}; }
hipError_t launch_with(const ScratchUse* use, const void* kern, dim3 grid, dim3 block, void** args, size_t lds_bytes, hipStream_t stream) {
    return use ? use->launch(kern, grid, block, args, lds_bytes, stream) : hipLaunchKernel(kern, grid, block, args, lds_bytes, stream);
}

}  // namespace pbk

extern "C" pbk_status pbk_release_scratch(void) {
    using namespace pbk;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return PBK_ERR_HIP;
    if (dev < 0 || dev >= kDevices) return PBK_OK;
    std::lock_guard<std::mutex> lock(g_mutex);
    Pool& pool = g_pools[dev];
    if (pool.n && allocation_id(pool.entries[0].base) != pool.entries[0].id) pool.n = 0;
    if (pool.n && hipDeviceSynchronize() != hipSuccess) return PBK_ERR_HIP;
    for (int i = 0; i < pool.n; ++i) {
        (void)hipEventDestroy(pool.entries[i].done);
        (void)hipFree(pool.entries[i].base);
    }
    pool.n = 0;
    return PBK_OK;
}
