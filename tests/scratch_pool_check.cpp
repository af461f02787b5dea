// The library's scratch memory per stream against a model of the runtime in which nothing ends unless it is told to: every two launches
// that use the same memory have to be ordered, whatever becomes of the streams.  Exits with 0 if they are.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
#include <vector>
#include "../paper_2603_06731_amd/csrc/scratch.h"

using pbk::ScratchUse;

#define CHECK(x) do { if (!(x)) { std::fprintf(stderr, "%s:%d: %s\n", __FILE__, __LINE__, #x); std::exit(1); } } while (0)

// ---- the model
struct Work { bool ended = false; std::set<int> after; char* memory = nullptr; };
static std::vector<Work> g_work;
static std::map<hipStream_t, std::set<int>> g_order;       // what the next work of the stream with this handle comes after
static std::map<hipEvent_t, int> g_events;                 // -> work
static std::map<char*, unsigned long long> g_memory;       // -> id
static unsigned long long g_ids = 0;
static hipError_t g_last = hipSuccess;
static bool g_capturing = false, g_full = false;
static int g_frees = 0;
static hipStream_t g_foreign = nullptr;                    // a stream of device 1

static int enqueue(hipStream_t s, char* memory) {
    Work w;
    w.after = g_order[s];
    w.memory = memory;
    if (memory)
        for (size_t i = 0; i < g_work.size(); ++i)
            CHECK(g_work[i].memory != memory || g_work[i].ended || w.after.count((int)i));
    const int id = (int)g_work.size();
    g_work.push_back(w);
    g_order[s].insert(id);
    return id;
}
static void end_all() { for (Work& w : g_work) w.ended = true; }
static void end_last() {                                   // and what it comes after
    g_work.back().ended = true;
    for (int i : g_work.back().after) g_work[i].ended = true;
}
static void destroy_and_create(hipStream_t s) { g_order[s].clear(); }     // the handle comes back, the work goes on

extern "C" {
hipError_t hipGetLastError() { const hipError_t e = g_last; g_last = hipSuccess; return e; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) { *d = s == g_foreign ? 1 : 0; return hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t) {
    if (g_full) return g_last = hipErrorOutOfMemory;
    *p = std::malloc(64);                       // (only its address is used)
    g_memory[(char*)*p] = ++g_ids;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    CHECK(g_memory.erase((char*)p) == 1);
    ++g_frees;
    return hipSuccess;
}
hipError_t hipPointerGetAttribute(void* data, hipPointer_attribute, hipDeviceptr_t p) {
    const auto at = g_memory.find((char*)p);
    if (at == g_memory.end()) return g_last = hipErrorInvalidValue;
    *(unsigned long long*)data = at->second;
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int, size_t, hipStream_t s) { enqueue(s, (char*)p); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    static char next;
    *e = (hipEvent_t)(&next + g_events.size() + 1);
    g_events[*e] = -1;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) { CHECK(g_events.count(e)); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { g_events[e] = enqueue(s, nullptr); return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e) {
    const int w = g_events[e];
    return w < 0 || g_work[w].ended ? hipSuccess : (g_last = hipErrorNotReady);
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    const int w = g_events[e];
    if (w >= 0) {
        g_order[s].insert(w);
        g_order[s].insert(g_work[w].after.begin(), g_work[w].after.end());
    }
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3, dim3, void** args, size_t, hipStream_t s) { enqueue(s, (char*)args[0]); return hipSuccess; }
hipError_t hipExtLaunchKernel(const void*, dim3, dim3, void** args, size_t, hipStream_t s, hipEvent_t, hipEvent_t stop, int) {
    g_events[stop] = enqueue(s, (char*)args[0]);
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceSynchronize() { end_all(); return hipSuccess; }
int pbk_release_scratch();
}

static char g_handles[256];
static hipStream_t stream(int i) { return (hipStream_t)(g_handles + i); }
static char* launch(const ScratchUse& use, hipStream_t s) {
    CHECK(use);
    void* args[] = {use.mem().tickets};                          // the start of the memory
    CHECK(pbk::launch_with(&use, nullptr, dim3(1), dim3(64), args, 0, s) == hipSuccess);
    return (char*)use.mem().tickets;
}
static char* call(hipStream_t s) { const ScratchUse use(0, s); return use ? launch(use, s) : nullptr; }

int main() {
    // a stream keeps its memory; another has other memory
    char* a = call(stream(0));
    char* null_stream = call(nullptr);
    CHECK(a && call(stream(0)) == a && null_stream && null_stream != a && call(nullptr) == null_stream);
    // the handle comes back while the first stream's work goes on
    for (int i = 0; i < 5; ++i) { destroy_and_create(stream(0)); CHECK(call(stream(0)) == a && call(stream(0)) == a); }
    // none for the handles of each thread's own stream, under capture, or on a device out of range
    CHECK(!call(hipStreamPerThread) && !call(hipStreamLegacy));
    g_capturing = true;
    CHECK(!call(stream(0)) && !call(stream(1)));
    g_capturing = false;
    CHECK(!ScratchUse(-1, stream(0)) && !ScratchUse(32, stream(0)));
    g_foreign = stream(0);                                       // the handle comes back with a stream of another device
    CHECK(!call(stream(0)));
    g_foreign = nullptr;
    // no memory: no scratch, and no error left behind
    g_full = true;
    CHECK(!call(stream(1)) && g_last == hipSuccess);
    g_full = false;

    // as many streams as there is memory for (stream(0) and the null stream have theirs)
    std::map<char*, int> owner;
    for (int i = 1; i < pbk::kScratchStreams - 1; ++i) CHECK(owner.emplace(call(stream(i)), i).second);
    CHECK(g_memory.size() == (size_t)pbk::kScratchStreams);
    // one more: nothing while all are at work, then what has been idle longest, but not what a call is about to use
    CHECK(!call(stream(100)) && g_last == hipSuccess);
    end_last();
    char* last = call(stream(100));
    CHECK(last && owner[last] == pbk::kScratchStreams - 2);
    end_all();
    call(stream(0));
    end_all();
    char* b = call(stream(101));                                 // (stream(1)'s was used longest ago but for the null stream's, which stays)
    CHECK(b && b != a && b != last && owner[b] == 1);
    {
        end_all();
        const ScratchUse held(0, stream(0));
        call(stream(100)), call(stream(101));
        for (int i = 2; i < pbk::kScratchStreams - 2; ++i) call(stream(i));
        CHECK(!call(stream(102)));                               // idle is what the call in between is about to use, and nothing else
        CHECK(launch(held, stream(0)) == a);
    }
    end_all();
    CHECK(g_memory.size() == (size_t)pbk::kScratchStreams);
    // streams that come and go
    for (int i = 0; i < 100; ++i) { CHECK(call(stream(120 + i))); if (i % 3 == 0) end_all(); }
    CHECK(g_memory.size() == (size_t)pbk::kScratchStreams && call(nullptr) == null_stream);

    // after hipDeviceReset: nothing of what was there is used or given back
    std::set<char*> old;
    for (auto& m : g_memory) old.insert(m.first);
    end_all();
    g_memory.clear();
    char* c = call(stream(0));
    CHECK(c && !old.count(c) && g_memory.size() == 1 && g_frees == 0);
    g_memory[c] = ++g_ids;                                       // other memory at the same address
    char* d = call(stream(0));
    CHECK(d && d != c);
    // a call that obtains memory and does not come to its launch: the memory is still being cleared when the handle comes back
    CHECK(ScratchUse(0, stream(1)));
    destroy_and_create(stream(1));
    CHECK(call(stream(1)));
    // given back, and obtained again
    CHECK(pbk_release_scratch() == 0 && g_frees == 2 && g_memory.size() == 1 && call(stream(0)));
    return 0;
}
