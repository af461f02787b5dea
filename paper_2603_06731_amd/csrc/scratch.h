// Scratch memory of a stream, and the meeting of the workgroups that share one output tile.
//
// A problem with few output tiles leaves most of the chip idle unless several workgroups share a tile, each with its part of the
// contraction (or of the keys).  Their partial results are put into scratch memory; the workgroup that arrives last adds them, in
// the order of the parts and not of arrival, so that a call repeats itself bit for bit.  No workgroup waits for another one.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pbk {

constexpr size_t kScratchBytes = (size_t)8 << 20;    // partial results
constexpr int kScratchTickets = 4096;                // one per output tile; every launch leaves them at zero

struct Scratch {
    char* data;
    unsigned* tickets;
};

// The scratch memory of `stream` on device `dev` (the current one) for one launch, which has to go through launch_with() while this object lives.
// False where there is none: the caller then takes a kernel that needs none.
// - Not while the stream is being captured: a graph is replayed on any stream, and next to eager work on this one.
// - Not for the handles that stand for another stream in each thread, and not for a stream of another device.
// - Up to kScratchStreams streams per device; another one takes over the memory that has been idle longest, if any is idle.
// A handle says little about a stream: it may come back with another one after hipStreamDestroy, which need not wait for the work of the
// first.  So every launch records an event, and the next one with the same memory waits for it on the device, which on one and the same stream
// is no wait.  The null stream is always the same, and does without.
// How the event is recorded: behind the launch, where the launches before have ended, and otherwise as the launch's stop event.  In a stream of launches of
// 2.5 us, one takes 6.4 us with hipEventRecord and 4.0 with a stop event (55 us: 58 and 55), but where each is waited for, the stop event costs 2 to 5 us
// and hipEventRecord nothing.  Attention 29 x 4 x 1959, D = 128, without events, with them: 10.65 and 10.64 us in a stream, 22.3 and 22.9 waited for; 32 x 1024 x
// 1536: 7.10 and 7.14, 18.8 and 19.5.
struct ScratchEntry;
class ScratchUse {
public:
    ScratchUse(int dev, hipStream_t stream);
    ~ScratchUse();
    ScratchUse(const ScratchUse&) = delete;
    ScratchUse& operator=(const ScratchUse&) = delete;
    explicit operator bool() const { return entry != nullptr; }
    Scratch mem() const;
    hipError_t launch(const void* kern, dim3 grid, dim3 block, void** args, size_t lds_bytes, hipStream_t stream) const;
private:
    ScratchEntry* entry = nullptr;
    bool idle = false;              // the launches before have ended
};
constexpr int kScratchStreams = 32;

// hipLaunchKernel, of a kernel that uses scratch memory (`use`) or none (null)
hipError_t launch_with(const ScratchUse* use, const void* kern, dim3 grid, dim3 block, void** args, size_t lds_bytes, hipStream_t stream);

typedef __attribute__((ext_vector_type(4))) float scratch_f32x4;

// Partial results pass between compute units that do not share a cache: stores and loads of device scope (cache policy sc1), which go
// to the memory that all of them see, instead of ordinary ones with a write-back of the whole L2.  16 bytes a lane, whole lines a
// wave: as two 8-byte atomic stores a lane, 6 MB of partial results took some 10 us longer.
// Buffer over a workgroup-uniform base; offsets in bytes below 2^31.
constexpr int kScratchDeviceScope = 16;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t scratch_buffer(const void* base) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)0x80000000u, 0x00020000);
}
__device__ __forceinline__ void scratch_put(__amdgpu_buffer_rsrc_t buf, int offset, scratch_f32x4 v) {
    typedef __attribute__((ext_vector_type(4))) unsigned u4;
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), buf, offset, 0, kScratchDeviceScope);
}
__device__ __forceinline__ scratch_f32x4 scratch_get(__amdgpu_buffer_rsrc_t buf, int offset) {
    return __builtin_bit_cast(scratch_f32x4, __builtin_amdgcn_raw_buffer_load_b128(buf, offset, 0, kScratchDeviceScope));
}

// Called by all threads of a workgroup after they have put their partial results: true in the workgroup that arrives last of
// `parts`, which then finds all of them in scratch memory.  `flag`: a word of LDS.
__device__ __forceinline__ bool scratch_last(unsigned* ticket, int parts, int* flag) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this thread's stores have arrived in memory
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned before = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *flag = before == (unsigned)(parts - 1);
        // nobody else comes to this ticket: the next launch finds it at zero
        if (before == (unsigned)(parts - 1)) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    asm volatile("" ::: "memory");
    return *flag != 0;
}

}  // namespace pbk
