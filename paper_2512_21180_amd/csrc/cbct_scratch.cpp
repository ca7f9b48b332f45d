// Library-owned device scratch, one buffer per device and use, reused across
// calls (see cbct_internal.h).  A call takes the buffer under a lock,
// makes its stream wait for the previous user's completion event, enqueues
// its work and records the event again before releasing the lock, so calls
// on different streams never overlap on the buffer.  The buffer grows (once,
// after the previous user has finished) when a call needs more; an outgrown
// buffer is freed unless a captured call used it, whose graph names it for as
// long as it may be replayed.
#include <hip/hip_runtime.h>

#include <mutex>

#include "cbct_internal.h"

namespace cbct {
namespace {

constexpr int kMaxDevices = 64, kUses = 2;

struct DevScratch {
    void *ptr = nullptr;
    size_t bytes = 0;
    bool captured = false;       // a graph may name the buffer
    hipEvent_t last = nullptr;   // completion of the latest user's work
};

std::mutex g_mutex[kMaxDevices * kUses];
DevScratch g_scratch[kMaxDevices * kUses];

}  // namespace

hipError_t scratch_acquire(size_t bytes, hipStream_t s, ScratchLease &lease, ScratchUse use)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return e;
    if (dev < 0 || dev >= kMaxDevices)
        return hipErrorInvalidDevice;
    lease.slot = dev * kUses + use;
    lease.lock = std::unique_lock<std::mutex>(g_mutex[lease.slot]);
    DevScratch &S = g_scratch[lease.slot];
    if (!S.last) {
        e = hipEventCreateWithFlags(&S.last, hipEventDisableTiming);
        if (e != hipSuccess)
            return e;
    } else {
        e = hipStreamWaitEvent(s, S.last, 0);
        if (e != hipSuccess)
            return e;
    }
    if (S.bytes < bytes) {
        if (S.ptr) {
            e = hipEventSynchronize(S.last);
            if (e != hipSuccess)
                return e;
            e = S.captured ? hipSuccess : hipFree(S.ptr);
            S.ptr = nullptr;
            S.bytes = 0;
            S.captured = false;
            if (e != hipSuccess)
                return e;
        }
        e = hipMalloc(&S.ptr, bytes);
        if (e != hipSuccess) {
            S.ptr = nullptr;
            return e;
        }
        S.bytes = bytes;
    }
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) != hipSuccess)
        (void)hipGetLastError();   // the null stream beside another stream's capture
    else if (cap != hipStreamCaptureStatusNone)
        S.captured = true;
    lease.ptr = S.ptr;
    return hipSuccess;
}

hipError_t scratch_release(hipStream_t s, ScratchLease &lease)
{
    hipError_t e = hipSuccess;
    if (lease.slot >= 0 && g_scratch[lease.slot].last)
        e = hipEventRecord(g_scratch[lease.slot].last, s);
    lease.ptr = nullptr;
    lease.slot = -1;
    if (lease.lock.owns_lock())
        lease.lock.unlock();
    return e;
}

}  // namespace cbct
