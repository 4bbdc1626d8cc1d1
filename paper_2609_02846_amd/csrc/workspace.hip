// Library-owned device workspaces (see Workspace in launch.hpp).
//
// A workspace that has to grow is replaced by a larger allocation and the
// old one is kept, never freed, until the process ends: launches already
// enqueued on the stream, or recorded in a captured graph, may still use it.
// Nothing here synchronizes.  A stream that is being captured cannot
// allocate (hipMalloc is not a capturable operation), so a call that would
// need a new or larger workspace during capture fails instead.
//
// A call that passes data from one launch to the next through a workspace
// holds it from before the first of them is enqueued until after the last:
// host threads that share a stream would otherwise enqueue one call's launch
// between another's, and the stream would run them in that order.
#include "launch.hpp"

#include <mutex>

namespace ue5m3 {

struct WorkspaceSlot {
    int dev = -1;
    hipStream_t stream = nullptr;
    std::mutex held;                             // by the call that uses the buffer
    void* ptr = nullptr;                         // ptr and bytes change under `held`
    size_t bytes = 0;
};

namespace {

// The slot of (kind, dev, s), created on first use unless s is capturing.
hipError_t find_slot(int kind, int dev, hipStream_t s, WorkspaceSlot** out) {
    static std::mutex mu;
    static WorkspaceSlot ws[kWsKinds][64];
    std::lock_guard<std::mutex> lock(mu);
    for (auto& x : ws[kind])
        if (x.dev == dev && x.stream == s) {
            *out = &x;
            return hipSuccess;
        }
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    const hipError_t e = hipStreamIsCapturing(s, &cs);
    if (e != hipSuccess) return e;
    if (cs != hipStreamCaptureStatusNone) return hipErrorStreamCaptureUnsupported;
    for (auto& x : ws[kind])
        if (x.dev < 0) {
            x.dev = dev;
            x.stream = s;
            *out = &x;
            return hipSuccess;
        }
    return hipErrorOutOfMemory;                  // more than 64 (device, stream) pairs
}

hipError_t grow(WorkspaceSlot& x, hipStream_t s, size_t bytes) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    hipError_t e = hipStreamIsCapturing(s, &cs);
    if (e != hipSuccess) return e;
    if (cs != hipStreamCaptureStatusNone) return hipErrorStreamCaptureUnsupported;
    void* p = nullptr;
    if ((e = hipMalloc(&p, bytes)) != hipSuccess) return e;
    x.ptr = p;                                   // a replaced buffer stays allocated
    x.bytes = bytes;
    return hipSuccess;
}

}  // namespace

hipError_t Workspace::take(int kind, hipStream_t s, size_t bytes, void** out) {
    if (kind < 0 || kind >= kWsKinds || slot_ != nullptr) return hipErrorInvalidValue;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    WorkspaceSlot* slot = nullptr;
    if ((e = find_slot(kind, dev, s, &slot)) != hipSuccess) return e;
    slot->held.lock();
    slot_ = slot;
    if (slot->bytes < bytes && (e = grow(*slot, s, bytes)) != hipSuccess) return e;
    *out = slot->ptr;
    return hipSuccess;
}

Workspace::~Workspace() {
    if (slot_ != nullptr) slot_->held.unlock();
}

}  // namespace ue5m3
