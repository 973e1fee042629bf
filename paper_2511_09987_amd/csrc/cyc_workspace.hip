// cyc_workspace.hip -- device memory for the partial products of the k-in-space matmul and for the inverses of the triangular solve (see cyc_internal.h).
//
// Two sources.  WorkspaceHold: one hipMalloc'd buffer per (device, stream), so that calls on different streams never share
// one; grown when a call needs more, never shrunk, kept until the process ends.  The object keeps that buffer's lock while it
// lives, so that of two threads that call on one stream each has all its launches in the stream before the other's begin.
// static_workspace(): a fixed array in the library's own device image, for callers that must not allocate.
#include "cyc_internal.h"

#include <map>
#include <mutex>

namespace cyc {
namespace {

constexpr int MAX_DEVICES = 64;

// The fixed workspace of the allocation-free entry point: every device the library runs on holds its own copy
// until the process ends.  In host code the name below is only a handle for hipGetSymbolAddress; kernels are
// given the address obtained from it.
constexpr int64_t SCRATCH_BYTES = (int64_t)32 << 20;
static __device__ __align__(256) unsigned char scratch[SCRATCH_BYTES];

struct PerDevice {
    bool tried = false;
    void *scratch_ptr = nullptr;                        // this device's address of `scratch`
    struct Buffer {
        std::mutex lock;                                // of the call that uses it, and of the fields below
        void *ptr = nullptr;
        int64_t bytes = 0;
        bool captured = false;                          // some graph holds its address
        void *former = nullptr;                         // outgrown under a capture, which cannot free it
    };
    std::map<hipStream_t, Buffer> cache;
};
PerDevice g_dev[MAX_DEVICES];
std::mutex g_mutex;                                     // of g_dev; held for look-ups only

PerDevice *current_device()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return nullptr;
    return &g_dev[dev];
}

}  // namespace

void *static_workspace(int64_t *bytes)
{
    *bytes = SCRATCH_BYTES;
    std::lock_guard<std::mutex> hold(g_mutex);
    PerDevice *d = current_device();
    if (!d) return nullptr;
    if (!d->tried) {
        // once per device, with that device current: each device has the array at an address of its own
        d->tried = true;
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) == hipSuccess) d->scratch_ptr = p;
    }
    return d->scratch_ptr;
}

static void release(void *p)
{
    if (hipFree(p) != hipSuccess) (void)hipGetLastError();
}

bool is_capturing(hipStream_t s)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError();                            // (the caller is answered by what follows, not by the next launch check)
    return false;
}

void *WorkspaceHold::acquire(hipStream_t s, int64_t bytes)
{
    if (held_ || bytes <= 0) return nullptr;            // one buffer per object
    PerDevice::Buffer *slot = nullptr;
    try {
        std::lock_guard<std::mutex> lookup(g_mutex);
        if (PerDevice *d = current_device()) slot = &d->cache[s];   // (stays where it is: nothing is ever taken out of the map)
    } catch (...) {
    }
    if (!slot) return nullptr;
    slot->lock.lock();
    held_ = &slot->lock;
    const bool capturing = is_capturing(s);
    if (slot->bytes < bytes) {
        const int64_t want = (bytes + ((int64_t)1 << 20) - 1) >> 20 << 20;
        void *p = nullptr;
        // A buffer that a graph was captured with stays: the graph may be launched at any time.  Any other goes when the new one is
        // there, or before where there is no room for both.  (hipFree waits for the device, so nothing enqueued earlier still uses
        // it.  Under a capture it is left to a later call; the next to grow the buffer is one, as this one will be captured.)
        const bool old = slot->ptr && !slot->captured;
        if (capturing) {
            // an allocation is no part of the capture: this thread says so for its duration
            hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
            const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
            if (hipMalloc(&p, (size_t)want) != hipSuccess) p = nullptr;
            if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
            if (p && old) slot->former = slot->ptr;
        } else {
            if (slot->former) release(slot->former);
            slot->former = nullptr;
            const hipError_t e = hipMalloc(&p, (size_t)want);
            if (e != hipSuccess) p = nullptr;
            if (old && (p || e == hipErrorOutOfMemory)) {   // (other refusals, a capture elsewhere say, leave it as it is)
                release(slot->ptr);
                slot->ptr = nullptr;
                slot->bytes = 0;
                if (!p) (void)hipGetLastError();
                if (!p && hipMalloc(&p, (size_t)want) != hipSuccess) p = nullptr;
            }
        }
        if (!p) {
            (void)hipGetLastError();                    // (reported by the status of the call, or by nothing where it does without)
            return nullptr;
        }
        slot->ptr = p;
        slot->bytes = want;
        slot->captured = false;
    }
    slot->captured = slot->captured || capturing;
    return slot->ptr;
}

WorkspaceHold::~WorkspaceHold()
{
    if (held_) held_->unlock();
}

}  // namespace cyc
