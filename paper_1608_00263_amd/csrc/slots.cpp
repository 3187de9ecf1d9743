// Pinned result slots of the synchronous calls (ResultSlot).
#include <hip/hip_runtime.h>

#include <mutex>

#include "internal.h"

namespace svi {

static std::mutex g_slot_mu;
static uint8_t *g_slots = nullptr;
static bool g_slots_tried = false;
static uint32_t g_slots_free = (1u << ResultSlot::COUNT) - 1;

ResultSlot::ResultSlot(size_t need, hipStream_t s) : stream(s) {
    if (need > (size_t)BYTES) return;
    std::lock_guard<std::mutex> lock(g_slot_mu);
    if (!g_slots_tried) {
        g_slots_tried = true;
        void *p = nullptr;
        if (hipHostMalloc(&p, (size_t)COUNT * BYTES, hipHostMallocPortable | hipHostMallocMapped) == hipSuccess)
            g_slots = (uint8_t *)p;
        else
            (void)hipGetLastError();   // the calls copy
    }
    if (!g_slots || !g_slots_free) return;
    const int i = __builtin_ctz(g_slots_free);
    g_slots_free &= ~(1u << i);
    ptr = g_slots + (size_t)i * BYTES;
}

void ResultSlot::release() {
    if (!ptr) return;
    std::lock_guard<std::mutex> lock(g_slot_mu);
    g_slots_free |= 1u << (((uint8_t *)ptr - g_slots) / BYTES);
    ptr = nullptr;
}

// A call that failed waits for what it had launched.  Where the wait fails, its
// kernel may still write to the slot, which stays out; not after a capture that
// the wait broke off, whose kernels never run.
ResultSlot::~ResultSlot() {
    if (!ptr) return;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamSynchronize(stream) == hipSuccess ||
        (hipStreamIsCapturing(stream, &cap) == hipSuccess && cap == hipStreamCaptureStatusInvalidated))
        release();
}

}  // namespace svi
