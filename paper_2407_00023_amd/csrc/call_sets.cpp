// Which set of the matcher's shared scratch memory a call may use (see common.h).
#include <mutex>

#include "common.h"

namespace pa {
namespace {
constexpr int kMaxDevices = 64;
struct DeviceSets {
    void* base = nullptr;
    struct { const void* stream; uint64_t used; unsigned calls; } of[kStreamSets / 2] = {};  // (used = 0: free)
    uint64_t clock = 0;
    int captured = 0;
};
std::mutex g_mu;
DeviceSets g_sets[kMaxDevices];
}  // namespace

int call_set_for(const char* fn, const void* symbol, hipStream_t stream, void** base, int* set) {
    *set = -1;
    int dev = -1;
    PA_HIP(hipGetDevice(&dev));
    PA_REQUIRE(dev >= 0 && dev < kMaxDevices, "%s: device ordinal %d not supported", fn, dev);
    const void* key = stream == hipStreamLegacy ? nullptr : static_cast<const void*>(stream);
    static thread_local char this_thread;
    if (stream == hipStreamPerThread) key = &this_thread;  // (one handle, a stream for every thread)
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (key != nullptr) PA_HIP(hipStreamIsCapturing(stream, &capture));  // (the default stream cannot be captured)
    std::lock_guard<std::mutex> lk(g_mu);
    DeviceSets& d = g_sets[dev];
    if (d.base == nullptr) {
        void* ptr = nullptr;
        PA_HIP(hipGetSymbolAddress(&ptr, symbol));
        PA_REQUIRE(ptr != nullptr, "%s: no address for the library's scratch array", fn);
        d.base = ptr;
    }
    *base = d.base;
    if (capture != hipStreamCaptureStatusNone) {
        if (d.captured < kGraphSets) *set = kStreamSets + d.captured++;
        return PA_OK;
    }
    int at = 0;
    for (int i = 0; i < kStreamSets / 2; ++i) {
        if (d.of[i].used != 0 && d.of[i].stream == key) {
            at = i;
            break;
        }
        if (d.of[i].used < d.of[at].used) at = i;
    }
    d.of[at].stream = key;
    d.of[at].used = ++d.clock;
    *set = 2 * at + static_cast<int>(d.of[at].calls++ & 1);
    return PA_OK;
}

}  // namespace pa
