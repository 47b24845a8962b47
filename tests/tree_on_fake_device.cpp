// The tree's host code on a device made of host memory, for tests of its error paths without a GPU: the runtime calls that
// tree.cpp makes, of which any can be told to fail.  Copies and launches are queued and done when something waits for them.
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <string>

#include "../paper_2407_00023_amd/csrc/tree.cpp"

namespace {
std::deque<std::function<void()>> g_queue;
std::map<const unsigned char*, size_t> g_host, g_device;  // live allocations
std::map<hipEvent_t, size_t> g_recorded;                  // commands enqueued before the event
size_t g_done = 0, g_enqueued = 0;
std::string g_fail;   // the call that fails, and how many of them are let through first
int g_let_through = 0, g_bad = 0;

bool fails(const char* name) { return g_fail == name && g_let_through-- <= 0; }
void drain(size_t upto) {
    for (; g_done < upto; ++g_done) {
        g_queue.front()();
        g_queue.pop_front();
    }
}
void enqueue(std::function<void()> f) {
    g_queue.push_back(std::move(f));
    ++g_enqueued;
}
bool within(const std::map<const unsigned char*, size_t>& live, const void* p, size_t n) {
    const unsigned char* x = static_cast<const unsigned char*>(p);
    auto it = live.upper_bound(x);
    if (it == live.begin()) return false;
    --it;
    return x >= it->first && x + n <= it->first + it->second;
}
}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "made to fail"; }
hipError_t hipMalloc(void** p, size_t n) {
    if (fails("hipMalloc")) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    g_device[static_cast<unsigned char*>(*p)] = n;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    drain(g_enqueued);
    g_device.erase(static_cast<unsigned char*>(p));
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    if (fails("hipHostMalloc")) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    g_host[static_cast<unsigned char*>(*p)] = n;
    return hipSuccess;
}
hipError_t hipHostFree(void* p) {
    drain(g_enqueued);
    g_host.erase(static_cast<unsigned char*>(p));
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
    if (fails("hipHostGetDevicePointer")) return hipErrorInvalidValue;
    return *d = h, hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    if (fails("hipEventCreateWithFlags")) return hipErrorOutOfMemory;
    *e = reinterpret_cast<hipEvent_t>(std::malloc(1));
    return g_recorded[*e] = 0, hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) { return std::free(e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
    if (fails("hipEventRecord")) return hipErrorInvalidHandle;
    return g_recorded[e] = g_enqueued, hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    if (fails("hipEventSynchronize")) return hipErrorInvalidHandle;
    return drain(g_recorded[e]), hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return drain(g_enqueued), hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* h, size_t n, hipMemcpyKind, hipStream_t) {
    if (fails("hipMemcpyAsync")) return hipErrorInvalidValue;
    enqueue([=] {
        if (!within(g_device, d, n) || !within(g_host, h, n)) ++g_bad;
        else std::memcpy(d, h, n);
    });
    return hipSuccess;
}
}

int pa::launch_apply_changes(const ChangePiece* piece, const uint32_t* words, int n, void* mirror, hipStream_t) {
    if (fails("launch")) return pa::fail(PA_EHIP, "made to fail");
    enqueue([=] {
        if (!within(g_host, piece, sizeof(ChangePiece) * n) || !within(g_host, words, sizeof(uint32_t) * kChangeWords * n)) {
            ++g_bad;
            return;
        }
        for (int i = 0; i < n; ++i) {
            uint32_t* to = static_cast<uint32_t*>(mirror) + piece[i].to;
            if (piece[i].words > kChangeWords || !within(g_device, to, sizeof(uint32_t) * piece[i].words)) ++g_bad;
            else std::memcpy(to, words + static_cast<size_t>(i) * kChangeWords, sizeof(uint32_t) * piece[i].words);
        }
    });
    return PA_OK;
}

extern "C" void fake_fail(const char* call, int let_through) { g_fail = call, g_let_through = let_through; }
// Everything that is queued is done; 0: the device holds the tree as it is, 1: it does not, 2: a command was out of bounds.
extern "C" int fake_check(const pa_tree* tree) {
    drain(g_enqueued);
    if (g_bad) return 2;
    return !tree->uploaded || !tree->d_blob || std::memcmp(tree->d_blob, tree->h_stage, tree->flat.total) != 0;
}
