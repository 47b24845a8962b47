// Shared host-side helpers of libprefixattn: error reporting, argument checks, and the
// device-side view of the flattened radix tree.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdint>
#include <cstdio>

#include "../../include/prefixattn.h"

namespace pa {

// Records a message for pa_last_error() and returns `code`.
int fail(int code, const char* fmt, ...);

#define PA_HIP(expr)                                                                         \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess) return pa::fail(PA_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

#define PA_REQUIRE(cond, ...)                                \
    do {                                                     \
        if (!(cond)) return pa::fail(PA_EINVAL, __VA_ARGS__); \
    } while (0)

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t elt_size(int dtype) { return dtype == PA_F32 ? 4 : 2; }
inline bool shape_ok(int Hq, int Hkv, int D) {
    return Hkv > 0 && Hq > 0 && Hq % Hkv == 0 && (D == 64 || D == 128);
}

// What the positional index of the flattened tree holds of a node (see DeviceTree).
struct __attribute__((aligned(32))) PathEntry {
    unsigned long long hash;     // of the token path up to and including the first token of the node's edge
    unsigned long long endhash;  // ... and the last one
    int32_t depth;               // depth of the first one; -1: the node is gone
    int32_t edge_start;          // index of the node's first edge token in edge_tok / edge_slot
    int32_t edge_len;
    int32_t parent;
};
struct PathSlot {
    uint32_t tag;  // path_tag of the node's (hash, depth)
    int32_t node;  // -1: empty; kGoneNode: the node was removed
};
constexpr int32_t kGoneNode = -2;

// Entry of the child table of the flattened tree: all that a walk needs to know of the child, so that a step of it is
// one round trip to memory.
struct __attribute__((aligned(32))) ChildEntry {
    unsigned long long key;      // (parent node id << 32) | first token of the child's edge; kEmptyKey, kDeletedKey
    int32_t node;
    int32_t edge_start;          // index of the first edge token in edge_tok / edge_slot
    unsigned long long endhash;  // hash of the path up to and including the edge's last token
    int32_t edge_len;
    int32_t pad;
};

// Flattened radix tree in device memory.
//   Every node but the empty virtual root 0 owns a run of edge tokens in edge_tok and, in parallel, the KV slot of each
//   of those tokens in edge_slot.
//   Children are found through one open-addressing hash table for the whole tree; linear probing, empty key = all
//   ones, capacity a power of two (mask = capacity - 1), at least 64.
struct DeviceTree {
    const int32_t* edge_tok;
    const int32_t* edge_slot;
    const ChildEntry* child;
    uint32_t ht_mask;
    // Second index, by position: a node is also reachable through the hash of the whole token path from
    // the root up to and including the FIRST token of its edge, together with the depth of that token.
    // A prompt can therefore look up every node boundary on its path at once from its own prefix hashes.
    //   path_slot: buckets of four slots (one read settles most lookups), the bucket from path_bucket, the next
    //              bucket where one is full; ph_mask = slots - 1, a power of two less one
    //   path[n]:   the node's entry (node 0: the root, endhash 0)
    const PathSlot* path_slot;
    const PathEntry* path;
    uint32_t ph_mask;
};

// A piece of the changes to a DeviceTree (tree_changes.hip): where its words go, counted from the start of the mirror in words
// of 32 bits.  The words of piece i lie at i * kChangeWords of the transfer buffer.
constexpr int kChangeWords = 256;
struct __attribute__((aligned(16))) ChangePiece {
    uint64_t to;
    uint32_t words, pad;
};
// piece, words: device addresses of pinned host memory.
int launch_apply_changes(const ChangePiece* piece, const uint32_t* words, int n, void* mirror, hipStream_t stream);

constexpr unsigned long long kEmptyKey = ~0ull;
constexpr unsigned long long kDeletedKey = ~0ull - 1;  // child table: an entry that was removed (never a real key)

// 64-bit mix (splitmix64 finaliser) used identically by the host builder and the device lookup.
__host__ __device__ inline uint32_t hash_key(unsigned long long k) {
    k ^= k >> 30; k *= 0xbf58476d1ce4e5b9ull;
    k ^= k >> 27; k *= 0x94d049bb133111ebull;
    k ^= k >> 31;
    return static_cast<uint32_t>(k);
}

// Polynomial hash of a token path: h(empty) = 0, h(p + t) = h(p) * kPathHashBase + (uint32(t) + 1), mod 2^64.
constexpr unsigned long long kPathHashBase = 0x9E3779B97F4A7C15ull;  // odd
__host__ __device__ inline unsigned long long path_hash_push(unsigned long long h, int32_t tok) {
    return h * kPathHashBase + (static_cast<unsigned long long>(static_cast<uint32_t>(tok)) + 1ull);
}
// 64 mixed bits of (path hash, depth): the low half picks the bucket, the high half is the tag kept in the slot.
__host__ __device__ inline unsigned long long path_mix(unsigned long long h, int32_t depth) {
    unsigned long long k = h ^ (static_cast<unsigned long long>(static_cast<uint32_t>(depth)) * 0xD6E8FEB86659FD93ull);
    k ^= k >> 30; k *= 0xbf58476d1ce4e5b9ull;
    k ^= k >> 27; k *= 0x94d049bb133111ebull;
    return k ^ (k >> 31);
}
__host__ __device__ inline uint32_t path_bucket(unsigned long long mix, uint32_t mask) { return static_cast<uint32_t>(mix) & mask & ~3u; }
__host__ __device__ inline uint32_t path_tag(unsigned long long mix) { return static_cast<uint32_t>(mix >> 32); }

// Pool layout: [page][K=0 | V=1][kv head][token in page][D] elements.
// Element index of the first element of (slot, which, head).
__host__ __device__ inline int64_t pool_row(int64_t slot, int which, int g, int Hkv, int D, int page_size) {
    int64_t page = slot / page_size;
    int64_t o = slot - page * page_size;
    return (((page * 2 + which) * Hkv + g) * page_size + o) * D;
}

// Per-kernel event timing (profile.cpp).  A ProfScope around a launch records a start/stop event
// pair on the stream while profiling is switched on, and does nothing otherwise.
// Byte offset, in the workspace of pa_extend_attention, of the two 64-bit counters of the clock probe (the header
// of the workspace is 256 bytes; the first 20 hold the work-list counts).
constexpr size_t kClockProbeOffset = 128;
bool prof_clock_enabled();

enum ProfKernel { kProfMatch = 0, kProfPlan, kProfExtend, kProfMerge, kProfExtendF32, kProfAppend, kProfGather, kProfCalibCopy, kProfCalibMfma, kProfKernels };
bool prof_begin(int kernel, hipStream_t stream, size_t* slot);
void prof_end(size_t slot, hipStream_t stream);
struct ProfScope {
    hipStream_t stream;
    size_t slot = 0;
    bool on;
    ProfScope(int kernel, hipStream_t s) : stream(s), on(prof_begin(kernel, s, &slot)) {}
    ~ProfScope() { if (on) prof_end(slot, stream); }
    ProfScope(const ProfScope&) = delete;
    ProfScope& operator=(const ProfScope&) = delete;
};

// ---- scratch memory that the workgroups of one match share (counters, summaries): sets in an array of the code object ----
// No two matches that can be in flight at once may meet in one set.  Matches on one stream follow one another, so a stream has
// sets of its own (two in turn: a new stream may be given the handle of one just destroyed), those of the stream that has not
// matched for longest going to a new one: matches in flight at once on more than 64 streams are excluded by the interface.  A
// captured call keeps its set for good, since its graph may be replayed at any time beside any other call (two replays of one
// captured call would meet in its output as well); where no such set is left, it takes the form without shared state.
constexpr int kStreamSets = 128;  // sets for calls on streams, two to a stream ...
constexpr int kGraphSets = 128;   // ... and for captured calls, one each
constexpr int kCallSets = kStreamSets + kGraphSets;
// The set for a call on `stream` of the current device (`fn` names the entry point in messages); *set = -1: none.
// *base: the device address of the array, looked up once per device from `symbol`.
int call_set_for(const char* fn, const void* symbol, hipStream_t stream, void** base, int* set);

}  // namespace pa

// Internal: device view of an uploaded tree (PA_ESTATE if it is stale or was never uploaded).
int pa_tree_device(const pa_tree* tree, const pa::DeviceTree** out);
