// Batched longest-prefix match of prompts against the flattened radix tree.
//
// Algorithm 1 of the paper starts by matching the request to the radix tree and taking
// cached_len = the sum of the matched lengths along the path; Sec. 3.2 defines the match as
// running from the beginning until no match exists, a partly matched node counting for the
// tokens that do match.  A request's walk has two forms.  Most paths are a few nodes long: the first
// nodes are found one after the other through the (parent, first token) table, WITHOUT comparing their edges
// (one round trip to memory per node), and then all of their tokens are compared with the prompt at once.  Where the path
// goes on, windows of prompt positions are resolved at once through a positional index (below), in small batches with a
// workgroup per window.
//
// What bounds it: the number of dependent round trips to memory and, in large batches, how many requests are in flight
// on a compute unit.  Hence workgroups of 256 threads with 10 (windows of 512 positions) to 19 KB of LDS.  Measured on a
// 256-unit chip against workgroups of 1,024 threads that compared every edge before they looked for the next one: 4,096
// prompts of 2,650 tokens over four edges of 512 each 150 -> 24 us; 64 prompts over three or four edges 18 -> 9; a path of
// 541 nodes (32 prompts of 8,483 tokens) 41 -> 23; one long edge of 16,384 tokens (16 prompts) 24 -> 13; the smallest call
// 13 -> 5.
#include "common.h"

namespace pa {

struct Child {
    int32_t node, start, len;    // (start: index of the first edge token in the tree's arrays)
    unsigned long long endhash;
};

// Child of `node` whose edge starts with `tok`; false if there is none.  Executed by full waves; every lane gets the result.
__device__ __forceinline__ bool find_child(const DeviceTree& t, int32_t node, int32_t tok, Child& c) {
    const unsigned long long key =
        (static_cast<unsigned long long>(static_cast<uint32_t>(node)) << 32) | static_cast<uint32_t>(tok);
    const uint32_t sub = threadIdx.x & 15;  // (sixteen entries per probe, the same ones in each quarter of the wave)
    uint32_t h = hash_key(key) & t.ht_mask;
    // The table is at most half full, so an empty entry ends the probe sequence soon.
    for (uint32_t probed = 0; probed <= t.ht_mask; probed += 16) {
        const uint4* e = reinterpret_cast<const uint4*>(t.child + ((h + sub) & t.ht_mask));
        const uint4 lo = e[0], hi = e[1];
        const unsigned long long k = (static_cast<unsigned long long>(lo.y) << 32) | lo.x;
        const unsigned hit = static_cast<unsigned>(__ballot(k == key)) & 0xFFFFu;
        if (hit) {
            const int src = __ffs(hit) - 1;
            auto lane = [&](uint32_t x) { return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x), src)); };
            c.node = static_cast<int32_t>(lane(lo.z));
            c.start = static_cast<int32_t>(lane(lo.w));
            c.endhash = (static_cast<unsigned long long>(lane(hi.y)) << 32) | lane(hi.x);
            c.len = static_cast<int32_t>(lane(hi.z));
            return true;
        }
        if (__ballot(k == kEmptyKey)) return false;
        h = (h + 16) & t.ht_mask;
    }
    return false;
}

// ---------------------------------------------------------------------------------------------------
// Windows: all node boundaries of a stretch of the prompt's path at once, instead of one node after the
// other (a path through a tree with many branch points has hundreds of nodes).
//
// The tree carries a second index: (hash of the token path up to and including the first token of a node's
// edge, depth of that token) -> node.  A window is the kWinP prompt positions from the current match position
// on.  The workgroup forms the prefix hash of the prompt at every position of the window (a scan seeded with
// the stored hash of the path that ends at the current node) and looks every (hash, position) up: a hit
// NOMINATES a node whose edge would start there.  The nominated nodes are the path's nodes in order, hash
// collisions apart, so every position of the window belongs to the last node nominated at or before it, and
// all positions are compared with their nodes' edges in one round trip, the slots copied along.  The match in
// the window ends at the first position whose token differs or that no edge covers, or at the first nominated
// node that is not linked to the one before it ("that one ends where this one starts, and is this one's
// parent"), starting from position 0, which holds the child found exactly.  Whatever ends it, the loop head
// takes over from the last confirmed position with an exact child lookup where one is needed, so the result
// never depends on the hash being free of collisions: a collision can only cost time.
// What bounds it: four dependent round trips to memory (tokens, buckets of the index, entries of the nominated
// nodes, edges) and five barriers, about 8 us with the caches cold.
// ---------------------------------------------------------------------------------------------------
constexpr int kWalk = 16;         // nodes found one after the other before windows are opened, at most ...
constexpr int kWalkFree = 4;      // ... and beyond this many only while their edges hold kWalkEdge tokens on average: a node
constexpr int kWalkEdge = 128;    // costs one round trip, 0.8 us, a window four of them and several barriers, 8 us
constexpr int kSweep = 8;         // tokens per thread and round of the comparison of what the walk found
// kT = threads per workgroup; kPos = prompt positions per thread and window (consecutive ones), kWinP = kT * kPos positions
// per window
constexpr int kDirectEdge = 256;  // a next edge at least this long is compared directly, without opening a window
constexpr int kSplitSweep = 4096; // a walked path longer than this is compared by several workgroups, where a request has them

// Several workgroups per request (batches of up to kMultiMaxB).  The hashes of a window depend on the prompt alone, so the
// windows of a long path need not wait for one another.  All workgroups of a request make the same walk of kWalk nodes; if
// the path ends there the first one compares it and the others leave (one longer than kSplitSweep is compared by as many as
// make the shares 2,048 tokens or fewer, if there are so many; the last of them to finish takes the first mismatch).
// Otherwise the windows lie at fixed places [k * kWinP, (k + 1) * kWinP): workgroup 0 goes on walking as long as it begins a
// step inside the window where the walk stands, workgroup w takes the w-th window after that one, from the first node
// nominated in it, its entry hash formed from the prompt's tokens before the window - and leaves a summary: where its chain
// begins, the parent its first node names, and where the walk would stand after it.  The workgroup that finishes last (a
// counter per request) joins the summaries in order - a window's chain is accepted if it begins exactly where the walk stands
// and names the walk's node as parent: the same exact link as inside a window - and walks on alone from where the chain of
// accepted windows ends.  Nobody waits for anybody.  Slot ids that a window writes before it is accepted are those of a chain of linked nodes, confirmed
// token by token, behind a first node whose path hashes like the prompt; where that node proves to be none of the path, the
// last workgroup writes what the chain has written, and all that lies behind it, again: its writes come after all others.
constexpr int kMaxW = 16;        // workgroups per request at most; a longer path's rest is walked by the last one
constexpr int kMultiMaxB = 256;  // batches of up to this many requests take this form
constexpr int kMultiWgs = 1024;  // ... with up to this many workgroups (four on a compute unit)
constexpr int kWideMaxB = 1024;  // one workgroup per request: wide windows up to this many requests
struct MatchSummary {
    int32_t f_pos, f_parent;     // position of the first node of the chain (-1: none), the parent it names
    int32_t exit_pos, exit_cur;  // matched length and current node after the chain
    int32_t done;                // 1: the walk ends there (mismatch inside an edge, or no child)
    int32_t last_es, last_start; // the chain's last edge: index of its first token in the tree's arrays, its position
    int32_t pad;
};
struct MatchScratch {
    MatchSummary sum[kMultiWgs];   // workgroup w of request r: r * (workgroups per request) + w
    unsigned counter[kMultiMaxB];  // workgroups of the request that have finished; back to 0 with the last one
};

// Workgroup barrier that orders LDS accesses only.  __syncthreads() also waits until the global stores of
// the slot ids are acknowledged, a long round trip the matcher has no reason to wait for.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int kT, int kPos, bool kMulti>
__global__ __launch_bounds__(kT, kPos == 4 ? 4 : 8) void match_prefixes_kernel(DeviceTree t, const int32_t* __restrict__ tokens,
                                                            const int32_t* __restrict__ offsets,
                                                            int32_t* __restrict__ prefix_len,
                                                            int32_t* __restrict__ slot_idx, int n_req, MatchScratch* scratch) {
    constexpr int kWinP = kT * kPos;
    constexpr int kWaves = kT / 64;
    constexpr int kLogT = 8;
    static_assert(kT == 1 << kLogT, "256 threads");
    // The first kStage tokens of the prompt during the walk; afterwards, per window position: {nominated node or -1, its
    // parent, its edge length, index of its first edge token}
    constexpr int kStage = 4 * kWinP;
    __shared__ __attribute__((aligned(16))) int32_t s_raw[kStage];
    int32_t* const s_tok = s_raw;
    int4* const s_rec = reinterpret_cast<int4*>(s_raw);
    __shared__ int16_t s_cv[kWinP];      // per window position: the last nominated position at or before it, -1: none
    __shared__ unsigned long long s_wtot[kWaves];
    __shared__ int32_t s_wmax[kWaves];
    __shared__ int32_t s_wpos[kWalk], s_wes[kWalk];  // the walk: where an edge begins; what to add to a position for its place in the tree's arrays
    __shared__ int32_t s_red[2][kWaves], s_red2[2][kWaves];
    __shared__ int32_t s_last_one;  // this workgroup is the last of its request to finish
    __shared__ int32_t s_sum[kMulti ? kMaxW * 8 : 1];  // ... and then holds the request's summaries here
    // (the records of a thread's consecutive positions lie kT apart: neighbouring threads then use neighbouring words)
    auto at_rec = [](int rel) __attribute__((always_inline)) { return (rel % kPos) * kT + rel / kPos; };
    // (multi-workgroup form: the first workgroups of the grid are the requests' workgroups 0, which have the longest way
    // to go, then come all workgroups 1, and so on)
    const int n_w = kMulti ? gridDim.x / n_req : 1;
    const int r = kMulti ? blockIdx.x % n_req : blockIdx.x;
    const int w = kMulti ? blockIdx.x / n_req : 0;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int32_t base = offsets[r];
    const int32_t n = offsets[r + 1] - base;
    const int32_t* __restrict__ prompt = tokens + base;
    int32_t* __restrict__ out_slots = slot_idx + base;
    int red_round = 0;
    // minimum over the workgroup, in every thread
    auto wg_min = [&](int32_t x) __attribute__((always_inline)) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) x = min(x, __shfl_xor(x, off));
        if (lane == 0) s_red[red_round & 1][wave] = x;
        lds_barrier();
        int32_t m = INT32_MAX;
#pragma unroll
        for (int v = 0; v < kWaves; ++v) m = min(m, s_red[red_round & 1][v]);
        ++red_round;
        return m;
    };
    auto put_slot = [&](int32_t p, int32_t v, bool through) __attribute__((always_inline)) {
        // Slot ids written by a lone window go straight through to memory (stores of device scope leave no dirty line in
        // this XCD's L2), so that waiting for them to be acknowledged is all it takes for the last workgroup's own writes to
        // come after them; a fence of device scope would write the whole L2 back and costs 100 us and more here.  (The walk
        // from the root writes the slots of nodes that are linked to it, up to where they differ from the prompt: final
        // ones, or past the end of the match.)
        if (kMulti && through) __hip_atomic_store(out_slots + p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else out_slots[p] = v;
    };
    // Compares tokens [from, lim) of the edge at es with the prompt from `at` on (token k of the edge against prompt[at + k]) and
    // copies their slots; the first that differs, or lim.
    auto compare_run = [&](int32_t es, int32_t at, int32_t from, int32_t lim, bool through) __attribute__((always_inline)) {
        for (int32_t c0 = from; c0 < lim; c0 += kT * 4) {
            int32_t et[4], pt[4], sl[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int32_t k = min(c0 + u * kT + tid, lim - 1);
                et[u] = t.edge_tok[es + k];
                pt[u] = prompt[at + k];
                sl[u] = t.edge_slot[es + k];
            }
            int32_t mine = INT32_MAX;
#pragma unroll
            for (int u = 3; u >= 0; --u) {
                const int32_t k = c0 + u * kT + tid;
                if (k < lim) {
                    put_slot(at + k, sl[u], through);  // entries past the final match are unspecified by contract
                    if (et[u] != pt[u]) mine = k;
                }
            }
            const int32_t first = wg_min(mine);
            if (first != INT32_MAX) return first;
        }
        return lim;
    };

    int32_t pos = 0, cur = 0;        // matched so far; node whose edge ends at pos
    bool done = n <= 0;
    int32_t last_es = 0, last_start = 0;  // the last edge walked: its first token in the tree's arrays, its position
    int32_t walked = 0;  // where the walk stands, the same in all workgroups of the request
    // ---- the walk: up to kWalk nodes, edges taken on trust ----
    if (!done) {
        const int32_t tok0 = prompt[0];
        if (kMulti && w > 0 && n <= kWinP) return;  // (no window for this workgroup whatever the walk finds)
        if (kMulti) {
#pragma unroll 4
            for (int32_t p = tid; p < min(n, kStage); p += kT) s_tok[p] = prompt[p];
        }
        int32_t tok = tok0;
        int nk = 0;
        while (nk < kWalk && (nk < kWalkFree || pos >= nk * kWalkEdge)) {
            Child c;
            if (!find_child(t, cur, tok, c)) {
                done = true;
                break;
            }
            if (tid == 0) {
                s_wpos[nk] = pos;
                s_wes[nk] = c.start - pos;
            }
            last_es = c.start;
            last_start = pos;
            if (kMulti && nk == 0) lds_barrier();  // (the staged tokens, first looked at below)
            ++nk;
            cur = c.node;
            if (c.len >= n - pos) {  // the prompt ends inside this edge or with it
                pos = n;
                done = true;
                break;
            }
            pos += c.len;
            tok = __builtin_amdgcn_readfirstlane(kMulti && pos < kStage ? s_tok[pos] : prompt[pos]);
        }
        walked = pos;
        // ---- compare the walked edges with the prompt and copy their slots ----
        const int n_sw = kMulti && done && pos > kSplitSweep ? min(n_w, (pos + kT * kSweep - 1) / (kT * kSweep)) : 1;
        if (kMulti && done && w >= n_sw) return;
        lds_barrier();  // (the list of nodes is complete; the staged tokens make room for the records of a window)
        if (w < n_sw) {
            const int32_t share = ((pos + n_sw - 1) / n_sw + 63) & ~63;
            const int32_t lo = w * share, hi = min(pos, lo + share);
            int32_t mine = INT32_MAX;
            for (int32_t c0 = lo; c0 < hi; c0 += kT * kSweep) {
                int32_t et[kSweep], pt[kSweep], sl[kSweep];
                int32_t at[kSweep];
#pragma unroll
                for (int u = 0; u < kSweep; ++u) {
                    const int32_t p = min(c0 + u * kT + tid, hi - 1);
                    pt[u] = prompt[p];
                    at[u] = s_wes[0] + p;
                }
                for (int k = 1; k < nk; ++k) {
                    const int32_t from = s_wpos[k], es = s_wes[k];
#pragma unroll
                    for (int u = 0; u < kSweep; ++u) {
                        const int32_t p = min(c0 + u * kT + tid, hi - 1);
                        at[u] = p >= from ? es + p : at[u];
                    }
                }
#pragma unroll
                for (int u = 0; u < kSweep; ++u) {
                    et[u] = t.edge_tok[at[u]];
                    sl[u] = t.edge_slot[at[u]];
                }
#pragma unroll
                for (int u = kSweep - 1; u >= 0; --u) {
                    const int32_t p = c0 + u * kT + tid;
                    if (p < hi) {
                        out_slots[p] = sl[u];  // entries past the final match are unspecified by contract
                        if (et[u] != pt[u]) mine = p;
                    }
                }
                if (__any(mine != INT32_MAX)) break;  // (this wave's later positions lie behind the mismatch)
            }
            int32_t first = wg_min(mine);
            if (kMulti && n_sw > 1) {
                if (tid == 0) {
                    __hip_atomic_store(&scratch->sum[r * n_w + w].f_pos, first, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    s_last_one = atomicInc(&scratch->counter[r], n_sw - 1) == static_cast<unsigned>(n_sw - 1);
                }
                lds_barrier();
                if (!s_last_one) return;
                if (tid < n_sw) mine = __hip_atomic_load(&scratch->sum[r * n_w + tid].f_pos, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                first = wg_min(mine);
            }
            if (done || (!kMulti && first < pos)) {  // the path ends here, or sooner
                if (tid == 0) prefix_len[r] = min(first, pos);
                return;
            }
            if (first < pos) {
                pos = first;
                done = true;
            }
        }
    }

    if (n <= 0) {
        if (w == 0 && tid == 0) prefix_len[r] = 0;
        return;
    }

    // What this workgroup's pass over the loop below is: 0 the whole walk (the only pass of the single-workgroup form, the
    // last workgroup's second pass otherwise), 1 the walk as long as it begins a step inside the window where it stands, 2 one
    // window at a fixed place.
    const int32_t win0 = walked / kWinP;  // the window in which the walk stands
    // (a request takes one workgroup per window that is left of its prompt; the others leave at once)
    const int n_wg = !kMulti ? 1 : max(1, min(n_w, (n + kWinP - 1) / kWinP - win0));
    if (w >= n_wg) return;
    int role = n_wg == 1 ? 0 : w == 0 ? 1 : 2;
    const int32_t first_end = (win0 + 1) * kWinP;
    // With b = B^kPos (a thread's positions hash as one step of the scan): b^(2^k), and b^lane
    unsigned long long bp2[7];
    bp2[0] = 1ull;
#pragma unroll
    for (int i = 0; i < kPos; ++i) bp2[0] *= kPathHashBase;
#pragma unroll
    for (int k = 1; k < 7; ++k) bp2[k] = bp2[k - 1] * bp2[k - 1];
    unsigned long long bpow_lane = 1ull;
#pragma unroll
    for (int k = 0; k < 6; ++k)
        if (lane >> k & 1) bpow_lane *= bp2[k];
    int32_t f_pos = role == 2 ? -1 : 0, f_parent = 0;
    unsigned long long seed = 0ull;  // role 2: hash of the prompt before the window
    bool active = true;
    if (kMulti && role == 2) {
        pos = (win0 + w) * kWinP;
        // The hash of the pos = kT * L tokens before the window is sum_j (token_j + 1) B^(pos - 1 - j).  Thread t takes
        // the tokens t, t + kT, t + 2 kT, ... (neighbouring lanes read neighbouring tokens): its share is
        // B^(kT - 1 - t) times a fold of its L tokens with B^kT as the step; the shares are then joined in thread
        // order, a scan with B as the step.
        const int L = pos / kT;
        unsigned long long big = kPathHashBase;  // B^kT
#pragma unroll
        for (int k = 0; k < kLogT; ++k) big *= big;
        unsigned long long c = 0ull;
        constexpr int kAhead = 16;  // (loads in flight per thread)
        for (int i0 = 0; i0 < L; i0 += kAhead) {
            int32_t tk[kAhead];
#pragma unroll
            for (int i = 0; i < kAhead; ++i) tk[i] = prompt[min(i0 + i, L - 1) * kT + tid];
#pragma unroll
            for (int i = 0; i < kAhead; ++i)
                if (i0 + i < L) c = c * big + (static_cast<unsigned long long>(static_cast<uint32_t>(tk[i])) + 1ull);
        }
        unsigned long long step = kPathHashBase;  // B^(2^k)
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const unsigned long long left = __shfl_up(c, 1u << k);
            if (lane >= (1 << k)) c = left * step + c;
            step *= step;
        }
        if (lane == 63) s_wtot[wave] = c;
        lds_barrier();
        for (int v = 0; v < kWaves; ++v) seed = seed * step + s_wtot[v];  // (step = B^64 by now)
        lds_barrier();
    }
    bool direct = false;  // the next edge is to be compared directly, whatever its length
    for (;;) {
    while (active && !done && pos < n && (role != 1 || pos < first_end)) {
        // The next node, found exactly (child table keyed by parent and first token).  A long edge is compared
        // right away by the whole workgroup; a short one opens a window.  (A lone window has no node to start from: its
        // first node is whatever the hashes nominate first.)
        unsigned long long h = seed;  // hash of prompt[0 .. pos)
        Child child{-1, 0, 0, 0ull};
        if (role != 2) {
            h = t.path[cur].endhash;  // (asked for ahead of its use below)
            if (!find_child(t, cur, prompt[pos], child)) {
                done = true;
                break;
            }
            if (direct || child.len >= kDirectEdge) {
                direct = false;
                last_es = child.start;
                last_start = pos;
                const int32_t m = compare_run(child.start, pos, 0, min(child.len, n - pos), false);
                pos += m;
                if (m < child.len) {  // mismatch inside the edge, or the prompt ended inside it
                    done = true;
                    break;
                }
                cur = child.node;
                continue;
            }
        }
        const int32_t w0 = pos;
        // (workgroup 0 of several nominates nodes inside its first window only, so that its chain ends where the next
        // workgroup's begins)
        const int32_t n_nom = role == 1 ? min(n, first_end) : n;
        const int32_t rel0 = tid * kPos;  // this thread's first position in the window; its positions are rel0 + i
        // ---- A. prefix hashes of the window: inclusive scan of x -> x * B + (token + 1).  A thread folds its own
        // positions, then the scan runs over threads with B^kPos as the step: within a wave by shuffles, then
        // across waves ----
        unsigned long long loc[kPos];  // hash of this thread's positions 0 .. i
        {
            unsigned long long run = 0ull;
#pragma unroll
            for (int i = 0; i < kPos; ++i) {
                const int32_t p = w0 + rel0 + i;
                run = run * kPathHashBase + (p < n ? static_cast<unsigned long long>(static_cast<uint32_t>(prompt[p])) + 1ull : 0ull);
                loc[i] = run;
            }
        }
        unsigned long long c = loc[kPos - 1];
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const unsigned long long left = __shfl_up(c, 1u << k);
            if (lane >= (1 << k)) c = left * bp2[k] + c;
        }
        if (lane == 63) s_wtot[wave] = c;
        unsigned long long excl = __shfl_up(c, 1);  // hash of the wave's positions before this thread's
        if (lane == 0) excl = 0ull;
        lds_barrier();
        unsigned long long before = h;  // hash of everything before this wave's positions
        for (int v = 0; v < wave; ++v) before = before * bp2[6] + s_wtot[v];
        const unsigned long long upto = before * bpow_lane + excl;  // hash of prompt[0 .. w0 + rel0)
        // ---- B. nominations: nodes whose edge starts at p after exactly this prefix (by hash) ----
        // A bucket of the index (four slots) is one 32-byte read and settles its position unless it is full; the reads of all
        // of a thread's positions are in flight together, and so are those of the entries that the hits name.
        int32_t lastc = -1;  // the last nominated position among the thread's own
        {
            unsigned long long hps[kPos];
            uint32_t tags[kPos], ats[kPos];
            int32_t nd[kPos];
            unsigned pending = 0;  // positions not settled yet
            unsigned long long bi = 1ull;
#pragma unroll
            for (int i = 0; i < kPos; ++i) {
                bi *= kPathHashBase;
                const int32_t p = w0 + rel0 + i;
                hps[i] = upto * bi + loc[i];  // hash of prompt[0 .. p]
                const unsigned long long mix = path_mix(hps[i], p);
                tags[i] = path_tag(mix);
                ats[i] = path_bucket(mix, t.ph_mask);
                nd[i] = -1;
                if (p < n_nom) pending |= 1u << i;
            }
            for (uint32_t probed = 0; pending != 0 && probed <= t.ph_mask; probed += 4) {
                uint4 a[kPos], b[kPos];
#pragma unroll
                for (int i = 0; i < kPos; ++i) {
                    const uint4* e = reinterpret_cast<const uint4*>(t.path_slot + (pending >> i & 1 ? ats[i] : 0u));
                    a[i] = e[0];
                    b[i] = e[1];
                }
#pragma unroll
                for (int i = 0; i < kPos; ++i) {
                    if (pending >> i & 1) {
                        const uint32_t tg[4] = {a[i].x, a[i].z, b[i].x, b[i].z};
                        const int32_t ids[4] = {static_cast<int32_t>(a[i].y), static_cast<int32_t>(a[i].w), static_cast<int32_t>(b[i].y), static_cast<int32_t>(b[i].w)};
                        bool open = false;
#pragma unroll
                        for (int j = 3; j >= 0; --j) {
                            if (ids[j] >= 0 && tg[j] == tags[i]) nd[i] = ids[j];
                            open |= ids[j] == -1;
                        }
                        if (nd[i] >= 0 || open) pending &= ~(1u << i);
                        ats[i] = (ats[i] + 4) & t.ph_mask;
                    }
                }
            }
            int4 recs[kPos];
            uint4 lo[kPos], hi[kPos];
#pragma unroll
            for (int i = 0; i < kPos; ++i) {
                const uint4* e = reinterpret_cast<const uint4*>(t.path + max(nd[i], 0));  // (without branches: all in flight)
                lo[i] = e[0];
                hi[i] = e[1];
            }
#pragma unroll
            for (int i = 0; i < kPos; ++i) {
                const int32_t p = w0 + rel0 + i;
                recs[i] = make_int4(-1, -1, 0, 0);
                if (nd[i] >= 0) {
                    const unsigned long long eh = (static_cast<unsigned long long>(lo[i].y) << 32) | lo[i].x;
                    // (a node that shares no more than the tag may hide the right one: it is nominated as one that covers
                    // nothing and that nothing is linked to, so that the exact lookup decides what begins here)
                    recs[i] = make_int4(nd[i], -1, 0, 0);
                    if (eh == hps[i] && static_cast<int32_t>(hi[i].x) == p)
                        recs[i] = make_int4(nd[i], static_cast<int32_t>(hi[i].w), static_cast<int32_t>(hi[i].z), static_cast<int32_t>(hi[i].y));
                }
                // position 0 holds the node found exactly above, whatever the index said
                if (role != 2 && rel0 + i == 0) recs[i] = make_int4(child.node, cur, child.len, child.start);
                s_rec[i * kT + tid] = recs[i];
                if (recs[i].x >= 0) lastc = rel0 + i;
            }
            // ---- C. the last nominated position at or before every position: a maximum scan ----
            int32_t cm = lastc;
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                const int32_t left = __shfl_up(cm, 1u << k);
                if (lane >= (1 << k)) cm = max(cm, left);
            }
            if (lane == 63) s_wmax[wave] = cm;
            int32_t run = __shfl_up(cm, 1);
            if (lane == 0) run = -1;
            lds_barrier();
            for (int v = 0; v < wave; ++v) run = max(run, s_wmax[v]);
            // a nominated node that is not linked to the one before it breaks the chain
            int32_t brk = INT32_MAX;
#pragma unroll
            for (int i = 0; i < kPos; ++i) {
                const int rel = rel0 + i;
                if (recs[i].x >= 0) {
                    if (run >= 0) {
                        const int4 pr = s_rec[at_rec(run)];
                        if (!(run + pr.z == rel && recs[i].y == pr.x)) brk = min(brk, rel);
                    }
                    run = rel;
                }
                s_cv[rel] = static_cast<int16_t>(run);
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) brk = min(brk, __shfl_xor(brk, off));
            if (lane == 0) s_red2[red_round & 1][wave] = brk;
        }
        lds_barrier();
        // ---- D. every position against the edge of its node; slots of what the chain holds.  (Not before it is known how far
        // the chain goes: the edge of a node nominated by a colliding hash may reach over positions of other windows, whose
        // workgroups write the right slots meanwhile.) ----
        const int32_t lim_end = min(kWinP, n - w0);
        int32_t bad = INT32_MAX;
        int32_t head = -1;  // first nominated position
        int32_t sl[kPos];
        unsigned in = 0;
        {
            int32_t et[kPos], pt[kPos];
#pragma unroll
            for (int i = 0; i < kPos; ++i) {
                const int rel = i * kT + tid;
                const int32_t cv = s_cv[rel];
                const int4 cr = s_rec[at_rec(max(cv, 0))];
                const bool on = cv >= 0 && rel < lim_end, covered = on && rel < cv + cr.z;
                in |= covered ? 1u << i : 0u;
                bad = on && !covered ? min(bad, rel) : bad;
                const int32_t at = covered ? cr.w + (rel - cv) : 0;  // (loads without branches: all in flight)
                et[i] = t.edge_tok[at];
                sl[i] = t.edge_slot[at];
                pt[i] = prompt[w0 + min(rel, lim_end - 1)];
            }
#pragma unroll
            for (int i = 0; i < kPos; ++i)
                if ((in >> i & 1) && et[i] != pt[i]) bad = min(bad, i * kT + tid);
        }
        const int round = red_round & 1;
        bad = wg_min(bad);
        int32_t brk = INT32_MAX;
#pragma unroll
        for (int v = 0; v < kWaves; ++v) brk = min(brk, s_red2[round][v]);
        // ---- E. where the walk stands after this window (the same in every thread) ----
        const int32_t end = min(min(bad, brk), lim_end);
#pragma unroll
        for (int i = 0; i < kPos; ++i)
            if ((in >> i & 1) && i * kT + tid < end) put_slot(w0 + i * kT + tid, sl[i], role == 2);
        if (role == 2) {
            // the first nominated position: the first whose last nomination is itself (every thread looks at its share)
            int32_t f = INT32_MAX;
#pragma unroll
            for (int i = kPos - 1; i >= 0; --i)
                if (s_cv[i * kT + tid] == i * kT + tid) f = i * kT + tid;
            f = wg_min(f);
            head = f == INT32_MAX ? -1 : f;
        } else {
            head = 0;
        }
        if (head < 0) {  // (a lone window in which nothing was nominated)
            active = false;
        } else {
            if (role == 2) {
                f_pos = w0 + head;
                f_parent = s_rec[at_rec(head)].y;
            }
            if (end <= head) {  // (only a colliding hash nominates a node that does not begin with the prompt's token)
                pos = w0 + head;
                cur = f_parent;
            } else {
                const int32_t z = s_cv[end - 1];
                const int4 zr = s_rec[at_rec(z)];
                last_es = zr.w;
                last_start = w0 + z;
                pos = w0 + end;
                if (z + zr.z == end) {  // the node's whole edge
                    cur = zr.x;
                    // (every node that begins at a position of the window was nominated there: if nothing was where this
                    // edge ends, no child continues the walk, and the lookup that would say so is saved)
                    if (end < kWinP && pos < n_nom && s_rec[at_rec(end)].x < 0) done = true;
                } else if (end == brk) {  // a colliding hash nominated a node inside this one's edge: compare it by itself
                    pos = w0 + z;
                    cur = zr.y;
                    direct = true;
                } else if (end == kWinP && pos < n) {  // the edge reaches past the window
                    const int32_t m = compare_run(zr.w, w0 + z, kWinP - z, min(zr.z, n - w0 - z), role == 2);
                    pos = w0 + z + m;
                    if (m == zr.z) cur = zr.x;
                    else done = true;
                } else {
                    done = true;  // mismatch inside the edge, or the prompt ended inside it
                }
            }
        }
        lds_barrier();  // the window arrays are rebuilt next
        if (role == 2) break;  // one window only
    }
    if (!kMulti || role == 0) break;
    if constexpr (kMulti) {
    // ---- leave the summary; the last workgroup of the request to get here joins them ----
    // (the summary goes out behind the slot ids and all of it is awaited at once: what the count says has arrived)
    if (tid == 0) {
        int32_t* sm = reinterpret_cast<int32_t*>(&scratch->sum[r * n_w + w]);
        const int32_t vals[7] = {f_pos, f_parent, pos, cur, done ? 1 : 0, last_es, last_start};
#pragma unroll
        for (int i = 0; i < 7; ++i) __hip_atomic_store(sm + i, vals[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (role == 2 || tid == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    if (tid == 0) s_last_one = atomicInc(&scratch->counter[r], n_wg - 1) == static_cast<unsigned>(n_wg - 1);
    lds_barrier();
    if (!s_last_one) return;
    {
        // (fetched at once, by loads of device scope: past this XCD's L2, which may hold what the array said during an
        // earlier call)
        static_assert(sizeof(MatchSummary) == 8 * sizeof(int32_t), "eight words per summary");
        if (tid < n_wg * 8)
            s_sum[tid] = __hip_atomic_load(reinterpret_cast<int32_t*>(&scratch->sum[r * n_w]) + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        lds_barrier();
        auto field = [&](int ww, int i) __attribute__((always_inline)) { return s_sum[ww * 8 + i]; };
        auto accept = [&](int ww) __attribute__((always_inline)) {
            pos = field(ww, 2);
            cur = field(ww, 3);
            done = field(ww, 4) != 0;
            last_es = field(ww, 5);
            last_start = field(ww, 6);
        };
        // A window that is no part of the walk may still have written slot ids, from its first nominated position on: only a
        // chain that begins with a node nominated by a colliding hash does (no node of the path begins inside an edge).  What
        // it wrote below the walk's position is put right from the edge the walk took; what it wrote beyond may lie over a
        // later window's slots, so no later window is accepted then and the walk goes on by itself, writing all of them.
        bool stray = false;
        auto repair = [&](int ww) __attribute__((always_inline)) {
            const int32_t fp = field(ww, 0);
            stray |= fp >= 0;
            if (fp >= 0)
                for (int32_t k = max(fp, last_start) + tid; k < pos; k += kT) out_slots[k] = t.edge_slot[last_es + (k - last_start)];
        };
        accept(0);
        int wlast = 0;  // the last window (counted from the one where the first walk stood) whose chain is part of the walk
        for (;;) {
            // the window the walk stands in (n_wg: past all of them; 0 also for a walk that met a mismatch further up)
            const int ww = max(0, min(pos / kWinP - win0, n_wg));
            for (int x = wlast + 1; x < ww; ++x) repair(x);  // (windows that lie inside the last edge)
            if (ww >= n_wg || ww == wlast) break;
            if (!stray && !done && pos < n && field(ww, 0) == pos && field(ww, 1) == cur && field(ww, 2) > pos) {
                accept(ww);  // the walk's next node begins this window's chain
                wlast = ww;
                continue;
            }
            // (the window nominated every node that begins in it: none where the walk stands means no child goes on)
            if (!done && pos < n && (field(ww, 0) < 0 || field(ww, 0) > pos)) done = true;
            repair(ww);
            break;  // the walk goes on by itself, if it goes on
        }
    }
    role = 0;
    active = true;
    direct = false;
    }
    }
    if (tid == 0) prefix_len[r] = pos;
}

}  // namespace pa

// Summaries and counters of the multi-workgroup form: part of the library's code object (each GPU holds its own copy;
// in host code the array's name is only a handle for hipGetSymbolAddress).
static __device__ pa::MatchScratch g_match_scratch[pa::kCallSets];

extern "C" int pa_match_prefixes(const pa_tree* tree, const int32_t* tokens, const int32_t* offsets, int B,
                                 int32_t* prefix_len, int32_t* slot_idx, void* stream) {
    const pa::DeviceTree* view = nullptr;
    int rc = pa_tree_device(tree, &view);
    if (rc != PA_OK) return rc;
    PA_REQUIRE(B >= 0, "pa_match_prefixes: B = %d", B);
    if (B == 0) return PA_OK;
    PA_REQUIRE(offsets && prefix_len, "pa_match_prefixes: offsets or prefix_len is NULL");
    // tokens / slot_idx may be NULL only if every prompt is empty (offsets[B] == 0), which the host cannot see
    // Up to kMultiMaxB requests: several workgroups per request, four on a compute unit in all.  Larger batches: one workgroup
    // per request and no copy of the prompt in LDS; while four on a unit hold them all (kWideMaxB), windows of 1,024 positions,
    // beyond that of 512, eight on a unit.  Measured (us, 1,024 | 512): 257 requests with paths of 250 nodes in 2,100 tokens
    // 19.3 | 25.8, of 540 in 8,448 51 | 60; 1,024 of these 81 | 87; short paths the same.
    pa::MatchScratch* scratch = nullptr;
    if (B <= pa::kMultiMaxB) {
        void* base = nullptr;
        int set = -1;
        rc = pa::call_set_for("pa_match_prefixes", HIP_SYMBOL(g_match_scratch), static_cast<hipStream_t>(stream), &base, &set);
        if (rc != PA_OK) return rc;
        if (set >= 0) scratch = static_cast<pa::MatchScratch*>(base) + set;
    }
    {
        pa::ProfScope prof(pa::kProfMatch, static_cast<hipStream_t>(stream));
        if (scratch != nullptr) {
            const int per = pa::kMultiWgs / B < pa::kMaxW ? pa::kMultiWgs / B : pa::kMaxW;
            hipLaunchKernelGGL((pa::match_prefixes_kernel<256, 4, true>), dim3(B * per), dim3(256), 0, static_cast<hipStream_t>(stream),
                               *view, tokens, offsets, prefix_len, slot_idx, B, scratch);
        } else if (B <= pa::kWideMaxB) {
            hipLaunchKernelGGL((pa::match_prefixes_kernel<256, 4, false>), dim3(B), dim3(256), 0, static_cast<hipStream_t>(stream),
                               *view, tokens, offsets, prefix_len, slot_idx, B, scratch);
        } else {
            hipLaunchKernelGGL((pa::match_prefixes_kernel<256, 2, false>), dim3(B), dim3(256), 0, static_cast<hipStream_t>(stream),
                               *view, tokens, offsets, prefix_len, slot_idx, B, scratch);
        }
    }
    PA_HIP(hipGetLastError());
    return PA_OK;
}
