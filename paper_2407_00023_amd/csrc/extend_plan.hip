// The planner of the bf16 extend attention: builds the work list of one launch on the device, from the lengths and slot
// lists that the matcher left there.
//
// A row tile = up to 128 packed query rows (row = (extend token, query head of the group)) of one request, or rows of several
// requests with a common prefix; a work item = a row tile x a contiguous part of its key range; one workgroup per (item, KV
// head).  Workgroups cost about the same per key tile whatever the number of their rows, and the hardware starts them in
// index order as slots fall free, so the list is built for an even finish: requests with the same prefix together, the
// longest first, every tile cut into parts of about 1 / rounds of a slot's share of the whole work.  (Cutting the end of the
// list finer still evens the finish further and was measured to gain nothing: while every slot is busy the chip is at its
// power limit, and the extra parts cost a merge.)
//
// Kinds of tile.
//   Whole: rows of one request over all its keys.
//   Shared, whole prefix: the left-over rows of a request - those past its last full tile - cost a workgroup as much per key
//     tile as a full tile, so where two or more requests share their whole prefix (at least kPackMinPrefix keys) their
//     left-over rows are laid end to end and cut into tiles.  Such a tile walks the common prefix, every key of it visible to
//     every row, and then the extend tokens of each request that has rows in it, one request's after the other's, visible to
//     that request's rows only (and causally).  Its members are consecutive entries of the member table.
//   Shared, common first part: requests may also share only the first part of their prefixes (a decode batch: a common system
//     and tool prompt, then tokens of each request's own).  Those of few rows (first_part_rows), whose whole prefix nobody
//     shares, are grouped by the deepest of a few fixed depths at which another such request has the same slot (slots
//     name cached tokens: the same slot at a depth means the same tokens up to there); the group's common part is then
//     measured, to a thirteenth of the distance to the next probe, against the group's first member.  Their rows are packed into tiles
//     over the common keys, and again, request by request, into own-key tiles over the rest; the merge joins the two.
//   Narrow: a tile of at most 32 rows, of any of these kinds.  Its workgroup splits the keys over its four waves.
//
// What bounds it: one workgroup's chain of dependent steps - two round trips to memory, about twelve barriers, for common
// first parts one more round trip and six barriers - so equal keys are found through hash tables in LDS instead of all-pairs comparisons, a
// scan costs one barrier, and small batches use four waves.  Kernel times against a planner that
// compared all pairs in sixteen waves (us): 12 requests 14 -> 7, 64 requests 18 -> 10, 256 decode requests 51 -> 21.  Counted in
// cycles, 256 decode requests: lengths and slots from memory 8,400, whole prefixes 3,200, probes 6,000, places compared 12,000 (3,000
// of them for 8 requests: one compute unit fetches 14 lines per request), order 4,300, tiles and items 15,000.
#include "extend_plan.h"

#include <type_traits>

namespace pa {

constexpr int kWgSlots = 512;            // workgroups resident at once: two on each of the 256 compute units
constexpr int kMinChunkTiles = 16;       // never split below this many key tiles (1,024 keys) per part (with 512 keys a decode
                                         // batch's step took 3 % longer) ...
constexpr int kMinChunkCommon = 8;       // ... unless the tile leaves partial results anyway (or is narrow: kMinChunkNarrow)
constexpr int kItemOverhead = 4;         // fixed cost of a work item, in key tiles (its prologue and epilogue)
constexpr int kItemFixed = 6;            // ... as the time of a workgroup goes: 9 us, a key tile 1.6
constexpr int kLengthRounds = 6;         // lists of up to this many rounds of workgroups are ordered by length (7 to 41: nothing either way):
constexpr float kLengthFirst = 1.1f;     // first the items longer than so many times the average, last those shorter than so many
constexpr float kLengthLast = 0.75f;
constexpr float kLengthNarrow = 0.7f;    // what a key tile of a narrow item counts there
constexpr int kMergeCost = 4;            // what partial results cost a launch, in key tiles
constexpr int kMaxParts = 64;            // parts of one tile at most
constexpr int kSortMax = 1024;           // ... and up to this many are ordered
constexpr int kPackMinPrefix = 512;      // prefixes, or first parts of them, are shared from this many keys on ...
constexpr int kPackOwnCost = 2;          // ... and, whole ones, if the members' own keys, which a shared tile walks in the general
                                         // tile for the few rows that see them, cost less than walking the prefix per member:
                                         // this factor x their sum <= (members - 1) x the shared prefix
// Rows of a request at most that are shared over a common first part, and the keys it has to have for a request of more rows
// than a narrow tile.  Every 32 of these rows walk the request's own keys in a tile of their own and leave fp32 partial results
// twice, while they save the less of the common keys' tiles the more they are.  Measured (us, shared | not; 256 requests, 2,000
// common and 300 own keys): heads of 128, 8 rows 117 | 234, 32 rows 195 | 237, 48 rows 288 | 301, 64 rows 339 | 304, 96 rows
// 472 | 339; heads of 64, 48 rows 175 | 239, 64 rows 193 | 236, 80 rows 257 | 227; with 600 common keys, heads of 128, 8 rows
// 85 | 103, 48 rows 207 | 141.
static inline int first_part_rows(int D) { return D == 128 ? 48 : 64; }
constexpr int kPackWidePrefix = 1024;
constexpr int kProbes = 12;              // depths looked at for common first parts, and which
__device__ __forceinline__ constexpr int probe_depth(int k) {
    constexpr int in512[kProbes] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64};
    return kPackMinPrefix * in512[k];
}

// Batches whose tiles fill the chip a few times at most need no work list: a workgroup can find its item from the lengths alone - the
// parts of the first request's tiles, then the second's, and so on - and the workgroup that finishes a tile last joins its parts.
// That saves the launches of the planner and of the merge (13 and 5 us of the 42 of a step of four decode requests) and gives up
// what the planner knows: rows of different requests never share a tile.  A common prefix is then read once per request (from the
// L2s, which hold it), and left-over rows have tiles of their own; but a shared tile walks the own keys of all its members in the
// general tile, 5 us per 64 keys, and with few rounds of workgroups the longest decides.  Measured (us, the call alone, 32 heads over 8
// KV heads of 128 unless said otherwise, random lengths in the ranges given, list | direct, in brackets with 512 MB written in between, so that
// nothing is in the caches):
//   decode, 4 requests behind 1,800 common and 50 to 3,000 own keys 27.4 | 17.0 (34.9 | 24.0); behind 2,200 and up to 350 own ones 8
//   27.4 | 17.7 (32.6 | 23.2), 16 33.3 | 25.2 (44.8 | 32.6); heads of 64 behind 900 and up to 900, 16 35.6 | 15.0 (49.1 | 21.6)
//   50 to 150 new tokens behind 800 keys, 8 requests 63.6 | 34.7 (70.5 | 39.6), 16 71.9 | 38.3, 32 82.2 | 68.7, 52 114.6 | 109.1 (122.9 | 119.1)
//   ... behind 2,200, 8 79.9 | 65.0 (87.0 | 69.4), 16 (five draws) 90 to 109 | 72 to 98; 18 to 22, about a
//   round of workgroups, as the lengths fall: 26 draws 87 to 141 | 74 to 118, 1.09 times as fast in the mean (1.11), nine slower, by up to 20 %
//   20 to 60 new tokens of 32 requests behind 2,200 keys 99.8 | 69.8 (106.8 | 75.0); 100 to 300 of 8 129.2 | 108.5 (138.9 | 115.4)
//   three and four rounds: 73 to 219 new tokens of 40 requests behind 1,500 keys 201.9 | 187.5 (210.2 | 197.5), 25 to 478 of 24 behind
//   800 150.1 | 138.0; heads of 64, 11 to 220 of 46 behind 800 87.8 | 83.5 (99.5 | 95.5), 152 to 457 of 16 behind 400 63.2 | 61.3, 403 to
//   492 of 12 behind 800 82.1 | 79.5 (91.4 | 89.5)
//   218 random batches of 1 to 72 requests, bf16 and fp8 pool, that go without a list: 1.52 times as fast (1.44)
// Hence the limits:
constexpr int kDirectMaxB = 64;            // one request per lane
constexpr int kDirectFewRows = 16;         // rows per request on average: up to this many in narrow tiles; more, but too few not to
                                           // be shared over a common first part (first_part_rows): with a work list
constexpr int kDirectKeyTilesNarrow = 16;  // narrow tiles: key tiles per workgroup slot, at the longest lengths the host was told (fp8
                                           // pool: kDirectKeyTilesFp8)
constexpr int kDirectKeyTilesWide = 24;    // the same for wide tiles, where a slot has half a tile at most
constexpr int kDirectRounds = 3;           // wide tiles per slot at most, or where requests have up to direct_short_rows on average, so
constexpr int kDirectRoundsShort = 4;      // that what their left-over rows cost a list weighs more than what cutting would give, this many ...
static inline int direct_short_rows(int D) { return D == 128 ? 1536 : 1024; }
constexpr int kDirectLongest = 48;         // ... of up to this many key tiles where a slot has more than half a tile (longer ones want
                                           // cutting: 20 requests behind 8,000 keys 168 | 208)
constexpr int kDirectPartNarrow = 34;      // key tiles of a part at most, so that few long requests on few KV heads do not leave most of the
constexpr int kDirectPartIdle = 20;        // chip empty: narrow tiles, and with less than an eighth of the slots taken (list | direct, cold in
                                           // brackets; decode, 1 KV head, 1 request of 16,384 keys 31.6 | 24.1 (36 | 32), 32,768 35.1 | 36.6
                                           // (42 | 51), 262,144 93 | 232; 4 requests of 32,768 46.9 | 39.6 (61 | 59), 65,536 57.8 | 68.6)
constexpr int kDirectPartWide = 32;        // wide tiles, where one part more of each would still leave half of the slots empty (30 new tokens,
                                           // 4 KV heads, 18 requests of 3,000 keys, uncut 48 | 54 (71 | 84), 5,600 62 | 87; 12 of 4,400, two
                                           // parts, 44 | 54 (70 | 82), of 3,000 46.4 | 44.8)
constexpr int kDirectFewTiles = 6;         // batches of more requests only where a tile's share of the slots is no more than the parts there
                                           // may be (kMaxDirectParts, kDirectWideParts); up to this many also beyond it (1 KV head, 5 of
                                           // 4,000 keys 27.0 | 15.9, 6 of 12,000 36.5 | 22.0; more have not been measured without a list)
// and no more than kDirectWideParts parts of a tile of 128 rows where a list would make more: one workgroup joins them, 64 KB a part.
static void make_direct(ExtendPlan& p, int B, int64_t rows, int64_t max_kv_len, int Hkv, int D) {
    p.direct_parts = 0;
    if (B < 1 || B > kDirectMaxB) return;
    const bool few = rows <= int64_t{kDirectFewRows} * B;
    if (!few && rows <= int64_t{first_part_rows(D)} * B) return;
    const int tile_rows = few ? kNarrowRows : kTileRows;
    const int64_t tiles = rows / tile_rows + B, key_tiles = (max_kv_len + kKT - 1) / kKT, per_tile = p.slots / tiles;
    const auto least = [](int64_t a, int64_t b) { return a < b ? a : b; };
    if (few || per_tile >= 2) {
        if (per_tile < 1) return;
        if (tiles * key_tiles > int64_t{p.slots} * (few ? kDirectKeyTilesNarrow : kDirectKeyTilesWide)) return;
        if (!few && least(per_tile, key_tiles / kMinChunkTiles) > kDirectWideParts) return;
        if (B > kDirectFewTiles && (few ? per_tile > kMaxDirectParts : per_tile / 2 > kDirectWideParts)) return;
    } else if (tiles > int64_t{p.slots} * (rows <= int64_t{direct_short_rows(D)} * B ? kDirectRoundsShort : kDirectRounds) || key_tiles > kDirectLongest) {
        return;
    }
    // (wide tiles: one workgroup on a compute unit; a second one there slows the first by what it does itself)
    int64_t parts = least(least(few ? per_tile : per_tile / 2, key_tiles / (few ? kMinChunkNarrow : kDirectMinChunkWide)), few ? kMaxDirectParts : kDirectWideParts);
    parts = least(parts, p.tile_parts);
    if (parts < 1) parts = 1;
    const int64_t part_tiles = (key_tiles + parts - 1) / parts;
    p.direct_idle = 8 * tiles * parts < p.slots;
    if (few) {
        if (part_tiles > (p.direct_idle ? kDirectPartIdle : kDirectPartNarrow)) return;
    } else if (per_tile >= 2 && part_tiles > kDirectPartWide) {
        const int64_t rows_each = int64_t{B} * kTileRows, likely = B * ((rows + rows_each - 1) / rows_each);  // tiles of requests of like length
        if (2 * likely * (parts + 1) <= p.slots) return;
    }
    if (p.prows_cap / parts < rows) return;
    // (the words that count a tile's parts lie where a list would: always enough room, see make_extend_plan)
    if (parts > 1 && static_cast<size_t>(tiles) * Hkv * sizeof(unsigned long long) > p.off_part_o - p.off_tile) return;
    p.direct_parts = static_cast<int>(parts);
    p.direct_tile_rows = tile_rows;
    p.direct_tiles = static_cast<int>(tiles);
    p.direct_key_tiles = static_cast<int>((tiles * key_tiles + p.slots - 1) / p.slots);
    p.direct_part_tiles = static_cast<int>(part_tiles);
    p.direct_stride = static_cast<int>(p.prows_cap / parts);
}

static inline size_t up256(size_t x) { return (x + 255) & ~size_t(255); }

ExtendPlan make_extend_plan(int B, int64_t T, int64_t max_kv_len, int Hq, int Hkv, int D, int rounds, size_t limit) {
    ExtendPlan p{};
    const int G = Hq / Hkv;
    const int64_t rows = T * G;
    p.rounds = rounds;
    p.slots = kWgSlots / Hkv > 0 ? kWgSlots / Hkv : 1;
    p.resident = D == 128 ? p.slots : p.slots + p.slots / 2;
    p.pack = B <= kPackMax;
    p.tiles_cap = static_cast<int>((rows + kTileRows - 1) / kTileRows + B);  // (packing only lowers the number of row tiles)
    p.chunk_rows = 256 / (D / 4);
    // The number of parts of a tile is at most its cost over the target cost of an item + 3/4, so the sum of (parts - 1) over
    // the tiles stays below whole cost / target = slots * rounds; and no part is shorter than the minimum.
    const int64_t by_rule = static_cast<int64_t>(p.slots) * rounds + 1;
    // (the key range of a shared tile holds the own keys of every member: of up to kTileRows requests)
    const int64_t longest = p.pack ? max_kv_len * (B < kTileRows ? (B > 0 ? B : 1) : kTileRows) : max_kv_len;
    const int64_t per_tile = (longest / kKT) / kMinChunkNarrow > 1 ? (longest / kKT) / kMinChunkNarrow : 1;
    p.tile_parts = static_cast<int>(per_tile < kMaxParts ? per_tile : kMaxParts);
    for (p.first_part = p.pack && B > 1 ? first_part_rows(D) : 0; ; p.first_part = 0) {
        // (rows of requests grouped by a common first part: once per shared tile, once per own-key tile)
        const int64_t fp_rows = rows < int64_t{B} * p.first_part ? rows : int64_t{B} * p.first_part;
        p.own_cap = static_cast<int>(p.first_part ? fp_rows / kNarrowRows + B : 0);
        const int64_t by_size = (static_cast<int64_t>(p.tiles_cap) + p.own_cap) * p.tile_parts;
        const int64_t more = by_rule < by_size ? by_rule : by_size;
        p.items_cap = static_cast<int>(p.tiles_cap + p.own_cap + more);
        const int64_t split_parts = 2 * by_rule < by_size ? 2 * by_rule : by_size;
        // Rows of partial results, the smallest of three bounds: every part of a split tile full (n <= 2 (n - 1) for n >= 2
        // parts) and the rows of common first parts twice; each row once, those of common first parts twice, and 128 rows
        // more for every part beyond a tile's first; each of these rows in as many parts as a tile may have.
        const int64_t once = rows + fp_rows;
        int64_t prows = split_parts * kTileRows + 2 * fp_rows;
        prows = by_rule * kTileRows + once < prows ? by_rule * kTileRows + once : prows;
        prows = p.tile_parts * once < prows ? p.tile_parts * once : prows;
        p.prows_cap = static_cast<int>(prows);
        p.chunks_cap = static_cast<int>((split_parts / 2 + 1) * (kTileRows / p.chunk_rows) + fp_rows / p.chunk_rows + 2 * p.own_cap);
        p.off_tile = 256;
        p.off_member = p.off_tile + up256(sizeof(int2) * (static_cast<size_t>(p.tiles_cap) + p.own_cap));
        p.off_item = p.off_member + up256(p.pack ? sizeof(int4) * 2 * (B > 0 ? B : 1) : 0);
        p.off_chunk = p.off_item + up256(sizeof(int4) * 3 * p.items_cap);
        p.off_part_o = p.off_chunk + up256(sizeof(int4) * 3 * p.chunks_cap);
        const size_t head_rows = static_cast<size_t>(p.prows_cap) * Hkv;
        p.off_part_ml = p.off_part_o + up256(head_rows * D * sizeof(float));
        p.total = p.off_part_ml + up256(head_rows * 2 * sizeof(float));
        if (!p.first_part || limit == 0 || p.total <= limit) break;
    }
    make_direct(p, B, rows, max_kv_len, Hkv, D);
    return p;
}

PlanTables plan_tables(const ExtendPlan& p, void* workspace) {
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    return {reinterpret_cast<int32_t*>(ws), reinterpret_cast<int2*>(ws + p.off_tile), reinterpret_cast<int4*>(ws + p.off_member),
            reinterpret_cast<int4*>(ws + p.off_item), reinterpret_cast<int4*>(ws + p.off_chunk), reinterpret_cast<float*>(ws + p.off_part_o),
            reinterpret_cast<float*>(ws + p.off_part_ml)};
}

// Where a pair (place, slot) is looked for in a table in LDS of a power of two of entries.  (One multiplication: the 64-bit mix
// that the tree's tables use costs this kernel, which forms twelve of them per request, 2,500 cycles.)
__device__ __forceinline__ unsigned lds_hash(unsigned place, unsigned slot) {
    const unsigned x = (slot ^ (place << 24) ^ (place >> 8)) * 0x9E3779B1u;
    return x ^ (x >> 15);
}

struct PlanArgs {
    const int32_t *prefix_len, *ext_len, *ext_offsets, *slot_offsets, *slot_idx;
    int32_t* hdr;
    int2* tile;
    int4 *member, *item, *chunk;
    int B, G, tiles_cap, own_cap, items_cap, prows_cap, chunks_cap, slots, resident, slot_items, pack, first_part, tile_parts, chunk_rows;
};

// All of a kernel's arguments asked for at its start: where they are looked at for the first time later on, each cache line of
// them is another round trip to host memory.
__device__ __forceinline__ void touch_args(const PlanArgs& a) {
    asm volatile("" ::"s"(a.prefix_len), "s"(a.hdr), "s"(a.item), "s"(a.chunk), "s"(a.tile_parts), "s"(a.chunk_rows));
}

// The largest of the wave's values, none negative, in its last lane; by the same moves as wave_scan.
__device__ __forceinline__ int wave_max(int x) {
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));
    return x;
}

// Exclusive prefix sums of N ints per thread over the workgroup, and their totals: a scan inside each wave, then the
// totals of the waves.  s_w is used by this call only (one barrier).
template <int NT, int N>
__device__ __forceinline__ void block_scan(int (&v)[N], int (&total)[N], int (*s_w)[NT / 64]) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = wave_scan(v[i]);
    if (lane == 63)
#pragma unroll
        for (int i = 0; i < N; ++i) s_w[i][w] = x[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        int before = 0, all = 0;
#pragma unroll
        for (int k = 0; k < NT / 64; ++k) {
            const int c = s_w[i][k];
            before += k < w ? c : 0;
            all += c;
        }
        v[i] = x[i] - v[i] + before;
        total[i] = all;
    }
}

struct TileDesc {
    int r, row0, kv_lo, kv_end;      // request (a shared tile: one that has the common keys), first packed row, keys
    int rows_here, e_or_rows, P;     // rows; extend length or rows of the group; prefix length or common part
    int member0, n_members;          // shared tiles: the entries of the member table whose rows meet the tile
    // own-key tiles: the shared tile of their group's first rows, their own first row counted from there, the group's rows
    int common_tile, common_row, group_rows;
    int e0, slot_off;
    bool partial_only;               // a shared tile over a common first part: leaves partial results for the own-key tiles to join
    bool own;
};

// The second half of every planner: costs, parts, items and pieces of the merge of tiles [0, n_all), of which n_rows are row
// tiles.  describe(t) says what tile t is; tile_tab: room for what own-key tiles look up of their shared tile.
template <int NT, class Describe>
__device__ __forceinline__ void emit_items(const PlanArgs& a, int n_rows, int n_all, bool over, int2* tile_tab, Describe describe) {
    __shared__ int s_cost[2][NT / 64];
    __shared__ int s_sum[3][NT / 64], s_class[2][NT / 64];
    const int tid = threadIdx.x;
    // thread i owns tiles [i * per, (i + 1) * per); where there are fewer tiles than threads, S threads (a power of two, up to
    // 16, neighbours in a wave) share one and write its records in turn.  What a thread's first tile is (often its only one)
    // is worked out once
    const int per = (n_all + NT - 1) / NT;
    int S = 1;
    while (S < 16 && 2 * S * n_all <= NT) S *= 2;
    const int sub = tid & (S - 1);
    const int t_lo = min(n_all, S > 1 ? tid / S : tid * per), t_hi = min(n_all, t_lo + per);
    const TileDesc d_first = t_lo < t_hi ? describe(t_lo) : TileDesc{};
    auto tile_desc = [&](int t) { return t == t_lo ? d_first : describe(t); };
    auto key_tiles = [](const TileDesc& d) { return (d.kv_end - d.kv_lo + kKT - 1) / kKT; };
    auto narrow = [](const TileDesc& d) { return d.rows_here <= kNarrowRows; };
    // (a narrow tile's waves do four blocks of 32 keys in the time of one)
    auto cost_of = [&](const TileDesc& d) { return (narrow(d) ? (key_tiles(d) + 1) / 2 : key_tiles(d)) + kItemOverhead; };
    int cost = 0, longest = 0;
    for (int t = t_lo; t < t_hi; ++t) {
        const int c = cost_of(tile_desc(t));
        cost += sub == 0 ? c : 0;
        longest = max(longest, c);
    }
    cost = wave_scan(cost);
    longest = wave_max(longest);
    if ((tid & 63) == 63) {
        s_cost[0][tid >> 6] = cost;
        s_cost[1][tid >> 6] = longest;
    }
    __syncthreads();
    int W = 0;
#pragma unroll
    for (int k = 0; k < NT / 64; ++k) {
        W += s_cost[0][k];
        longest = max(longest, s_cost[1][k]);
    }
    // parts of a tile: its cost over the target cost of an item, rounded up from a quarter past a whole number (an item
    // of 1.5 targets at the end of the list is a tail of its own)
    const float target = fmaxf(static_cast<float>(W) / static_cast<float>(a.slot_items), 1.f);
    bool whole = false;  // no tile is cut (decided below)
    auto parts_of = [&](const TileDesc& d) {
        if (whole) return 1;
        const int n = static_cast<int>(static_cast<float>(cost_of(d)) / target + 0.75f);
        const int shortest = narrow(d) ? kMinChunkNarrow : d.partial_only ? kMinChunkCommon : kMinChunkTiles;
        return max(min(min(n, key_tiles(d) / shortest), a.tile_parts), 1);
    };
    // pieces of the merge of a tile: up to chunk_rows rows each; those of an own-key tile inside one shared tile
    auto next_piece = [&](const TileDesc& d, int row) {
        int n = min(a.chunk_rows, d.rows_here - row);
        if (d.own) n = min(n, kTileRows - (d.common_row + row) % kTileRows);
        return n;
    };
    auto chunks_of = [&](const TileDesc& d, int n) {
        if (d.partial_only || (n == 1 && !d.own)) return 0;
        if (!d.own) return (d.rows_here + a.chunk_rows - 1) / a.chunk_rows;
        int c = 0;
        for (int row = 0; row < d.rows_here; row += next_piece(d, row)) ++c;
        return c;
    };
    int v[3] = {0, 0, 0}, total[3];  // items, rows of partial results, pieces of the merge
    for (int t = t_lo; t < t_hi; ++t) {
        const TileDesc d = tile_desc(t);
        const int n = parts_of(d);
        v[0] += n;
        v[1] += n > 1 || d.partial_only || d.own ? n * d.rows_here : 0;
        v[2] += chunks_of(d, n);
    }
    if (sub > 0) v[0] = v[1] = v[2] = 0;
    block_scan<NT, 3>(v, total, s_sum);
    if (S > 1)  // (to the other threads of the tile)
#pragma unroll
        for (int i = 0; i < 3; ++i) v[i] = __shfl(v[i], (tid & 63) - sub);
    // ---- cut or not: where the tiles as they are fill the slots about once or twice, cutting them can make one round of
    // workgroups more than it shortens them.  Compared in key tiles: whole rounds of workgroups of the average cost, a last
    // round that leaves half of the slots empty at two thirds of that (a workgroup alone on its compute unit is faster), the
    // fixed cost of an item, and what the partial results cost.  Steps in us, always cut | by this rule: 16 requests of 50 to 150
    // new tokens behind 2,200 keys (50 tiles for 64 slots) 124.6 | 112.0, 24 160.9 | 149.2; 32 on 2 KV heads 128.2 | 114.9. ----
    // Narrow tiles are bound by memory, and with slots empty by the time a workgroup waits for it: they are cut as they were before,
    // unless every round of them uncut is at least half full (us, cut | uncut; 8 KV heads: 16 decode requests with 4,000 keys each 68 | 85
    // (4 KV heads, 32), 70 with 2,500 151 | 165, but 48 with 1,000 51 | 42, 64 56 | 48; 2 KV heads: 64 with 4,000 69 | 85, 100 with
    // 2,500 62 | 69, but 160 with 1,000 53 | 44).
    auto may_stay = [&] {
        const int last_round = n_all % a.slots;
        return total[1] > kNarrowRows * total[0] || last_round == 0 || 2 * last_round >= a.slots;
    };
    if (n_all == n_rows && total[0] > n_all && may_stay()) {
        const float inv_slots = __builtin_amdgcn_rcpf(static_cast<float>(a.resident));
        const float keys_cost = static_cast<float>(W - n_all * kItemOverhead);  // without the items' fixed cost
        auto finish = [&](int items) {
            const float n = static_cast<float>(items), rounds = n * inv_slots, whole_rounds = floorf(rounds + 0.001f), rest = rounds - whole_rounds;
            const float one = keys_cost * __builtin_amdgcn_rcpf(n) + static_cast<float>(kItemFixed);
            return one * (whole_rounds + (rest < 0.001f ? 0.f : rest < 0.501f ? 0.65f : 1.f));
        };
        const float cut = finish(total[0]) + static_cast<float>(kMergeCost);
        const float uncut = fmaxf(finish(n_all), (2 * n_all <= a.resident ? 0.65f : 1.f) * static_cast<float>(longest - kItemOverhead + kItemFixed));
        if (uncut < cut) {
            whole = true;
            v[0] = t_lo;
            v[1] = v[2] = 0;
            total[0] = n_all;
            total[1] = total[2] = 0;
        }
    }
    // The capacities follow from the host's T and max_kv_len: a batch on the device that is larger than they say does
    // not fit.  Nothing is computed then (an empty list: no output row is written) and hdr[3] says so, which
    // pa_extend_status reports.
    const bool overflow = over || total[0] > a.items_cap || total[1] > a.prows_cap || total[2] > a.chunks_cap;
    if (tid == 0) {
        a.hdr[0] = overflow ? 0 : n_rows;
        a.hdr[1] = overflow ? 0 : total[0];
        a.hdr[2] = overflow ? 0 : total[2];
        a.hdr[3] = overflow;
        a.hdr[4] = overflow ? 0 : total[1];
        a.hdr[5] = 0;
    }
    if (overflow) return;
    if (n_all > n_rows) {  // (own-key tiles look up the parts of their shared tile)
        int prow = v[1];
        for (int t = t_lo; t < t_hi; ++t) {
            const TileDesc d = tile_desc(t);
            const int n = parts_of(d);
            if (d.partial_only && sub == 0) tile_tab[t] = make_int2(n, prow);
            prow += n > 1 || d.partial_only || d.own ? n * d.rows_here : 0;
        }
        __syncthreads();
    }
    // ---- where a tile's items stand: workgroups start in the list's order, and what starts last alone decides when the launch ends.
    // In up to kLengthRounds rounds of them the items of more than the average length come first, the short ones last.  Longer lists stay
    // in order: their last items are a small part.  So do those of more tiles than the planner has threads, whose tiles would be described
    // once more (2 us).  Only three classes, because requests with a common prefix find each other's keys in the L2 while they run together.
    // The average is that of the planner's costs, where a narrow item counts half its key tiles, as where it has the memory to itself;
    // beside wide ones it takes nearly all of their time, and in the classes counts more.  (With half there, too, three whole new problems
    // beside 61 requests of a few new tokens, 190 tiles of 24 to 98 key tiles for 64 slots, gain nothing: 315.6.)
    // Steps in us, in order | so: these 313.6 | 285.8, a video of 8,192 keys 489.2 | 484.8, 256 decode requests 109.1 | 107.5, 80 of 500 to
    // 6,200 keys 221.4 | 217.7, 6 documents of 2,000 to 16,000 keys 212.1 | 204.6, 4 of 4,000 to 20,000 213.6 | 220.4, on the fp8 pool
    // 258.3 | 255.4.  572 random lists: 1.007 times as fast in the mean, with new problems 1.022, documents of unlike length 1.003.  Lists of
    // one length gain nothing and pay the scan (0.4 us); asking for the longest item first costs all others a reduction. ----
    const float average = static_cast<float>(W - n_all * kItemOverhead) / static_cast<float>(max(total[0], 1));
    const bool by_length = per == 1 && total[0] > a.resident && total[0] <= kLengthRounds * a.resident;
    auto class_of = [&](const TileDesc& d, int n) {
        const float len = static_cast<float>(key_tiles(d)) * (narrow(d) ? kLengthNarrow : 1.f), scale = average * static_cast<float>(n);
        return len >= kLengthFirst * scale ? 0 : len >= kLengthLast * scale ? 1 : 2;
    };
    int c[2] = {0, 0}, c_total[2] = {0, 0};
    if (by_length) {
        if (t_lo < t_hi && sub == 0) {
            const int n = parts_of(d_first), k = class_of(d_first, n);
            c[0] = k == 0 ? n : 0;
            c[1] = k == 1 ? n : 0;
        }
        block_scan<NT, 2>(c, c_total, s_class);
        if (S > 1) c[0] = __shfl(c[0], (tid & 63) - sub), c[1] = __shfl(c[1], (tid & 63) - sub);
    }
    for (int t = t_lo; t < t_hi; ++t) {
        const TileDesc d = tile_desc(t);
        const int K = key_tiles(d), n = parts_of(d), k = by_length ? class_of(d, n) : 2;
        const bool partial = n > 1 || d.partial_only || d.own;
        const int item0 = k == 0 ? c[0] : k == 1 ? c_total[0] + c[1] : c_total[0] + c_total[1] + v[0] - c[0] - c[1];
        for (int j = sub; j < n; j += S) {
            // (K < 2^24 key tiles and n <= 64 parts: the products fit 32 bits)
            const int lo = d.kv_lo + static_cast<int>(static_cast<unsigned>(K) * static_cast<unsigned>(j) / static_cast<unsigned>(n)) * kKT;
            const int hi = min(d.kv_end, d.kv_lo + static_cast<int>(static_cast<unsigned>(K) * static_cast<unsigned>(j + 1) / static_cast<unsigned>(n)) * kKT);
            int4* rec = a.item + 3 * static_cast<size_t>(item0 + j);
            rec[0] = make_int4(d.r, d.row0, lo, hi);
            rec[1] = make_int4(partial ? v[1] + j * d.rows_here : -1, d.P, d.e_or_rows, d.e0);
            rec[2] = make_int4(d.slot_off, narrow(d) ? 1 : 0, d.member0, d.n_members);
        }
        if (chunks_of(d, n) > 0) {
            auto write = [&](int c, int row, int len, int n_common, int4 c2) {
                int4* rec = a.chunk + 3 * static_cast<size_t>(v[2] + c);
                rec[0] = make_int4(n, v[1], d.rows_here, row | len << 16);
                rec[1] = make_int4(d.n_members == 0 ? d.e0 : d.member0, d.row0, d.n_members, n_common);
                rec[2] = c2;
            };
            if (!d.own) {
                for (int c = sub; c * a.chunk_rows < d.rows_here; c += S)
                    write(c, c * a.chunk_rows, min(a.chunk_rows, d.rows_here - c * a.chunk_rows), 0, make_int4(0, 0, 0, 0));
            } else if (sub == 0) {
                for (int row = 0, c = 0, len; row < d.rows_here; row += len, ++c) {
                    len = next_piece(d, row);
                    const int at = d.common_row + row, k = at / kTileRows;
                    const int2 ct = tile_tab[d.common_tile + k];
                    write(c, row, len, ct.x, make_int4(ct.y, min(kTileRows, d.group_rows - k * kTileRows), at % kTileRows, 0));
                }
            }
        }
        v[2] += chunks_of(d, n);
        v[0] += n;
        v[1] += partial ? n * d.rows_here : 0;
    }
}

// Batches of up to MAXB requests.  MAXB = kPackMax: with the search for common prefixes; kSortMax: ordered only.
template <int MAXB, int NT>
__global__ __launch_bounds__(NT) void extend_plan_kernel(PlanArgs a) {
    constexpr bool kPack = MAXB <= kPackMax;
    constexpr int HT = (kPack ? 4 : 2) * MAXB;              // hash table of whole prefixes
    constexpr int PT = kPack ? 4096 : 1;      // ... of (probe depth, slot)
    static_assert(!kPack || PT >= kProbes * MAXB + 1, "the table of probes is never full");
    constexpr int NG = kPack ? 2 * MAXB : MAXB;  // groups: [0, MAXB) by whole prefix, [MAXB, 2 MAXB) by common first part
    __shared__ int s_P[MAXB], s_E[MAXB], s_e0[MAXB], s_so[MAXB];
    __shared__ int4 s_id[MAXB];               // prefix length, last, first and middle slot of it
    __shared__ int s_ht[HT], s_hlead[HT], s_hcnt[HT];  // a request with the prefix (-1: none), the first one, how many
    __shared__ __attribute__((aligned(16))) int s_pt[PT], s_pc[PT];  // a pair (request, probe) (-1: none), later the first request that chose it;
                                              // how many requests, and how many chose it << 16
    __shared__ int s_pslot[kPack ? (kProbes + 2) * MAXB : 1];  // slots at the probes; later, of leaders, at the places compared
    __shared__ int s_cutg[kPack ? MAXB : 1];  // per leader: at how many of these places its group agrees
    __shared__ int s_cut[MAXB];               // per request: the same; its whole prefix otherwise
    __shared__ int s_gid[MAXB];
    __shared__ int s_gkey[NG];                // per group: the most keys of any of its requests
    __shared__ int s_gn[NG], s_gL[NG], s_gown[NG];         // packable members, their rows, their extend tokens
    __shared__ int s_gR[NG], s_gm[NG], s_go[NG], s_gt[NG]; // what the groups before it hold: rows, members, tokens; its first tile
    using SortKey = std::conditional_t<kPack, unsigned, unsigned long long>;
    __shared__ __attribute__((aligned(16))) SortKey s_sk[MAXB];
    __shared__ int s_order[MAXB];             // position in the list -> request
    __shared__ int s_first[MAXB], s_ofirst[MAXB];  // per position: its first row tile and own-key tile
    __shared__ int4 s_req[MAXB];              // ... its request, its group, the shared tiles in front of its own ones, and the
                                              // first of its packed rows among the group's (-1: not packed)
    __shared__ int s_mR[MAXB], s_mO[MAXB], s_mE[MAXB];     // per member: that; extend tokens of the members before it; its own
    __shared__ int s_any;
    __shared__ int s_scan[5][NT / 64];
    const int tid = threadIdx.x, B = a.B, G = a.G, mt = kTileRows;
    touch_args(a);
    const bool first_part = kPack && a.first_part;
    const int32_t* const slot_idx = a.slot_idx;
    // ---- lengths, the slots that name a prefix, the probes ----
    const bool on = tid < B;
    int P = 0, E = 0, e0 = 0, so = 0;
    if (on) {
        P = a.prefix_len[tid];
        E = a.ext_len[tid];
        e0 = a.ext_offsets[tid];
        so = a.slot_offsets[tid];
    }
    const int pmask = [&] {  // (a table of about sixteen entries per request, cleared below)
        int n = 64;
        while (n < 16 * B && n < PT) n <<= 1;
        return n - 1;
    }();
    for (int i = tid; i < HT; i += NT) s_ht[i] = -1, s_hlead[i] = 0x7fffffff, s_hcnt[i] = 0;
    for (int i = tid; i < NG; i += NT) s_gkey[i] = 0, s_gn[i] = 0, s_gL[i] = 0, s_gown[i] = 0;
    if (first_part)
        for (int i = tid; i <= pmask; i += NT) s_pt[i] = -1, s_pc[i] = 0;
    if (tid == 0) s_any = 0;
    const int rows = on ? max(E, 0) * G : 0, full = rows / mt, left = rows - full * mt;
    const bool small = on && first_part && rows > 0 && rows <= a.first_part && P >= kPackMinPrefix;
    [[maybe_unused]] int probe[kProbes];  // this request's slots at the probes (-1: none)
#pragma unroll
    for (int k = 0; k < kProbes; ++k) probe[k] = -1;
    if (on) {
        s_P[tid] = P;
        s_E[tid] = E;
        s_e0[tid] = e0;
        s_so[tid] = so;
        s_cut[tid] = P;
        if (kPack) s_cutg[tid] = 0x7fffffff;
        const int32_t* list = slot_idx + so;
        int4 id = make_int4(P, -1 - tid, 0, 0);
        if (P > 0) id = make_int4(P, list[P - 1], list[0], list[P / 2]);
        if constexpr (kPack) {
            if (small) {
#pragma unroll
                for (int k = 0; k < kProbes; ++k)
                    if (probe_depth(k) <= P) probe[k] = list[probe_depth(k) - 1];
#pragma unroll
                for (int k = 0; k < kProbes; ++k) s_pslot[(kProbes + 2) * tid + k] = probe[k];
            }
        }
        s_id[tid] = id;
    }
    __syncthreads();
    // ---- requests share their whole prefix if it has the same length and the same slots.  Slot lists that name the tokens of
    // one prefix tree are equal as soon as their last slots are; the length, the first and the middle slot are compared as
    // well, so that lists of other origin that merely end in the same slot stay apart ----
    int hslot = 0;
    if (rows > 0) {
        const int4 id = s_id[tid];
        hslot = lds_hash(static_cast<unsigned>(id.x), static_cast<unsigned>(id.y)) & (HT - 1);
        for (int step = 0; step < HT; ++step) {
            const int old = atomicCAS(&s_ht[hslot], -1, tid);
            if (old < 0 || old == tid) break;
            const int4 o = s_id[old];
            if (o.x == id.x && o.y == id.y && o.z == id.z && o.w == id.w) break;
            hslot = (hslot + 1) & (HT - 1);
        }
        atomicMin(&s_hlead[hslot], tid);
        atomicAdd(&s_hcnt[hslot], 1);
    }
    __syncthreads();
    int gid = tid;
    if (rows > 0) gid = s_hlead[hslot];
    if constexpr (kPack) {
        const bool cand = small && s_hcnt[hslot] == 1;
        if (cand) s_any = 1;
        if (first_part) __syncthreads();
        if (first_part && s_any) {
            // ---- common first parts: the deepest probe at which another candidate has the same slot ----
            // (The first look into the table goes out for all probes together; few need another.)
            // (Of the lanes of a wave that have the same slot as its first one - a system prompt common to the batch - only that
            // one goes to the table, and counts for all: 256 atomic operations on one entry follow one another.)
            int at[kProbes], old[kProbes], theirs[kProbes], first_lane[kProbes];
            unsigned with_first = 0;  // bit k: same slot at probe k as the wave's first lane with one
            const int lane = tid & 63;
#pragma unroll
            for (int k = 0; k < kProbes; ++k) {
                const bool has = cand && probe_depth(k) <= P && (rows <= kNarrowRows || probe_depth(k) >= kPackWidePrefix);
                const unsigned long long any = __ballot(has);
                at[k] = old[k] = -1;
                first_lane[k] = -1;
                if (any) {
                    const int slot = has ? probe[k] : -1;
                    first_lane[k] = __ffsll(any) - 1;
                    const bool same = has && slot == __builtin_amdgcn_readlane(slot, first_lane[k]);
                    with_first |= same ? 1u << k : 0u;
                    if (has && (!same || lane == first_lane[k])) {
                        at[k] = lds_hash(static_cast<unsigned>(k), static_cast<unsigned>(slot)) & pmask;
                        old[k] = atomicCAS(&s_pt[at[k]], -1, (1 << 16) | (tid * kProbes + k));
                    }
                }
            }
            auto slot_of = [&](int pair) { return s_pslot[(kProbes + 2) * (pair / kProbes) + pair % kProbes]; };
#pragma unroll
            for (int k = 0; k < kProbes; ++k) theirs[k] = old[k] >= 0 ? slot_of(old[k] & 0xFFFF) : 0;
#pragma unroll
            for (int k = 0; k < kProbes; ++k) {
                if (first_lane[k] < 0) continue;
                const unsigned long long sharers = __ballot(with_first >> k & 1);
                if (at[k] >= 0) {
                    const int slot = probe[k];
                    for (int step = 0; step <= pmask && old[k] >= 0; ++step) {
                        const int who = old[k] & 0xFFFF;
                        if (who % kProbes == k && (step == 0 ? theirs[k] : slot_of(who)) == slot) break;
                        at[k] = (at[k] + 1) & pmask;
                        old[k] = atomicCAS(&s_pt[at[k]], -1, (1 << 16) | (tid * kProbes + k));
                    }
                    atomicAdd(&s_pc[at[k]], lane == first_lane[k] ? __popcll(sharers) : 1);
                }
                const int theirs_at = __builtin_amdgcn_readlane(at[k], first_lane[k]);
                if (with_first >> k & 1) at[k] = theirs_at;
            }
            __syncthreads();
            int chosen = -1, depth = 0, next = 0x7fffffff;
            int with[kProbes];
#pragma unroll
            for (int k = 0; k < kProbes; ++k) with[k] = s_pc[max(at[k], 0)] & 0xFFFF;
#pragma unroll
            for (int k = 0; k < kProbes; ++k)
                if (at[k] >= 0 && with[k] >= 2) {
                    chosen = at[k];
                    depth = probe_depth(k);
                    next = k + 1 < kProbes ? probe_depth(k + 1 < kProbes ? k + 1 : k) : 0x7fffffff;
                }
            __syncthreads();
            // the group: the candidates that chose this probe; its first member leads
            if (chosen >= 0) {
                atomicMin(&s_pt[chosen], tid);
                atomicAdd(&s_pc[chosen], 1 << 16);
            }
            __syncthreads();
            const bool grouped = chosen >= 0 && (s_pc[chosen] >> 16) >= 2;
            const int lead = grouped ? s_pt[chosen] : tid;
            // The slot lists agree up to the probe.  Beyond it, up to the next probe or the end of the leader's prefix, kProbes
            // places are compared with the leader's list; what all members agree on is common (the tokens between the last
            // place they agree at and the first they do not, a thirteenth of the interval, are each member's own).  (Lists of
            // one prefix tree agree on everything before a place where they agree; for lists of other origin two more places
            // and the first slot are compared, and a request that differs there stays on its own.)
            const int pl = grouped ? s_P[lead] : 0, stride = static_cast<int>(static_cast<unsigned>(max(min(pl, next) - depth, 0)) / (kProbes + 1));
            auto place = [&](int j) { return depth + stride * (j + 1); };
            int mine[kProbes + 2];
            if (grouped) {
                const int32_t* x = slot_idx + so;
#pragma unroll
                for (int j = 0; j < kProbes; ++j) mine[j] = place(j) < min(P, pl) ? x[place(j)] : -2;
                mine[kProbes] = x[depth / 3];
                mine[kProbes + 1] = x[2 * (depth / 3)];
                if (lead == tid)
#pragma unroll
                    for (int j = 0; j < kProbes + 2; ++j) s_pslot[(kProbes + 2) * tid + j] = mine[j];
            }
            __syncthreads();
            bool agree = false;
            if (grouped) {
                const int* y = s_pslot + (kProbes + 2) * lead;
                int same = 0;
#pragma unroll
                for (int j = kProbes - 1; j >= 0; --j) same = mine[j] == y[j] && mine[j] != -2 ? same + 1 : 0;  // (from place 0 on)
                agree = mine[kProbes] == y[kProbes] && mine[kProbes + 1] == y[kProbes + 1] && s_id[tid].z == s_id[lead].z;
                if (agree) atomicMin(&s_cutg[lead], same);
            }
            __syncthreads();
            if (agree) {
                const int same = s_cutg[lead];
                gid = MAXB + lead;
                s_cut[tid] = same > 0 ? place(same - 1) + 1 : depth;
            }
        }
    }
    // ---- what the groups hold ----
    const bool fp = kPack && gid >= MAXB;  // grouped by a common first part
    const int keys = rows > 0 ? P + E : 0;
    if (on) {
        s_gid[tid] = gid;
        atomicMax(&s_gkey[gid], keys);
        if (kPack && a.pack && left > 0 && (fp || P >= kPackMinPrefix)) {
            atomicAdd(&s_gn[gid], 1);
            atomicAdd(&s_gL[gid], left);
            atomicAdd(&s_gown[gid], fp ? 0 : E);
        }
    }
    __syncthreads();
    // ---- order: groups with the most keys first, inside a group the request with the most keys first.  In batches of up to
    // kPackMax in a sort key of 32 bits, all different (the comparison of every request with every other is what this costs,
    // and one of 64 bits takes three times as long): the group's most keys, in tiles, on a scale of 64 steps per doubling (16 of
    // them: 64 requests on 16 tools 302.5 -> 306.4 us); the group's leader, which heads no other; the request's keys as a
    // fraction of the group's most; its number ----
    if constexpr (kPack) {
        static_assert(MAXB <= 256, "eight bits");
        if (on) {
            constexpr unsigned kTop = (1u << 20) - 1;
            const unsigned most = max(1u, min(kTop, static_cast<unsigned>(s_gkey[gid] + 63) >> 6)), mine = min(most, static_cast<unsigned>(max(keys, 0) + 63) >> 6);
            const unsigned e = max(0, 25 - static_cast<int>(__clz(static_cast<int>(most))));
            const unsigned gk = (e << 6) + (most >> e);  // (below 15 x 64)
            const unsigned part = static_cast<unsigned>(63.f * __builtin_amdgcn_rcpf(static_cast<float>(most)) * static_cast<float>(mine));
            s_sk[tid] = ((1023u - gk) << 22) | (static_cast<unsigned>(gid & 255) << 14) | ((63u - min(63u, part)) << 8) | static_cast<unsigned>(tid);
        }
        for (int i = B + tid; i < ((B + 3) & ~3); i += NT) s_sk[i] = 0xFFFFFFFFu;
    } else if (on) {
        constexpr unsigned kTop = (1u << 22) - 1;
        const unsigned gk = min(kTop, static_cast<unsigned>(s_gkey[gid] + 63) >> 6), mine = min(kTop, static_cast<unsigned>(keys + 63) >> 6);
        s_sk[tid] = (static_cast<unsigned long long>(kTop - gk) << 42) | (static_cast<unsigned long long>(gid) << 32) |
                    (static_cast<unsigned long long>(kTop - mine) << 10) | static_cast<unsigned>(tid);
    }
    static_assert(NG <= 1024 && MAXB <= 1024, "the fields of the sort key");
    __syncthreads();
    {
        // tpr threads per request (a power of two, neighbours in a wave), each over its share of the others, four at a time
        int tpr = 1;
        while (tpr < 16 && 2 * tpr * B <= NT) tpr *= 2;
        const int q = tid / tpr, first = tid & (tpr - 1);
        const SortKey mine = s_sk[min(q, B - 1)];
        int rank = 0;
        if constexpr (kPack) {
#pragma unroll 8
            for (int i = 4 * first; i < B; i += 4 * tpr) {
                const uint4 k = *reinterpret_cast<const uint4*>(&s_sk[i]);
                rank += (k.x < mine) + (k.y < mine) + (k.z < mine) + (k.w < mine);
            }
        } else {
#pragma unroll 8
            for (int i = first; i < B; i += tpr) rank += s_sk[i] < mine;
        }
        for (int off = 1; off < tpr; off <<= 1) rank += __shfl_xor(rank, off);
        if (q < B && first == 0) s_order[rank] = q;
        __syncthreads();
    }
    // (the tables of the probes are free by now)
    constexpr int kTileTab = kPack ? PT / 2 : 0;
    int2* const s_tpart = reinterpret_cast<int2*>(s_pt);       // per row tile: what own-key tiles look up of their shared one
    short* const s_tpos = reinterpret_cast<short*>(s_pc);      // per tile: its position in the list
    short* const s_tmem = s_tpos + kTileTab;                   // per shared tile: its first member
    // ---- one thread per position of the list: tiles, packed rows, members ----
    bool over;
    int n_rows, n_own;
    {
        int r = 0, g = 0, pE = 0, pfull = 0, pleft = 0;
        bool packed = false, pfp = false, head = false;
        if (on) {
            r = s_order[tid];
            g = s_gid[r];
            pE = s_E[r];
            const int prow = max(pE, 0) * G;
            pfull = prow / mt;
            pleft = prow - pfull * mt;
            pfp = kPack && g >= MAXB;
            head = tid == 0 || s_gid[s_order[tid - 1]] != g;
            // (requests with long extends behind a short common prefix stay on their own)
            packed = kPack && s_gn[g] >= 2 && (pfp || static_cast<int64_t>(kPackOwnCost) * s_gown[g] <= static_cast<int64_t>(s_gn[g] - 1) * s_P[r]);
        }
        const int nshared = head && packed ? (s_gL[g] + mt - 1) / mt : 0;
        packed = packed && pleft > 0;
        int v[5] = {packed ? pleft : 0, packed ? 1 : 0, packed && !pfp ? pE : 0, nshared + pfull + (pleft > 0 && !packed ? 1 : 0),
                    packed && pfp ? (pleft + kNarrowRows - 1) / kNarrowRows : 0};
        int total[5];
        const int n_mine = v[3], n_mine_own = v[4];
        block_scan<NT, 5>(v, total, s_scan);
        const int first_mine = v[3], first_own = v[4];
        if (head) {
            s_gR[g] = v[0];
            s_gm[g] = v[1];
            s_go[g] = v[2];
            s_gt[g] = v[3];
            s_gL[g] = nshared > 0 ? s_gL[g] : 0;  // (0 from here on: not packed)
        }
        if (on) {
            s_first[tid] = v[3];
            s_ofirst[tid] = v[4];
        }
        __syncthreads();
        if (on) s_req[tid] = make_int4(r, g, nshared, packed ? v[0] - s_gR[g] : -1);
        if constexpr (kPack) {
            // which position a tile belongs to, and the first member of a shared one, where the tables hold all tiles
            if (total[3] + total[4] <= kTileTab) {
                for (int i = 0; i < n_mine; ++i) s_tpos[first_mine + i] = static_cast<short>(tid);
                for (int i = 0; i < n_mine_own; ++i) s_tpos[total[3] + first_own + i] = static_cast<short>(tid);
                const int R0 = packed ? v[0] - s_gR[g] : 0, k = (R0 + mt - 1) / mt;
                if (packed && k * mt < R0 + pleft) s_tmem[s_gt[g] + k] = static_cast<short>(v[1]);
            }
        }
        if (packed) {
            a.member[2 * v[1]] = make_int4(v[0] - s_gR[g], s_e0[r], pfull * mt, pE);
            a.member[2 * v[1] + 1] = make_int4(v[2] - s_go[g], 0, 0, 0);
            s_mR[v[1]] = v[0] - s_gR[g];
            s_mO[v[1]] = v[2] - s_go[g];
            s_mE[v[1]] = pfp ? 0 : pE;
        }
        n_rows = total[3];
        n_own = total[4];
        over = n_rows > a.tiles_cap || n_own > a.own_cap;
    }
    __syncthreads();
    if (over) n_rows = n_own = 0;
    const bool tabled = kPack && n_rows + n_own <= kTileTab;
    // the last position whose first tile is <= t
    auto position = [&](const int* first, int t) {
        if (tabled) return static_cast<int>(s_tpos[first == s_ofirst ? n_rows + t : t]);
        int lo = 0, hi = B;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (first[mid] <= t) lo = mid; else hi = mid;
        }
        return lo;
    };
    auto describe = [&](int t) {
        TileDesc d{};
        const bool own = t >= n_rows;
        const int pos = own ? position(s_ofirst, t - n_rows) : position(s_first, t);
        const int4 rq = s_req[pos];
        const int r = rq.x, g = rq.y;
        const int nrow = s_E[r] * G, full_r = nrow / mt;
        int j = own ? t - n_rows - s_ofirst[pos] : t - s_first[pos];
        d.r = r;
        d.P = s_P[r];
        d.e0 = s_e0[r];
        d.slot_off = s_so[r];
        if (own) {  // rows of one request over the keys behind its group's common part
            d.own = true;
            d.row0 = j * kNarrowRows;
            d.rows_here = min(kNarrowRows, nrow - d.row0);
            d.e_or_rows = s_E[r];
            d.kv_lo = s_cut[r];
            d.kv_end = d.P + (d.row0 + d.rows_here - 1) / G + 1;
            d.common_tile = s_gt[g];
            d.common_row = rq.w + d.row0;
            d.group_rows = s_gL[g];
            return d;
        }
        const int nshared = kPack ? rq.z : 0;
        if (j < nshared) {  // a shared tile of the group this position heads
            const int m0 = s_gm[g], nm = s_gn[g], L = s_gL[g];
            d.row0 = j * mt;
            d.rows_here = min(mt, L - d.row0);
            d.e_or_rows = L;
            // the members whose rows meet the tile: the one holding its first row ... the one holding its last
            auto member_of = [&](int row) {
                int lo = 0, hi = nm;
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (s_mR[m0 + mid] <= row) lo = mid; else hi = mid;
                }
                return m0 + lo;
            };
            int ma, mb;
            if (tabled) {
                ma = s_tmem[t];
                const bool last = d.row0 + mt >= L;  // (the next tile's first member may have rows in this one)
                mb = last ? m0 + nm - 1 : s_tmem[t + 1];
                if (!last && s_mR[mb] >= d.row0 + mt) --mb;
            } else {
                ma = member_of(d.row0);
                mb = member_of(d.row0 + d.rows_here - 1);
            }
            d.member0 = ma;
            d.n_members = mb - ma + 1;
            d.P = s_cut[r];
            d.kv_end = d.P + s_mO[mb] + s_mE[mb] - s_mO[ma];
            d.partial_only = kPack && g >= MAXB;
            return d;
        }
        j -= nshared;
        d.e_or_rows = s_E[r];
        // the request's last rows - the most keys - first: its left-over rows, if they were not packed, then the
        // full tiles from the last one down
        const int left_r = nrow - full_r * mt;
        if (left_r > 0 && rq.w < 0) {
            if (j == 0) {
                d.row0 = full_r * mt;
                d.rows_here = left_r;
                d.kv_end = d.P + (nrow - 1) / G + 1;
                return d;
            }
            --j;
        }
        d.row0 = (full_r - 1 - j) * mt;
        d.rows_here = mt;
        d.kv_end = d.P + (d.row0 + mt - 1) / G + 1;
        return d;
    };
    emit_items<NT>(a, n_rows, n_rows + n_own, over, tabled ? s_tpart : a.tile, describe);
}

// Batches of more than kSortMax requests: in the order given, tables in global memory.
template <int NT>
__global__ __launch_bounds__(NT) void extend_plan_large_kernel(PlanArgs a) {
    __shared__ int s_scan[2][1][NT / 64];
    touch_args(a);
    const int tid = threadIdx.x, G = a.G, mt = kTileRows;
    int n_rows = 0;
    for (int base = 0, round = 0; base < a.B; base += NT, ++round) {
        const int r = base + tid;
        int cnt = 0;
        if (r < a.B) {
            const int e = a.ext_len[r];
            cnt = e > 0 ? (e * G + mt - 1) / mt : 0;
        }
        int v[1] = {cnt}, total[1];
        block_scan<NT, 1>(v, total, s_scan[round & 1]);
        for (int j = 0; j < cnt; ++j)  // a request's last rows - the most keys - first
            if (n_rows + v[0] + j < a.tiles_cap) a.tile[n_rows + v[0] + j] = make_int2(r, (cnt - 1 - j) * mt);
        n_rows += total[0];
    }
    __syncthreads();
    const bool over = n_rows > a.tiles_cap;
    if (over) n_rows = 0;
    auto describe = [&](int t) {
        TileDesc d{};
        const int2 tt = a.tile[t];
        d.r = tt.x;
        d.row0 = tt.y;
        d.P = a.prefix_len[d.r];
        d.e_or_rows = a.ext_len[d.r];
        d.e0 = a.ext_offsets[d.r];
        d.slot_off = a.slot_offsets[d.r];
        d.rows_here = min(mt, d.e_or_rows * G - d.row0);
        d.kv_end = d.P + (d.row0 + d.rows_here - 1) / G + 1;
        return d;
    };
    emit_items<NT>(a, n_rows, n_rows, over, a.tile, describe);
}

int launch_extend_plan(const ExtendPlan& p, const PlanTables& t, const int32_t* prefix_len, const int32_t* ext_len, const int32_t* ext_offsets,
                       const int32_t* slot_offsets, const int32_t* slot_idx, int B, int G, hipStream_t stream) {
    const PlanArgs a{prefix_len, ext_len, ext_offsets, slot_offsets, slot_idx, t.hdr, t.tile, t.member, t.item, t.chunk, B, G, p.tiles_cap,
                     p.own_cap, p.items_cap, p.prows_cap, p.chunks_cap, p.slots, p.resident, p.slots * p.rounds, p.pack, p.first_part, p.tile_parts, p.chunk_rows};
    ProfScope prof(kProfPlan, stream);
    // (few requests and tiles: four waves meet at a barrier sooner than sixteen)
    const int most = p.tiles_cap + p.own_cap;
    if (B <= kPackMax && most <= 512)
        hipLaunchKernelGGL((extend_plan_kernel<kPackMax, 256>), dim3(1), dim3(256), 0, stream, a);
    else if (B <= kPackMax && most <= 1024)
        hipLaunchKernelGGL((extend_plan_kernel<kPackMax, 512>), dim3(1), dim3(512), 0, stream, a);
    else if (B <= kPackMax)
        hipLaunchKernelGGL((extend_plan_kernel<kPackMax, 1024>), dim3(1), dim3(1024), 0, stream, a);
    else if (B <= kSortMax)
        hipLaunchKernelGGL((extend_plan_kernel<kSortMax, 1024>), dim3(1), dim3(1024), 0, stream, a);
    else
        hipLaunchKernelGGL((extend_plan_large_kernel<1024>), dim3(1), dim3(1024), 0, stream, a);
    return PA_OK;
}

}  // namespace pa
