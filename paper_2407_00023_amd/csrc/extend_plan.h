// The work list of a bf16 extend-attention launch: what the planner (extend_plan.hip) writes and the attention and merge
// kernels (extend_bf16.hip) read.
#pragma once

#include "common.h"

namespace pa {

constexpr int kKT = 64;          // key tokens per tile
constexpr int kTileRows = 128;   // packed query rows of a wide row tile (four waves, 32 rows each, every wave all keys)
constexpr int kNarrowRows = 32;  // ... of a narrow one (four waves, the same rows each, every wave a quarter of the keys)
constexpr int kPackMax = 256;    // batches of up to this many requests are looked through for common prefixes

struct ExtendPlan {
    int tiles_cap;   // upper bound on the number of row tiles
    int own_cap;     // ... on the number of own-key tiles (rows of shared tiles again, over the keys that are theirs alone)
    int items_cap;   // ... on the number of work items (tile x part of its key range)
    int prows_cap;   // ... on the number of rows of partial results, per KV head
    int chunks_cap;  // ... on the number of pieces of the merge
    int slots;       // workgroup slots per KV head, two on a compute unit
    int resident;    // workgroups per KV head that are resident at once (heads of 64: three on a compute unit)
    int rounds;      // work items aimed at per workgroup slot
    int pack;        // 1: rows of requests with a common prefix may be packed
    int first_part;  // ... of requests of up to this many rows also where they have only the first part of it in common (0: not)
    int tile_parts;  // parts of one tile at most
    int chunk_rows;  // rows per piece of the merge
    // small batches: no work list is built, every workgroup finds its own item (see make_direct in extend_plan.hip)
    int direct_parts;      // parts of a tile at most; 0: a work list
    int direct_tile_rows;  // rows of a tile
    int direct_tiles;      // upper bound on the number of tiles
    int direct_key_tiles;  // key tiles per workgroup slot
    int direct_part_tiles; // ... and of a part
    bool direct_idle;      // the parts take less than an eighth of the slots
    int direct_stride;     // rows of partial results of one part of all tiles, per KV head
    size_t off_tile, off_member, off_item, off_chunk, off_part_o, off_part_ml, total;
};

// limit: bytes that the plan may take (0: no limit); what may be left out to stay below it is.
ExtendPlan make_extend_plan(int B, int64_t T, int64_t max_kv_len, int Hq, int Hkv, int D, int rounds, size_t limit);
constexpr int kRounds = 2;        // the plan aims at about this many work items per workgroup slot (measured: with 3 a kernel
                                  // over long shared documents took 6 % longer - every item pays its start-up, its partial
                                  // results and their merge - with 1.5 its last round ran thin; the rest did not care)
constexpr int kRoundsStatic = 1;  // ... with the library's own scratch buffer as workspace (fewer partial results)

constexpr int kMinChunkNarrow = 4;      // a part of a narrow tile has at least this many key tiles: 64 keys for each of its waves
constexpr int kDirectMinChunkWide = 8;  // ... of a wide one in a launch without a work list, or twice as many where the rows of a
constexpr int kDirectJoinRows = 2048;   // request, in all KV heads, are more than this: the partial results are stored through to
                                        // memory and read again (100 to 300 new tokens behind 2,200 keys, 8 KV heads, 46.7 us, with
                                        // parts of 8 50.8; 20 to 60 new tokens 36.3, with parts of 16 43.4)
constexpr int kDirectKeyTilesFp8 = 9;   // key tiles per workgroup slot that go without a work list where the pool is in fp8 (a narrow
                                        // tile takes longer there: 12 decode requests, 8.5 a slot, 41.4 us with list | 39.5 without;
                                        // 16, 11.8 a slot, 42.2 | 47.2)
constexpr int kDirectPartFp8 = 20;      // ... and key tiles of a part (as kDirectPartNarrow and kDirectPartIdle for bf16 ones): one
constexpr int kDirectPartIdleFp8 = 16;  // decode request, 8 KV heads, 20,000 keys 39.6 | 40.3, 32,000 44.2 | 57.3; 1 KV head, 16,000 33.5 | 34.2,
                                        // 20,000 34.7 | 39.0
constexpr int kMaxDirectParts = 16;     // parts of a tile at most in such a launch ...
constexpr int kDirectWideParts = 4;     // ... and of a wide one

// Inclusive prefix sum over the wave, by the cross-lane moves of the vector ALU (rows of 16 lanes, then row to row).
__device__ __forceinline__ int wave_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
    return x;
}

// Workspace: a header of 256 bytes - hdr[0] = row tiles, hdr[1] = work items, hdr[2] = pieces of the merge, hdr[3] = 1 if
// the batch on the device does not fit the plan (nothing is computed then), hdr[4] = rows of partial results, per KV head (without a
// work list: at most that many), hdr[5] = parts of a tile at most without a work list, 0 with one - and, without a work list, a word of 64 bits per tile and KV head that counts the tile's finished
// parts, from off_tile on, or the tables of the list, of int4:
//   member[2 m]     = (first row among its group's packed rows, first extend token, first packed row of the request,
//                      extend length)
//   member[2 m + 1] = (extend tokens of the group's members before it, 0, 0, 0)
//   item[3 i ..]    = (request, first packed row, first key, end key),
//                     (first row of its partial result or -1: writes the output, prefix length or common part, extend
//                      length or rows of the group, first extend token),
//                     (first slot-list entry, 1: narrow, first member, members or 0)
//   chunk[3 c ..]   = (parts, first partial row, rows of the tile, first row | number of rows << 16),
//                     (first extend token or first member, first packed row of the tile, members or 0, parts of the shared
//                      tile that holds the common keys of these rows, or 0),
//                     (its first partial row, its rows, these rows' first one in it, 0)
// The partial result of part p of a tile: row (first partial row + p * rows of the tile) * Hkv + g * rows of the tile + row in
// the tile, for KV head g.
struct PlanTables {
    int32_t* hdr;
    int2* tile;    // (parts, first partial row); for tables that do not fit LDS, (request, first packed row) at first
    int4* member;
    int4* item;
    int4* chunk;
    float* part_o;
    float* part_ml;
};
PlanTables plan_tables(const ExtendPlan& p, void* workspace);

int launch_extend_plan(const ExtendPlan& p, const PlanTables& t, const int32_t* prefix_len, const int32_t* ext_len, const int32_t* ext_offsets,
                       const int32_t* slot_offsets, const int32_t* slot_idx, int B, int G, hipStream_t stream);

}  // namespace pa
