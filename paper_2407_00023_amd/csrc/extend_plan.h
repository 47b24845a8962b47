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
    int slots;       // workgroup slots per KV head
    int rounds;      // work items aimed at per workgroup slot
    int pack;        // 1: rows of requests with a common prefix may be packed
    int first_part;  // ... of requests of up to this many rows also where they have only the first part of it in common (0: not)
    int tile_parts;  // parts of one tile at most
    int chunk_rows;  // rows per piece of the merge
    size_t off_tile, off_member, off_item, off_chunk, off_part_o, off_part_ml, total;
};

// limit: bytes that the plan may take (0: no limit); what may be left out to stay below it is.
ExtendPlan make_extend_plan(int B, int64_t T, int64_t max_kv_len, int Hq, int Hkv, int D, int rounds, size_t limit);
constexpr int kRounds = 2;        // the plan aims at about this many work items per workgroup slot (measured: with 3 a kernel
                                  // over long shared documents took 6 % longer - every item pays its start-up, its partial
                                  // results and their merge - with 1.5 its last round ran thin; the rest did not care)
constexpr int kRoundsStatic = 1;  // ... with the library's own scratch buffer as workspace (fewer partial results)

// Workspace: a header of 256 bytes - hdr[0] = row tiles, hdr[1] = work items, hdr[2] = pieces of the merge, hdr[3] = 1 if
// the batch on the device does not fit the plan (nothing is computed then), hdr[4] = rows of partial results, per KV head - and
// tables of int4:
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
