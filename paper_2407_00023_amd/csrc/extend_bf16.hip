// Extend attention on the bf16 matrix cores (MFMA 16x16x32, fp32 accumulate), gfx950.
//
// What is computed (Sec. 3.2 and Sec. 5 of the paper: only the missed tokens of a prompt
// are prefilled, the cached prefix KV is reused losslessly): extend row i of request r
// attends to the P_r prefix tokens, whose K/V rows are gathered from the paged pool
// through slot_idx, and causally to extend tokens 0..i.
//
// Decomposition.  The G = Hq/Hkv query heads of one KV head are packed with the extend
// rows into one row axis rho = i * G + (h mod G), so a K/V tile is read once per KV head.
// A workgroup of four waves owns 128 packed rows of one (request, KV head) and walks the
// key axis in tiles of kKT = 64 tokens: prefix positions first, then the extend tokens
// (the same loop; only the row address differs); where there are at most 32 rows, its waves share the keys
// instead (narrow tiles).  A planning kernel (extend_plan.hip) builds the list of work items per launch - row tile x part of
// its key range - from the lengths on the device; the parts of a split tile are merged by a third kernel.  Small batches go
// without list and merge: a workgroup finds its item from the lengths, the last one of a tile joins its parts (kDirect).
//
// Data movement.  K and V tiles go from global memory straight into LDS (16 bytes per
// lane, no register staging), one tile ahead of the arithmetic, into a ring of LDS
// buffers.  A wave's load lands as 1 KB of consecutive LDS bytes, so the bank-conflict
// swizzle is applied on the global-address side: the lane that owns LDS chunk c of a row
// fetches the row's chunk c ^ swizzle(row).
//
// MFMA formulation.  Scores are produced TRANSPOSED, S^T = K * Q^T, so that in the
// accumulator layout every lane holds two query rows (l % 16 and 16 more of the wave's 32) and 8 of the 32
// keys of a block for each: row statistics of the online softmax are per-lane scalars plus two
// exchanges between the lanes l, l ^ 16, l ^ 32, l ^ 48, and the probabilities are already laid out as the
// B operand of the second product O^T = V^T * P^T.  The V^T fragments are read from the
// row-major V tile with the transposing LDS read of gfx950.  (16x16x32 rather than 32x32x16: less energy for the same
// product, see gen_fast_run.py.)
//
// Two kinds of tile.  The general tile (general_block below) takes any mix of pool and extend rows, masks and
// ragged ends, and moves the running maximum; it runs where nothing else applies (heads of 64 on the fp8 pool or on
// pools of 4 GB and more, pages that are no power of two, the extend tokens in shared tiles, a tile that outgrew the frozen
// maximum, a first tile too short to seed one).  The rest executes in one assembly statement (fast_run.inc, written by
// gen_fast_run.py) with the running maximum frozen: runs of consecutive unmasked tiles, and single tiles, plain or on the
// causal diagonal.
#include <hip/hip_bf16.h>

#include <unistd.h>

#include <atomic>
#include <chrono>
#include <mutex>
#include <type_traits>

#include "extend_plan.h"
#include "fp8_rows.h"

namespace pa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

typedef __bf16 bf16x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x32 __attribute__((ext_vector_type(32)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

// the tiles as assembly with fixed registers, for heads of 128 and of 64
#include "fast_run.inc"

constexpr int kStages = 2;               // LDS ring: one tile being read, one being filled
constexpr float kRescaleThreshold = 8.f; // log2 units: the running maximum may lag the true one by this much
constexpr float kLargest = 3.4028234663852886e38f;  // the largest finite float
// The steady-state tiles (fast_run.inc) never move the running maximum: a run is left, for the general tile, when
// the probabilities of one row and key block sum to more than 2^40.  The exponent range of fp32 and bf16 leaves that
// much room: a probability of 2^40 is as precise as one of 1, and what then underflows next to it is < 2^-100 of it.

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    // round to nearest even; inputs are finite probabilities or outputs
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    f32x2 v = {a, b};
    bf16x2_t r = __builtin_convertvector(v, bf16x2_t);
    return __builtin_bit_cast(uint32_t, r);
}

// XOR swizzles of the 16-byte chunks of a K/V row in LDS, chosen so that the two read patterns of the
// arithmetic are free of bank conflicts: K is read 16 bytes per lane down 16 consecutive rows, V is read 8 bytes per lane across
// 32 bytes of 8 consecutive rows (by half a wave).
template <int D>
__device__ __forceinline__ int swz_k(int row) {
    return D == 128 ? (row & 15) : ((row >> 1) & 7);
}
template <int D>
__device__ __forceinline__ int swz_v(int row) {
    return ((D == 128 ? row & 3 : (row >> 1) & 1) << 2) | (((row >> 2) & 1) << 1) | ((row >> 3) & 1);
}

// The V^T fragments come from the transposing LDS read ds_read_b64_tr_b16: within each group of 16 lanes the
// 16 x 4 16-bit values addressed by the lanes form a flat array F (lane-major); lane i of the group receives
// F[i], F[16 + i], F[32 + i], F[48 + i].

// The largest of a query row's values, which lie in the lanes l, l ^ 16, l ^ 32 and l ^ 48, in all of them, without going through
// LDS.  v_permlane32_swap exchanges lanes 32..63 of its first operand with lanes 0..31 of its second, v_permlane16_swap the odd
// rows of 16 lanes of the first with the even ones of the second: fed the same value twice they leave both values of a pair in
// every lane.  Written as inline assembly (the compiler builtin folded its two results into one); the s_nop pairs cover the
// wait states the instructions need after a VALU write of their operands and before a VALU read of them.
__device__ __forceinline__ float row_max(float x) {
    float a = x, b = x;
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
    a = b = fmaxf(a, b);
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
    return fmaxf(a, b);
}
// ... and their sum.
__device__ __forceinline__ float row_sum(float x) {
    float a = x, b = x;
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
    a = b = a + b;
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
    return a + b;
}

// The lane's number, worked out anew: what is derived from it here is held by no register before.
__device__ __forceinline__ unsigned lane_here() {
    unsigned x;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(x));
    return x;
}

// Workgroup barrier without the memory fence of __syncthreads(): the fence would make the compiler wait
// for every outstanding global->LDS load, including the ones meant to stay in flight.  Completion of
// the loads that must be visible is awaited explicitly (wait_vm_all) before the barrier.
__device__ __forceinline__ void wg_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
// s_waitcnt vmcnt(0) (expcnt and lgkmcnt left alone), as the builtin so that the compiler's own wait
// bookkeeping sees it and does not repeat it later.
__device__ __forceinline__ void wait_vm_all() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);
    asm volatile("" ::: "memory");
}

// Direct global -> LDS load of 16 bytes per lane: lane l of the wave writes LDS bytes
// [lds_addr + 16 l, lds_addr + 16 l + 16) with the 16 bytes at its own global address g.  lds_addr is
// wave-uniform.  Issued as inline assembly so that the compiler does not see an LDS store in flight: it
// would otherwise wait for it before every later LDS read, and the load could not overlap the
// arithmetic on the other ring slot.  The explicit wait_vm_all() + wg_barrier() order it instead.
__device__ __forceinline__ void load_to_lds_16(const void* g, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(lds_addr) : "memory");
}
// The same with the global address given as a wave-uniform base plus a 32-bit unsigned byte offset per lane.
__device__ __forceinline__ void load_to_lds_16(const void* base, unsigned off, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds_addr) : "memory");
}
// One byte per lane: lane l of the wave writes the 32-bit word at lds_addr + 4 l (the byte in its low 8 bits).
__device__ __forceinline__ void load_to_lds_1(const void* g, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_ubyte %0, off" ::"v"(g), "s"(lds_addr) : "memory");
}
// Four bytes per lane, past the L2: lane l of the wave writes the 32-bit word at lds_addr + 4 l.
__device__ __forceinline__ void load_to_lds_4(const void* g, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off sc1" ::"v"(g), "s"(lds_addr) : "memory");
}
__device__ __forceinline__ unsigned lds_address(const void* p) {
    return static_cast<unsigned>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const unsigned char*)(p)));
}

// The K fragments of a block of 32 keys, all asked for before the first product, so that their LDS round trips overlap
// instead of following one another (the compiler, short of registers, reads one fragment at a time into the same four
// registers).  The wait stands in the same statement: no register of a read in flight is ever the compiler's to use.
// kf[2 s + kb]: k-slice s of the keys 16 kb .. 16 kb + 15, which lie kHalf bytes apart.
template <int kHalf, int KS>
__device__ __forceinline__ void read_k_block(bf16x8 (&kf)[2 * KS], const unsigned (&at)[KS], unsigned off) {
    static_assert(KS == 4 || KS == 2, "head dimension 128 or 64");
    if constexpr (KS == 4)
        asm volatile(
            "ds_read_b128 %0, %8\n\tds_read_b128 %1, %8 offset:%12\n\tds_read_b128 %2, %9\n\tds_read_b128 %3, %9 offset:%12\n\t"
            "ds_read_b128 %4, %10\n\tds_read_b128 %5, %10 offset:%12\n\tds_read_b128 %6, %11\n\tds_read_b128 %7, %11 offset:%12\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(kf[0]), "=&v"(kf[1]), "=&v"(kf[2]), "=&v"(kf[3]), "=&v"(kf[4]), "=&v"(kf[5]), "=&v"(kf[6]), "=&v"(kf[7])
            : "v"(at[0] + off), "v"(at[1] + off), "v"(at[2] + off), "v"(at[3] + off), "n"(kHalf)
            : "memory");
    else
        asm volatile(
            "ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:%6\n\tds_read_b128 %2, %5\n\tds_read_b128 %3, %5 offset:%6\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(kf[0]), "=&v"(kf[1]), "=&v"(kf[2]), "=&v"(kf[3])
            : "v"(at[0] + off), "v"(at[1] + off), "n"(kHalf)
            : "memory");
}

// A store of 16 bytes that goes through to memory: the workgroup that joins the parts of a tile may run on another XCD, whose
// L2 does not see this one's.  (The s_nop: a vector-ALU write of the data registers must stay two slots away.)
__device__ __forceinline__ void store_through_16(float* p, float4 v) {
    const f32x4 x = {v.x, v.y, v.z, v.w};
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(x) : "memory");
}
__device__ __forceinline__ float2 load_through_8(const float* p) {
    const unsigned long long x = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__uint_as_float(static_cast<unsigned>(x)), __uint_as_float(static_cast<unsigned>(x >> 32)));
}
__device__ __forceinline__ void store_through_8(float* p, float2 v) {
    const unsigned long long x = static_cast<unsigned long long>(__float_as_uint(v.x)) | static_cast<unsigned long long>(__float_as_uint(v.y)) << 32;
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What a workgroup of a launch without a work list needs to find its item (parts = 0: there is a work list).
struct DirectArgs {
    const int32_t *prefix_len, *ext_len, *ext_offsets, *slot_offsets;
    unsigned long long *join, tag;  // a word in the workspace per tile and KV head, and this call's number in its upper 56 bits (join_parts)
    int32_t* hdr;
    int B, parts, tile_rows, tiles, stride;
};

struct NoArgs {};

// The item of a workgroup of a launch without a work list, in the form of a record of the list: the parts of the first
// request's tiles, then the second's, and so on.  (Every request cuts all of its tiles into the same number of parts, so that
// the workgroups without an item are the last ones: scattered between the others, they left compute units empty while others
// had two items.)  *n_parts = parts of the tile, *tile = its number.  false: there is no such item.  Wave-uniform.
__device__ __forceinline__ bool direct_item(const DirectArgs& a, int item, int G, int Hkv, int4& rec0, int4& rec1, int4& rec2, int* n_parts, int* tile) {
    const int lane = threadIdx.x & 63;
    int P = 0, E = 0, e0 = 0, so = 0;
    if (lane < a.B) {
        P = a.prefix_len[lane];
        E = a.ext_len[lane];
        e0 = a.ext_offsets[lane];
        so = a.slot_offsets[lane];
    }
    // (a length that cannot fit counts as one that just does not: the sums stay small)
    const int rows = min(max(E, 0), a.stride / G + 1) * G;
    const int shortest = a.tile_rows == kNarrowRows ? kMinChunkNarrow : rows * Hkv <= kDirectJoinRows ? kDirectMinChunkWide : 2 * kDirectMinChunkWide;
    const int parts = max(1, min(a.parts, (P + E + kKT - 1) / kKT / shortest)), tiles = (rows + a.tile_rows - 1) / a.tile_rows;
    const int tiles_incl = wave_scan(tiles), rows_incl = wave_scan(rows), items_incl = wave_scan(tiles * parts);
    const int n_tiles = __builtin_amdgcn_readlane(tiles_incl, 63), n_rows = __builtin_amdgcn_readlane(rows_incl, 63);
    const int n_items = __builtin_amdgcn_readlane(items_incl, 63);
    const bool over = n_tiles > a.tiles || n_rows > a.stride;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.hdr[0] = over ? 0 : n_tiles;
        a.hdr[1] = over ? 0 : n_items;
        a.hdr[2] = 0;
        a.hdr[3] = over;
        a.hdr[4] = over || n_items == n_tiles ? 0 : n_rows * a.parts;  // (at most)
        a.hdr[5] = a.parts;
    }
    if (over || item >= n_items) return false;
    const int r = __popcll(__ballot(items_incl <= item));  // (the items of the requests up to this one are all before it)
    auto of = [&](int x) __attribute__((always_inline)) { return __builtin_amdgcn_readlane(x, r); };
    // (a request's last rows, the most keys, first)
    const int n_req = of(parts), local = item - (of(items_incl) - of(tiles) * n_req), at = local / n_req, j = local - at * n_req, t = of(tiles) - 1 - at;
    const int rP = of(P), all = of(rows);
    const int row0 = t * a.tile_rows, rows_here = min(a.tile_rows, all - row0);
    const int end = rP + (row0 + rows_here - 1) / G + 1, K = (end + kKT - 1) / kKT;
    const int n = min(n_req, K);
    if (j >= n) return false;
    // (K < 2^24 key tiles, n <= 16: the products fit 32 bits)
    const int lo = static_cast<int>(static_cast<unsigned>(K) * static_cast<unsigned>(j) / static_cast<unsigned>(n)) * kKT;
    const int hi = min(end, static_cast<int>(static_cast<unsigned>(K) * static_cast<unsigned>(j + 1) / static_cast<unsigned>(n)) * kKT);
    const int first = of(rows_incl) - all + row0;  // this tile's first row among the partial rows of a part
    rec0 = make_int4(first, row0, lo, hi);
    rec1 = make_int4(n > 1 ? j * a.stride + first : -1, rP, of(E), of(e0));
    rec2 = make_int4(of(so), rows_here <= kNarrowRows ? 1 : 0, 0, 0);
    *n_parts = n;
    *tile = of(tiles_incl) - of(tiles) + t;
    return true;
}

// LDS behind the K/V ring: the table of a shared tile's members (two ints each, one int more), two ints per wave, and, from
// kLdsMl on, what the waves of a narrow tile leave for one another.
constexpr int kLdsMl = ((2 * kTileRows + 1 + 2 * 4) * 4 + 15) & ~15;
constexpr int kLdsRows = kLdsMl + 4 * kNarrowRows * 8;
constexpr int kLdsTail = kLdsRows + kTileRows * 4;

// KV8: the pool holds one-byte codes and row exponents (fp8_rows.h) instead of bfloat16; its rows are decoded into the
// bfloat16 tiles in LDS, and everything from there on is the same arithmetic.
// kForm: a launch with a work list, or one without (DirectArgs, direct_item), of tiles of 128 rows (narrow where a tile has few) or of
// narrow ones only.  Kernels of their own, so that none of them keeps the registers and code of the others.
constexpr int kList = 0, kDirectWide = 1, kDirectNarrow = 2;
template <int D, bool KV8, int kForm>
__global__ __launch_bounds__(256, D == 64 ? (KV8 ? 4 : 3) : 2) void extend_bf16_kernel(
    const __hip_bfloat16* __restrict__ q_ext, const __hip_bfloat16* __restrict__ k_ext,
    const __hip_bfloat16* __restrict__ v_ext, const __hip_bfloat16* __restrict__ pool, const signed char* __restrict__ pool_exp,
    const int32_t* __restrict__ slot_idx, int Hq, int Hkv, int page_size, int page_shift, unsigned page_magic,
    int page_mshift, int num_slots, int fast_ok, float scale_log2e, __hip_bfloat16* __restrict__ out, const int32_t* __restrict__ hdr,
    const int4* __restrict__ item_tab, const int4* __restrict__ member_tab, float* __restrict__ part_o,
    float* __restrict__ part_ml, unsigned long long* __restrict__ clk, std::conditional_t<kForm != kList, DirectArgs, NoArgs> direct) {
    constexpr bool kDirect = kForm != kList;
    constexpr int NW = 4;                    // waves
    constexpr int MT = kTileRows;            // packed query rows per wide row tile, 32 per wave
    constexpr int RB = 2;                    // row blocks of a wave: its rows 0..15 and 16..31
    constexpr int NB = D / 16;               // MFMA row blocks of the head dimension in O^T
    constexpr int KS = D / 32;               // k-slices of the QK^T product
    constexpr int CPR = D / 8;               // 16-byte chunks per K/V row
    constexpr int ROWB = D * 2;              // bytes per row
    constexpr int TILEB = kKT * ROWB;        // bytes of one K (or V) tile
    constexpr int STAGEB = 2 * TILEB;        // one ring slot: K tile, V tile
    constexpr int RPB = 1024 / ROWB;         // rows per 1 KB block (what one wave-wide 16-byte load fills)
    constexpr int UPW = kKT / RPB / NW;      // blocks per wave, tile and tensor
    constexpr bool kAsm = D == 128 || !KV8;  // there are assembly tiles for this kernel
    static_assert(UPW >= 1, "tile too small for this many waves");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];  // [kStages][K tile | V tile]

    // block -> (work item, kv head); the kv head varies fastest so that with 8 kv heads every XCD (blocks are
    // dealt round-robin to the 8 XCDs) serves one head and keeps its shared prefixes in L2
    const int g = blockIdx.x % Hkv;
    const int item = blockIdx.x / Hkv;
    int4 rec0, rec1, rec2;
    [[maybe_unused]] int n_join = 0, join_tile = 0;  // parts of the tile, and its number, if its workgroups join them themselves
    if constexpr (kDirect) {
        if (!direct_item(direct, item, Hq / Hkv, Hkv, rec0, rec1, rec2, &n_join, &join_tile)) return;
    } else {
        if (item >= hdr[1]) return;
        rec0 = item_tab[3 * static_cast<size_t>(item)];
        rec1 = item_tab[3 * static_cast<size_t>(item) + 1];
        rec2 = item_tab[3 * static_cast<size_t>(item) + 2];
    }
    const int slot_off = rec2.x;
    const int row0 = rec0.y, kv_lo = rec0.z, kv_hi = rec0.w;
    const int prow = rec1.x;  // first row of this item's partial result; -1: the item covers all keys and writes the output
    const int P = rec1.y;  // keys of the prefix; in a shared tile: of the part of it that all members have in common
    const int G = Hq / Hkv;
    // packed rows by the size of the group: a shift where that is a power of two, as it mostly is (a division by a number that is
    // not known at compile time is thirty instructions)
    const int g_shift = (G & (G - 1)) == 0 ? __builtin_ctz(static_cast<unsigned>(G)) : -1;
    auto by_group = [&](int x) __attribute__((always_inline)) { return g_shift >= 0 ? x >> g_shift : x / G; };
    // a shared tile: rows of n_members requests with this prefix, laid end to end; after the common keys come the members'
    // extend tokens, member after member (unless only the first part of their prefixes is common: the tile ends there)
    const int member0 = __builtin_amdgcn_readfirstlane(rec2.z), n_members = kDirect ? 0 : __builtin_amdgcn_readfirstlane(rec2.w);
    const bool shared = n_members > 0;
    // Wide and narrow tiles have nothing but this in common, not even the code of their set-up: written once, compiled for each (values
    // of the one kept across the assembly of the other were spilled, and reloaded in the narrow tiles' loop behind its loads: 256
    // decode requests 69 -> 73 us).
    auto tile = [&](auto narrow_c) __attribute__((always_inline)) {
    constexpr bool narrow = decltype(narrow_c)::value;
    const int rows_total = shared ? rec1.z : rec1.z * G;
    const int rows_here = min(narrow ? kNarrowRows : MT, rows_total - row0);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g4 = lane >> 4;
    const int64_t e0 = rec1.w;
    const int32_t* __restrict__ slots = slot_idx + slot_off;

    // this lane's query rows are wave_row0 + 16 rb + n (a narrow tile: the same rows in every wave)
    const int wave_row0 = narrow ? 0 : wave * 32;
    const bool wave_on = wave_row0 < rows_here;
    // (the rows of a shared tile are their requests' last ones: no tile of its key range is skipped)
    const int wave_i_last = shared ? max(0, kv_hi - P) : by_group(row0 + min(rows_here, wave_row0 + 32) - 1);
    // the members of a shared tile: where a member's extend tokens begin on the tile's key axis (and, one past the last
    // member, where they end) and its first extend token counted from this item's
    // (behind the K/V ring in the dynamic LDS, which thereby keeps its alignment)
    int* const s_mseg = reinterpret_cast<int*>(smem + kStages * STAGEB);
    int* const s_mx0 = s_mseg + (MT + 1);
    int* const s_wave_own = s_mx0 + MT;  // per wave: the key range that holds the extend tokens of its rows' members
    float2* const s_ml = reinterpret_cast<float2*>(smem + kStages * STAGEB + kLdsMl);  // narrow tiles: (maximum, sum) per wave and row
    // the tile's rows of q and of the output; -1: none.  (Needed again behind the key loop only: kept in LDS, since a register
    // held across the loop was spilled, and asked back from memory.)
    int* const s_row = reinterpret_cast<int*>(smem + kStages * STAGEB + kLdsRows);
    // (a launch without a work list has no members: what is needed to join the parts of the tile, read behind the key loop)
    if constexpr (kDirect) {
        if (tid == 0) {
            s_mseg[0] = n_join;
            s_mseg[2] = join_tile;
            s_mseg[3] = rec0.x;
        }
        // (what the tile's word holds now, into s_mseg[4] and [5]: it flies during the key loop and takes no register)
        if (n_join > 1 && tid < 2)
            load_to_lds_4(reinterpret_cast<const unsigned*>(direct.join + join_tile * Hkv + g) + tid, __builtin_amdgcn_readfirstlane(lds_address(s_mseg + 4)));
    }
    if (shared) {
        if (tid < n_members) {  // (a member has at least one row in the tile: there are at most MT)
            const int4 mem = member_tab[2 * (member0 + tid)];
            const int at = P + member_tab[2 * (member0 + tid) + 1].x - member_tab[2 * member0 + 1].x;
            s_mseg[tid] = at;
            s_mx0[tid] = mem.y - static_cast<int>(rec1.w);
            if (tid == n_members - 1) s_mseg[n_members] = at + mem.w;
        }
        __syncthreads();
    }
    bf16x8 qreg[RB][KS];
    int vis_lo[RB], vis_end[RB]; // keys [.., vis_end) are visible to the row; in a shared tile [P, vis_lo) are other members' and hidden
    const int blk_vis_min = shared ? min(kv_hi, P) : min(kv_hi, P + by_group(row0 + wave_row0) + 1);  // every row of the wave sees keys [.., this)
    int rho[RB], e0_row[RB];     // packed row of its request; that one's first extend token
    bool row_ok[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        rho[rb] = row0 + wave_row0 + 16 * rb + n;
        row_ok[rb] = wave_row0 + 16 * rb + n < rows_here;
        e0_row[rb] = static_cast<int>(e0);
        vis_lo[rb] = P;
    }
    if (shared) {
        // whose rows these are: the last member that starts at or before a row; its place in that request; where
        // that member's extend tokens begin on the tile's key axis
        const int first = member_tab[2 * member0].x;
        const int want[RB] = {row_ok[0] ? rho[0] : first, row_ok[1] ? rho[1] : first};
        for (int k = 0; k < n_members; ++k) {
            const int4 mem = member_tab[2 * (member0 + k)];  // (same address in every lane)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                if (mem.x <= want[rb]) {
                    e0_row[rb] = mem.y;
                    rho[rb] = mem.z + (want[rb] - mem.x);
                    vis_lo[rb] = s_mseg[k];
                }
        }
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int r = row_ok[rb] ? rho[rb] : 0;
        const int qi = by_group(r), qh = g * G + (r - qi * G);  // extend index and query head
        vis_end[rb] = min(kv_hi, vis_lo[rb] + qi + 1);
        // (q and the output, of 64 elements a row and more, both have to fit the memory: fewer than 2^31 rows)
        const int q_row = (e0_row[rb] + qi) * Hq + qh;
        s_row[wave_row0 + 16 * rb + n] = row_ok[rb] ? q_row : -1;
        const uint4* qp = reinterpret_cast<const uint4*>(q_ext + q_row * static_cast<int64_t>(D));
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            uint4 v = make_uint4(0, 0, 0, 0);
            if (row_ok[rb]) v = qp[4 * s + g4];
            qreg[rb][s] = __builtin_bit_cast(bf16x8, v);
        }
    }

    // In a shared tile the keys past the common part concern one member each: the wave skips the arithmetic of a tile
    // that holds no key of the members its rows belong to (uniform over the wave).
    if (shared) {
        int wave_own_lo = min(vis_lo[0], vis_lo[1]), wave_own_hi = max(vis_end[0], vis_end[1]);
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            wave_own_lo = min(wave_own_lo, __shfl_xor(wave_own_lo, off));
            wave_own_hi = max(wave_own_hi, __shfl_xor(wave_own_hi, off));
        }
        if (lane == 0) {  // (kept in LDS, not in registers: read, by this wave only, in the own-key part of a shared tile)
            s_wave_own[2 * wave] = wave_own_lo;
            s_wave_own[2 * wave + 1] = wave_own_hi;
        }
    }

    // ---- global -> LDS tile loads.  Wave w fills blocks w * UPW + u: rows blk * RPB + lane / CPR, and the
    // lane lands on chunk position lane % CPR of its row.
    const int ld_pos = lane % CPR;
    const int ld_rowl = lane / CPR;
    const unsigned char* pool_g = reinterpret_cast<const unsigned char*>(pool) + static_cast<size_t>(g) * page_size * ROWB;
    const unsigned page_stride = 2u * Hkv * page_size * ROWB;  // bytes from one page to the next (< 4 GB, checked on the host)
    const unsigned v_off32 = static_cast<unsigned>(Hkv) * page_size * ROWB;      // from a K row to its V row
    const unsigned char* kx_g = reinterpret_cast<const unsigned char*>(k_ext) + (e0 * Hkv + g) * static_cast<int64_t>(ROWB);
    const unsigned char* vx_g = reinterpret_cast<const unsigned char*>(v_ext) + (e0 * Hkv + g) * static_cast<int64_t>(ROWB);
    // (strides within a page and a token fit 31 bits, checked on the host: products with them are one 32 x 32 bit multiplication)
    const int x_stride = Hkv * ROWB;  // bytes from one extend token to the next
    const unsigned smem_addr = __builtin_amdgcn_readfirstlane(lds_address(smem));
    // Pool slots of rows of the tile after the one in flight.  Heads of 128: of one row of the wave's sixteen, 4 (lane % 4) + lane / 16; the
    // lanes 16 j .. 16 j + 15, which load row 4 u + j in block u, have it from lane 16 j + u.  Heads of 64: of the rows that the lane loads.
    constexpr int NSL = D == 128 ? 1 : UPW;
    int32_t sl_next[NSL];
    const int sl_row = D == 128 ? 4 * (lane & 3) + (lane >> 4) : ld_rowl;
    // The lane's number where a tile's general loads and slot ids need it: asked for anew in the kernels with assembly tiles, whose
    // registers that fills.  (What the loads derive from it was kept from tile to tile, spilled, and each reload waited for the loads
    // issued just before it: 16 questions to long documents on the fp8 pool 281 us a step, so 278.  Heads of 64 on the fp8 pool run
    // this code for every tile and have the registers: 17 questions to a document 232, so 236.)
    auto lane_again = [&]() __attribute__((always_inline)) { return kAsm ? static_cast<int>(lane_here() & 63) : lane; };
    auto slot_row = [&]() __attribute__((always_inline)) {
        if constexpr (!kAsm) return sl_row;
        const int l = lane_again();
        return D == 128 ? 4 * (l & 3) + (l >> 4) : l / CPR;
    };
    auto slot_of = [&](int u) __attribute__((always_inline)) -> int {  // (all lanes; u known at compile time)
        if constexpr (D == 128)
            return u == 0   ? __builtin_amdgcn_update_dpp(0, sl_next[0], 0x150, 0xf, 0xf, false)
                   : u == 1 ? __builtin_amdgcn_update_dpp(0, sl_next[0], 0x151, 0xf, 0xf, false)
                   : u == 2 ? __builtin_amdgcn_update_dpp(0, sl_next[0], 0x152, 0xf, 0xf, false)
                            : __builtin_amdgcn_update_dpp(0, sl_next[0], 0x153, 0xf, 0xf, false);
        else
            return sl_next[u];
    };

    // (first member of a shared tile whose own keys reach the tile asked for; the tiles are asked for in order)
    int cur_member = 0;
    auto member_at = [&](int cur, int p) __attribute__((always_inline)) {  // the member whose own keys hold key p >= P
        int k = cur;
        while (k + 1 < n_members && p >= s_mseg[k + 1]) ++k;
        return k;
    };
    auto load_slots = [&](int p0) __attribute__((always_inline)) {
        const int row = slot_row();
#pragma unroll
        for (int u = 0; u < NSL; ++u) {
            // positions past the end of the key range repeat the last valid one (see issue)
            const int p = min(p0 + (wave * UPW + u) * RPB + row, kv_hi - 1);
            sl_next[u] = p < P ? slots[p] : 0;
        }
    };
    // Byte offset, inside its K (V) row, of the 16 bytes this lane fetches for block u.  Block u of the wave holds
    // rows 16 w + 4 u + lane / 16 (D = 128), so its swizzle differs from that of block 0 by an XOR with 4 u (K) or
    // 2 (u % 2) + u / 2 (V); for D = 64 (rows 16 w + 8 u + lane / 8) by an XOR with 4 u (K) or u (V).
    const unsigned ld_koff0 = (ld_pos ^ swz_k<D>(wave * UPW * RPB + ld_rowl)) * 16;
    const unsigned ld_voff0 = (ld_pos ^ swz_v<D>(wave * UPW * RPB + ld_rowl)) * 16;
    // (Worked out where they are used, from a value the compiler cannot see through: left to itself it keeps all eight
    // of them as 64-bit addends, spills them, and each reload waits for the tile load issued just before it - eight
    // loads in a row, one memory round trip each.)
    auto opaque = [](unsigned x) __attribute__((always_inline)) {
        asm volatile("" : "+v"(x));
        return x;
    };
    auto ld_koff = [&](int u) __attribute__((always_inline)) { return opaque(ld_koff0) ^ (64u * u); };
    auto v_swizzle = [](int u) __attribute__((always_inline)) { return 16u * (D == 128 ? 2 * (u & 1) + (u >> 1) : u); };
    auto ld_voff = [&](int u) __attribute__((always_inline)) { return opaque(ld_voff0) ^ v_swizzle(u); };
    // The next tile's loads, general: every lane takes its row from the pool (through the slot prefetched for it) or
    // from the extend tensors, by position; rows past the end of the key range repeat the last valid row (finite
    // values that the mask zeroes).  The page of a slot: a shift where the page size is a power of two
    // (page_shift >= 0), otherwise the exact quotient by a multiplication (see page_divider).
    auto issue = [&](int p0, int ring) __attribute__((always_inline)) {
        const unsigned sk = __builtin_amdgcn_readfirstlane(smem_addr + ring * STAGEB);  // wave-uniform (goes to M0)
        if (shared)
            while (cur_member + 1 < n_members && s_mseg[cur_member + 1] <= p0) ++cur_member;
        const int rowl = lane_again() / CPR;
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
            const int blk = wave * UPW + u;
            const int p = min(p0 + blk * RPB + rowl, kv_hi - 1);
            const bool ext = p >= P;
            const unsigned sl = static_cast<unsigned>(min(max(slot_of(u), 0), num_slots - 1));  // never outside the pool
            const unsigned pg = page_shift >= 0 ? sl >> page_shift : __umulhi(sl, page_magic) >> page_mshift;
            const size_t pool_off = static_cast<size_t>(pg) * page_stride +
                                    (sl - pg * static_cast<unsigned>(page_size)) * static_cast<unsigned>(ROWB);
            int xrow = p - P;  // extend token, counted from the first one of the request of this item
            if (shared && ext) {
                // the member whose extend tokens hold key p, and that token relative to e0
                const int k = member_at(cur_member, p);
                xrow = s_mx0[k] + (p - s_mseg[k]);
            }
            const size_t off = ext ? static_cast<size_t>(static_cast<int64_t>(xrow) * x_stride) : pool_off;
            const unsigned char* ka = (ext ? kx_g : pool_g) + off + ld_koff(u);
            const unsigned char* va = (ext ? vx_g : pool_g + v_off32) + off + ld_voff(u);
            load_to_lds_16(ka, sk + blk * 1024);
            load_to_lds_16(va, sk + TILEB + blk * 1024);
        }
    };

    // ---- fp8 pool.  A pool row arrives as its D codes, in the first half of the LDS bytes its bfloat16 form will take
    // (the lanes that would fetch the second half stay idle), and its exponent as one byte in a small staging area of
    // the wave; rows of the extend tensors arrive as before.  Once the loads have landed, landed8() turns the codes
    // into bfloat16 in place: the lanes of a row (one wave, in step) all read their 8 codes before any of them writes,
    // and no other wave touches the row until the barrier that follows.
    constexpr int EXPB = 256 * 2 * UPW;  // staging bytes per wave: one 32-bit word per lane, load block and tensor
    constexpr int EX_OFF = (kStages * STAGEB + kLdsTail + 255) & ~255;
    const unsigned char* pool8_g = reinterpret_cast<const unsigned char*>(pool) + static_cast<size_t>(g) * page_size * D;
    const unsigned page_stride8 = 2u * Hkv * page_size * D;
    const unsigned v_off8 = static_cast<unsigned>(Hkv) * page_size * D;
    const signed char* exp_g = pool_exp + static_cast<size_t>(g) * page_size;
    const unsigned exp_page = 2u * Hkv * page_size, exp_v = static_cast<unsigned>(Hkv) * page_size;
    int raw_mask = 0;  // bit u: this lane's row of load block u is a pool row (codes to be decoded)
    auto issue8 = [&](int p0, int ring) __attribute__((always_inline)) {
        const unsigned sk = __builtin_amdgcn_readfirstlane(smem_addr + ring * STAGEB);
        const unsigned ex = __builtin_amdgcn_readfirstlane(smem_addr + EX_OFF + wave * EXPB);
        if (shared)
            while (cur_member + 1 < n_members && s_mseg[cur_member + 1] <= p0) ++cur_member;
        raw_mask = 0;
        const int l_here = lane_again(), pos = l_here % CPR, rowl = l_here / CPR;
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
            const int blk = wave * UPW + u;
            const int p = min(p0 + blk * RPB + rowl, kv_hi - 1);
            const bool ext = p >= P;
            const unsigned sl = static_cast<unsigned>(min(max(slot_of(u), 0), num_slots - 1));  // never outside the pool
            const unsigned pg = page_shift >= 0 ? sl >> page_shift : __umulhi(sl, page_magic) >> page_mshift;
            const unsigned o = sl - pg * static_cast<unsigned>(page_size);
            int xrow = p - P;
            if (shared && ext) {
                const int k = member_at(cur_member, p);
                xrow = s_mx0[k] + (p - s_mseg[k]);
            }
            if (ext) {
                const size_t off = static_cast<size_t>(static_cast<int64_t>(xrow) * x_stride);
                load_to_lds_16(kx_g + off + ld_koff(u), sk + blk * 1024);
                load_to_lds_16(vx_g + off + ld_voff(u), sk + TILEB + blk * 1024);
            } else {
                raw_mask |= 1 << u;
                if (pos < CPR / 2) {
                    const unsigned char* ka = pool8_g + static_cast<size_t>(pg) * page_stride8 + o * static_cast<unsigned>(D) + pos * 16;
                    load_to_lds_16(ka, sk + blk * 1024);
                    load_to_lds_16(ka + v_off8, sk + TILEB + blk * 1024);
                }
                if (D == 64 && pos == 0) {
                    const signed char* ea = exp_g + static_cast<size_t>(pg) * exp_page + o;
                    load_to_lds_1(ea, ex + (2 * u) * 256);
                    load_to_lds_1(ea + exp_v, ex + (2 * u + 1) * 256);
                }
            }
        }
        if constexpr (D == 128) {  // (lane 16 j + u those of row 4 u + j, as the assembly does)
            if (pos < UPW && min(p0 + wave * UPW * RPB + 4 * (l_here & 3) + (l_here >> 4), kv_hi - 1) < P) {
                const unsigned sl = static_cast<unsigned>(min(max(sl_next[0], 0), num_slots - 1));
                const unsigned pg = page_shift >= 0 ? sl >> page_shift : __umulhi(sl, page_magic) >> page_mshift;
                const signed char* ea = exp_g + static_cast<size_t>(pg) * exp_page + (sl - pg * static_cast<unsigned>(page_size));
                load_to_lds_1(ea, ex);
                load_to_lds_1(ea + exp_v, ex + 256);
            }
        }
    };
    // the tile in ring slot `ring` has landed (this wave's loads have been waited for): decode this wave's pool rows
    auto landed8 = [&](int ring) __attribute__((always_inline)) {
        unsigned char* const sk = smem + ring * STAGEB;
        const int* const ex = reinterpret_cast<const int*>(smem + EX_OFF + wave * EXPB);
        const int l_here = lane_again();
        uint2 kraw[UPW], vraw[UPW];
        int ke[UPW], ve[UPW];
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
            if ((raw_mask >> u) & 1) {
                const unsigned char* row = sk + (wave * UPW + u) * 1024 + l_here / CPR * ROWB;
                kraw[u] = *reinterpret_cast<const uint2*>(row + (ld_koff(u) >> 1));
                vraw[u] = *reinterpret_cast<const uint2*>(row + TILEB + (ld_voff(u) >> 1));
                ke[u] = D == 128 ? ex[(l_here & ~15) + u] : ex[(2 * u) * 64 + (l_here & ~(CPR - 1))];
                ve[u] = D == 128 ? ex[64 + (l_here & ~15) + u] : ex[(2 * u + 1) * 64 + (l_here & ~(CPR - 1))];
            }
        }
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
            if ((raw_mask >> u) & 1) {
                unsigned char* dst = sk + (wave * UPW + u) * 1024 + l_here * 16;
                const float ks = fp8_scale(static_cast<int>(static_cast<signed char>(ke[u] & 0xFF)));
                const float vs = fp8_scale(static_cast<int>(static_cast<signed char>(ve[u] & 0xFF)));
                const uint2 ka = fp8_decode4(kraw[u].x, ks), kb = fp8_decode4(kraw[u].y, ks);
                const uint2 va = fp8_decode4(vraw[u].x, vs), vb = fp8_decode4(vraw[u].y, vs);
                *reinterpret_cast<uint4*>(dst) = make_uint4(ka.x, ka.y, kb.x, kb.y);
                *reinterpret_cast<uint4*>(dst + TILEB) = make_uint4(va.x, va.y, vb.x, vb.y);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the barrier that follows does not wait for LDS writes
    };
    auto issue_any = [&](int p0, int ring) __attribute__((always_inline)) {
        if constexpr (KV8) issue8(p0, ring);
        else issue(p0, ring);
    };

    f32x4 oacc[RB][NB];
    float m_run[RB] = {-INFINITY, -INFINITY}, l_run[RB] = {0.f, 0.f};  // running maximum (scaled, log2 domain) and this lane's share of the sum
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int b = 0; b < NB; ++b) oacc[rb][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    // ---- LDS read addresses of this lane in the ring slot that holds the current tile (toggled after every tile).
    // K: row n (+16 for the second half of a block, +32 for the second block), 16-byte chunk 4 s + g4 of the row.
    // V, transposing read: group lane i = 4 e + c reads key row 4 g4 + e (+ 16 for the second half, + 32 for the second block) and
    // 8 bytes at head-dim offset 16 b + 4 c.  The swizzles do not depend on halves and blocks, which become immediates.
    typedef __attribute__((address_space(3))) const unsigned char lds_cbyte;
    lds_cbyte* lds = (lds_cbyte*)nullptr;  // k_rd / v_rd hold absolute LDS addresses
    unsigned k_rd[KS], v_rd[NB];
    {
        const int tr_e = (lane >> 2) & 3, tr_c = lane & 3;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            k_rd[s] = smem_addr + n * ROWB + (((4 * s + g4) ^ swz_k<D>(n)) * 16);
            asm volatile("" : "+v"(k_rd[s]));  // keep it in a register instead of recomputing it every tile
        }
        const int vrow = 4 * g4 + tr_e;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            v_rd[b] = smem_addr + TILEB + vrow * ROWB + (((2 * b + (tr_c >> 1)) ^ swz_v<D>(vrow)) * 16) + (tr_c & 1) * 8;
            asm volatile("" : "+v"(v_rd[b]));
        }
    }

    const bf16x2_t ones = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};

    // ---- One block of 32 keys of the current tile, general: masks, any running maximum.  Kept small in registers
    // (one score block alive, no overlap of its phases inside the wave; the other wave of the SIMD fills the gaps):
    // it runs wherever the assembly tiles do not apply.  mb = 0 / 1: first / second block of the tile.
    auto general_block = [&](int p0, int mb, bool need_mask) __attribute__((always_inline)) {
        const unsigned off = static_cast<unsigned>(mb) * (32 * ROWB);
        const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
        f32x4 sacc[2][RB];  // [half of the block's keys][row block]
        // S^T = K Q^T
        bf16x8 kf[2 * KS];
        read_k_block<16 * ROWB>(kf, k_rd, off);
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
                    sacc[kb][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[2 * s + kb], qreg[rb][s], s == 0 ? zero4 : sacc[kb][rb], 0, 0, 0);
        const int pb0 = p0 + 32 * mb;
        // the keys a row must not see (only where the block crosses a visibility limit)
        // (register i of half kb holds the key at offset 16 kb + i from the lane's first key of the block:
        // compared, without branches, against the row's limits counted from that key)
        if (need_mask && pb0 + 32 > blk_vis_min) {
            const int first = pb0 + 4 * g4;
            if (!shared) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    const int lim_end = vis_end[rb] - first;
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int i = 0; i < 4; ++i) sacc[kb][rb][i] = (16 * kb + i < lim_end) ? sacc[kb][rb][i] : -INFINITY;
                }
            } else {
                const int lim_p = P - first;
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    const int lim_end = vis_end[rb] - first, lim_lo = vis_lo[rb] - first;
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int o = 16 * kb + i;
                            const bool hide = (o >= lim_end) | ((o >= lim_p) & (o < lim_lo));
                            sacc[kb][rb][i] = hide ? -INFINITY : sacc[kb][rb][i];
                        }
                }
            }
        }
        // largest score of the block that this lane holds, by row
        float mx[RB], neg_m[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            mx[rb] = sacc[0][rb][0];
#pragma unroll
            for (int i = 1; i < 8; ++i) mx[rb] = fmaxf(mx[rb], sacc[i / 4][rb][i % 4]);
            // (no maximum yet: any finite score exceeds it, and of hidden keys, -inf, the probability is 0 whatever stands here)
            neg_m[rb] = fminf(-m_run[rb], kLargest);
        }
        // The running maximum may lag the true one by kRescaleThreshold (probabilities then reach 2^threshold,
        // harmless in bf16/fp32).  If some row of the wave outgrew it by more, raise it and rescale what was
        // accumulated so far.  With a stable maximum this happens for the first block only, so only there are the lanes of a row
        // brought together.  (What bounds heads of 64 on the fp8 pool, which run this code for every tile with four waves a SIMD, is
        // its vector instructions: 78 a block, exponentials aside, with the maxima of all rows, the dot products and one address per fragment,
        // now 46.)
        const float over = fmaxf(fmaf(mx[0], scale_log2e, neg_m[0]), fmaf(mx[1], scale_log2e, neg_m[1]));  // log2 domain (scale > 0)
        if (__builtin_amdgcn_ballot_w64(over > kRescaleThreshold) != 0) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const float m_new = fmaxf(m_run[rb], row_max(mx[rb]) * scale_log2e);
                const float alpha = __builtin_amdgcn_exp2f(m_run[rb] - ((m_new == -INFINITY) ? 0.f : m_new));
                l_run[rb] *= alpha;
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int i = 0; i < 4; ++i) oacc[rb][b][i] *= alpha;
                m_run[rb] = m_new;
                neg_m[rb] = fminf(-m_new, kLargest);
            }
        }
        // probabilities, packed to bf16 pairs (the B operand of the second product: its k-slots of lane group g4 are the keys
        // 4 g4 .. 4 g4 + 3 of the block's halves, and so are those of the V^T fragments); the row sum takes the
        // ROUNDED probabilities, the values the numerator uses
        // ... wide tiles that have no others (heads of 64 on the fp8 pool): by a product with a row of ones, two matrix instructions in
        // place of twelve vector ones.  (In narrow tiles, which wait for memory, it costs registers: 103 decode requests 57.0 -> 58.4 us.)
        constexpr bool kSumProduct = !kAsm && !narrow;
        bf16x8 pop[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            uint32_t pb[4];
            float acc = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float a = __builtin_amdgcn_exp2f(fmaf(sacc[k / 2][rb][2 * (k % 2)], scale_log2e, neg_m[rb]));
                const float b = __builtin_amdgcn_exp2f(fmaf(sacc[k / 2][rb][2 * (k % 2) + 1], scale_log2e, neg_m[rb]));
                pb[k] = pack_bf16x2(a, b);
                if constexpr (!kSumProduct) acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, pb[k]), ones, acc, false);
            }
            pop[rb] = __builtin_bit_cast(bf16x8, make_uint4(pb[0], pb[1], pb[2], pb[3]));
            if constexpr (!kSumProduct) l_run[rb] += acc;
        }
        f32x4 sums[RB];
        if constexpr (kSumProduct) {
            const uint32_t one2 = n == 0 ? 0x3f803f80u : 0u;
            const bf16x8 one = __builtin_bit_cast(bf16x8, make_uint4(one2, one2, one2, one2));
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) sums[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(one, pop[rb], zero4, 0, 0, 0);
        }
        // O^T += V^T P^T
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            s16x4 frag[2];
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2)
                frag[h2] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(lds + (v_rd[b] + off + h2 * 16 * ROWB)));
            const bf16x8 vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(frag[0], frag[1], 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) oacc[rb][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pop[rb], oacc[rb][b], 0, 0, 0);
        }
        if constexpr (kSumProduct) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) l_run[rb] += sums[rb][0];
        }
    };

    // One tile, general: any mix of prefix and extend rows, masks, ragged ends, any page size.  from = 1: the first
    // key block is already accumulated; issue_next = false: the next tile's loads are already in flight.
    auto tile_general = [&](int p0, int ring, int from, bool issue_next) __attribute__((always_inline)) {
        if (issue_next && p0 + kKT < kv_hi) {
            issue_any(p0 + kKT, ring ^ 1);  // the next tile flies during this tile's arithmetic
            load_slots(p0 + 2 * kKT);
        } else if (issue_next) {
            raw_mask = 0;  // (the last tile: nothing lands after it)
        }
        const bool not_ours = shared && p0 >= P && (p0 >= s_wave_own[2 * wave + 1] || p0 + kKT <= s_wave_own[2 * wave]);
        if (wave_on && p0 <= P + wave_i_last && !not_ours) {
            const bool need_mask = p0 + kKT > blk_vis_min;
#pragma unroll 1
            for (int mb = from; mb < 2; ++mb) general_block(p0, mb, need_mask);
        }
    };
    // 0: the tile at p0 takes the general code; 1 / 2: the hand-scheduled one, the next tile lying wholly in the
    // prefix / wholly in the extend tokens (its rows clamp to the last valid key).  Uniform over the wave.
    auto tile_kind = [&](int p0) __attribute__((always_inline)) -> int {
        if (!(fast_ok && kAsm && (smem_addr & 255u) == 0)) return 0;
        if (!(wave_on && p0 <= P + wave_i_last && p0 + kKT <= blk_vis_min)) return 0;
        const int first = min(p0 + kKT, kv_hi - 1), last = min(p0 + 2 * kKT - 1, kv_hi - 1);
        // (after the common keys of a shared tile come several requests' keys: never one run of extend tokens)
        // (fp8 pool: fast_ok bit 0 allows runs over the extend tokens, bit 1 runs over the pool)
        if (last < P) return !KV8 || (fast_ok & 2) ? 1 : 0;
        return (first >= P && !shared && (!KV8 || (fast_ok & 1))) ? 2 : 0;
    };

    // ---- a launch without a work list: the parts of a tile are joined by the workgroup that finishes last.  A word of the
    // workspace per tile and KV head counts the parts that have finished.  It may hold anything beforehand: every part first
    // sees to it that it holds this call's number and a count of 0 (claim_word; whoever comes first exchanges what was there
    // for that, for the others the exchange fails), and the last one leaves 0, so that a captured call, whose number is the
    // same in every replay, finds no count of its own.  The library keeps nothing outside the workspace, so calls with workspaces
    // of their own never meet, whatever their streams, threads and graphs.  (Counters in arrays of the library's, a set per
    // stream, were shared as soon as more streams called than there were sets.)  Nobody waits for anybody; partial results are stored
    // through to memory and awaited before the count, and read past this XCD's L2, which may hold what an earlier call left
    // there.  The word is asked for before the key loop and claimed ahead of the stores, so that its
    // round trips hide behind them: a step of four decode requests takes 28.9 us with counters known to be 0, 29.2 so. ----
    [[maybe_unused]] auto claim_word = [&]() __attribute__((always_inline)) {
        if constexpr (kDirect) {
            if (prow >= 0 && tid == 0) {
                wait_vm_all();
                const unsigned long long seen = static_cast<unsigned long long>(static_cast<unsigned>(s_mseg[5])) << 32 | static_cast<unsigned>(s_mseg[4]);
                unsigned long long expected = seen;
                if ((seen ^ direct.tag) >> 8 != 0)
                    (void)__hip_atomic_compare_exchange_strong(direct.join + s_mseg[2] * Hkv + g, &expected, direct.tag, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    };
    // All threads; prow >= 0.
    [[maybe_unused]] auto join_parts = [&]() __attribute__((always_inline)) {
        if constexpr (kDirect) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            const int n = __builtin_amdgcn_readfirstlane(s_mseg[0]);
            if (tid == 0) {
                unsigned long long* const word = direct.join + s_mseg[2] * Hkv + g;
                const unsigned long long before = __hip_atomic_fetch_add(word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const bool last = static_cast<int>(before & 255) == n - 1;
                if (last) __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s_mseg[1] = last;
            }
            __syncthreads();
            if (!s_mseg[1]) return;
            const size_t base = static_cast<size_t>(s_mseg[3]) * Hkv + static_cast<size_t>(g) * rows_here;
            const size_t step = static_cast<size_t>(direct.stride) * Hkv;
            // what each part of a row counts for: 2^(its maximum - the row's), over the row's sum (the LDS ring is free by now)
            constexpr int kW = kDirectWideParts * MT;
            static_assert(kMaxDirectParts * kNarrowRows <= kW && 2 * kW * 4 <= kStages * STAGEB, "fits the ring");
            float* const s_w = reinterpret_cast<float*>(smem);  // [part][row]: maximum, then weight
            float* const s_l = s_w + kW;                        // ... sum
            auto weigh = [&]() __attribute__((always_inline)) {
                for (int x = tid; x < rows_here * n; x += 256) {
                    const int s = x / rows_here;
                    const float2 ml = load_through_8(part_ml + 2 * (base + (x - s * rows_here) + s * step));
                    s_w[x] = ml.x;
                    s_l[x] = ml.y;
                }
                __syncthreads();
                if (tid < rows_here) {
                    float m = -INFINITY, l = 0.f;
                    for (int s = 0; s < n; ++s) m = fmaxf(m, s_w[s * rows_here + tid]);  // (some part has seen a key)
                    for (int s = 0; s < n; ++s) {
                        const float w = __builtin_amdgcn_exp2f(s_w[s * rows_here + tid] - m);
                        s_w[s * rows_here + tid] = w;
                        l += w * s_l[s * rows_here + tid];
                    }
                    const float inv = 1.f / l;
                    for (int s = 0; s < n; ++s) s_w[s * rows_here + tid] *= inv;
                }
                __syncthreads();
            };
            constexpr int V4 = D / 4;   // 16-byte pieces per partial row: one thread per (row, piece)
            const int n_x = rows_here * V4;
            auto store_row = [&](int x, float4 acc) __attribute__((always_inline)) {
                const int rr = row0 + x / V4;
                reinterpret_cast<uint2*>(out + ((e0 + rr / G) * Hq + g * G + rr % G) * static_cast<int64_t>(D))[x % V4] =
                    make_uint2(pack_bf16x2(acc.x, acc.y), pack_bf16x2(acc.z, acc.w));
            };
            // kX (row, piece) pairs of a thread and kS parts of each in flight
            auto sum_parts = [&](auto k_x, auto k_s, int x0, int s0, float4* acc, auto before_use) __attribute__((always_inline)) {
                constexpr int kX = decltype(k_x)::value, kS = decltype(k_s)::value;
                float2 a[kX][kS], b[kX][kS];
#pragma unroll
                for (int k = 0; k < kX; ++k) {
                    const int x = min(x0 + 256 * k, n_x - 1);
#pragma unroll
                    for (int u = 0; u < kS; ++u) {
                        const float* from = part_o + (base + x / V4 + min(s0 + u, n - 1) * step) * D + 4 * (x % V4);
                        a[k][u] = load_through_8(from);
                        b[k][u] = load_through_8(from + 2);
                    }
                }
                before_use();
#pragma unroll
                for (int k = 0; k < kX; ++k) {
                    const int x = min(x0 + 256 * k, n_x - 1);
#pragma unroll
                    for (int u = 0; u < kS; ++u) {
                        if (s0 + u >= n) continue;  // (the last part again: 0 times it is no 0 where it holds an infinity)
                        const float w = s_w[(s0 + u) * rows_here + x / V4];
                        acc[k].x += w * a[k][u].x; acc[k].y += w * a[k][u].y; acc[k].z += w * b[k][u].x; acc[k].w += w * b[k][u].y;
                    }
                }
            };
            const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
            if (n_x <= 256) {
                // (few rows: everything a thread sums is asked for at once, the maxima and sums behind it)
                static_assert(kMaxDirectParts == 16, "in one go");
                float4 acc[1] = {zero};
                sum_parts(std::integral_constant<int, 1>{}, std::integral_constant<int, 16>{}, tid, 0, acc, weigh);
                if (tid < n_x) store_row(tid, acc[0]);
            } else {
                constexpr int kX = 4, kS = 4;
                weigh();
                for (int x0 = tid; x0 < n_x; x0 += 256 * kX) {
                    float4 acc[kX] = {zero, zero, zero, zero};
                    for (int s0 = 0; s0 < n; s0 += kS)
                        sum_parts(std::integral_constant<int, kX>{}, std::integral_constant<int, kS>{}, x0, s0, acc, [] {});
#pragma unroll
                    for (int k = 0; k < kX; ++k)
                        if (x0 + 256 * k < n_x) store_row(x0 + 256 * k, acc[k]);
                }
            }
        }
    };

    // ---- narrow tiles: at most 32 rows, so that one wave's registers hold them all, and the four waves take the keys in
    // turn, 32 at a time, each through a quarter of the LDS ring of its own: no barrier until the end, where the four partial
    // results are joined.  What bounds them is memory (a few rows make little arithmetic): eight waves of a compute unit have
    // 16 KB each on the way.  (As a wide tile, one wave at work between two barriers per 64 keys, they took three times as
    // long.) ----
    if constexpr (narrow) {
        constexpr int NLB = 32 / RPB;           // 1 KB load blocks of 32 rows, per tensor
        constexpr int VOFF = 32 * ROWB;         // the V rows lie behind the K rows
        constexpr int WB = kStages * STAGEB / NW;
        static_assert(WB == 2 * VOFF, "a quarter of the ring holds 32 K rows and 32 V rows");
        const unsigned wbase = __builtin_amdgcn_readfirstlane(smem_addr + wave * WB);
#pragma unroll
        for (int s = 0; s < KS; ++s) k_rd[s] += wave * WB;
#pragma unroll
        for (int b = 0; b < NB; ++b) v_rd[b] += wave * WB + VOFF - TILEB;
        // (rows RPB u + lane / CPR: the swizzles repeat after 4 (D = 128) or 2 (D = 64) load blocks)
        const unsigned koff0 = (ld_pos ^ swz_k<D>(ld_rowl)) * 16, voff0 = (ld_pos ^ swz_v<D>(ld_rowl)) * 16;
        auto koff = [&](int u) __attribute__((always_inline)) { return opaque(koff0) ^ (64u * (u & (D == 128 ? 3 : 1))); };
        auto voff = [&](int u) __attribute__((always_inline)) { return opaque(voff0) ^ v_swizzle(u & (D == 128 ? 3 : 1)); };
        int32_t sl[NLB];
        auto ask_slots = [&](int p0) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < NLB; ++u) {
                const int p = min(p0 + u * RPB + ld_rowl, kv_hi - 1);
                sl[u] = p < P ? slots[p] : 0;
            }
        };
        int p = kv_lo + 32 * wave;
        if (wave_on && p < kv_hi) ask_slots(p);
        for (; wave_on && p < kv_hi; p += 32 * NW) {
            p = __builtin_amdgcn_readfirstlane(p);
            int raw = 0;                      // fp8 pool: bit u: this lane's row of load block u is a pool row
            int ke[KV8 ? NLB : 1], ve[KV8 ? NLB : 1];
#pragma unroll
            for (int u = 0; u < NLB; ++u) {
                const int pr = min(p + u * RPB + ld_rowl, kv_hi - 1);
                const bool ext = pr >= P;
                const unsigned slot = static_cast<unsigned>(min(max(sl[u], 0), num_slots - 1));  // never outside the pool
                const unsigned pg = page_shift >= 0 ? slot >> page_shift : __umulhi(slot, page_magic) >> page_mshift;
                const unsigned o = slot - pg * static_cast<unsigned>(page_size);
                int xrow = pr - P;
                if (shared && ext) {
                    const int k = member_at(0, pr);
                    xrow = s_mx0[k] + (pr - s_mseg[k]);
                }
                if constexpr (KV8) {
                    const signed char* ea = exp_g + static_cast<size_t>(pg) * exp_page + o;  // (slot 0 where the row is no pool row)
                    ke[u] = ea[0];
                    ve[u] = ea[exp_v];
                    if (ext) {
                        const size_t off = static_cast<size_t>(static_cast<int64_t>(xrow) * x_stride);
                        load_to_lds_16(kx_g + off + koff(u), wbase + u * 1024);
                        load_to_lds_16(vx_g + off + voff(u), wbase + VOFF + u * 1024);
                    } else {
                        raw |= 1 << u;
                        if (ld_pos < CPR / 2) {
                            const unsigned char* ka = pool8_g + static_cast<size_t>(pg) * page_stride8 + o * static_cast<unsigned>(D) + ld_pos * 16;
                            load_to_lds_16(ka, wbase + u * 1024);
                            load_to_lds_16(ka + v_off8, wbase + VOFF + u * 1024);
                        }
                    }
                } else {
                    const size_t off = ext ? static_cast<size_t>(static_cast<int64_t>(xrow) * x_stride)
                                           : static_cast<size_t>(pg) * page_stride + o * static_cast<unsigned>(ROWB);
                    load_to_lds_16((ext ? kx_g : pool_g) + off + koff(u), wbase + u * 1024);
                    load_to_lds_16((ext ? vx_g : pool_g + v_off32) + off + voff(u), wbase + VOFF + u * 1024);
                }
            }
            ask_slots(p + 32 * NW);
            wait_vm_all();
            if constexpr (KV8) {  // codes to bfloat16 in place, as in landed8
                unsigned char* const base = smem + wave * WB;
                uint2 kraw[NLB], vraw[NLB];
#pragma unroll
                for (int u = 0; u < NLB; ++u) {
                    if ((raw >> u) & 1) {
                        const unsigned char* row = base + u * 1024 + ld_rowl * ROWB;
                        kraw[u] = *reinterpret_cast<const uint2*>(row + (koff(u) >> 1));
                        vraw[u] = *reinterpret_cast<const uint2*>(row + VOFF + (voff(u) >> 1));
                    }
                }
#pragma unroll
                for (int u = 0; u < NLB; ++u) {
                    if ((raw >> u) & 1) {
                        unsigned char* dst = base + u * 1024 + lane * 16;
                        const float ks = fp8_scale(ke[u]), vs = fp8_scale(ve[u]);
                        const uint2 ka = fp8_decode4(kraw[u].x, ks), kb = fp8_decode4(kraw[u].y, ks);
                        const uint2 va = fp8_decode4(vraw[u].x, vs), vb = fp8_decode4(vraw[u].y, vs);
                        *reinterpret_cast<uint4*>(dst) = make_uint4(ka.x, ka.y, kb.x, kb.y);
                        *reinterpret_cast<uint4*>(dst + VOFF) = make_uint4(va.x, va.y, vb.x, vb.y);
                    }
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
            const bool not_ours = shared && p >= P && (p >= s_wave_own[2 * wave + 1] || p + 32 <= s_wave_own[2 * wave]);
            if (p <= P + wave_i_last && !not_ours) general_block(p, 0, p + 32 > blk_vis_min);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (nothing still reads what the next loads overwrite)
        }
        claim_word();
        // ---- join the waves: each leaves its sums in its quarter of the ring (16-byte pieces of a row XORed with the row's
        // number, so that the lanes of a store meet different banks) ----
        constexpr int V4 = D / 4;  // pieces per row
        const float l_row[RB] = {row_sum(l_run[0]), row_sum(l_run[1])};
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int row = 16 * rb + n;
            if (row >= rows_here) continue;
            float4* mine = reinterpret_cast<float4*>(smem + wave * WB) + row * V4;
#pragma unroll
            for (int b = 0; b < NB; ++b)
                mine[(4 * b + g4) ^ (row & (V4 - 1))] = make_float4(oacc[rb][b][0], oacc[rb][b][1], oacc[rb][b][2], oacc[rb][b][3]);
            if (g4 == 0) s_ml[wave * kNarrowRows + row] = make_float2(m_run[rb], l_row[rb]);
        }
        const int jr = tid >> 3, sub = tid & 7;  // eight threads per row
        __syncthreads();
        const int64_t out_row = s_row[jr];
        if (jr < rows_here) {
        float2 ml[NW];
        float m = -INFINITY, l = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            ml[w] = s_ml[w * kNarrowRows + jr];
            m = fmaxf(m, ml[w].x);
        }
        float wgt[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            wgt[w] = ml[w].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[w].x - m);
            l += wgt[w] * ml[w].y;
        }
        const float inv = prow < 0 ? 1.f / l : 1.f;
        const size_t part_row = static_cast<size_t>(prow < 0 ? 0 : prow) * Hkv + static_cast<size_t>(g) * rows_here + jr;
#pragma unroll
        for (int i = 0; i < V4 / 8; ++i) {
            const int c = sub + 8 * i;
            float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float4 o = reinterpret_cast<const float4*>(smem + w * WB)[jr * V4 + (c ^ (jr & (V4 - 1)))];
                acc.x += wgt[w] * o.x; acc.y += wgt[w] * o.y; acc.z += wgt[w] * o.z; acc.w += wgt[w] * o.w;
            }
            if (prow < 0) {
                uint2 v;
                v.x = pack_bf16x2(acc.x * inv, acc.y * inv);
                v.y = pack_bf16x2(acc.z * inv, acc.w * inv);
                reinterpret_cast<uint2*>(out + out_row * D)[c] = v;
            } else if constexpr (kDirect) {
                store_through_16(part_o + part_row * D + 4 * c, acc);
            } else {
                reinterpret_cast<float4*>(part_o + part_row * D)[c] = acc;
            }
        }
        if (prow >= 0 && sub == 0) {
            if constexpr (kDirect) store_through_8(part_ml + 2 * part_row, make_float2(m, l));
            else reinterpret_cast<float2*>(part_ml)[part_row] = make_float2(m, l);
        }
        }
        if constexpr (kDirect)
            if (prow >= 0) join_parts();
    } else {
    // ---- prologue: first tile into ring slot 0 ----
    load_slots(kv_lo);
    issue_any(kv_lo, 0);
    load_slots(kv_lo + kKT);
    wait_vm_all();
    if constexpr (KV8) landed8(0);
    wg_barrier();

    // clock probe (benchmarks only): shader cycles and ticks of the constant 100 MHz counter across the key loop
    long long clk_c0 = 0, clk_w0 = 0;
    if (clk) {
        clk_c0 = clock64();
        clk_w0 = wall_clock64();
    }
    int p0 = kv_lo, ring = 0;  // the tile at p0 sits in ring slot `ring`
    // the LDS read addresses follow the ring: from slot `from_ring` to the other one
    auto move_read_addresses = [&](int from_ring) __attribute__((always_inline)) {
        const int d = from_ring ? -STAGEB : STAGEB;
#pragma unroll
        for (int s = 0; s < KS; ++s) k_rd[s] += d;
#pragma unroll
        for (int b = 0; b < NB; ++b) v_rd[b] += d;
    };
    // this wave's part of the next tile has landed, and so has everyone else's; nobody still reads the tile just
    // finished; then on to the next tile
    auto next_tile = [&]() __attribute__((always_inline)) {
        wait_vm_all();
        if constexpr (KV8) landed8(ring ^ 1);
        wg_barrier();
        move_read_addresses(ring);
        ring ^= 1;
        p0 += kKT;
    };
    // Tiles in assembly (one statement, see fast_run.inc).  A run: consecutive tiles that need no mask
    // and whose successors lie wholly in the prefix (mode 1, or 3 for pools of 4 GB and more) or wholly in the extend
    // tokens (2); it issues its tiles' loads itself.  A single tile: arithmetic only, with the keys a row must not see
    // hidden if there are any (5, else 4), the next tile's loads issued from here by the general code - for the tiles
    // that no run takes because of what their successor is (prefix and extend rows mixed) or because they touch the
    // causal diagonal; in shared tiles only where all keys are common (a second visibility bound otherwise).  Neither before the
    // running maximum exists.  (Last tiles of common first parts so, 256 decode requests: 3.5 us in the general tile.)
    auto single_tile_ok = [&](int p0) __attribute__((always_inline)) -> bool {
        return (fast_ok || KV8) && kAsm && (smem_addr & 255u) == 0 && (!shared || min(p0 + kKT, kv_hi) <= P) && wave_on && p0 <= P + wave_i_last;
    };
    // The assembly tiles want a running maximum to start from, and any lower bound of the true one will do as long as it
    // is not 2^40 short (then the tile is handed to the general code, as always): the largest score of the first 32 keys,
    // where every row of the wave sees all of them.  The first tile then runs in assembly like the others (its first
    // key block is multiplied twice) instead of in the general code, which establishes the maximum otherwise.
    if constexpr (kAsm) {
        // (also in shared tiles: the keys of the common prefix are visible to every row)
        if ((fast_ok || KV8) && (smem_addr & 255u) == 0 && wave_on && kv_lo <= P + wave_i_last && kv_lo + 32 <= blk_vis_min && kv_lo + 32 <= kv_hi) {
            const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
            bf16x8 kf[2 * KS];
            read_k_block<16 * ROWB>(kf, k_rd, 0);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                f32x4 s0 = zero4, s1 = zero4;
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[2 * s], qreg[rb][s], s0, 0, 0, 0);
                    s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[2 * s + 1], qreg[rb][s], s1, 0, 0, 0);
                }
                float mx = fmaxf(s0[0], s1[0]);
#pragma unroll
                for (int i = 1; i < 4; ++i) mx = fmaxf(mx, fmaxf(s0[i], s1[i]));
                m_run[rb] = row_max(mx) * scale_log2e;
            }
        }
    }
    bool fast_allowed = true;
    while (p0 < kv_hi) {
        p0 = __builtin_amdgcn_readfirstlane(p0);  // wave-uniform, said so to the compiler
        ring = __builtin_amdgcn_readfirstlane(ring);
        int from = 0;
        bool issue_next = true;
        int mode = 0, kind = 0;
        const bool idle = !wave_on || p0 > P + wave_i_last;
        if (idle && fast_ok && kAsm && (smem_addr & 255u) == 0) {
            // Nothing to compute, in this tile or any later one: only its share of the loads.  (In the general code they held up the other
            // waves: 16 questions to long documents, items of 68 to 92 rows 110 us instead of 90, with the fp8 pool 210 instead of 100.)
            kind = min(p0 + 2 * kKT - 1, kv_hi - 1) < P ? (!KV8 || (fast_ok & 2) ? 1 : 0) : min(p0 + kKT, kv_hi - 1) >= P && !shared && (!KV8 || (fast_ok & 1)) ? 2 : 0;
            mode = kind == 0 ? 0 : kind == 2 ? 8 : KV8 ? 10 : fast_ok == 2 ? 9 : 7;
        } else if (fast_allowed && __all(m_run[0] != -INFINITY && m_run[1] != -INFINITY)) {  // (every row has a running maximum)
            kind = tile_kind(p0);
            mode = kind == 1 ? (KV8 ? 6 : fast_ok == 2 ? 3 : 1) : kind == 2 ? 2 : single_tile_ok(p0) ? (p0 + kKT > blk_vis_min ? 5 : 4) : 0;
        }
        if (mode != 0) {
            if constexpr (kAsm) {
                // Against the running maximum as it stands: scores never move it in there (a row's probabilities may
                // reach 2^40 instead), the output accumulators are touched by MFMAs only.
                int p_end = p0 + kKT;
                if (mode != 4 && mode != 5) {
                    // (as far as tile_kind() stays what it is: every condition in it, once it fails, fails for all later tiles.  Asked
                    // tile by tile this took 2 us of a workgroup's 60.)
                    int last = idle ? kv_hi - 1 : min(P + wave_i_last, blk_vis_min - kKT);
                    if (kind == 1 && kv_hi > P) last = min(last, P - 2 * kKT);
                    p_end += (last - p0) & ~(kKT - 1);
                    raw_mask = 0;  // (fp8 pool: a run decodes what it loads itself)
                } else if (p0 + kKT < kv_hi) {
                    issue_any(p0 + kKT, ring ^ 1);
                    load_slots(p0 + 2 * kKT);
                } else {
                    raw_mask = 0;
                }
                const int p_start = p0, ring_start = ring;
                int st = 0;
                auto fragments = [&](int rb) __attribute__((always_inline)) {  // the query fragments of a row block in a row
                    const bf16x16 a = __builtin_shufflevector(qreg[rb][0], qreg[rb][1], 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
                    if constexpr (KS == 2) {
                        return a;
                    } else {
                        const bf16x16 b = __builtin_shufflevector(qreg[rb][2], qreg[rb][3], 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
                        return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17, 18, 19, 20, 21, 22, 23, 24,
                                                       25, 26, 27, 28, 29, 30, 31);
                    }
                };
                // wave-uniform values, said so to the compiler (they go to scalar registers)
                auto uni = [](int x) __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane(x); };
                auto uni_ptr = [&](const void* q) __attribute__((always_inline)) {
                    const uint64_t a = reinterpret_cast<uint64_t>(q);
                    const uint64_t lo = static_cast<uint32_t>(uni(static_cast<int>(a))), hi = static_cast<uint32_t>(uni(static_cast<int>(a >> 32)));
                    return reinterpret_cast<const void*>(lo | (hi << 32));
                };
                // (mode 3: the pool is too large for 32-bit byte offsets; rows are then counted in units of 256 bytes)
                // (mode 6, the fp8 pool: strides of the codes and of the row exponents, and where the latter lie)
                const uint64_t exp_addr = reinterpret_cast<uint64_t>(exp_g);
                // (the single tiles look at none of the bases and strides: the fp8 pool's kernels need not keep those of a bf16 pool for them,
                // 18 scalars that were spilled around the statement)
                const bool is8 = mode == 6 || mode == 10;
                const i32x8 c = {uni(page_shift), uni(page_size - 1),
                                 uni(static_cast<int>(KV8 ? page_stride8 : mode == 3 || mode == 9 ? page_stride / ROWB : page_stride)), uni(num_slots - 1),
                                 uni(P - 1), uni(static_cast<int>(is8 ? exp_page : x_stride)),
                                 uni(is8 ? static_cast<int>(exp_v) : kv_hi - 1 - P),
                                 uni(static_cast<int>(smem_addr) + wave * (UPW * 1024))};
                const i32x4 c2 = {uni(is8 ? static_cast<int>(exp_addr) : 128), uni(is8 ? static_cast<int>(exp_addr >> 32) : 192), uni(P),
                                  uni(__float_as_int(scale_log2e))};
                p0 = uni(p0);
                ring = uni(ring);
                p_end = uni(p_end);
                const int row_in_tile = wave * (UPW * RPB) + slot_row();
                const void* base_k = kind == 2 ? static_cast<const void*>(kx_g) : KV8 ? static_cast<const void*>(pool8_g) : static_cast<const void*>(pool_g);
                const void* base_v = kind == 2 ? static_cast<const void*>(vx_g) : KV8 ? static_cast<const void*>(pool8_g + v_off8) : static_cast<const void*>(pool_g + v_off32);
                const int lim[RB] = {vis_end[0] - p0 - 4 * g4, vis_end[1] - p0 - 4 * g4};
                if constexpr (KV8)  // (single tiles only; they end with this wave's loads landed and leave the barrier to the caller)
                    fast_tiles_d128_kv8(uni(mode), oacc, fragments(0), fragments(1), l_run, -m_run[0], -m_run[1], sl_next, k_rd[0], v_rd[0], ld_koff0,
                                        ld_voff0, row_in_tile, p0, ring, st, p_end, uni_ptr(slots), uni_ptr(base_k), uni_ptr(base_v), lim[0], lim[1], c, c2,
                                        uni(static_cast<int>(smem_addr) + EX_OFF + wave * EXPB));
                else if constexpr (D == 128)
                    fast_tiles_d128(uni(mode), oacc, fragments(0), fragments(1), l_run, -m_run[0], -m_run[1], sl_next, k_rd[0], v_rd[0], ld_koff0,
                                    ld_voff0, row_in_tile, p0, ring, st, p_end, uni_ptr(slots), uni_ptr(base_k), uni_ptr(base_v), lim[0], lim[1], c, c2);
                else
                    fast_tiles_d64(uni(mode), oacc, fragments(0), fragments(1), l_run, -m_run[0], -m_run[1], sl_next, k_rd[0], v_rd[0], ld_koff0,
                                   ld_voff0, row_in_tile, p0, ring, st, p_end, uni_ptr(slots), uni_ptr(base_k), uni_ptr(base_v), lim[0], lim[1], c, c2);
                if constexpr (KV8) {
                    if (mode == 6 && st != 0) raw_mask = (1 << UPW) - 1;  // left inside a tile: the next one's rows are still codes
                    if (st == 0 && (mode == 4 || mode == 5)) {
                        landed8(ring);
                        wg_barrier();
                    }
                }
                if (((p0 - p_start) / kKT) & 1) move_read_addresses(ring_start);
                if (st == 0) continue;
                // the tile outgrew the maximum: the general code does what is left of it, and stays (rare enough)
                from = st - 1;
                issue_next = false;
                fast_allowed = false;
            }
        }
        tile_general(p0, ring, from, issue_next);
        next_tile();
    }

    if (clk && blockIdx.x % 997 == 7 && tid == 0) {
        atomicAdd(clk, static_cast<unsigned long long>(clock64() - clk_c0));
        atomicAdd(clk + 1, static_cast<unsigned long long>(wall_clock64() - clk_w0));
    }
    claim_word();
    // ---- epilogue: lane holds, for block b and register i, head-dim element 16 b + 4 g4 + i of its rows ----
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int row = wave_row0 + 16 * rb + n;
        const float l_row = row_sum(l_run[rb]);
        const int64_t q_row = s_row[row];
        if (q_row < 0) {
            // (no row of its own: helps to join the parts, below)
        } else if (prow < 0) {
            const float inv = 1.f / l_row;
            __hip_bfloat16* orow = out + q_row * D;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                uint2 v;
                v.x = pack_bf16x2(oacc[rb][b][0] * inv, oacc[rb][b][1] * inv);
                v.y = pack_bf16x2(oacc[rb][b][2] * inv, oacc[rb][b][3] * inv);
                *reinterpret_cast<uint2*>(orow + 16 * b + 4 * g4) = v;
            }
        } else {
            const size_t part_row = static_cast<size_t>(prow) * Hkv + static_cast<size_t>(g) * rows_here + row;
            const float2 ml = make_float2(m_run[rb], l_row);
            if constexpr (kDirect) {
                // (through LDS, the pieces of a row XORed with its number as where narrow tiles join their waves: the stores that go
                // through to memory then write whole lines; the ring is free, the last tile ended with a barrier)
                float4* const mine = reinterpret_cast<float4*>(smem) + row * (D / 4);
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    mine[(4 * b + g4) ^ (row & 31 & (D / 4 - 1))] = make_float4(oacc[rb][b][0], oacc[rb][b][1], oacc[rb][b][2], oacc[rb][b][3]);
                if (g4 == 0) store_through_8(part_ml + 2 * part_row, ml);
            } else {
                float* po = part_o + part_row * D;
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    *reinterpret_cast<float4*>(po + 16 * b + 4 * g4) = make_float4(oacc[rb][b][0], oacc[rb][b][1], oacc[rb][b][2], oacc[rb][b][3]);
                if (g4 == 0) reinterpret_cast<float2*>(part_ml)[part_row] = ml;
            }
        }
    }
    if constexpr (kDirect) {
        if (prow < 0) return;
        __syncthreads();
        float* const po = part_o + (static_cast<size_t>(prow) * Hkv + static_cast<size_t>(g) * rows_here) * D;
        for (int x = tid; x < rows_here * (D / 4); x += 256) {
            const int row = x / (D / 4), c = x % (D / 4);
            store_through_16(po + 4 * static_cast<size_t>(x), reinterpret_cast<const float4*>(smem)[row * (D / 4) + (c ^ (row & 31 & (D / 4 - 1)))]);
        }
        join_parts();
    }
    }
    };
    if constexpr (kForm == kDirectNarrow) {
        tile(std::true_type{});
    } else {
        if (__builtin_amdgcn_readfirstlane(rec2.y) != 0) tile(std::true_type{});
        else tile(std::false_type{});
    }
}

// Merge of partial results: out = sum_s 2^(m_s - m) O_s / sum_s 2^(m_s - m) l_s over the parts s of a row: those of its tile,
// and of the shared tile that holds the common keys, if its tile is an own-key one.  A block per (piece, KV head); a piece is
// described by one record, whatever kind of tile it comes from.
template <int D>
__global__ __launch_bounds__(256) void extend_merge_kernel(int Hq, int Hkv, __hip_bfloat16* __restrict__ out, const int32_t* __restrict__ hdr,
                                                          const int4* __restrict__ chunk_tab, const int4* __restrict__ member_tab,
                                                          const float* __restrict__ part_o, const float* __restrict__ part_ml) {
    constexpr int V4 = D / 4;           // 16-byte pieces per partial row: one thread per (row, piece)
    constexpr int kAhead = 4;           // parts in flight per thread
    const int G = Hq / Hkv;
    const int i = threadIdx.x / V4, c = threadIdx.x % V4;
    const float2* ml_tab = reinterpret_cast<const float2*>(part_ml);
    // a fixed grid strides over (piece, kv head): how many there are is known on the device only
    const int n_work = hdr[2] * Hkv;
    int w = blockIdx.x;
    if (w >= n_work) return;
    const int4* rec = chunk_tab + 3 * static_cast<size_t>(w / Hkv);
    int4 c0 = rec[0], c1 = rec[1], c2 = rec[2];
    for (;;) {
        const int g = w % Hkv;
        const int4 d0 = c0, d1 = c1, d2 = c2;
        w += gridDim.x;
        const bool more = w < n_work;
        if (more) {  // (the next piece's record flies meanwhile)
            rec = chunk_tab + 3 * static_cast<size_t>(w / Hkv);
            c0 = rec[0], c1 = rec[1], c2 = rec[2];
        }
        if (i < d0.w >> 16) {
            const int lrow = (d0.w & 0xFFFF) + i;
            // whose row it is: the tile's request, or in a shared tile the last member that starts at or before it
            int64_t e0 = d1.x;
            int rho = d1.y + lrow;
            for (int k = 0; k < d1.z; ++k) {
                const int4 mem = member_tab[2 * (d1.x + k)];
                if (mem.x <= d1.y + lrow) {
                    e0 = mem.y;
                    rho = mem.z + (d1.y + lrow - mem.x);
                }
            }
            const size_t own0 = static_cast<size_t>(d0.y) * Hkv + static_cast<size_t>(g) * d0.z + lrow, own_step = static_cast<size_t>(d0.z) * Hkv;
            const size_t com0 = static_cast<size_t>(d2.x) * Hkv + static_cast<size_t>(g) * d2.y + d2.z + i, com_step = static_cast<size_t>(d2.y) * Hkv;
            const int n = d0.x + d1.w;
            float m = -INFINITY, l = 0.f;
            float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
            for (int s0 = 0; s0 < n; s0 += kAhead) {  // (maxima, sums and rows of kAhead parts in one round trip)
                float2 ml[kAhead];
                float4 o[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const int s = min(s0 + u, n - 1);
                    const size_t at = s < d0.x ? own0 + s * own_step : com0 + (s - d0.x) * com_step;
                    ml[u] = ml_tab[at];
                    o[u] = reinterpret_cast<const float4*>(part_o + at * D)[c];
                }
                float m_new = m;
#pragma unroll
                for (int u = 0; u < kAhead; ++u) m_new = fmaxf(m_new, ml[u].x);
                const float old = m == -INFINITY ? 0.f : exp2f(m - m_new);
                l *= old;
                acc.x *= old; acc.y *= old; acc.z *= old; acc.w *= old;
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const bool again = s0 + u >= n;  // (the last part once more: 0 times it would be no 0 where it holds an infinity)
                    const float wgt = again || ml[u].x == -INFINITY ? 0.f : exp2f(ml[u].x - m_new);
                    o[u].x = again ? 0.f : o[u].x; o[u].y = again ? 0.f : o[u].y; o[u].z = again ? 0.f : o[u].z; o[u].w = again ? 0.f : o[u].w;
                    l += wgt * ml[u].y;
                    acc.x += wgt * o[u].x; acc.y += wgt * o[u].y; acc.z += wgt * o[u].z; acc.w += wgt * o[u].w;
                }
                m = m_new;
            }
            const float inv = 1.f / l;
            __hip_bfloat16* orow = out + ((e0 + rho / G) * Hq + g * G + rho % G) * static_cast<int64_t>(D);
            uint2 v;
            v.x = pack_bf16x2(acc.x * inv, acc.y * inv);
            v.y = pack_bf16x2(acc.z * inv, acc.w * inv);
            reinterpret_cast<uint2*>(orow)[c] = v;
        }
        if (!more) break;
    }
}

// How the kernel divides a slot id (< 2^31) by the page size d.  A power of two: *shift = log2 d.  Otherwise
// *shift = -1 and slot / d = umulhi(slot, *magic) >> *mshift exactly: with l = ceil(log2 d), k = 31 + l and
// magic = floor(2^k / d) + 1 (< 2^32 since 2^l < 2 d), the error magic * d - 2^k is at most d <= 2^l = 2^(k - 31),
// which keeps the quotient exact for every numerator below 2^31; mshift = k - 32.
static void page_divider(int d, int* shift, unsigned* magic, int* mshift) {
    *shift = -1;
    *magic = 0;
    *mshift = 0;
    if ((d & (d - 1)) == 0) {
        *shift = 0;
        while ((1 << *shift) < d) ++*shift;
        return;
    }
    int l = 0;
    while ((int64_t{1} << l) < d) ++l;
    const int k = 31 + l;
    *magic = static_cast<unsigned>((static_cast<unsigned __int128>(1) << k) / static_cast<unsigned>(d) + 1);
    *mshift = k - 32;
}

template <int D, bool KV8>
static int launch_extend(const ExtendPlan& p, const PlanTables& t, const void* q_ext, const void* k_ext, const void* v_ext,
                         const void* kv_pool, const int32_t* slot_idx, int Hq, int Hkv, int page_size, int64_t num_slots, int64_t T_total,
                         float scale_log2e, void* out, unsigned long long* clk, const DirectArgs& direct, hipStream_t stream) {
    // the K/V ring and what lies behind it (fp8 pool: rounded up to 256 bytes, then one 32-bit word per lane, load block of a
    // wave and tensor for the row exponents)
    constexpr size_t lds_plain = static_cast<size_t>(kStages) * 2 * kKT * D * 2 + kLdsTail;
    constexpr size_t lds_bytes = KV8 ? ((lds_plain + 255) & ~size_t{255}) + static_cast<size_t>(4) * 256 * 2 * (kKT / (1024 / (D * 2)) / 4) : lds_plain;
    int page_shift = -1, page_mshift = 0;
    unsigned page_magic = 0;
    page_divider(page_size, &page_shift, &page_magic, &page_mshift);
    const dim3 grid(static_cast<unsigned>(direct.parts > 0 ? direct.tiles * direct.parts : p.items_cap) * Hkv);
    // The hand-scheduled tiles multiply in 24 bits and take a power-of-two page size.  They address pool rows by
    // 32-bit byte offsets where the pool is below 4 GB (1); by row numbers in units of 256 bytes, the byte address
    // formed in 64 bits, where it is larger (2: D = 128, a pool base aligned to 256 bytes, up to 64 GB).  The extend
    // tensors are addressed by 32-bit byte offsets in either case.
    const int64_t rowb = static_cast<int64_t>(D) * 2;
    const int64_t pool_bytes = num_slots * 2 * Hkv * rowb;
    const int64_t page_bytes = static_cast<int64_t>(page_size) * 2 * Hkv * rowb;
    const bool common_ok = page_shift >= 0 && num_slots / page_size < (1 << 24) && T_total < (1 << 24) &&
                           T_total * Hkv * rowb < (int64_t{1} << 32);
    const bool ok32 = common_ok && pool_bytes < (int64_t{1} << 32) && page_bytes < (1 << 24);
    const bool ok64 = common_ok && rowb == 256 && (reinterpret_cast<uintptr_t>(kv_pool) & 255u) == 0 &&
                      page_bytes / rowb < (1 << 24) && pool_bytes / rowb < (int64_t{1} << 28);
    // (fp8 pool: 1 = the extend tensors can be addressed by 32-bit offsets, all that its runs of tiles ask for)
    // (fp8 pool: bit 0 = the extend tensors can be addressed by 32-bit offsets, as the runs over extend tokens do; bit 1 =
    // so can the codes, with page numbers and page strides that fit the 24-bit multiplications of the runs over the pool)
    const bool ext_ok = T_total < (1 << 24) && T_total * Hkv * rowb < (int64_t{1} << 32);
    const bool pool8_ok = page_shift >= 0 && num_slots / page_size < (1 << 24) && pool_bytes / 2 < (int64_t{1} << 32) && page_bytes / 2 < (1 << 24);
    const int fast_ok = KV8 ? (ext_ok ? 1 : 0) | (pool8_ok ? 2 : 0) : ok32 ? 1 : ok64 ? 2 : 0;
    // (fp8 pool: the row exponents lie behind the codes)
    const signed char* pool_exp = KV8 ? static_cast<const signed char*>(kv_pool) + static_cast<size_t>(num_slots) * 2u * Hkv * D : nullptr;
    const auto launch = [&](auto kernel, auto args) {
        ProfScope prof(kProfExtend, stream);
        hipLaunchKernelGGL(kernel, grid, dim3(256), lds_bytes, stream,
                           static_cast<const __hip_bfloat16*>(q_ext), static_cast<const __hip_bfloat16*>(k_ext),
                           static_cast<const __hip_bfloat16*>(v_ext), static_cast<const __hip_bfloat16*>(kv_pool), pool_exp, slot_idx,
                           Hq, Hkv, page_size, page_shift, page_magic, page_mshift, static_cast<int>(num_slots), fast_ok,
                           scale_log2e, static_cast<__hip_bfloat16*>(out), t.hdr, t.item, t.member, t.part_o, t.part_ml, clk, args);
    };
    if (direct.parts > 0) {
        if (direct.tile_rows == kNarrowRows) launch(extend_bf16_kernel<D, KV8, kDirectNarrow>, direct);
        else launch(extend_bf16_kernel<D, KV8, kDirectWide>, direct);
    } else {
        launch(extend_bf16_kernel<D, KV8, kList>, NoArgs{});
        // whether any tile was split is known on the device only: otherwise the merge's blocks leave at once
        ProfScope prof(kProfMerge, stream);
        const int64_t most = static_cast<int64_t>(p.chunks_cap) * Hkv;
        hipLaunchKernelGGL((extend_merge_kernel<D>), dim3(static_cast<unsigned>(most < 2048 ? most : 2048)), dim3(256), 0, stream,
                           Hq, Hkv, static_cast<__hip_bfloat16*>(out), t.hdr, t.chunk, t.member, t.part_o, t.part_ml);
    }
    return PA_OK;
}

}  // namespace pa

// A number that no other call has, in the upper 56 bits (DirectArgs::tag): counted up from a start that differs from process to
// process, since memory may come from another one's workspace.
static unsigned long long next_call_tag() {
    static std::atomic<unsigned long long> next{[] {
        const int on_stack = 0;
        unsigned long long x = static_cast<unsigned long long>(std::chrono::system_clock::now().time_since_epoch().count()) ^
                               static_cast<unsigned long long>(std::chrono::steady_clock::now().time_since_epoch().count()) << 32 ^
                               reinterpret_cast<uintptr_t>(&on_stack) << 16 ^ static_cast<unsigned long long>(getpid()) << 40;
        return pa::path_mix(x, 0);
    }()};
    return next.fetch_add(1, std::memory_order_relaxed) << 8;
}

// Process-wide switch: 0 = every request gets row tiles of its own (no grouping by equal slots).
static std::atomic<int> g_row_sharing{1};
extern "C" int pa_extend_set_row_sharing(int on) {
    g_row_sharing.store(on != 0);
    return PA_OK;
}

// Whether the last bf16 launch that used this workspace found room for its work list.
extern "C" int pa_extend_status(const void* workspace, void* stream) {
    PA_REQUIRE(workspace != nullptr, "pa_extend_status: workspace is NULL");
    int32_t hdr[4] = {0, 0, 0, 0};
    hipStream_t s = static_cast<hipStream_t>(stream);
    PA_HIP(hipMemcpyAsync(hdr, workspace, sizeof hdr, hipMemcpyDeviceToHost, s));
    PA_HIP(hipStreamSynchronize(s));
    if (hdr[3] != 0)
        return pa::fail(PA_EOVERFLOW, "pa_extend_attention: the batch on the device is larger than the T and max_kv_len "
                                      "the call was given; its work list did not fit and no output was written");
    return PA_OK;
}

// What the largest plan of up to B requests takes: a plan of more requests than the planner looks through for common prefixes
// can be smaller than one of fewer, and a workspace is good for both.
size_t pa_extend_workspace_bytes_bf16(int B, int64_t T, int64_t max_kv_len, int Hq, int Hkv, int D) {
    const size_t all = pa::make_extend_plan(B, T, max_kv_len, Hq, Hkv, D, pa::kRounds, 0).total;
    if (B <= pa::kPackMax) return all;
    const size_t packed = pa::make_extend_plan(pa::kPackMax, T, max_kv_len, Hq, Hkv, D, pa::kRounds, 0).total;
    return packed > all ? packed : all;
}

// The work of a bf16 call once its plan and its workspace are settled.
static int run_extend_bf16(pa::ExtendPlan p, const void* q_ext, const void* k_ext, const void* v_ext, const void* kv_pool,
                           const int32_t* slot_idx, const int32_t* slot_offsets, const int32_t* prefix_len,
                           const int32_t* ext_len, const int32_t* ext_offsets, int B, int64_t T, int Hq, int Hkv, int D,
                           int page_size, int64_t num_slots, bool kv8, float scale, void* out, void* workspace, hipStream_t stream) {
    using namespace pa;
    if (!g_row_sharing.load()) p.pack = p.first_part = 0;
    const PlanTables t = plan_tables(p, workspace);
    // with the clock probe on, a few workgroups also add their cycle counts to two counters in the header
    unsigned long long* clk = prof_clock_enabled() ? reinterpret_cast<unsigned long long*>(static_cast<unsigned char*>(workspace) + kClockProbeOffset) : nullptr;
    const float scale_log2e = scale * 1.4426950408889634f;
    DirectArgs direct{prefix_len, ext_len, ext_offsets, slot_offsets, reinterpret_cast<unsigned long long*>(t.tile), 0, t.hdr, B, p.direct_parts, p.direct_tile_rows, p.direct_tiles,
                      p.direct_stride};
    if (kv8 && p.direct_tile_rows == kNarrowRows &&
        (p.direct_key_tiles > kDirectKeyTilesFp8 || p.direct_part_tiles > (p.direct_idle ? kDirectPartIdleFp8 : kDirectPartFp8)))
        direct.parts = 0;
    if (direct.parts > 1) direct.tag = next_call_tag();
    if (direct.parts == 0) launch_extend_plan(p, t, prefix_len, ext_len, ext_offsets, slot_offsets, slot_idx, B, Hq / Hkv, stream);
    const auto launch = D == 64 ? (kv8 ? launch_extend<64, true> : launch_extend<64, false>) : (kv8 ? launch_extend<128, true> : launch_extend<128, false>);
    launch(p, t, q_ext, k_ext, v_ext, kv_pool, slot_idx, Hq, Hkv, page_size, num_slots, T, scale_log2e, out, clk, direct, stream);
    PA_HIP(hipGetLastError());
    return PA_OK;
}

static int check_bf16_args(float scale, int64_t num_slots, int page_size, int Hkv, int D) {
    PA_REQUIRE(scale > 0.f && scale < INFINITY, "pa_extend_attention: scale must be positive and finite");
    PA_REQUIRE(num_slots <= INT32_MAX, "pa_extend_attention: num_slots exceeds the int32 range of slot ids");
    PA_REQUIRE(static_cast<int64_t>(page_size) * Hkv * D * 4 < (int64_t{1} << 31), "pa_extend_attention: a page of %d tokens x %d heads is too large", page_size, Hkv);
    return PA_OK;
}

// Called by pa_extend_attention after argument validation.
int pa_extend_attention_bf16(const void* q_ext, const void* k_ext, const void* v_ext, const void* kv_pool,
                             const int32_t* slot_idx, const int32_t* slot_offsets, const int32_t* prefix_len,
                             const int32_t* ext_len, const int32_t* ext_offsets, int B, int64_t T, int64_t max_kv_len,
                             int Hq, int Hkv, int D, int page_size, int64_t num_slots, bool kv8, float scale, void* out,
                             void* workspace, size_t workspace_bytes, hipStream_t stream) {
    using namespace pa;
    if (const int rc = check_bf16_args(scale, num_slots, page_size, Hkv, D)) return rc;
    // (sized for shared row tiles whether or not they are on; a smaller workspace that does for a plan without grouping by
    // common first parts gets that one)
    const ExtendPlan p = make_extend_plan(B, T, max_kv_len, Hq, Hkv, D, kRounds, workspace_bytes);
    if (workspace_bytes < p.total || workspace == nullptr)
        return fail(PA_ENOMEM, "pa_extend_attention: workspace of %zu bytes given, at least %zu needed", workspace_bytes, p.total);
    PA_REQUIRE((reinterpret_cast<uintptr_t>(workspace) & 255u) == 0, "pa_extend_attention: workspace must be 256-byte aligned");
    return run_extend_bf16(p, q_ext, k_ext, v_ext, kv_pool, slot_idx, slot_offsets, prefix_len, ext_len, ext_offsets, B, T, Hq,
                           Hkv, D, page_size, num_slots, kv8, scale, out, workspace, stream);
}

// ---------------------------------------------------------------------------------------
// The variant for callers that cannot allocate: its workspace is a buffer that is part of the library's code object.
// Every GPU that loads the library holds its own copy of the array at its own address; in host code the array's name
// is only a handle for hipGetSymbolAddress, never a device address.
// ---------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[PA_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per device.
int scratch_of_current_device(void** out) {
    int dev = -1;
    PA_HIP(hipGetDevice(&dev));
    PA_REQUIRE(dev >= 0 && dev < kMaxDevices, "pa_extend_attention_static: device ordinal %d not supported", dev);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (g_scratch_ptr[dev] == nullptr) {
        void* ptr = nullptr;
        PA_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        PA_REQUIRE(ptr != nullptr && (reinterpret_cast<uintptr_t>(ptr) & 255u) == 0, "pa_extend_attention_static: bad scratch address");
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return PA_OK;
}
}  // namespace

// Called by pa_extend_attention_static after argument validation.
int pa_extend_attention_bf16_static(const void* q_ext, const void* k_ext, const void* v_ext, const void* kv_pool,
                                    const int32_t* slot_idx, const int32_t* slot_offsets, const int32_t* prefix_len,
                                    const int32_t* ext_len, const int32_t* ext_offsets, int B, int64_t T,
                                    int64_t max_kv_len, int Hq, int Hkv, int D, int page_size, int64_t num_slots,
                                    bool kv8, float scale, void* out, hipStream_t stream) {
    using namespace pa;
    if (const int rc = check_bf16_args(scale, num_slots, page_size, Hkv, D)) return rc;
    // (one work item per workgroup slot is aimed at instead of two: half of the partial results at most)
    const ExtendPlan p = make_extend_plan(B, T, max_kv_len, Hq, Hkv, D, kRoundsStatic, PA_STATIC_SCRATCH_BYTES);
    if (p.total > PA_STATIC_SCRATCH_BYTES)
        return fail(PA_ENOMEM, "pa_extend_attention_static: this batch needs %zu bytes of workspace, the library's own buffer holds %zu; "
                               "use pa_extend_attention with a workspace of the caller's", p.total, static_cast<size_t>(PA_STATIC_SCRATCH_BYTES));
    void* ws = nullptr;
    if (const int rc = scratch_of_current_device(&ws)) return rc;
    return run_extend_bf16(p, q_ext, k_ext, v_ext, kv_pool, slot_idx, slot_offsets, prefix_len, ext_len, ext_offsets, B, T, Hq,
                           Hkv, D, page_size, num_slots, kv8, scale, out, ws, stream);
}
