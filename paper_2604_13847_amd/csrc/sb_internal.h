// Internal declarations shared by the translation units of libsparsebal (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <string>
#include <vector>

#include "sparsebal.h"

namespace sb {

typedef __bf16 bf16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

void set_error(const char* fmt, ...);

#define SB_CHECK_HIP(expr)                                                         \
  do {                                                                             \
    hipError_t e_ = (expr);                                                        \
    if (e_ != hipSuccess) {                                                        \
      ::sb::set_error("%s failed: %s", #expr, hipGetErrorString(e_));              \
      return SB_ERR_HIP;                                                           \
    }                                                                              \
  } while (0)

#define SB_LAUNCH_CHECK(name)                                                      \
  do {                                                                             \
    hipError_t e_ = hipGetLastError();                                             \
    if (e_ != hipSuccess) {                                                        \
      ::sb::set_error("launch of %s failed: %s", name, hipGetErrorString(e_));     \
      return SB_ERR_HIP;                                                           \
    }                                                                              \
  } while (0)

// Host-side geometry derived from sb_problem in O(S).
struct Geo {
  int T = 0, S = 0, Hq = 0, Hkv = 0, G = 1, D = 0, B = 64, Hs = 0, mode = 0, dtype = 0;
  float softmax_scale = 0.f, score_scale = 0.f;
  int64_t NQB = 0;          // total query blocks
  int n_max = 0;            // largest n_s
  int64_t scores_unit = 0;  // sum n_s^2 (per selection head)
  int64_t nnz_unit = 0;     // sum_s (k n - k(k-1)/2) (per selection head)
  int64_t bm_words_unit = 0;  // sum_s n_s * ceil(n_s/32) (per selection head)
  int64_t pairs_unit = 0;   // unmasked (query,key) pairs per query head
  // The attention kernels always work on 64-row tiles.  With a selection block of B = 64*r rows a kept
  // block stands for r consecutive key tiles and a query block for r query tiles (see plan_expand_kernel).
  int r = 1;                // tiles per block
  int64_t NT = 0;           // total 64-row tiles
  int nt_max = 0;           // largest tile count of a sequence
  int64_t nnzT_unit = 0;    // tile-level selection entries per selection head
  int64_t bmT_words_unit = 0;  // sum_s nt_s * ceil(nt_s/32)
  int rowT_max = 0;         // most tiles that a row keeps
};
// The same problem as the attention kernels see it: 64-row blocks, tile counts in the block fields.
inline Geo tile_geo(const Geo& g) {
  Geo t = g;
  t.B = 64; t.r = 1; t.NQB = g.NT; t.n_max = g.nt_max; t.nnz_unit = g.nnzT_unit; t.bm_words_unit = g.bmT_words_unit;
  return t;
}
// Tile-level selection entries of the first `it` query tiles of a sequence with budget k (in blocks):
// query tile it' of block I = it'/r keeps r tiles for each of its min(k, I+1)-1 earlier blocks plus the
// tiles r*I .. it' of its own block.
inline __host__ __device__ int64_t tile_entries_before(int64_t it, int64_t k, int64_t r) {
  const int64_t I = it / r, a = it % r;
  const int64_t sumc = I <= k ? I * (I - 1) / 2 : k * (k - 1) / 2 + (I - k) * (k - 1);  // sum_{I'<I} (min(k, I'+1) - 1)
  const int64_t cI = (k < I + 1 ? k : I + 1) - 1;
  return r * r * sumc + I * (r * (r + 1) / 2) + a * cI * r + a * (a + 1) / 2;
}

// Validates p and fills g; returns SB_OK or an error (message set).
int make_geo(const sb_problem* p, Geo* g);

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }
constexpr int kMaxDevices = 64;  // per-device state (attributes set, symbol addresses) is kept for this many ordinals

// Device tables computed by geom_kernel from cu_seqlens_dev / topk_dev.
struct TableOffsets {
  size_t qb_off;     // int32 [S+1]   prefix of n_s
  size_t sc_off;     // int64 [S+1]   prefix of n_s^2
  size_t row_base;   // int32 [S+1]   prefix of c-sums (k n - k(k-1)/2)
  size_t bm_off;     // int64 [S+1]   prefix of n_s*ceil(n_s/32)
  size_t kclamp;     // int32 [S]     min(k_s, n_s)
  size_t qb_seq;     // int32 [NQB]   sequence of each query block
  size_t bytes;
};
TableOffsets table_offsets(const Geo& g);

struct Tables {  // device pointers into a tables area
  const int32_t* cu;
  const int32_t* qb_off;
  const int64_t* sc_off;
  const int32_t* row_base;
  const int64_t* bm_off;
  const int32_t* kclamp;
  const int32_t* qb_seq;
};
Tables make_tables(const Geo& g, const sb_problem* p, void* base);
struct GeomArgs;
GeomArgs make_geom_args(const Geo& g, const sb_problem* p, const Tables& t);
// The device arrays that the geometry comes from, whether a kernel works it out itself or reads tables: every call that launches
// either checks them here first.
int check_device_arrays(const sb_problem* p);
int launch_geom(const Geo& g, const sb_problem* p, void* base, hipStream_t st);
// geometry tables of `g` and (unless it is null) of `g2`, and two fills, as one launch; the fills' sizes are multiples of 16 bytes
int launch_geom_and_fills(const Geo& g, void* base, const Geo* g2, void* base2, const sb_problem* p, void* zeros, size_t zero_bytes,
                          void* ones, size_t ones_bytes, hipStream_t st);

// Layout of the opaque plan buffer.
struct PlanOffsets {
  size_t tables;     // TableOffsets area
  size_t work_fwd;   // int32 [Hs*NQB]   row ids, longest first
  size_t colcost;    // int32 [Hkv*NQB]  tiles in each key-major column (summed over the group's heads)
  size_t zeros_end;  // end of colcost
  size_t bwd_items;  // ColItem [Hkv*(NQB+E)]  key-major items: entry r*Hkv + g is the r-th heaviest item of KV head g (col = -1: none)
  size_t counters;   // int32 [4]  {partial slots in use, split columns, sub-part slots in use, most key-major items of a KV head}, zeroed by every plan call
  size_t split_cols; // int32 [3*E]  (column, first partial slot, parts) of every split column
  size_t sub_base;   // int32 [Hkv*(NQB+E)]  first sub-part slot of every key-major item (see sub_weight), -1: none
  size_t sub_items;  // SubItem [Hkv*sub_slots_max]  the sub-parts: entry r*Hkv + g, those of KV head g's heaviest items first (col = -1: none)
  size_t part_item;  // int32 [2*E]  key-major item (index into bwd_items) of every partial slot
  size_t bitmap;     // uint32 [Hs * bm_words_unit] transpose bitmap: bit i of column (s,hs,j)
  size_t items;      // WorkItem [Hs*NQB]  descriptors of the query-major items, in work_fwd order
  // only for selection blocks larger than a tile (r > 1); everything above is then at tile level
  size_t blk_tables; // TableOffsets area of the block-level geometry
  size_t t_rowptr;   // int32 [Hs*NT+1]  tile-level selection CSR
  size_t t_idx;      // int32 [Hs*nnzT]
  size_t bytes;
};
constexpr int kBwdBins = 4096;
// A key-major column (s, g, j) is one work item unless it is heavier than split_weight() tiles: then it is cut, at the
// granularity of 32 query blocks, into parts of at least that weight that are separate work items; the parts leave
// fp32 partial dK/dV in the backward workspace and a reduction adds them in part order.  The bounds below follow from
// "every part but a column's last has at least split_weight() tiles": at most split_extra_max() parts close, so there are
// at most that many split columns, that many items more than columns (per KV head and overall), and twice that many
// partial slots.  All three are functions of the problem's sizes alone, so the host can size buffers and grids.
struct ColItem {
  int32_t col;     // g * NQB + global block index of the key block, or -1
  int32_t wrange;  // bitmap words [lo, hi) of the column this item covers: lo | hi << 16
  int32_t slot;    // partial slot of this part, or -1: the item is the whole column and writes dK/dV itself
  int32_t weight;  // (query block, query head) tiles of the item
};
static_assert(sizeof(ColItem) == 16, "ColItem is loaded as 4 dwords");
struct SubItem { ColItem item; int32_t sub, pad[3]; };  // sub-part `sub` of an item
static_assert(sizeof(SubItem) == 32, "SubItem is loaded as 8 dwords");
inline int64_t bwd_total_tiles(const Geo& tg) { return (int64_t)tg.Hq * tg.nnz_unit; }  // tg = tile_geo(...)
// Total / 2048: at most an eighth of what each of the 512 workgroup slots has to do.  Half of that cut every second column of the
// block-256 workloads (each cut costs 128 KiB of partial sums written and read) and made the plan walk them (131072-token sequence:
// plan 150 -> 77 us, dK/dV the same within 1 %); twice it makes the 65536-token batch with 28/4 heads 4 % slower.
inline int split_weight(const Geo& tg) { const int64_t w = (bwd_total_tiles(tg) + 2047) / 2048; return (int)(w < 512 ? 512 : w); }
inline int split_extra_max(const Geo& tg) { return (int)(bwd_total_tiles(tg) / split_weight(tg)); }
// Small problems: fewer columns than the chip has workgroup slots (two per CU) leave most of it idle while the heaviest column
// is walked (37 blocks on 2 KV heads with 8 query heads each: 74 workgroups, up to 88 tiles in a row, 115 us).  Items of more
// than sub_weight() tiles are then walked by several workgroups, each an equal run of the item's tiles in walk order; they leave
// fp32 partial sums that the reduction adds in walk order (the same problem: 44 us with the reduction; at least 4, 6 or 12 tiles a
// workgroup: 44, 43 and 46 us).  A heaviest column of at most twice the weight is left alone (16 tiles: 25 us whole, 24 us cut, and
// plan and reduction longer by as much).
// From sub_min_columns() columns on nothing is cut this way.  At D = 128 that is 1024: two rounds of workgroups are there, heaviest
// first.  (A line at 512 columns is slower on all that lies between: 30000 tokens of one long and many short dense sequences with 16/2
// heads 1.56 -> 1.95 ms a step, 16000 tokens with 28/4 heads 0.96 -> 1.10, 30000 with 14/2 heads at D = 64 0.88 -> 1.22.  So is cutting
// only items above twice the weight: 1.52 -> 1.78, 0.96 -> 1.05 and 0.88 -> 1.10 ms, the step of 37 blocks 120 -> 128 us.)
// At D = 64 a CU holds four workgroups, which with fewer than three rounds of them (3 * 1024 columns) are handed out at once or nearly
// so, and nothing evens out unequal columns then: uncut, the kernel was slower than with the two workgroups per CU it had when it took
// more registers.  From 1024 columns on the weight is half, or hardly an item would exceed it.  dK/dV with two workgroups per CU / four
// and uncut / four and cut: 12500 tokens with 32/8 heads 328 / 367 / 260 us, 40000 tokens of one long and many short dense sequences with
// 14/2 heads 907 / 986 / 485 us, 40000 tokens with 28/4 heads and a sink 1005 / 1051 / 773 us; at 3250 columns the sink gains 14 %, other
// selections are equal or 2 % slower.
constexpr int64_t kSubMinColumns = 1024, kSubSlots = 512;
inline int64_t sub_min_columns(const Geo& tg) { return (tg.D == 64 ? 3 : 1) * kSubMinColumns; }
inline int sub_weight(const Geo& tg) {
  const int64_t slots = ((int64_t)tg.Hkv * tg.NQB >= kSubMinColumns ? 2 : 1) * kSubSlots, w = (bwd_total_tiles(tg) + slots - 1) / slots;
  return (int)(w < 8 ? 8 : w);
}
// Slots of one KV head's sub-parts (0: nothing is cut).  An item has at most all tiles of its column, and less than split_weight()
// plus one bitmap word's; one of t > w tiles takes ceil(t / w) < 2 t / w slots, and a KV head has 1 / Hkv of the tiles.  The sub-parts'
// workgroups lead the key-major launch, one per slot, interleaved by KV head like the items and a multiple of 8 in all, so that item
// r * Hkv + g behind them is still on KV head g's XCD.
inline int sub_slots_max(const Geo& tg) {
  if ((int64_t)tg.Hkv * tg.NQB >= sub_min_columns(tg)) return 0;
  const int64_t w = sub_weight(tg), col = (int64_t)tg.n_max * tg.G, part = (int64_t)split_weight(tg) + 32 * tg.G;
  if ((col < part ? col : part) <= 2 * w) return 0;
  int slots = (int)(2 * bwd_total_tiles(tg) / tg.Hkv / w) + 1;
  while (slots * tg.Hkv % 8 != 0) ++slots;
  return slots;
}
// Everything a query-major workgroup needs to know about its item, so that it starts with one
// 32-byte load instead of a chain of dependent table lookups.
struct WorkItem {
  int32_t row;     // hs * NQB + query block (index into sel_rowptr)
  int32_t seq0;    // first token of the sequence
  int32_t len;     // tokens in the sequence
  int32_t i;       // query block inside the sequence
  int32_t e0;      // first selection entry of the row
  int32_t ntiles;  // selected blocks of the row
  int32_t hs;      // selection head
  int32_t s;       // sequence
};
static_assert(sizeof(WorkItem) == 32, "WorkItem is loaded as 8 dwords");
PlanOffsets plan_offsets(const Geo& g);

struct WsOffsets {
  size_t cu_busy;    // uint64 [SB_CU_SLOTS]
  size_t qc, kc, vc, oc, doc;  // bf16 copies when dtype == SB_F32 (0 size otherwise)
  size_t drow;       // float [Hq][T]
  size_t lse2;       // float [Hq][T]
  size_t ticket;     // int32 [kTicketPlanes][kTicketInts] work tickets of the attention kernels
  size_t partials;   // float [2*E + sub-parts][dK, dV][64][D]  partial sums of the parts of split key-major columns, then of the sub-parts
  size_t bytes;
};
WsOffsets fwd_ws_offsets(const Geo& g);
WsOffsets bwd_ws_offsets(const Geo& g);
// Launches whose list is handed out by ticket (see sb_attn_common.h): its first *_lead items are tied to workgroups,
// and there are more workgroups than items, for XCDs that draw more than their share.  Where the lines lie: what is drawn must be
// enough to even out what the XCDs' paces differ by (up to 10 %).  Key-major items are columns, few and heavy: half of them; an
// eighth or a quarter of the list by ticket is 4 and 1 % slower (65536 tokens, 28/4 heads: 7.26 and 7.08 ms against 6.97), three quarters and
// all of it equal or slower; and none where head_dim 64 makes columns light (by position / drawn, 32/8 heads: columns of 4 tiles 126 / 133 us, 16
// 908 / 932, 64 2.67 / 2.67 ms; 8 tiles, 8/8 heads 207 / 219 us).  Query-major launches that do not draw item after item: a quarter, where a draw (1 us, or 5 for a
// workgroup that finds nothing left) is to a workgroup's 20 us and more.
constexpr int64_t kTicketMinItems = 4096;  // shorter lists are dealt by position only
constexpr int kTicketPlanes = 16;          // of 8 counters, which are cache lines apart (in one line 8 XCDs' draws waited for each other: 15 us each)
constexpr int kTicketPitch = 64, kTicketInts = 8 * kTicketPitch;
inline bool use_tickets(int64_t n) { return n >= kTicketMinItems; }
inline __host__ __device__ int query_lead(int n) { return n / 32 * 24; }
inline __host__ __device__ int64_t held_items(int64_t n) { return n >> 7 << 3; }
inline int64_t held_grid(int64_t n) { return (n + held_items(n) + 7) / 8 * 8; }
inline int64_t last_grid(int64_t n) { return (n + n / 64 + 7) / 8 * 8; }
inline __host__ __device__ int key_lead(int n) { return n / 16 * 8; }
inline __host__ __device__ int64_t key_extra(int64_t n) { return n / 8; }
inline bool use_key_tickets(const Geo& tg, int64_t n) {
  return use_tickets(n) && n + key_extra(n) < (1ll << 24) && (tg.D == 128 || bwd_total_tiles(tg) >= 32 * (int64_t)tg.Hkv * tg.NQB);  // (a launch has fewer than 2^32 threads)
}
// Is a query-major item of one query head one wavefront's work, or two's?  Of `items` with at most `most` tiles, w wavefronts each, the
// chip works on 1024 / w at a time (head_dim 64: twice as many); an item costs about `fixed` tile times of two wavefronts besides its
// tiles (where the chip is not full and its clock is high: forward 16, dQ and head_dim 64 24), and the launch takes as long as its share
// of all items, as the longest item, or, where there are more items than fit, as two short ones.  So one wavefront each where there are
// enough items, two where the longest would stick out.  One / two wavefronts at head_dim 128: forward, 1280 items of 1 - 11 tiles
// 45.6 / 46.6 us, 1056 of 1 - 8 tiles 26 / 34, 592 of 1 - 11 tiles 25.4 / 26.8, 1248 of 1 - 78 tiles 126 / 113, 432 of 1 - 54 tiles 78 / 47;
// dQ, 1230 items of 1 - 11 tiles 31 / 41, 592 of them 24.2 / 26.5, 1248 items of 1 - 78 tiles 162 / 152, 432 of 1 - 54 tiles 92 / 59.
// At head_dim 64 the SIMD's other wavefront works through three quarters of the fixed part.  The sixteenth added to one wavefront's time
// there is a tie-break: where the two terms are about equal, two wavefronts, which gather for half as many items at a time, were the
// faster ones in what was measured, for reasons not shown (65536 tokens, 14/2 heads, blocks of 256: forward 1482 / 1436 us, dQ 1812 / 1767; 24551
// tokens, 32/8 heads, rows of up to 256 tiles: dQ 1156 / 1066, 24576 tokens: forward 2424 / 2227); where one wavefront wins it does so by more
// (6144 items of 1 - 16 tiles: forward 121 / 131, dQ 131 / 143).
inline bool one_wavefront_per_item(const Geo& tg, int64_t items, int fixed) {
  const bool d64 = tg.D == 64;
  const int64_t tiles = (int64_t)tg.Hq * tg.nnz_unit, most = tg.rowT_max, slots = d64 ? 2048 : 1024;
  auto time = [&](int64_t w) {  // of the launch, in 1/32 of the time that two wavefronts take for a tile
    int64_t t = 32 * ((d64 ? fixed / 4 : fixed) * items * w + 2 * tiles) / slots;
    if (d64 && w == 1) t += t / 16;
    const int64_t longest = 32 * (fixed + 2 * most / w), two = 32 * (2 * fixed + 2);
    if (longest > t) t = longest;
    if (items * w > slots && two > t) t = two;
    return t;
  };
  return time(1) <= time(2);
}
// How the items of a query-major launch of one query head each are handed out (see ItemQueue in sb_attn_common.h): all by position, one in
// sixteen held back, the last quarter drawn, or drawn one after the other by as many workgroups as the chip runs at a time (head_dim 128).
// Draws keep an item near its head's L2 and end the launch evenly, but each is an atomic across the chip, 1 - 2 us of its workgroup, which
// rows of a few tiles do not earn back unless there are many of them.  In us, alone, 32/8 heads, one sequence:
//   forward, D = 128  position / drawn:  9024 items of 1, 4, 16, 32 tiles 105 / 123, 165 / 177, 351 / 355, 596 / 588; 20000 items of 1, 8, 16, 32 tiles 206 / 218,
//                     525 / 524, 819 / 803, 1367 / 1360; 65536 items of 1, 2, 8 tiles 611 / 612, 805 / 797, 2071 / 1960; 16384 of 8 (8/8 heads) 557 / 537
//   forward, D = 64   position / last:   9024 items of 1, 4, 16, 32 tiles 44 / 51, 72 / 77, 184 / 190, 334 / 330; 65536 items of 1, 4, 16, 32 tiles 284 / 311, 596 / 612,
//                     1780 / 1693, 3175 / 3026; 20000 of 8 266 / 277, 16384 (8/8 heads) 279 / 272
//   dQ, D = 128       held / drawn:      9024 items of 1, 4, 16, 32 tiles 169 / 180, 212 / 219, 447 / 452, 772 / 752; 20000 of 2 402 / 382
//   dQ, D = 64        held / last:       9024 items of 1, 4, 16, 32 tiles 81 / 85, 97 / 103, 227 / 233, 428 / 418; 65536 items of 1, 4, 8 tiles 552 / 600, 769 / 779, 1226 / 1202
// (dQ by position: 180, 232, 472 and 795; 85, 102, 242 and 433.)  What is held back are items of every weight: where the longest is not small
// against a workgroup's share of all, they are the launch's end (head_dim 64, 7600 items of 1 - 21 tiles, 44 a workgroup: dQ 184 / 161; 6208 of 1 - 16,
// 23 a workgroup: 106 / 96).
enum Deal { kDealPosition, kDealHeld, kDealLast, kDealDraw };
inline __host__ __device__ int64_t head_ids(int64_t n_items, int heads) { return (n_items + 7) / 8 * 8 * heads; }
inline bool may_deal(int64_t n_items, int heads) { return use_tickets(n_items) && head_ids(n_items, heads) < (1ll << 30); }
inline bool rows_of(const Geo& tg, int64_t tiles) { return tg.nnz_unit >= tiles * tg.NQB; }  // mean
inline Deal forward_deal(const Geo& tg, int64_t n_items, int heads) {
  if (!may_deal(n_items, heads)) return kDealPosition;
  const int64_t items = (int64_t)tg.Hq * tg.NQB;
  if (tg.D == 128) return rows_of(tg, 15) || (rows_of(tg, 7) && items >= 16384) || items >= 32768 ? kDealDraw : kDealPosition;
  return rows_of(tg, 24) || (rows_of(tg, 12) && items >= 16384) ? kDealLast : kDealPosition;
}
inline Deal dq_deal(const Geo& tg, int64_t n_items, int heads) {
  if (!may_deal(n_items, heads)) return kDealPosition;
  const int64_t items = (int64_t)tg.Hq * tg.NQB;
  const bool even = (int64_t)tg.rowT_max * (tg.D == 64 ? 3 * 2048 : 2 * 1024) <= tg.nnz_unit * tg.Hq;
  if (tg.D == 128) return rows_of(tg, 24) || items >= 16384 || !even ? kDealDraw : kDealHeld;
  return rows_of(tg, 24) || (rows_of(tg, 7) && items >= 32768) || !even ? kDealLast : kDealHeld;
}
size_t scores_ws_bytes(const Geo& g);
size_t coverage_ws_bytes(const Geo& g);

// Zero `bytes` (a multiple of 4) at `dst` with a small kernel on `st`: unlike a memset node this is safe to record
// into a HIP graph.
int fill_zero(void* dst, size_t bytes, hipStream_t st);
int fill_words(void* dst, size_t bytes, uint32_t value, hipStream_t st);

extern std::atomic<int> g_instrument;  // bit 0: per-CU busy ticks, bit 1: HIP events around each kernel

// HIP-event bracket around one kernel launch on its own stream (only when bit 1 is set).
enum KernelSlot { K_POOL = 0, K_SCORE, K_TOPK, K_PLAN, K_FWD, K_BWD_PREP, K_BWD_DQ, K_BWD_DKV, K_COVERAGE, K_SCORE_SELECT, K_NUM };
static_assert(K_NUM == SB_NUM_KERNELS, "kernel slots");
struct KernelTimer {
  int slot; hipStream_t st; void* start = nullptr;
  KernelTimer(int slot, hipStream_t st);
  ~KernelTimer();
};

}  // namespace sb
