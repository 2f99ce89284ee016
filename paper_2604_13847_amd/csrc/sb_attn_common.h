// Device helpers shared by the forward and backward attention kernels (gfx950, wave64).
//
// MFMA used: v_mfma_f32_32x32x16_bf16.  Operand layout per lane (half = lane/32):
//   A (32 x 16): row = lane%32, the 8 elements are contraction slots (half, 0..7)
//   B (16 x 32): col = lane%32, the 8 elements are contraction slots (half, 0..7)
//   C (32 x 32): col = lane%32, register v is row 8*(v/4) + 4*half + v%4
// A and B only have to agree on which contraction index sits in slot (half, e); the kernels choose
// that mapping freely (see c_row below).
#pragma once

#include "sb_internal.h"

namespace sb {

struct AttnParams {
  const bf16* q; const bf16* k; const bf16* v; const bf16* d_o;
  void* o;            // forward output (bf16 or float per out_f32)
  float* lse;         // [Hq][T]
  float* drow;        // [Hq][T] rowsum(dO * O): written by the dQ kernel, read by the dK/dV kernel
  float* lse2;        // [Hq][T] lse * log2(e), likewise
  void* dq; void* dk; void* dv;
  const int32_t* idx;  // the selected tiles
  const WorkItem* items;  // descriptors of the query-major items, in work order
  const uint32_t* bitmap;
  const ColItem* bwd_items;    // key-major items (whole columns or parts of heavy ones), see ColItem
  const int32_t* split_cols;   // (column, first partial slot, parts) of the split columns; counters[1] of them
  const int32_t* counters;
  float* partials;             // [slot][dK, dV][64][D] fp32 partial sums of the parts of split columns
  const int32_t* sub_base;     // of every key-major item of KV head g: its sub-parts have slots Hkv*(sub_base + 0, 1, ...) + g; -1: walked as a whole
  const int32_t* part_item;    // key-major item of every partial slot
  float* sub_partials;         // like partials, of the sub-parts
  const SubItem* sub_items;    // the sub-parts, sub_slots entries
  int sub_weight, sub_slots;   // sub-parts of an item: ceil(tiles / sub_weight); sub_slots = 0: no item has any
  const int32_t* cu; const int32_t* qb_off; const int32_t* qb_seq; const int64_t* bm_off;
  int64_t NQB;
  int T, Hq, Hkv, G, Hs, mode;
  float scale, scale_log2e;
  int out_f32;
  unsigned long long* cu_busy;  // null when instrumentation is off
  // Work distribution (see held_item, draw_item and ItemQueue)
  int* ticket;        // counters, zero at launch: 8, or one for items that are held back (the group kernel: one per head plane); null: every item is taken by position
  int n_items;        // query-major items
  int deal;           // Deal, of a launch of one query head per item
};
// float -> bf16 copies of one launch
struct Conversions {
  const void* src[4]; void* dst[4]; int64_t n4[4];
  int n;
  void add(const void* from, void* to, int64_t elems) { src[n] = from; dst[n] = to; n4[n++] = elems / 4; }
};
int convert_f32_to_bf16(const Conversions& c, hipStream_t st);

// Which item does a workgroup work on?
// Workgroup ids are dealt to the 8 XCDs in turn, so every XCD gets the same number of workgroups whatever its pace, and the XCDs do
// differ by several percent (the L2 hit rate depends on which heads an XCD serves, and the dies themselves differ): a launch that ties
// every item to a position ends when the slowest XCD is through its share.  Two ways round that (sb_internal.h has the lines between them):
// - One item in sixteen, the last 8 of every 128 in list order, is held back: the other items are tied to the leading positions and the
//   held-back ones handed out by one counter at the end, to whichever workgroup asks first, in twice as many workgroups (held_*).
// - Only the list's first part, the heavier items, is tied to positions (*_lead).  Of the rest every eighth item is an XCD's, as if it
//   were dealt by position, but handed out in list order by that XCD's own counter, and an XCD that is through its items takes the next one of the
//   XCD that has most left (draw_item).  An item so stays on the XCD whose L2 holds its head unless it is one of the launch's last, and those
//   are the lightest.
// (The first against the second: one 131072-token sequence, top 32: forward 6.20 -> 5.75 ms, dQ 6.39 -> 6.18.  dK/dV without any, against
// the second: that sequence 10.4 -> 10.15 ms, 65536 tokens with 28/4 heads 7.3 -> 6.9, with a sink 3.47 -> 3.28, the 262144-token batch 34.2 -> 33.3.)
// Which workgroup computes an item never changes its result.
__device__ inline int held_lead(int pos, int held) { return pos < 15 * held ? (pos / 120 << 7) + pos % 120 : pos + held; }  // item of a leading position
__device__ inline int held_item(int held, int* counter) {  // the next one that was held back, or -1; by one thread
  const int t = atomicAdd(counter, 1);
  return t < held ? (t >> 3 << 7) + 120 + (t & 7) : -1;
}
// draw_item: an index from `lead` on, or -1 if all have been drawn; by one thread.
__device__ inline int draw_item(int xcd, int lead, int n, int* counters) {
  for (int tries = 0; tries < 9; ++tries) {
    const int item = lead + 8 * atomicAdd(&counters[kTicketPitch * xcd], 1) + xcd;
    if (item < n) return item;
    int left[8], most = 0;
#pragma unroll
    for (int x = 0; x < 8; ++x) left[x] = (n - lead - x + 7) / 8 - __hip_atomic_load(&counters[kTicketPitch * x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int x = 0; x < 8; ++x)
      if (left[x] > most) { most = left[x]; xcd = x; }
    if (most == 0) break;
  }
  return -1;
}
// The item of the workgroup at position `pos` of a launch that holds one in sixteen back (or, without a counter, of any), or -1; every
// thread of the workgroup must call it (it has a barrier).
__device__ inline int claim_item(int pos, int n_items, int* counter) {
  if (!counter) return pos < n_items ? pos : -1;
  const int held = (int)held_items(n_items);
  if (pos < n_items - held) return held_lead(pos, held);
  __shared__ int sh_claim;
  if (threadIdx.x == 0) sh_claim = held_item(held, counter);
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(sh_claim);
}

// Descriptor `pos` (wave-uniform) by scalar loads, so that everything that follows from it is scalar work.
__device__ inline WorkItem uniform_item(const WorkItem* items, int pos) {
  typedef int i32x8 __attribute__((ext_vector_type(8)));
  const i32x8 x = ((const __attribute__((address_space(4))) i32x8*)(uintptr_t)items)[__builtin_amdgcn_readfirstlane(pos)];
  return WorkItem{x[0], x[1], x[2], x[3], x[4], x[5], x[6], x[7]};
}

// The items of a query-major launch of one query head each: id -> (position in the work list, query head of the group).  In per-KV-group
// mode the `heads` query heads of an item have ids that are 8 apart, so they run on the same XCD (workgroup ids are dealt to the XCDs in
// turn) and share its L2.
inline int64_t head_grid(const AttnParams& P, int heads, int nw) {
  const int64_t ids = head_ids(P.n_items, heads);
  return P.deal == kDealDraw ? 1024 / nw : P.deal == kDealLast ? last_grid(ids) : P.deal == kDealHeld ? held_grid(ids) : ids;
}
// The items of one workgroup.  By position: workgroup w takes item w.  Held back: one item each too, the last ones by ticket.  Drawn at D = 128, where a
// wavefront fills its SIMD: as many workgroups as the chip runs at a time, which draw one item after the other.  At D = 64 workgroups take one item each, the
// last quarter by ticket: there the next workgroup's start overlaps the end of the last (drawing all: forward of 65536 tokens, 14/2 heads,
// blocks of 256 1.40 -> 1.44 ms).  At D = 128 the draw takes the place of a workgroup's start, against a quarter of the items by ticket, one a
// workgroup: the forward of 65536 tokens whose selection is a sink and a window 1.76 -> 1.66 ms, dQ 2.13 -> 2.06, of 131072 items of one or
// four tiles 650 -> 613 us and 1.19 -> 1.15 ms.  (The draw ahead of an item's output: 2 % faster on rows of 32 tiles, 4 % slower on short ones.)
// LOOP: the launch draws item after item.  A kernel of its own, because the loop costs a launch without tickets up to 1.4 us (2039 tokens,
// 16/2 heads: forward 22.0 -> 20.7 us).
// `sh` is an LDS word for launches of two wavefronts per item, which only wavefronts other than the first write otherwise.
// HELD: the launch may hold one item in 16 back.
template <int D, int NW, bool LOOP, bool HELD>
struct ItemQueue {
  WorkItem item;
  int hh;  // query head of the group
  int id, ids, lead, heads;
  __device__ inline int pos_of(int id) const { return id / (8 * heads) * 8 + (id & 7); }
  __device__ inline int drawn(const AttnParams& P) const {
    if (HELD && P.deal == kDealHeld) return held_item((int)held_items(ids), P.ticket);
    return draw_item(blockIdx.x & 7, lead, ids, P.ticket);
  }
  __device__ inline void draw(const AttnParams& P, int* sh) {
    int t = 0;
    if (threadIdx.x == 0) {
      do t = drawn(P);
      while (t >= 0 && pos_of(t) >= P.n_items);  // (the last ids may have no item)
      if (NW == 2) *sh = t;
    }
    id = __builtin_amdgcn_readfirstlane(t);
    if (NW == 2) {
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) != 0) id = __builtin_amdgcn_readfirstlane(*sh);
    }
  }
  __device__ inline void descriptor(const AttnParams& P) {
    if (id < 0) return;
    item = uniform_item(P.items, pos_of(id));
    hh = (id >> 3) % heads;
  }
  __device__ inline void first(const AttnParams& P, int heads_, int* sh) {
    heads = heads_;
    ids = (int)head_ids(P.n_items, heads);
    id = (int)blockIdx.x;
    lead = LOOP ? (int)gridDim.x : ids;
    if (D == 64 && P.deal == kDealLast) lead = query_lead(ids);
    if (HELD && P.deal == kDealHeld) lead = ids - (int)held_items(ids);
    if ((LOOP || D == 64 || HELD) && id >= lead) {
      draw(P, sh);
    } else {
      if (HELD && P.deal == kDealHeld) id = held_lead(id, (int)held_items(ids));
      if (pos_of(id) >= P.n_items) id = -1;
    }
    descriptor(P);
  }
  __device__ inline void next(const AttnParams& P, int* sh) {
    if (NW == 2) __syncthreads();  // the item's LDS is free
    draw(P, sh);
    descriptor(P);
  }
};
// What does not depend on the item would otherwise be worked out and kept in registers from before the loop, ahead of what the item needs.
template <bool LOOP>
__device__ inline int item_tid() {
  int x = (int)threadIdx.x;
  if (LOOP) asm volatile("" : "+v"(x));
  return x;
}
__device__ inline AttnParams reloaded_params() {  // the kernel's first argument, by scalar loads
  const __attribute__((address_space(4))) AttnParams* p = (const __attribute__((address_space(4))) AttnParams*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const AttnParams*)p;
}
template <int D, int NW, bool LOOP, bool HELD, typename F>
__device__ __attribute__((always_inline)) inline void for_items(const AttnParams& P, int heads, int* sh, F work) {
  ItemQueue<D, NW, LOOP, HELD> queue;
  queue.first(P, heads, sh);
  if constexpr (LOOP) {
    for (; queue.id >= 0; queue.next(P, sh)) work(reloaded_params(), queue.item, queue.hh);
  } else {
    if (queue.id >= 0) work(P, queue.item, queue.hh);
  }
}

__device__ inline f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// The same with the accumulator in arithmetic registers and the B operand in accumulation registers: in a kernel that needs more
// than 256 registers the compiler would put every accumulator into accumulation registers and copy the scores out one by one.
// It does not see these as matrix instructions: the caller keeps at least 12 wait states (half a stage of matrix instructions)
// between the last of a chain and the first reader of its result.
__device__ inline void mfma32_first(f32x16& c, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "a"(b));
}
__device__ inline void mfma32_more(f32x16& c, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "a"(b));
}
__device__ inline void mfma32_more_v(f32x16& c, bf16x8 a, bf16x8 b) {  // all three in arithmetic registers
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
// The other way round, for a running sum: accumulator in accumulation registers, both operands in arithmetic registers.  The caller
// keeps two wait states between a vector instruction that wrote an operand and this, and 12 before the accumulator is read.
__device__ inline void mfma32_sum(f32x16& c, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}

__device__ inline f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.f;
  return z;
}

__device__ inline bf16x8 zero_bf16x8() {
  bf16x8 z;
#pragma unroll
  for (int i = 0; i < 8; ++i) z[i] = (bf16)0.f;
  return z;
}

// Row (0..31) of C register v for a lane in half `hf`.
__device__ inline int c_row(int v, int hf) { return 8 * (v >> 2) + 4 * hf + (v & 3); }

// A 64-long contraction axis (keys or queries of one block) is walked in 4 steps of 16; step kk,
// slot (hf, e) holds element 16*kk + 8*(e/4) + 4*hf + e%4, which is exactly the row of C register
// 8*(kk%2)+e of the (kk/2)-th 32x32 tile: a C tile converts to an A/B operand without any shuffle.

// ---------------------------------------------------------------------------------------------
// Asynchronous tile staging.  A 64 x D bf16 tile lives in LDS unpadded (row r at byte r*2D), with
// the 16-byte chunks of each row permuted by chunk_swizzle(r): chunk c of row r sits at chunk
// c ^ chunk_swizzle(r).  The permutation makes both access patterns of the MFMA operands free of
// bank conflicts: (a) 16 lanes reading the same chunk of 16 consecutive rows, (b) a transposing
// read where 16 lanes cover 4 consecutive rows x 32 bytes.
// Tiles are written by global_load_lds_dwordx4: each lane fetches 16 bytes from its own global
// address and the wavefront's 1 KiB lands at M0 + 16*lane, so no registers are spent on data in
// flight.  The instruction is issued through inline asm on purpose: the waits are placed by hand
// (wait_vmcnt) so that loads stay in flight across the compute on the previous tile.
template <int D>
__device__ inline int chunk_swizzle(int r) {
  // D = 128 (16 chunks, one row = all 64 banks): the two low row bits pick the 64-byte quarter of the
  // row, the next two the chunk inside it.  A transposing read (32 lanes = 4 rows x 64 bytes) then
  // covers 8 distinct 32-byte bank groups and a row-wise read (16 rows, same chunk) 16 distinct chunks.
  if (D == 128) return ((r & 3) << 2) | ((r >> 2) & 3);
  // D = 64 (8 chunks, two rows = all banks): row bit 0 already selects the bank half.
  return (((r >> 1) & 1) << 2) | ((r >> 2) & 3);
}

__device__ inline unsigned lds_offset(const void* p) {
  return (unsigned)(size_t)(const __attribute__((address_space(3))) char*)p;
}

__device__ inline void dma16(const void* gptr, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(gptr), "s"(lds_base) : "memory", "m0");
}

// s_waitcnt vmcnt(N) only (the other counters stay unconstrained).  The memory clobber keeps the
// compiler from moving LDS reads of the awaited tile above the wait.
template <int N>
__device__ inline void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// Per-lane byte offsets (from the tile's first row, head h) of the loads a loader wavefront issues for a tile: the first four wavefronts
// of the workgroup share them, and wavefront w takes the LPT consecutive KiB (LPT * w + a) of the tile, a = 0 .. LPT-1, i.e. tile rows
// (LPT * w + a) * RPI .. +RPI-1.  The offsets depend only on the lane and on the tensor's row pitch, so they are computed once per kernel.
template <int D>
struct TileLoader {
  static constexpr int NW = 4;
  static constexpr int C = D / 8;           // 16-byte chunks per row
  static constexpr int RPI = 64 / C;        // rows covered by one wavefront-wide load
  // Loads per loader wavefront and tile.  They land 1 KiB apart in LDS, so one M0 value serves all of them: the instruction's immediate
  // offset moves both the global and the LDS address, and voff is pre-biased for it.
  static constexpr int LPT = (D / 8) / NW;
  static_assert((LPT == 2 || LPT == 4) && LPT * NW * RPI == 64, "the loader wavefronts must cover the 64 rows exactly");
  unsigned voff[LPT];
  int rl, pc;  // row within a load's group of RPI rows, 16-byte chunk of this lane
  int wave;
  __device__ inline void init(int H, int wave_, int lane) {
    wave = wave_;
    rl = lane / C;
    pc = lane % C;
#pragma unroll
    for (int a = 0; a < LPT; ++a) {
      const int r = (LPT * (wave & (NW - 1)) + a) * RPI + rl;
      voff[a] = (unsigned)(r * H * D * 2 + 16 * (pc ^ chunk_swizzle<D>(r))) - 1024u * a;
    }
  }
  // Issue the copy of rows row0 .. row0+63 (head h) of `src` into `slot`.  Rows >= valid repeat the
  // last valid row; their data is always masked by the consumer.  Wavefronts 0 .. NW-1 issue LPT loads
  // each, the others none.  Full tiles (the common case) use a scalar base address plus the
  // precomputed lane offsets, so no vector arithmetic is spent per load.
  __device__ inline void issue(bf16* slot, const bf16* src, int64_t row0, int valid, int H, int h) const {
    if (wave >= NW) return;
    const unsigned base = lds_offset(slot) + LPT * (wave & (NW - 1)) * 1024;  // this wavefront's part of the tile
    const char* tile = (const char*)(src + (row0 * H + h) * D);
    if (valid >= 64) {
      const unsigned long long tv = (unsigned long long)tile;  // wave-uniform: move it to scalar registers
      // (readfirstlane returns int: go through unsigned so that the low half is not sign-extended)
      const unsigned t_hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(tv >> 32));
      const unsigned t_lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(tv & 0xffffffffull));
      const unsigned long long ts = ((unsigned long long)t_hi << 32) | (unsigned long long)t_lo;
      // The base is copied by a scalar instruction first: a scalar register written by a vector instruction
      // (readfirstlane) must not be read by a vector-memory instruction within 5 wait states, while scalar reads of
      // it are interlocked.  M0 needs one wait state (s_nop 0) before the load that uses it.
      unsigned long long sbase;
      if constexpr (LPT == 4)
        asm volatile("s_mov_b64 %0, %6\n\ts_mov_b32 m0, %5\n\ts_nop 0\n\t"
                     "global_load_lds_dwordx4 %1, %0\n\t"
                     "global_load_lds_dwordx4 %2, %0 offset:1024\n\t"
                     "global_load_lds_dwordx4 %3, %0 offset:2048\n\t"
                     "global_load_lds_dwordx4 %4, %0 offset:3072"
                     : "=&s"(sbase) : "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3]), "s"(base), "s"(ts) : "memory", "m0");
      else
        asm volatile("s_mov_b64 %0, %4\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\t"
                     "global_load_lds_dwordx4 %1, %0\n\t"
                     "global_load_lds_dwordx4 %2, %0 offset:1024"
                     : "=&s"(sbase) : "v"(voff[0]), "v"(voff[1]), "s"(base), "s"(ts) : "memory", "m0");
    } else {
#pragma unroll
      for (int a = 0; a < LPT; ++a) {  // ragged tile (rare): the lane offsets are recomputed instead of being kept in registers
        const int r = (LPT * (wave & (NW - 1)) + a) * RPI + rl;
        dma16(tile + (int64_t)min(r, valid - 1) * H * D * 2 + 16 * (pc ^ chunk_swizzle<D>(r)), base + a * 1024);
      }
    }
  }
};

typedef int i32x4 __attribute__((ext_vector_type(4)));

// One wavefront copies a strip of 32 rows of one head of a [T][H][D] tensor into LDS (layout as above) with buffer loads: the buffer
// resource covers the rows that exist, and rows past it arrive as zeros without a branch or a per-lane clamp.  The resource is four
// scalar registers that the caller keeps: a wavefront that has its SIMD to itself issues one instruction every four cycles whatever it
// is, so a scalar instruction there costs as much as a vector one.  The immediate offset moves both the global and the LDS address, so
// four loads in a row need one M0, and the lane offsets are pre-biased for it (row 4a of the strip starts at least 1024 a bytes in, so
// they stay positive).  The resource's words must come from scalar instructions: a scalar register written by a vector instruction
// (readfirstlane, readlane) must not be read by a vector-memory instruction within 5 wait states, and the compiler does not look into
// the block for that (tests/test_hazards.py looks at what it made).  M0 needs one wait state before the load that uses it.
template <int D>
struct QuadLoader {
  static constexpr int C = D / 8, RPI = 64 / C, LPS = 32 / RPI;  // 16-byte chunks per row, rows per load, loads per strip
  unsigned voff[LPS];
  __device__ inline void init(int H, int lane) {
#pragma unroll
    for (int a = 0; a < LPS; ++a) {
      const int r = a * RPI + lane / C;
      voff[a] = (unsigned)(r * H * D * 2 + 16 * ((lane % C) ^ chunk_swizzle<D>(r)) - 1024 * (a & 3));
    }
  }
  // the first `bytes` bytes from `base` on exist, the rest arrives as zeros; both wave-uniform
  __device__ static inline i32x4 resource(unsigned long long base, unsigned bytes) {
    return i32x4{(int)(unsigned)base, (int)(unsigned)(base >> 32), (int)bytes, 0x20000};
  }
  template <int A>
  __device__ inline void issue2(i32x4 rsrc, unsigned slot) const {  // loads A, A+1 (A even) of a strip
    asm volatile("s_add_u32 m0, %2, %4\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %0, %3, 0 offen offset:%5 lds\n\tbuffer_load_dwordx4 %1, %3, 0 offen offset:%6 lds"
                 : : "v"(voff[A]), "v"(voff[A + 1]), "s"(slot), "s"(rsrc), "n"(A / 4 * 4096), "n"(A % 4 * 1024), "n"(A % 4 * 1024 + 1024)
                 : "memory", "m0", "scc");
  }
  __device__ inline void issue(i32x4 rsrc, unsigned slot) const {
    issue2<0>(rsrc, slot);
    issue2<2>(rsrc, slot);
    if constexpr (LPS > 4) { issue2<4>(rsrc, slot); issue2<6>(rsrc, slot); }
  }
};
// The 32-key strips that a wavefront of a query-major item walks: with two wavefronts per item (NW = 2) wavefront w takes strip w of every
// tile the row keeps, with one it takes both, one after the other.
template <int D, int NW>
struct StripWalk {
  const int32_t* idx;  // the row's block indices
  int ntiles, nstrips;
  // Lane a holds index jb0 + a; refilled every ~64 tiles, which waits for all loads in flight.
  int jb0, jreg;
  unsigned block_pitch, half_pitch;     // bytes from one key block to the next, from one strip to the next
  // Bytes of a strip that exist.  Only the row's last tile, the diagonal one, can end with the sequence; the missing rows arrive as zeros
  // and are masked.  Strips past the last tile are requested like the others, with no byte in existence, so that the number of loads
  // in flight is the same everywhere and a loop has no branch for it.
  unsigned full_bytes, last_a, last_b;  // of any other strip, of the last tile's first (or this wavefront's) strip, of its second
  __device__ inline void init(const WorkItem& item, const int32_t* all_idx, int Hkv, int wave, int lane) {
    idx = all_idx + item.e0;
    ntiles = item.ntiles;
    nstrips = NW == 2 ? ntiles : 2 * ntiles;
    jb0 = 0;
    jreg = lane < ntiles ? idx[lane] : 0;
    const unsigned pitch = (unsigned)Hkv * D * 2;
    block_pitch = 64u * pitch;
    half_pitch = 32u * pitch;
    auto bytes = [&](int rows) { return rows > 0 ? (unsigned)(min(rows, 32) - 1) * pitch + D * 2 : 0u; };
    const int rows = item.len - item.i * 64;
    full_bytes = 31u * pitch + D * 2;
    last_a = bytes(rows - (NW == 2 ? 32 * wave : 0));
    last_b = bytes(rows - 32);
  }
  // strips t, t + 1, ... t + ahead are about to be asked for
  __device__ inline void window(int t, int ahead, int lane) {
    const int tile = NW == 2 ? t : t >> 1, end = NW == 2 ? t + ahead : (t + ahead) >> 1;
    if (end - jb0 < 64) return;
    jb0 = tile;
    jreg = jb0 + lane < ntiles ? idx[jb0 + lane] : 0;
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), here and not at the join behind this branch, where it would drain the loads in flight every time
  }
  __device__ inline unsigned bytes_of(int t) const {
    if (NW == 2) return t < nstrips - 1 ? full_bytes : t == nstrips - 1 ? last_a : 0u;
    return t < nstrips - 2 ? full_bytes : t == nstrips - 2 ? last_a : t == nstrips - 1 ? last_b : 0u;
  }
  // from the wavefront's strip of the sequence's first block
  __device__ inline unsigned long long offset_of(int t) const {
    const unsigned long long o = (unsigned long long)(unsigned)__builtin_amdgcn_readlane(jreg, (NW == 2 ? t : t >> 1) - jb0) * block_pitch;
    return NW == 2 ? o : o + (t & 1) * half_pitch;
  }
};
// 64 consecutive floats to LDS, those that the resource (see QuadLoader) does not cover as zeros
__device__ inline void load_floats(unsigned slot, i32x4 rsrc, int lane4) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dword %0, %2, 0 offen lds" : : "v"(lane4), "s"(slot), "s"(rsrc) : "memory", "m0");
}
// x * f for an accumulator element that lives in an accumulation register.  Written as one opaque
// block so that the copies to and from the arithmetic registers stay inside the (rarely taken)
// branch that needs them instead of being hoisted into the main loop.
__device__ inline float scale_acc(float x, float f) {
  float tmp;
  asm volatile("v_accvgpr_read_b32 %1, %0\n\tv_mul_f32 %1, %1, %2\n\tv_accvgpr_write_b32 %0, %1" : "+a"(x), "=&v"(tmp) : "v"(f));
  return x;
}

// max(a, b, c) in one instruction.  Written as asm because the compiler's fmax first quiets a possible
// signalling NaN in every operand it has not produced itself (an extra instruction per value read
// back from an accumulator); a NaN operand is simply dropped by the hardware instruction.
__device__ inline float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// acc + p[0] + p[1] in one instruction (fp32 accumulation of two bf16 values)
__device__ inline float sum2(bf16x2 p, float acc) {
  bf16x2 one;
  one[0] = (bf16)1.0f;
  one[1] = (bf16)1.0f;
  return __builtin_amdgcn_fdot2_f32_bf16(p, one, acc, false);
}

// max of x over the two lanes l and l + 32 (both receive it): one lane-half swap, no LDS round trip
__device__ inline float max_across_halves(float x) {
  const unsigned u = __float_as_uint(x);
  // returns {own low half | partner's low half, partner's high half | own high half}: element 0 holds
  // the low half's value in every lane, element 1 the high half's
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// A wavefront stores 32 rows of one head that it holds as C tiles (lane%32: row, value(dt, v): column 32dt + c_row(v, lane/32)): the
// rows go through LDS (`buf`, the wavefront's own, 32 rows), so that every store covers whole rows.  Straight from the registers a store
// would be 8 bytes here and there, 16 of them to a row.
template <int D, bool F32, typename V>
__device__ inline void store_rows(char* buf, void* out, int64_t first, int64_t pitch, int rows, int lane, V value) {
  constexpr int EB = F32 ? 4 : 2, C = D * EB / 16, RPI = 64 / C;  // bytes per element, 16-byte chunks per row, rows per store
  const int l32 = lane & 31, hf = lane >> 5;
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int vg = 0; vg < 4; ++vg) {
      const int byte = (32 * dt + 8 * vg + 4 * hf) * EB;
      char* const at = buf + l32 * (D * EB) + 16 * ((byte >> 4) ^ (l32 & (C - 1))) + (byte & 15);
      if constexpr (F32) {
        *(f32x4*)at = f32x4{value(dt, 4 * vg), value(dt, 4 * vg + 1), value(dt, 4 * vg + 2), value(dt, 4 * vg + 3)};
      } else {
        bf16x4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = (bf16)value(dt, 4 * vg + e);
        *(bf16x4*)at = y;
      }
    }
  asm volatile("" ::: "memory");  // (LDS operations of a wavefront complete in order)
#pragma unroll
  for (int a = 0; a < 32 / RPI; ++a) {
    const int r = a * RPI + lane / C, c = lane % C;
    const f32x4 x = *(const f32x4*)(buf + r * (D * EB) + 16 * (c ^ (r & (C - 1))));
    if (r < rows) *(f32x4*)((char*)out + (first + r * pitch) * EB + 16 * c) = x;
  }
}

struct BusyTimer {
  long long t0;
  __device__ inline void start(const AttnParams& P) {
    if (P.cu_busy && threadIdx.x == 0) t0 = wall_clock64();
  }
  __device__ inline void stop(const AttnParams& P) {
    if (P.cu_busy && threadIdx.x == 0) atomicAdd(&P.cu_busy[__smid() & (SB_CU_SLOTS - 1)], (unsigned long long)(wall_clock64() - t0));
  }
};

}  // namespace sb
