// Work plan: longest-first ordering of the query-major items, the key-major transpose of the
// selection as a bitmap, and heaviest-first ordering of the key-major columns (per KV head).
//
// Query-major items.  Item (s,hs,i) costs c = min(k_s, i+1) selected tiles.  Because the cost is a
// closed form of (k_s, n_s, i), the rank of an item in the order (cost descending, then sequence,
// then query block, then head with the KV head fastest) is a closed form too: every thread
// computes its own rank with one pass over the S sequences, without sorting or atomics.  Adjacent
// ranks differ in the KV head first, so with workgroups dealt round-robin to the 8 XCDs each XCD's
// L2 keeps seeing the same KV heads.
//
// Key-major transpose.  Bit i of word (s,hs,j,i/32) says query block i kept key block j; the bitmap
// is a pure function of the selection, so the backward pass walks a column's query blocks in a
// fixed order and accumulates deterministically.
#include "sb_geom.h"
#include "sb_internal.h"

namespace sb {

struct PlanArgs {
  const int32_t *rowptr, *idx;             // the selection, at block level
  const int32_t *cu, *qb_off, *kclamp, *qb_seq;  // tile-level tables (for 64-token selection blocks tiles are blocks)
  const int64_t* bm_off;
  const int32_t *b_qb_off, *b_kclamp;      // block-level tables
  int S, Hs, Hkv, G, mode, r;              // r: tiles per selection block
  int64_t NQB, bNQB, nnzT_unit;            // tiles, blocks, tile-level selection entries of one head
  int32_t *t_rowptr, *t_idx;               // tile-level selection (r > 1)
  int32_t* work_fwd;
  WorkItem* items;
  uint32_t* bitmap;
  int32_t* colcost;
  int64_t row_x;                           // grid columns of the query-major part (Hs workgroups each)
  int64_t words;                           // (sequence, 32 query tiles) pairs
  // a plan of two launches (see plan_in_two) works the tables out itself and leaves them, and the counters cleared, for those after it
  const int32_t* topk;
  int32_t *w_qb_off, *w_row_base, *w_kclamp, *w_qb_seq, *w_counters;
  int64_t *w_sc_off, *w_bm_off;
};

// Plans of few tiles are all launches: geometry and fills, lists, order, 3 - 5 us each.  Up to kLaneSeqs sequences every workgroup of the
// second can work the tables out for itself, and up to kTwoMaxTiles tiles one workgroup per KV head counts its columns from the bitmap, so
// that nothing has to be cleared for the counting: 4.2 us less for the first launch, 1.3 more for the last (2039 tokens, 16/2 heads), a
// step of 1024 tokens on one head 58.6 -> 56.2 us.  What it counts grows with the square of a sequence: three launches / two, one sequence of 128 tiles on
// 8 heads a KV head (4096 words) 15.7 / 15.5 us, 256 tiles on 2 (4096) 16.1 / 16.2, 192 on 4 (4608) 15.5 / 16.0, 384 on one (4608) 16.2 / 17.3, 192 on 8
// (9216) 15.9 / 18.0, 512 on 4 (32768) 17.6 / 28.5; 256 tiles in 48 short sequences on 8 (2100) 22.7 / 18.5.
constexpr int64_t kTwoMaxTiles = 512;
constexpr int64_t kTwoMaxWords = 4096;  // bitmap words of a KV head's columns
inline bool plan_in_two(const Geo& tg) {
  const int64_t heads = tg.mode == SB_SELECT_PER_QHEAD ? tg.G : 1;
  return tg.S <= kLaneSeqs && tg.NQB <= kTwoMaxTiles && heads * tg.bm_words_unit <= kTwoMaxWords;
}
// the sequence of tile qb: the last one that starts at or before it
__device__ inline int seq_of_tile(const PlanArgs& A, int qb) {
  if (A.qb_seq) return A.qb_seq[qb];
  int lo = 0, hi = A.S - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (A.qb_off[mid] <= qb) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// order of the selection heads inside one query block: KV head fastest
__device__ inline int head_rank(const PlanArgs& A, int hs) { return A.mode == SB_SELECT_PER_QHEAD ? (hs % A.G) * A.Hkv + hs / A.G : hs; }

// Query-major item of selection row `row` (r = 1), one thread per row.
__device__ inline void plan_row(const PlanArgs& A, int64_t row) {
  const int hs = (int)(row / A.NQB);
  const int qb = (int)(row - (int64_t)hs * A.NQB);
  const int s = seq_of_tile(A, qb);
  const int i = qb - A.qb_off[s];
  const int ks = A.kclamp[s];
  const int c = min(ks, i + 1);
  int64_t pos = 0;
  for (int t = 0; t < A.S; ++t) {
    const int nt = A.qb_off[t + 1] - A.qb_off[t], kt = A.kclamp[t];
    if (nt == 0) continue;
    if (kt > c) pos += (int64_t)A.Hs * (nt - c);                          // items of t with larger cost
    if (t < s) pos += (int64_t)A.Hs * (kt == c ? nt - c + 1 : (kt > c ? 1 : 0));  // equal cost, earlier sequence
  }
  const int hrank = head_rank(A, hs);
  pos += (c < ks) ? hrank : (int64_t)(i - (ks - 1)) * A.Hs + hrank;
  A.work_fwd[pos] = (int32_t)row;
  WorkItem it;
  it.row = (int32_t)row; it.seq0 = A.cu[s]; it.len = A.cu[s + 1] - A.cu[s]; it.i = i;
  it.e0 = A.rowptr[row]; it.ntiles = A.rowptr[row + 1] - it.e0; it.hs = hs; it.s = s;
  A.items[pos] = it;
}

// ---- selection blocks larger than a tile (B = 64 r, r > 1) -------------------------------------
// The attention kernels work on 64-row tiles.  Query tile it of block I = it / r keeps, for every
// earlier block J its block kept, the r key tiles rJ .. rJ+r-1 (whole blocks in the past), and of
// its own block the tiles rI .. it (causality inside the diagonal block, at tile granularity; the
// token-level mask stays inside tile it).  One wavefront per tile row writes the tile-level CSR and the row's
// query-major item.  The tile count of a row grows with the query tile until the budget
// saturates, so "later query tiles first" is close to longest-first, keeps the heads of one query
// tile adjacent (KV head fastest, see plan_row) and is a closed form again: the position of
// (s, it, hs) counts the rows of all sequences with a larger tile index, then the rows with the same
// tile index in earlier sequences.
__device__ inline void plan_tile_row(const PlanArgs& A, int64_t row) {
  const int lane = threadIdx.x & 63;
  const int hs = (int)(row / A.NQB);
  const int64_t qt = row - (int64_t)hs * A.NQB;
  const int s = A.qb_seq[qt];
  const int it = (int)(qt - A.qb_off[s]);
  // the sequences are dealt to the lanes: entries of the earlier ones (one selection head), and this row's rank
  int64_t base = 0, pos = 0;
  for (int t = lane; t < A.S; t += 64) {
    const int nt = A.qb_off[t + 1] - A.qb_off[t];
    if (t < s) base += tile_entries_before(nt, A.b_kclamp[t], A.r);
    if (nt > it + 1) pos += (int64_t)A.Hs * (nt - 1 - it);  // rows of t with a larger tile index
    if (t < s && nt > it) pos += A.Hs;                      // same tile index, earlier sequence
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) { base += __shfl_xor(base, off, 64); pos += __shfl_xor(pos, off, 64); }
  const int64_t e0 = (int64_t)hs * A.nnzT_unit + base + tile_entries_before(it, A.b_kclamp[s], A.r);
  const int r = A.r, I = it / r, a = it % r;
  const int64_t brow = (int64_t)hs * A.bNQB + A.b_qb_off[s] + I;
  const int be0 = A.rowptr[brow], past = A.rowptr[brow + 1] - be0 - 1;  // kept earlier blocks
  if (lane == 0) {
    A.t_rowptr[row] = (int32_t)e0;
    if (row == (int64_t)A.Hs * A.NQB - 1) A.t_rowptr[row + 1] = (int32_t)(e0 + (int64_t)past * r + a + 1);
    pos += head_rank(A, hs);
    A.work_fwd[pos] = (int32_t)row;
    WorkItem w;
    w.row = (int32_t)row; w.seq0 = A.cu[s]; w.len = A.cu[s + 1] - A.cu[s]; w.i = it;
    w.e0 = (int32_t)e0; w.ntiles = past * r + a + 1; w.hs = hs; w.s = s;
    A.items[pos] = w;
  }
  for (int x = lane; x < past * r; x += 64) A.t_idx[e0 + x] = A.idx[be0 + x / r] * r + x % r;
  for (int x = lane; x <= a; x += 64) A.t_idx[e0 + (int64_t)past * r + x] = I * r + x;
}

// One workgroup per (selection head, sequence, 32 consecutive query tiles) builds word it/32 of
// every column of the sequence in LDS (LDS atomics) and then stores it: every bitmap word has one
// owner, so the bitmap needs neither clearing nor global atomics; the column weights get one global
// add per non-empty word instead of one per selected tile.
constexpr int kTrChunk = 8192;  // columns handled per pass (32 KiB of LDS)
__device__ inline void plan_transpose(const PlanArgs& A, int64_t word, int hs) {
  __shared__ uint32_t wcol[kTrChunk];
  __shared__ int sh_s, sh_w;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  if (wave == 0) {  // which sequence: 64 of them at a time
    int64_t x = word;
    int s = A.S;
    for (int base = 0; base < A.S; base += 64) {
      const int t = base + lane;
      const int w = t < A.S ? (A.qb_off[t + 1] - A.qb_off[t] + 31) >> 5 : 0;
      int incl = w;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(incl, off, 64);
        if (lane >= off) incl += up;
      }
      const unsigned long long hit = __builtin_amdgcn_ballot_w64(x < incl);
      if (hit) {
        const int src = __builtin_ctzll(hit);
        s = base + src;
        x -= __shfl(incl - w, src, 64);
        break;
      }
      x -= __shfl(incl, 63, 64);
    }
    if (lane == 0) { sh_s = s; sh_w = (int)x; }
  }
  __syncthreads();
  const int s = sh_s, wi = sh_w;
  if (s >= A.S) return;
  const int n = A.qb_off[s + 1] - A.qb_off[s];
  const int w = (n + 31) >> 5;
  uint32_t* bm = A.bitmap + (int64_t)A.Hs * A.bm_off[s] + (int64_t)hs * n * w;
  const int g = A.mode == SB_SELECT_PER_QHEAD ? hs / A.G : hs;
  const int weight = A.mode == SB_SELECT_PER_QHEAD ? 1 : A.G;  // query-head tiles an entry stands for
  int32_t* cost = A.colcost + (int64_t)g * A.NQB + A.qb_off[s];
  const int nrows = min(32, n - 32 * wi), r = A.r;
  const int64_t row0 = (int64_t)hs * A.bNQB + A.b_qb_off[s];  // the sequence's first block row
  for (int j0 = 0; j0 < n; j0 += kTrChunk) {
    const int nj = min(kTrChunk, n - j0);
    for (int j = tid; j < nj; j += 256) wcol[j] = 0u;
    __syncthreads();
    auto mark = [&](int jt, uint32_t bit) {
      const int j = jt - j0;
      if (j >= 0 && j < nj) atomicOr(&wcol[j], bit);
    };
    for (int y = wave; y < nrows; y += 4) {
      const int it = 32 * wi + y;
      const int64_t row = row0 + it / r;
      const int e1 = A.rowptr[row + 1];
      for (int e = A.rowptr[row] + lane; e < e1; e += 64) {
        const int J = A.idx[e];
        if (r == 1) mark(J, 1u << y);
        else if (e + 1 == e1) for (int jt = J * r; jt <= it; ++jt) mark(jt, 1u << y);  // the row's own block
        else for (int u = 0; u < r; ++u) mark(J * r + u, 1u << y);
      }
    }
    __syncthreads();
    for (int j = tid; j < nj; j += 256) {
      const uint32_t x = wcol[j];
      bm[(int64_t)(j0 + j) * w + wi] = x;
      if (A.qb_seq && x) atomicAdd(&cost[j0 + j], weight * __popc(x));
    }
    __syncthreads();
  }
}

// The tables of a plan of two launches (tiles are blocks there), in LDS; one workgroup also writes them out.
struct LdsTables { int32_t qb_off[kLaneSeqs + 1], kclamp[kLaneSeqs]; int64_t bm_off[kLaneSeqs + 1]; };
__device__ inline void tables_in_lds(PlanArgs& A, LdsTables& t) {
  const int lane = threadIdx.x & 63;
  const bool writes = blockIdx.x == 0 && blockIdx.y == 0;
  if (threadIdx.x < 64) {
    int n = 0, k = 0;
    if (lane < A.S) {
      n = (A.cu[lane + 1] - A.cu[lane] + 63) / 64;
      k = max(min(A.topk[lane], n), min(n, 1));
    }
    int qb = n, row = k * n - k * (k - 1) / 2;
    int64_t bm = (int64_t)n * ((n + 31) >> 5), sc = (int64_t)n * n;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int q = __shfl_up(qb, off, 64), r = __shfl_up(row, off, 64);
      const int64_t b = __shfl_up(bm, off, 64), c = __shfl_up(sc, off, 64);
      if (lane >= off) { qb += q; row += r; bm += b; sc += c; }
    }
    if (lane == 0) { t.qb_off[0] = 0; t.bm_off[0] = 0; }
    t.qb_off[lane + 1] = qb;
    t.bm_off[lane + 1] = bm;
    t.kclamp[lane] = k;
    if (writes) {
      if (lane == 0) { A.w_qb_off[0] = 0; A.w_bm_off[0] = 0; A.w_sc_off[0] = 0; A.w_row_base[0] = 0; }
      if (lane < A.S) {
        A.w_qb_off[lane + 1] = qb; A.w_bm_off[lane + 1] = bm; A.w_sc_off[lane + 1] = sc; A.w_row_base[lane + 1] = row;
        A.w_kclamp[lane] = k;
      }
      if (lane < 4) A.w_counters[lane] = 0;
    }
  }
  __syncthreads();
  A.qb_off = A.b_qb_off = t.qb_off;
  A.kclamp = A.b_kclamp = t.kclamp;
  A.bm_off = t.bm_off;
  A.qb_seq = nullptr;
  if (writes)
    for (int qb = threadIdx.x; qb < A.NQB; qb += 256) A.w_qb_seq[qb] = seq_of_tile(A, qb);
}

// The query-major lists and the transpose, side by side: neither needs the other.  The selection heads are the grid's second
// dimension, so that half a million one-token sequences on 32 heads stay below the 2^32 threads of one dimension.
template <bool SELF>
__global__ __launch_bounds__(256) void plan_lists_kernel(PlanArgs A) {
  if constexpr (SELF) {
    __shared__ LdsTables tables;
    tables_in_lds(A, tables);
  }
  if ((int64_t)blockIdx.x < A.row_x) {
    const int64_t wg = (int64_t)blockIdx.x * A.Hs + blockIdx.y;
    if (A.r == 1) {
      const int64_t row = wg * 256 + threadIdx.x;  // row id = hs*NQB + qb
      if (row < (int64_t)A.Hs * A.NQB) plan_row(A, row);
    } else {
      const int64_t row = wg * 4 + (threadIdx.x >> 6);  // hs * NT + global tile
      if (row < (int64_t)A.Hs * A.NQB) plan_tile_row(A, row);
    }
  } else {
    plan_transpose(A, (int64_t)blockIdx.x - A.row_x, (int)blockIdx.y);
  }
}

// Key-major items are ordered heaviest first separately for every KV head g, and the Hkv lists are
// interleaved (position = rank_in_g * Hkv + g).  Neighbouring workgroups of one KV head then walk
// neighbouring key blocks of one sequence and meet the same Q/dO tiles in the L2 of their XCD at
// about the same time, while the heaviest-first rule still holds inside each list.
// An item is a whole column, or, for a column heavier than `wmax` tiles, one of its parts: the column's
// bitmap words are walked from the last query block down (the order the backward kernel uses) and a part
// closes as soon as it has gathered wmax tiles (see ColItem).  A column kept by every query block of a
// long sequence (an attention sink) would otherwise be one workgroup's job for longer than the rest of
// the launch takes.
// One workgroup per KV head: a counting sort on the item weight in LDS (histogram, suffix sums,
// scatter); items of equal weight end up in no particular order.
// Sub-parts (see sub_weight) get a list of their own, sorted and interleaved the same way, and lead the launch.  They used to be
// neighbours in a grid of (items x most parts an item could have), where a workgroup without a part exits at once: with two parts
// per item and few items cut, the work was on every second workgroup and so on four of the eight XCDs, with 68 on one.  A step of
// 7000 tokens with 32/8 heads: 1.26 -> 0.84 ms; 64000 tokens on one head with two blocks kept: 289 -> 173 us.
struct ColumnWalk {
  const uint32_t* bm;  // first bitmap word of the column's first selection head
  int64_t head_stride; // words between the same column of consecutive selection heads
  int nsel, hpe, words, wj;
  // calls emit(lo, hi, weight) for every part, last query blocks first; returns the number of parts
  template <typename F>
  __device__ inline int parts(int wmax, F emit) const {
    // the loads of four words' selection heads in flight together: one word after the other, a column of 32 words waited 32 times
    // (the order of 65536 tokens in blocks of 256, 14/2 heads: 55 -> 36 us, with a sink, 32/8 heads: 43 -> 26).
    int acc = 0, hi = words, np = 0;
    for (int w0 = words - 1; w0 >= wj; w0 -= 4) {
      int t[4] = {0, 0, 0, 0};
#pragma unroll 4
      for (int sel = 0; sel < nsel; ++sel) {
        uint32_t x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = bm[sel * head_stride + max(w0 - u, wj)];
#pragma unroll
        for (int u = 0; u < 4; ++u) t[u] += __popc(x[u]);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int w = w0 - u;
        if (w < wj) break;
        acc += t[u] * hpe;
        if (acc >= wmax && w > wj) { emit(w, hi, acc); hi = w; acc = 0; ++np; }
      }
    }
    emit(wj, hi, acc);
    return np + 1;
  }
};

// SELF: the second of two launches; it counts the columns' tiles and fills the lists' unused entries.
template <bool SELF>
__global__ __launch_bounds__(1024) void plan_bwd_order_kernel(int32_t* __restrict__ colcost, const uint32_t* __restrict__ bitmap,
                                                              const int32_t* __restrict__ qb_off, const int32_t* __restrict__ qb_seq,
                                                              const int64_t* __restrict__ bm_off, int64_t NQB, int Hkv, int Hs, int G,
                                                              int mode, int wmax, int wsub, int slots, int extra, ColItem* __restrict__ items,
                                                              int32_t* __restrict__ counters, int32_t* __restrict__ split_cols,
                                                              int32_t* __restrict__ sub_base, SubItem* __restrict__ sub_items,
                                                              int32_t* __restrict__ part_item) {
  __shared__ int bins[kBwdBins];
  __shared__ int sh[16], listed;
  const int tid = threadIdx.x;
  const int64_t g = blockIdx.x;
  __shared__ int32_t counted[SELF ? kTwoMaxTiles : 1];
  const int32_t* cost = SELF ? counted : colcost + g * NQB;
  auto walk_of = [&](int64_t c) {
    ColumnWalk cw;
    const int s = qb_seq[c], j = (int)(c - qb_off[s]), n = qb_off[s + 1] - qb_off[s];
    cw.words = (n + 31) >> 5;
    cw.wj = j >> 5;
    cw.nsel = mode == SB_SELECT_PER_QHEAD ? G : 1;
    cw.hpe = mode == SB_SELECT_PER_QHEAD ? 1 : G;
    const int64_t hs0 = mode == SB_SELECT_PER_QHEAD ? g * G : g;
    cw.head_stride = (int64_t)n * cw.words;
    cw.bm = bitmap + (int64_t)Hs * bm_off[s] + (hs0 * n + j) * cw.words;
    return cw;
  };
  // A bin counts its items, and from bit 16 on their sub-parts: where items are cut there are fewer than 3 * kSubMinColumns columns, so
  // at most 3072 + 2048 items and, but for the rounding, 4 * kSubSlots sub-parts.
  auto sub_parts = [&](int wt) { return wsub > 0 && wt > wsub ? (wt + wsub - 1) / wsub : 0; };
  auto count = [&](int wt) { return atomicAdd(&bins[min(wt, kBwdBins - 1)], 1 + (sub_parts(wt) << 16)); };
  // places an item and its sub-parts and returns where the item is
  auto emit = [&](ColItem it) {
    const int before = count(it.weight), n = sub_parts(it.weight);
    const int64_t at = (int64_t)(wsub > 0 ? before & 0xffff : before) * Hkv + g;
    items[at] = it;
    if (wsub > 0) {
      int base = n > 0 ? before >> 16 : -1;
      if (base + n > slots) {  // more entries on this KV head than the budgets give it: the item is walked as a whole
        if (SELF)
          for (int u = base; u < slots; ++u) sub_items[(int64_t)u * Hkv + g].item.col = -1;
        base = -1;
      }
      sub_base[at] = base;
      if (base >= 0) {
        atomicAdd(&counters[2], n);
        for (int u = 0; u < n; ++u) sub_items[(int64_t)(base + u) * Hkv + g] = SubItem{it, u, {}};
      }
    }
    return at;
  };
  for (int b = tid; b < kBwdBins; b += 1024) bins[b] = 0;
  if constexpr (SELF) {
    for (int64_t c = tid >> 3; c < (NQB + 127) / 128 * 128; c += 128) {  // eight lanes a column
      int t = 0;
      if (c < NQB) {
        const ColumnWalk cw = walk_of(c);
        for (int x = tid & 7; x < cw.nsel * cw.words; x += 8) t += __popc(cw.bm[x / cw.words * cw.head_stride + x % cw.words]);
        t *= cw.hpe;
      }
#pragma unroll
      for (int off = 4; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
      if (c < NQB && (tid & 7) == 0) { counted[c] = t; colcost[g * NQB + c] = t; }
    }
  }
  __syncthreads();
  for (int64_t c = tid; c < NQB; c += 1024) {
    if (cost[c] <= wmax) {
      count(cost[c]);
    } else {
      walk_of(c).parts(wmax, [&](int, int, int wt) { count(wt); });
    }
  }
  __syncthreads();
  // bins[b] <- number of items with a bin > b; thread t owns bins (kBwdBins-1 - t*per) downwards
  constexpr int per = kBwdBins / 1024;
  int v[per], sum = 0;
#pragma unroll
  for (int a = 0; a < per; ++a) { v[a] = bins[kBwdBins - 1 - (tid * per + a)]; sum += v[a]; }
  int incl = sum;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int t = __shfl_up(incl, off, 64);
    if ((tid & 63) >= off) incl += t;
  }
  if ((tid & 63) == 63) sh[tid >> 6] = incl;
  __syncthreads();
  int run = incl - sum;
  for (int w = 0; w < (tid >> 6); ++w) run += sh[w];
#pragma unroll
  for (int a = 0; a < per; ++a) { bins[kBwdBins - 1 - (tid * per + a)] = run; run += v[a]; }
  if (tid == 1023) {
    atomicMax(&counters[3], wsub > 0 ? run & 0xffff : run);
    listed = run;
  }
  __syncthreads();
  if constexpr (SELF) {
    const int placed = wsub > 0 ? listed & 0xffff : listed, cut = wsub > 0 ? listed >> 16 : 0;
    for (int64_t r = placed + tid; r < NQB + extra; r += 1024) items[r * Hkv + g].col = -1;
    for (int64_t r = cut + tid; r < slots; r += 1024) sub_items[r * Hkv + g].item.col = -1;
  }
  for (int64_t c = tid; c < NQB; c += 1024) {
    const int32_t col = (int32_t)(g * NQB + c);
    const ColumnWalk cw = walk_of(c);
    int np = 1;
    if (cost[c] > wmax) np = cw.parts(wmax, [](int, int, int) {});
    if (np == 1) {
      emit(ColItem{col, cw.wj | (cw.words << 16), -1, cost[c]});
    } else {
      const int slot0 = atomicAdd(&counters[0], np);
      const int si = atomicAdd(&counters[1], 1);
      split_cols[3 * si] = col; split_cols[3 * si + 1] = slot0; split_cols[3 * si + 2] = np;
      int part = 0;
      cw.parts(wmax, [&](int lo, int hi, int wt) {
        part_item[slot0 + part] = (int32_t)emit(ColItem{col, lo | (hi << 16), slot0 + part, wt});
        ++part;
      });
    }
  }
}

}  // namespace sb

using namespace sb;

extern "C" int sb_plan_worklist(const sb_problem* p, const int32_t* sel_rowptr, const int32_t* sel_idx, void* plan_out,
                                void* stream) {
  Geo gb;
  int rc = make_geo(p, &gb);
  if (rc != SB_OK) return rc;
  if (gb.S == 0 || gb.T == 0 || gb.NQB == 0) return SB_OK;
  if (!sel_rowptr || !sel_idx || !plan_out) { set_error("null sel_rowptr, sel_idx or plan_out"); return SB_ERR_INVALID_ARG; }
  hipStream_t st = (hipStream_t)stream;
  const Geo g = tile_geo(gb);  // everything below is at the granularity of the 64-row tiles
  PlanOffsets po = plan_offsets(gb);
  char* base = (char*)plan_out;
  Tables t = make_tables(g, p, base + po.tables);
  const Tables tb = gb.r == 1 ? t : make_tables(gb, p, base + po.blk_tables);
  int32_t* colcost = (int32_t*)(base + po.colcost);
  ColItem* bwd_items = (ColItem*)(base + po.bwd_items);
  int32_t* counters = (int32_t*)(base + po.counters);
  uint32_t* bitmap = (uint32_t*)(base + po.bitmap);
  KernelTimer kt(K_PLAN, st);
  // Three launches: tables and fills (unless plan_in_two), lists and transpose, order of the key-major items (each costs 4 - 5 us whatever
  // it does; as seven to nine launches the plan took 20 us of a 1024-token step and 43 us of a 32768-token one, as three 14 and 38 us).
  // The item lists are padded to their largest possible length; unused entries say "no item".
  const size_t n_items = (size_t)g.Hkv * ((size_t)g.NQB + (size_t)split_extra_max(g));
  if ((rc = check_device_arrays(p)) != SB_OK) return rc;
  const bool two = gb.r == 1 && plan_in_two(g);
  if (!two) {
    rc = launch_geom_and_fills(g, base + po.tables, gb.r > 1 ? &gb : nullptr, base + po.blk_tables, p, base + po.counters, po.zeros_end - po.counters,
                               base + po.sub_items, po.bwd_items - po.sub_items + sizeof(ColItem) * n_items, st);
    if (rc != SB_OK) return rc;
  }
  PlanArgs A{};
  A.rowptr = sel_rowptr; A.idx = sel_idx;
  A.cu = t.cu; A.qb_off = t.qb_off; A.kclamp = t.kclamp; A.qb_seq = t.qb_seq; A.bm_off = t.bm_off;
  A.b_qb_off = tb.qb_off; A.b_kclamp = tb.kclamp;
  A.S = g.S; A.Hs = g.Hs; A.Hkv = g.Hkv; A.G = g.G; A.mode = g.mode; A.r = gb.r;
  A.NQB = g.NQB; A.bNQB = gb.NQB; A.nnzT_unit = g.nnz_unit;
  A.t_rowptr = (int32_t*)(base + po.t_rowptr); A.t_idx = (int32_t*)(base + po.t_idx);
  A.work_fwd = (int32_t*)(base + po.work_fwd); A.items = (WorkItem*)(base + po.items);
  A.bitmap = bitmap; A.colcost = colcost;
  const int64_t rows = (int64_t)g.Hs * g.NQB;
  const int64_t row_wgs = gb.r == 1 ? (rows + 255) / 256 : (rows + 3) / 4;
  A.row_x = (row_wgs + g.Hs - 1) / g.Hs;
  for (int s = 0; s < g.S; ++s) {
    const int64_t L = (int64_t)p->cu_seqlens_host[s + 1] - p->cu_seqlens_host[s];
    A.words += ((L + g.B - 1) / g.B + 31) / 32;
  }
  if (two) {
    const TableOffsets to = table_offsets(g);
    char* tb = base + po.tables;
    A.topk = p->topk_dev;
    A.w_qb_off = (int32_t*)(tb + to.qb_off); A.w_row_base = (int32_t*)(tb + to.row_base); A.w_kclamp = (int32_t*)(tb + to.kclamp);
    A.w_qb_seq = (int32_t*)(tb + to.qb_seq); A.w_sc_off = (int64_t*)(tb + to.sc_off); A.w_bm_off = (int64_t*)(tb + to.bm_off);
    A.w_counters = counters;
  }
  hipLaunchKernelGGL(two ? plan_lists_kernel<true> : plan_lists_kernel<false>, dim3((unsigned)(A.row_x + A.words), (unsigned)g.Hs), dim3(256), 0, st, A);
  SB_LAUNCH_CHECK("plan_lists_kernel");
  hipLaunchKernelGGL(two ? plan_bwd_order_kernel<true> : plan_bwd_order_kernel<false>, dim3((unsigned)g.Hkv), dim3(1024), 0, st, colcost, bitmap,
                     t.qb_off, t.qb_seq, t.bm_off, g.NQB, g.Hkv, g.Hs, g.G, g.mode, split_weight(g), sub_slots_max(g) > 0 ? sub_weight(g) : 0,
                     sub_slots_max(g), split_extra_max(g), bwd_items, counters, (int32_t*)(base + po.split_cols), (int32_t*)(base + po.sub_base),
                     (SubItem*)(base + po.sub_items), (int32_t*)(base + po.part_item));
  SB_LAUNCH_CHECK("plan_bwd kernels");
  return SB_OK;
}
