// Geometry of a packed batch inside a kernel: which sequence a block belongs to, and where the sequence's rows start in the
// score and selection arrays.  Batches of up to 64 sequences need no tables in memory: lane s of every wavefront holds sequence
// s and the prefix sums are taken across the lanes, which costs about as much as one table lookup (a dependent load) and saves
// the launch that fills the tables (5 - 6 us of a call that takes 10 - 20 us on a small batch).  Larger batches read the tables
// of geom_kernel.
#pragma once

#include "sb_internal.h"

namespace sb {

constexpr int kLaneSeqs = 64;  // sequences that fit the lanes of a wavefront

struct SeqGeom {
  int qb0, n;        // first block of the sequence in the batch, its blocks
  int row_base, k;   // first selection entry (one head), budget
  int64_t sc_off;    // n^2 elements of the earlier sequences
};

// what a kernel needs to find its place: cu_seqlens and budgets, and the tables (used from kLaneSeqs + 1 sequences on)
struct GeomArgs {
  const int32_t *cu, *topk;
  const int32_t *qb_off, *row_base, *kclamp, *qb_seq;
  const int64_t* sc_off;
  int S, B;
};

// Entry i of a table.  The kernels only read the tables, but in a loop that stores results the compiler cannot know that: it would fetch
// them with vector loads behind those stores and take all that follows from them for different from lane to lane.  In the constant
// address space they are scalar loads (scoring and selection in one kernel, 262144 tokens in 109 sequences: 618 -> 610 us).
template <typename T>
__device__ inline T entry(const T* table, int64_t i) {
  return ((const __attribute__((address_space(4))) T*)(uintptr_t)table)[i];
}

struct BatchGeom {
  const GeomArgs& a;
  int n_, qb_, row_, k_;  // lane s: blocks, blocks up to and including s, selection entries before s, budget
  int64_t sc_;
  __device__ inline explicit BatchGeom(const GeomArgs& args) : a(args), n_(0), qb_(0), row_(0), k_(0), sc_(0) {
    if (a.S > kLaneSeqs) return;
    const int lane = threadIdx.x & 63;
    if (lane < a.S) {
      n_ = (a.cu[lane + 1] - a.cu[lane] + a.B - 1) / a.B;
      k_ = max(min(a.topk[lane], n_), min(n_, 1));
    }
    qb_ = n_;
    const int rows = k_ * n_ - k_ * (k_ - 1) / 2;
    const int64_t sq = (int64_t)n_ * n_;
    row_ = rows;
    sc_ = sq;
    for (int off = 1; off < a.S; off <<= 1) {
      const int q = __shfl_up(qb_, off, 64), r = __shfl_up(row_, off, 64);
      const int64_t s = __shfl_up(sc_, off, 64);
      if (lane >= off) { qb_ += q; row_ += r; sc_ += s; }
    }
    row_ -= rows;
    sc_ -= sq;
  }
  // The sequence that work item x of a launch belongs to, when a sequence of n blocks has count(n) items; x becomes the item's
  // number inside the sequence.  Returns S (and the number of items too many) past the last item.  Wave-uniform.
  template <typename F>
  __device__ inline int locate(int64_t& x, F count) const {
    const int lane = threadIdx.x & 63;
    for (int base = 0; base < a.S; base += 64) {
      int n = n_;
      if (a.S > kLaneSeqs) n = base + lane < a.S ? entry(a.qb_off, base + lane + 1) - entry(a.qb_off, base + lane) : 0;
      const int64_t c = count(n);
      int64_t incl = c;
      for (int off = 1; off < 64; off <<= 1) {
        const int64_t t = __shfl_up(incl, off, 64);
        if (lane >= off) incl += t;
      }
      const unsigned long long hit = __builtin_amdgcn_ballot_w64(x < incl);
      const int src = hit ? __builtin_ctzll(hit) : 63;
      x -= __shfl(hit ? incl - c : incl, src, 64);
      if (hit) return base + src;
    }
    return a.S;
  }
  // sequence of block qb (wave-uniform)
  __device__ inline int seq_of(int qb) const {
    if (a.S > kLaneSeqs) return entry(a.qb_seq, qb);
    return __builtin_ctzll(__builtin_amdgcn_ballot_w64(qb < qb_) | (1ull << 63));
  }
  __device__ inline SeqGeom get(int s) const {
    if (a.S > kLaneSeqs) {
      const int qb0 = entry(a.qb_off, s);
      return SeqGeom{qb0, entry(a.qb_off, s + 1) - qb0, entry(a.row_base, s), entry(a.kclamp, s), entry(a.sc_off, s)};
    }
    SeqGeom g;
    g.n = __builtin_amdgcn_readlane(n_, s);
    g.qb0 = __builtin_amdgcn_readlane(qb_, s) - g.n;
    g.row_base = __builtin_amdgcn_readlane(row_, s);
    g.k = __builtin_amdgcn_readlane(k_, s);
    g.sc_off = ((int64_t)__builtin_amdgcn_readlane((int)(sc_ >> 32), s) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)sc_, s);
    return g;
  }
};

}  // namespace sb
