// Budget controller around the attention path (paper section 4.1 and 4.2):
//   sb_score_coverage   coverage curves C_s(k) of the routing scores (Eq. 4) on the GPU
//   sb_perf_predict / sb_perf_align   the profiled latency table (Eq. 8-10), host
//   sb_dst_tune         Algorithm 1 (anchor, Perf.align, coverage threshold p, Eq. 3/5/7), host
//
// Coverage.  For one query block i and one selection head the candidates are the earlier blocks
// j < i; their scores are normalised by a softmax and sorted in descending order; a budget k keeps
// the diagonal block and the k-1 best candidates, so the row covers pref_i[min(k-1, i)], the sum of
// its min(k-1, i) largest shares (pref_i[i] = 1).  C_s(k) is the mean over the sequence's rows.
// All kernels are deterministic (fixed summation order, no atomics):
//   coverage_rows_regs_kernel   rows of at most 2048 candidates: one wavefront per (row, selection head) sorts the row in
//                           registers (long rows by a histogram, short ones by a bitonic network), then softmax and prefix sums; summed over the heads of a group into
//                           Pacc[s][i][m-1] = sum_hs pref_{hs,i}[m], m = 1..i
//   coverage_rows_kernel    longer rows: one workgroup per query block and group of selection heads, for every head in
//                           turn softmax + bitonic sort + prefix sum in LDS, into the same Pacc
//   coverage_partial_kernel / coverage_reduce_kernel   one thread per (s, k): column sums of Pacc over slabs of 32 query
//                           blocks, then C_s(k) = (Hs*k + sum_{i>=k} Pacc[s][i][k-2]) / (Hs*n) (the k rows i < k are fully covered)
#include <math.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "sb_geom.h"
#include "sb_internal.h"

namespace sb {

__device__ inline float block_reduce_256(float v, float* tmp, bool is_max) {
  const int tid = threadIdx.x;
  for (int off = 32; off > 0; off >>= 1) {
    const float o = __shfl_xor(v, off, 64);
    v = is_max ? fmaxf(v, o) : v + o;
  }
  __syncthreads();
  if ((tid & 63) == 0) tmp[tid >> 6] = v;
  __syncthreads();
  float r = tmp[0];
  for (int w = 1; w < 4; ++w) r = is_max ? fmaxf(r, tmp[w]) : r + tmp[w];
  return r;  // the same value, combined in the same order, in every thread
}

// P compare-exchanges of one bitonic stage per lane (pairs t, t + 64, ...): the pairs of a stage are disjoint, so all
// operands are read before anything is written back and the LDS latencies of the P pairs overlap.
template <int P>
__device__ inline void bitonic_pairs(float* keys, int t0, int j2, int k2) {
  int lo[P];
  float a[P], b[P];
#pragma unroll
  for (int u = 0; u < P; ++u) {
    const int t = t0 + 64 * u;
    lo[u] = ((t & ~(j2 - 1)) << 1) | (t & (j2 - 1));  // j2 is a power of two
    a[u] = keys[lo[u]];
    b[u] = keys[lo[u] + j2];
  }
#pragma unroll
  for (int u = 0; u < P; ++u) {  // branch-free: both elements are written back, swapped or not
    const bool lt = a[u] < b[u], gt = a[u] > b[u];
    const bool swap = (lo[u] & k2) == 0 ? lt : gt;
    keys[lo[u]] = swap ? b[u] : a[u];
    keys[lo[u] + j2] = swap ? a[u] : b[u];
  }
}

__global__ __launch_bounds__(256) void coverage_rows_kernel(const float* __restrict__ scores, const int32_t* __restrict__ qb_off,
                                                            const int64_t* __restrict__ sc_off, const int32_t* __restrict__ qb_seq,
                                                            int Hs, int64_t slab, int min_row, float* __restrict__ pacc) {
  extern __shared__ float smem[];  // keys[N], acc[N], tmp[260]
  const int tid = threadIdx.x;
  const int qb = blockIdx.x;
  const int s = qb_seq[qb];
  const int i = qb - qb_off[s];
  const int n = qb_off[s + 1] - qb_off[s];
  if (i == 0 || i < min_row) return;  // no candidates: the row is fully covered at every budget; short rows: the other kernel's
  int N = 1;
  while (N < i) N <<= 1;
  float* keys = smem;
  float* acc = smem + N;
  float* tmp = smem + 2 * N;
  for (int j = tid; j < i; j += 256) acc[j] = 0.f;
  const int chunk = (N + 255) / 256;  // contiguous elements per thread in the prefix sum
  const int hpg = (Hs + (int)gridDim.y - 1) / (int)gridDim.y;  // selection heads per group
  const int hs0 = blockIdx.y * hpg, hs1 = min(Hs, hs0 + hpg);
  for (int hs = hs0; hs < hs1; ++hs) {
    const float* row = scores + (int64_t)Hs * sc_off[s] + ((int64_t)hs * n + i) * n;
    float mx = -INFINITY;
    for (int j = tid; j < N; j += 256) {
      const float x = j < i ? row[j] : -INFINITY;
      keys[j] = x;
      mx = fmaxf(mx, x);
    }
    mx = block_reduce_256(mx, tmp, true);
    // Bitonic sort, descending.  Pair p of a stage with compare distance j2 is (lo, lo + j2), lo = (p / j2) * 2 j2 + p % j2.
    // The pairs are dealt to the four wavefronts in contiguous quarters: as long as j2 < N / 4 both elements of every
    // pair of wavefront w lie in its own quarter of the keys, and so did the pairs that last wrote them, so the stage
    // needs no workgroup barrier (the LDS operations of one wavefront complete in issue order); only the stages with
    // j2 >= N / 4 (three of 66 for 2048 keys) exchange data between wavefronts.
    {
      const int wave = tid >> 6, lane = tid & 63;
      const int ppw = N >> 3;  // pairs per wavefront (N >= 8 here: smaller rows take the plain loop)
      bool shared_prev = true;  // the keys were written by all threads above
      for (int k2 = 2; k2 <= N; k2 <<= 1) {
        for (int j2 = k2 >> 1; j2 > 0; j2 >>= 1) {
          const bool shared = N < 512 || j2 >= (N >> 2);
          if (shared || shared_prev) __syncthreads(); else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          shared_prev = shared;
          if (N < 512) {
            if (tid < (N >> 1)) bitonic_pairs<1>(keys, tid, j2, k2);  // at most 128 pairs
          } else if (ppw == 64) {
            bitonic_pairs<1>(keys, wave * ppw + lane, j2, k2);
          } else if (ppw == 128) {
            bitonic_pairs<2>(keys, wave * ppw + lane, j2, k2);
          } else {  // a multiple of 256 pairs per wavefront
            for (int t = wave * ppw + lane; t < (wave + 1) * ppw; t += 256) bitonic_pairs<4>(keys, t, j2, k2);
          }
        }
      }
    }
    __syncthreads();
    // shares in sorted order, their total, and the running sum
    float part = 0.f;
    const int c0 = tid * chunk, c1 = min(c0 + chunk, N);
    for (int j = c0; j < c1; ++j) {
      const float e = j < i ? __expf(keys[j] - mx) : 0.f;
      keys[j] = e;
      part += e;
    }
    // exclusive prefix of the 256 partial sums: shuffle scan inside each wavefront, then the four wavefront totals
    float incl = part;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const float up = __shfl_up(incl, off, 64);
      if ((tid & 63) >= off) incl += up;
    }
    __syncthreads();
    if ((tid & 63) == 63) tmp[tid >> 6] = incl;
    __syncthreads();
    float before = incl - part, total = 0.f;
    for (int w = 0; w < 4; ++w) {
      if (w < (tid >> 6)) before += tmp[w];
      total += tmp[w];
    }
    const float inv = 1.0f / total;
    float run = before;
    for (int j = c0; j < c1; ++j) {
      run += keys[j];
      if (j < i) acc[j] += j == i - 1 ? 1.0f : run * inv;
    }
    __syncthreads();
  }
  float* out = pacc + (int64_t)blockIdx.y * slab + sc_off[s] + (int64_t)i * n;
  for (int j = tid; j < i; j += 256) out[j] = acc[j];
}

// The same rows for sequences of at most kCovRegMax blocks, sorted in registers: one wavefront per (row, selection
// head), 64 E = N keys (N the row length rounded up to a power of two, at least 64), E per lane.  Key number lane * E + r
// of the bitonic network lives in register r of the lane, so the compare-exchanges at distances below E stay inside a lane
// (two instructions per pair, no memory) and only those at distances E and above cross lanes (cross_stage); a wavefront alone needs no
// barrier.  Keys are integers of the scores' order.  A block of the network that sorts ascending is handled by inverting its lanes' keys,
// so that every compare-exchange puts the larger key first.  The four wavefronts of a workgroup take the heads of the
// group in turn, keep their sums in registers and add them in wavefront order at the end: fixed summation order again.
// Scores must be numbers (a NaN counts as -infinity); sb_block_scores writes none for finite inputs.
// Row lengths share a kernel, whose longest form sets the registers of all: 168 with E = 32 for three wavefronts per SIMD, nothing spilled
// (four would leave 128 and 54 of them spilled: 131072 tokens 241 -> 261 us); batches without rows of more than 1024 keys take one that ends
// with E = 16, four wavefronts (32768 tokens: 42.8 -> 40.0 us).
constexpr int kCovRegMax = 2048;

// Scores as integers of the same order (and back): integer comparisons take a partner lane's key as an operand (DPP) as it is, float
// ones would first quiet a NaN in it.
__device__ __forceinline__ int ordered(int bits) { return bits ^ ((bits >> 31) & 0x7fffffff); }
template <int CTRL>
__device__ __forceinline__ int dpp(int x) {
  return __builtin_amdgcn_mov_dpp(x, CTRL, 0xf, 0xf, true);
}
// A reduction over each row of 16 lanes, and over the wavefront's four rows, without LDS.
template <typename F>
__device__ __forceinline__ int over_row(int x, F f) {
  x = f(x, dpp<0xB1>(x));
  x = f(x, dpp<0x4E>(x));
  x = f(x, dpp<0x141>(x));
  return f(x, dpp<0x140>(x));
}
template <typename F>
__device__ __forceinline__ int over_rows(int x, F f) {
  const auto s = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  x = f((int)s[0], (int)s[1]);
  const auto u = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return f((int)u[0], (int)u[1]);
}
// One stage of the network across lanes: lane l against lane l ^ d, lanes with (l & d) == 0 keep the larger key.  No LDS: at distances 1, 2
// and 8 the partner's key is an operand of the comparison, at 4 one move away; at 16 and 32 two registers swap halves, so that each
// then holds one side of every pair, are compared with each other and swap back.
template <int E, int D_>
__device__ __forceinline__ void cross_stage(int (&x)[E], int lane) {
  if constexpr (D_ >= 16 && E > 1) {
#pragma unroll
    for (int r = 0; r < E; r += 2) {
      const auto s = D_ == 32 ? __builtin_amdgcn_permlane32_swap(x[r], x[r + 1], false, false) : __builtin_amdgcn_permlane16_swap(x[r], x[r + 1], false, false);
      const int hi = max((int)s[0], (int)s[1]), lo = min((int)s[0], (int)s[1]);
      const auto u = D_ == 32 ? __builtin_amdgcn_permlane32_swap(hi, lo, false, false) : __builtin_amdgcn_permlane16_swap(hi, lo, false, false);
      x[r] = (int)u[0];
      x[r + 1] = (int)u[1];
    }
  } else {
    const bool first = (lane & D_) == 0;
#pragma unroll
    for (int r = 0; r < E; ++r) {
      int hi, lo;
      if constexpr (D_ == 1) { hi = max(dpp<0xB1>(x[r]), x[r]); lo = min(dpp<0xB1>(x[r]), x[r]); }
      else if constexpr (D_ == 2) { hi = max(dpp<0x4E>(x[r]), x[r]); lo = min(dpp<0x4E>(x[r]), x[r]); }
      else if constexpr (D_ == 4) { const int m = dpp<0x141>(x[r]); hi = max(dpp<0x1B>(m), x[r]); lo = min(dpp<0x1B>(m), x[r]); }
      else if constexpr (D_ == 8) { hi = max(dpp<0x128>(x[r]), x[r]); lo = min(dpp<0x128>(x[r]), x[r]); }
      else { const int m = __builtin_amdgcn_ds_bpermute((lane ^ D_) << 2, x[r]); hi = max(m, x[r]); lo = min(m, x[r]); }
      x[r] = first ? hi : lo;
    }
  }
}

// Rows of more than 256 keys: most of the sorting is done by a histogram.  The finite keys fall, by value, into 64 E bins between the smallest
// and the largest of them; a key's place is where its bin begins plus how many came before it in the bin, an LDS atomic each; what is left out of order,
// inside bins, an odd-even transposition network puts right in as many stages as the fullest bin has keys.  A bin with kCovBin keys or more
// (ties, heavy tails), a row with +infinity or one whose finite keys are all equal: false, and the network below does it all.
// Keys of -infinity (masked blocks, and what the row's end is filled with) take no part: their places, behind the finite keys', are filled.
// In which order a bin's keys are counted decides nothing: the result is the sorted row.  `lds`: cov_lds<E> words, the wavefront's own; a
// lane's E words are four words further from the next lane's than they would have to be, or all lanes would read from the same banks.
// What bounds both: instruction issue.  For 2048 keys the network takes 4000 vector instructions, this 1200 and 100 LDS operations: 131072
// tokens, 32 heads: 0.370 -> 0.240 ms; 65536 tokens 0.113 -> 0.078 (both with the launch saved below), 0.371 -> 0.254 where every row has an
// outlier (1e4 among N(0, 1)), 0.371 -> 0.236 where half of the keys are -infinity (0.444 where those were counted in one bin).
constexpr int kCovBin = 32;
// (comparisons of all keys' places with the row's length would be kept, 64 scalar registers of them, from one phase to the next)
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+s"(x));
  return x;
}
// keys lane, lane + 64, ... of a row of i (any placement will do for what is then sorted), -infinity past its end and for a NaN
template <int E>
__device__ __forceinline__ void load_keys(const float* __restrict__ row, int i, int lane, int (&x)[E]) {
  asm volatile("" : "+s"(row));
  i = opaque(i);
  // Buffers that end with the row: no branch and no address of its own for any of the loads.  Offsets are the lane's and an immediate, the
  // scalar offset is zero, because the bounds check leaves it out; an immediate reaches 4 KB, so the second half of 32 keys a lane has a buffer of its own.
  int at = 4 * lane;
  asm volatile("" : "+v"(at));  // (or every load's offset gets a register of its own)
#pragma unroll
  for (int r0 = 0; r0 < E; r0 += 16) {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(row + 64 * r0), 0, 4 * max(i - 64 * r0, 0), 0x20000);
#pragma unroll
    for (int r = r0; r < r0 + 16 && r < E; ++r) {
      const float f = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, at + 256 * (r - r0), 0, 0));
      x[r] = __float_as_int(fmaxf(lane < i - 64 * r ? f : -INFINITY, -INFINITY));
    }
  }
}
template <int E> constexpr int cov_lds = 64 * (E + 4) + 2 * E + 8;  // the places, and room for what has none
// `x`: the keys, lane, lane + 64, ..., still there where the result is false.  Where it is true they have been read from memory again for the last step: with
// them, their places and the sums of the heads in registers all the while, a hundred were spilled.
template <int E>
__device__ __forceinline__ bool bucket_sort(const float* __restrict__ row, int (&x)[E], int i, int lane, int* lds) {
  asm volatile("" : "+v"(lane));  // (what follows from the lane is not kept over the loop of rows)
  float hi = -INFINITY, lo = INFINITY;  // of the finite keys
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const float f = __int_as_float(x[r]);
    hi = fmaxf(hi, f);
    lo = f > -INFINITY ? fminf(lo, f) : lo;
  }
  const auto fmax_ = [](int a, int b) __attribute__((always_inline)) { return __float_as_int(fmaxf(__int_as_float(a), __int_as_float(b))); };
  const auto fmin_ = [](int a, int b) __attribute__((always_inline)) { return __float_as_int(fminf(__int_as_float(a), __int_as_float(b))); };
  const int hi_row = over_row(__float_as_int(hi), fmax_), lo_row = over_row(__float_as_int(lo), fmin_);
  hi = __int_as_float(over_rows(hi_row, fmax_)); lo = __int_as_float(over_rows(lo_row, fmin_));
  // what every quarter of the lanes has a key beyond
  const float hi4 = __int_as_float(over_rows(hi_row, fmin_)), lo4 = __int_as_float(over_rows(lo_row, fmax_));
  if (hi4 > lo4 && hi - lo > 2.f * (hi4 - lo4)) { hi = hi4; lo = lo4; }  // a few keys far from the others: they share the first or the last bin
  constexpr float last = 64 * E - 1;
  const float scale = last / (hi - lo);
  if (!__builtin_amdgcn_readfirstlane(hi < INFINITY && scale > 0.f && scale < 1e30f)) return false;  // (also a row without a finite key, and one of equal keys)
  typedef int i32x4s __attribute__((ext_vector_type(4)));
  i32x4s* const own = (i32x4s*)(lds + lane * (E + 4));
  // What is no finite key counts in a word between two lanes' that is no bin, and so far on that its place is none of the row's.
#pragma unroll
  for (int r = 0; r < E / 4; ++r) own[r] = i32x4s{0, 0, 0, 0};
  lds[lane * (E + 4) + E] = 32 * E;
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  int at[E], most = 0;  // word of the key's bin | keys before it << 16, then its place's word
#pragma unroll
  for (int r = 0; r < E; ++r) {
    asm volatile("" : "+v"(x[r]));  // (or what was compared above is kept)
    const unsigned bin = (unsigned)fminf(fmaxf((hi - __int_as_float(x[r])) * scale, 0.f), last);  // (no smaller for a smaller key)
    const bool key = __int_as_float(x[r]) > -INFINITY;
    int word = bin + bin / E * 4;
    asm volatile("" : "+v"(word));  // (or a branch round it)
    at[r] = key ? word : lane * (E + 4) + E;
    const int before = atomicAdd(&lds[at[r]], 1);
    most = max(most, key ? before : 0);
    at[r] |= before << 16;
    if (r % 8 == 7) __builtin_amdgcn_sched_barrier(0);
  }
  if (__builtin_amdgcn_ballot_w64(most + 1 >= kCovBin) != 0) return false;
  const auto imax = [](int a, int b) __attribute__((always_inline)) { return max(a, b); };
  most = __builtin_amdgcn_readfirstlane(over_rows(over_row(most, imax), imax));
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  int sum = 0;
#pragma unroll
  for (int r = 0; r < E / 4; ++r) { const i32x4s c = own[r]; sum += c[0] + c[1] + c[2] + c[3]; if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0); }
  int run = sum;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int up = __shfl_up(run, off, 64);
    if (lane >= off) run += up;
  }
  const int finite = __builtin_amdgcn_readlane(run, 63);
  run -= sum;
  asm volatile("" ::: "memory");  // (read again instead of kept)
#pragma unroll
  for (int r = 0; r < E / 4; ++r) {
    const i32x4s c = own[r];
    own[r] = i32x4s{run, run + c[0], run + c[0] + c[1], run + c[0] + c[1] + c[2]};
    run += c[0] + c[1] + c[2] + c[3];
    if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const unsigned place = ((volatile int*)lds)[at[r] & 0xffff] + ((unsigned)at[r] >> 16);
    at[r] = place + place / E * 4;
    if (r % 8 == 7) __builtin_amdgcn_sched_barrier(0);
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  if ((lane + 1) * E > finite) {  // the places behind the finite keys
    const int none = ordered(__float_as_int(-INFINITY));
#pragma unroll
    for (int r = 0; r < E / 4; ++r) own[r] = i32x4s{none, none, none, none};
  }
  asm volatile("" ::: "memory");
  load_keys<E>(row, opaque(i), lane, x);
#pragma unroll
  for (int r = 0; r < E; ++r)
    lds[at[r]] = ordered(x[r]);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
  for (int r = 0; r < E / 4; ++r) {
    const i32x4s c = own[r];
#pragma unroll
    for (int e = 0; e < 4; ++e) x[4 * r + e] = c[e];
    if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  }
  auto put = [](int& a, int& b) { const int big = max(a, b), small = min(a, b); a = big; b = small; };
#pragma unroll 1
  for (int stage = 0; stage <= most; stage += 2) {
#pragma unroll
    for (int r = 0; r < E; r += 2) put(x[r], x[r + 1]);
    __builtin_amdgcn_sched_barrier(0);
    const int next = __shfl_down(x[0], 1, 64), before = __shfl_up(x[E - 1], 1, 64);
#pragma unroll
    for (int r = 1; r + 1 < E; r += 2) put(x[r], x[r + 1]);
    x[E - 1] = lane < 63 ? max(x[E - 1], next) : x[E - 1];
    x[0] = lane > 0 ? min(x[0], before) : x[0];
  }
  return true;
}

template <int E>
__device__ __forceinline__ void bitonic_sort(int (&x)[E], int lane) {
  // phases k2 = 2 .. E/2: inside a lane, directions known at compile time (bit k2 of r)
#pragma unroll
  for (int k2 = 2; k2 < E; k2 <<= 1) {
#pragma unroll
    for (int j2 = k2 >> 1; j2 > 0; j2 >>= 1) {
#pragma unroll
      for (int r = 0; r < E; ++r) {
        if ((r & j2) == 0) {
          const int hi = max(x[r], x[r | j2]), lo = min(x[r], x[r | j2]);
          const bool desc = (r & k2) == 0;
          x[r] = desc ? hi : lo;
          x[r | j2] = desc ? lo : hi;
        }
      }
      __builtin_amdgcn_sched_barrier(0);  // (left alone, the scheduler interleaves the stages and triples the register count)
    }
  }
  // phases k2 = E .. 64 E: the direction is bit k2 / E of the lane; ascending lanes work on inverted keys
  bool inverted = false;
#pragma unroll 1
  for (int t = (E > 1 ? 0 : 1); t <= 6; ++t) {
    const bool want = ((lane >> t) & 1) != 0 && t < 6;  // (the last phase, k2 = N, is descending everywhere)
    const int flip = want != inverted ? -1 : 0;
    inverted = want;
#pragma unroll
    for (int r = 0; r < E; ++r) x[r] ^= flip;
    // distances d * E, d = 2^(t-1) .. 1
    if (t >= 6) { cross_stage<E, 32>(x, lane); __builtin_amdgcn_sched_barrier(0); }
    if (t >= 5) { cross_stage<E, 16>(x, lane); __builtin_amdgcn_sched_barrier(0); }
    if (t >= 4) { cross_stage<E, 8>(x, lane); __builtin_amdgcn_sched_barrier(0); }
    if (t >= 3) { cross_stage<E, 4>(x, lane); __builtin_amdgcn_sched_barrier(0); }
    if (t >= 2) { cross_stage<E, 2>(x, lane); __builtin_amdgcn_sched_barrier(0); }
    if (t >= 1) { cross_stage<E, 1>(x, lane); __builtin_amdgcn_sched_barrier(0); }
#pragma unroll
    for (int j2 = E >> 1; j2 > 0; j2 >>= 1) {
#pragma unroll
      for (int r = 0; r < E; ++r) {
        if ((r & j2) == 0) {
          const int hi = max(x[r], x[r | j2]), lo = min(x[r], x[r | j2]);
          x[r] = hi;
          x[r | j2] = lo;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <int E>
__device__ __forceinline__ void coverage_row_regs(const float* __restrict__ row, int i, int lane, int* lds, bool& spread, float (&acc)[E]) {
  int x[E];
  i = opaque(i);
  bool sorted = false;
  load_keys<E>(row, i, lane, x);
  if constexpr (E >= 8)
    if (spread) spread = sorted = bucket_sort<E>(row, x, i, lane, lds);
  if (!sorted) {
#pragma unroll
    for (int r = 0; r < E; ++r) x[r] = ordered(x[r]);
    bitonic_sort<E>(x, lane);
  }
  i = opaque(i);
  // shares in sorted order (key 0 is the row maximum), their running sum, the coverage of every prefix
  const float mx = __int_as_float(ordered(__shfl(x[0], 0, 64)));
  float run = 0.f, e[E];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    e[r] = lane * E + r < i ? __expf(__int_as_float(ordered(x[r])) - mx) : 0.f;
    run += e[r];
  }
  float incl = run;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const float up = __shfl_up(incl, off, 64);
    if (lane >= off) incl += up;
  }
  const float inv = 1.0f / __shfl(incl, 63, 64);
  run = incl - run;  // the shares of the lanes before this one
  i = opaque(i);
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int p = lane * E + r;
    run += e[r];
    if (p < i) acc[r] += p == i - 1 ? 1.0f : run * inv;
  }
}

template <int E, int LDS>
__device__ __forceinline__ void coverage_rows_regs_body(const float* __restrict__ scores_s, int n, int i, int hs0, int hs1, int* lds,
                                               float* __restrict__ out) {
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, waves = (int)blockDim.x >> 6;
  float acc[E];
#pragma unroll
  for (int r = 0; r < E; ++r) acc[r] = 0.f;
  // Once the histogram has failed for a head, it is not tried for the heads after it: what ties or far-off values these scores have, the others'
  // are likely to have too (131072 tokens, 32 heads, 40 different values: 404 us where every head tries it and then loads its keys again, so 372 - 379,
  // 371 with the network alone; all keys equal 382, 366 - 371 and 371).
  bool spread = true;
  for (int hs = hs0 + wave; hs < hs1; hs += waves) coverage_row_regs<E>(scores_s + ((int64_t)hs * n + i) * n, i, lane, lds + wave * LDS, spread, acc);
  float* const part = (float*)lds;
#pragma unroll
  for (int r = 0; r < E; ++r) part[wave * LDS + lane * E + r] = acc[r];
  __syncthreads();
  for (int p = tid; p < i; p += (int)blockDim.x) {
    float sum = part[p];
    for (int w = 1; w < waves; ++w) sum += part[w * LDS + p];
    out[p] = sum;
  }
}

template <int MAXE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MAXE == 32 ? 3 : 4))) void coverage_rows_regs_kernel(
    const float* __restrict__ scores, GeomArgs ga, int Hs, int64_t slab, int32_t* qb_off, int64_t* sc_off, int32_t* qb_seq,
    float* __restrict__ pacc) {
  constexpr int LDS = cov_lds<MAXE>;  // words of a wavefront
  extern __shared__ __attribute__((aligned(16))) int part[];
  const int qb = blockIdx.x;
  const BatchGeom bg(ga);
  const int s = bg.seq_of(qb);
  const SeqGeom sg = bg.get(s);
  const int i = qb - sg.qb0, n = sg.n;
  // Up to kLaneSeqs sequences nobody has filled the tables that the next kernels read: a launch of 4 - 5 us saved.
  if (ga.S <= kLaneSeqs && blockIdx.y == 0 && threadIdx.x == 0) {
    qb_seq[qb] = s;
    if (i == 0) { qb_off[s] = sg.qb0; qb_off[s + 1] = sg.qb0 + n; sc_off[s] = sg.sc_off; }
  }
  if (i == 0 || i > kCovRegMax) return;  // no candidates; longer rows are left to coverage_rows_kernel
  const int hpg = (Hs + (int)gridDim.y - 1) / (int)gridDim.y;  // selection heads per group
  const int hs0 = blockIdx.y * hpg, hs1 = min(Hs, hs0 + hpg);
  const float* scores_s = scores + (int64_t)Hs * sg.sc_off;
  float* out = pacc + (int64_t)blockIdx.y * slab + sg.sc_off + (int64_t)i * n;
  auto rows = [&](auto e) __attribute__((always_inline)) { coverage_rows_regs_body<decltype(e)::value, LDS>(scores_s, n, i, hs0, hs1, part, out); };
  if (i <= 64) rows(std::integral_constant<int, 1>());
  else if (i <= 128) rows(std::integral_constant<int, 2>());
  else if (i <= 256) rows(std::integral_constant<int, 4>());
  else if (i <= 512) rows(std::integral_constant<int, 8>());
  else if (MAXE == 16 || i <= 1024) rows(std::integral_constant<int, 16>());
  else rows(std::integral_constant<int, MAXE>());
}

// partial column sums over slabs of kCovSlab query blocks: part[y][qb] = sum over head groups and rows i of slab y, i >= k
constexpr int kCovSlab = 32;
__global__ __launch_bounds__(256) void coverage_partial_kernel(const float* __restrict__ pacc, const int32_t* __restrict__ qb_off,
                                                               const int64_t* __restrict__ sc_off, const int32_t* __restrict__ qb_seq,
                                                               int64_t NQB, int groups, int64_t slab, float* __restrict__ part) {
  const int64_t qb = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (qb >= NQB) return;
  const int s = qb_seq[qb];
  const int n = qb_off[s + 1] - qb_off[s];
  const int k = (int)(qb - qb_off[s]) + 1;
  const int i0 = max(k, (int)blockIdx.y * kCovSlab), i1 = min(n, ((int)blockIdx.y + 1) * kCovSlab);
  float sum = 0.f;
  if (k >= 2) {
    for (int gidx = 0; gidx < groups; ++gidx) {
      const float* col = pacc + (int64_t)gidx * slab + sc_off[s] + (k - 2);
      // eight rows in flight: one after the other, the latencies of up to 128 loads are all that a small problem waits for
      int i = i0;
      for (; i + 8 <= i1; i += 8) {
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = col[(int64_t)(i + u) * n];
#pragma unroll
        for (int u = 0; u < 8; ++u) sum += x[u];
      }
      for (; i < i1; ++i) sum += col[(int64_t)i * n];
    }
  }
  part[(int64_t)blockIdx.y * NQB + qb] = sum;
}

__global__ __launch_bounds__(256) void coverage_reduce_kernel(const float* __restrict__ part, const int32_t* __restrict__ qb_off,
                                                              const int32_t* __restrict__ qb_seq, int64_t NQB, int Hs,
                                                              float* __restrict__ cov) {
  const int64_t qb = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (qb >= NQB) return;
  const int s = qb_seq[qb];
  const int n = qb_off[s + 1] - qb_off[s];
  const int k = (int)(qb - qb_off[s]) + 1;
  double sum = (double)Hs * k;  // the k rows i < k are fully covered
  const int slabs = (n + kCovSlab - 1) / kCovSlab;
  int y = k / kCovSlab;
  for (; y + 8 <= slabs; y += 8) {
    float x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = part[(int64_t)(y + u) * NQB + qb];
#pragma unroll
    for (int u = 0; u < 8; ++u) sum += (double)x[u];
  }
  for (; y < slabs; ++y) sum += (double)part[(int64_t)y * NQB + qb];
  cov[qb] = (float)(sum / ((double)Hs * n));
}

// selection heads are processed in up to kCovGroups groups by separate workgroups (one slab of partial sums each)
constexpr int kCovGroups = 4;
static int coverage_groups(const Geo& g) { return g.Hs < kCovGroups ? g.Hs : kCovGroups; }
static size_t coverage_slab(const Geo& g) { return align_up(sizeof(float) * (size_t)(g.scores_unit + 1)) / sizeof(float); }
static int coverage_row_slabs(const Geo& g) { return (g.n_max + kCovSlab - 1) / kCovSlab; }
size_t coverage_ws_bytes(const Geo& g) {
  return align_up(table_offsets(g).bytes) + sizeof(float) * coverage_slab(g) * (size_t)coverage_groups(g) +
         align_up(sizeof(float) * (size_t)(coverage_row_slabs(g) * g.NQB + 1));
}

// ---- latency table (host, double arithmetic)
static void bracket(const float* grid, int n, double v, int* a, double* w) {
  if (n == 1 || v <= (double)grid[0]) { *a = 0; *w = 0.0; return; }
  if (v >= (double)grid[n - 1]) { *a = n - 2; *w = 1.0; return; }
  int lo = 0;
  while (lo + 1 < n && (double)grid[lo + 1] <= v) ++lo;  // last bucket edge <= v
  *a = lo;
  *w = (v - (double)grid[lo]) / ((double)grid[lo + 1] - (double)grid[lo]);
}

static int check_table(const sb_perf_table* t) {
  if (!t || t->num_lengths < 1 || t->num_budgets < 1 || !t->lengths || !t->budgets || !t->latency) {
    set_error("bad latency table");
    return SB_ERR_INVALID_ARG;
  }
  for (int a = 1; a < t->num_lengths; ++a)
    if (!(t->lengths[a] > t->lengths[a - 1])) { set_error("latency table: lengths must increase"); return SB_ERR_INVALID_ARG; }
  for (int b = 1; b < t->num_budgets; ++b)
    if (!(t->budgets[b] > t->budgets[b - 1])) { set_error("latency table: budgets must increase"); return SB_ERR_INVALID_ARG; }
  return SB_OK;
}

static double predict(const sb_perf_table* t, double x, double k) {
  int a, b;
  double wa, wb;
  bracket(t->lengths, t->num_lengths, x, &a, &wa);
  bracket(t->budgets, t->num_budgets, k, &b, &wb);
  const int a2 = a + 1 < t->num_lengths ? a + 1 : t->num_lengths - 1, b2 = b + 1 < t->num_budgets ? b + 1 : t->num_budgets - 1;
  const int nk = t->num_budgets;
  const double lo = (1.0 - wb) * (double)t->latency[a * nk + b] + wb * (double)t->latency[a * nk + b2];
  const double hi = (1.0 - wb) * (double)t->latency[a2 * nk + b] + wb * (double)t->latency[a2 * nk + b2];
  return (1.0 - wa) * lo + wa * hi;
}

static int align(const sb_perf_table* t, double x, double target, int kmax) {
  int best = 1;
  for (int k = 1; k <= kmax; ++k)
    if (predict(t, x, (double)k) <= target) best = k;
  return best;
}

}  // namespace sb

using namespace sb;

extern "C" {

int sb_score_coverage(const sb_problem* p, const float* scores, float* coverage_out, void* ws, void* stream) {
  Geo g;
  int rc = make_geo(p, &g);
  if (rc != SB_OK) return rc;
  if (g.S == 0 || g.T == 0 || g.NQB == 0) return SB_OK;
  if (!scores || !coverage_out || !ws) { set_error("null scores, coverage_out or ws"); return SB_ERR_INVALID_ARG; }
  hipStream_t st = (hipStream_t)stream;
  if ((rc = check_device_arrays(p)) != SB_OK) return rc;
  if (g.S > kLaneSeqs && (rc = launch_geom(g, p, ws, st)) != SB_OK) return rc;
  Tables t = make_tables(g, p, ws);
  float* pacc = (float*)((char*)ws + align_up(table_offsets(g).bytes));
  int N = 1;
  while (N < g.n_max) N <<= 1;
  const size_t smem = sizeof(float) * (size_t)(2 * N + 264);
  if (smem > 48 * 1024) {  // raise the kernel's dynamic LDS limit; once per device, whichever thread comes first
    static std::mutex mu;
    static bool attr_set[kMaxDevices] = {};
    int dev = 0;
    SB_CHECK_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) { set_error("device ordinal %d out of range", dev); return SB_ERR_UNSUPPORTED; }
    std::lock_guard<std::mutex> lock(mu);
    if (!attr_set[dev]) {
      SB_CHECK_HIP(hipFuncSetAttribute((const void*)coverage_rows_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)(sizeof(float) * (2 * SB_MAX_BLOCKS_PER_SEQ + 264))));
      attr_set[dev] = true;
    }
  }
  KernelTimer kt(K_COVERAGE, st);
  const int groups = coverage_groups(g);
  const int64_t slab = (int64_t)coverage_slab(g);
  // A wavefront per head of a group, four at most: one without a head would hold registers and LDS until the others are done (131072 tokens, 4
  // heads, which are groups of one: 118 -> 63 us, keys of 40 values 155 -> 90, with the network alone 127; 8 heads 128 -> 93).
  const int waves = std::min(4, (g.Hs + groups - 1) / groups);
  const bool short_rows = g.n_max <= 1025;
  hipLaunchKernelGGL(short_rows ? coverage_rows_regs_kernel<16> : coverage_rows_regs_kernel<32>, dim3((unsigned)g.NQB, (unsigned)groups), dim3(64 * waves),
                     sizeof(int) * waves * (short_rows ? cov_lds<16> : cov_lds<32>), st, scores, make_geom_args(g, p, t), g.Hs, slab,
                     (int32_t*)t.qb_off, (int64_t*)t.sc_off, (int32_t*)t.qb_seq, pacc);
  SB_LAUNCH_CHECK("coverage_rows_regs_kernel");
  if (g.n_max > kCovRegMax + 1) {  // rows with more than kCovRegMax candidates
    hipLaunchKernelGGL(coverage_rows_kernel, dim3((unsigned)g.NQB, (unsigned)groups), dim3(256), smem, st, scores, t.qb_off, t.sc_off,
                       t.qb_seq, g.Hs, slab, kCovRegMax + 1, pacc);
    SB_LAUNCH_CHECK("coverage_rows_kernel");
  }
  float* part = pacc + slab * groups;
  hipLaunchKernelGGL(coverage_partial_kernel, dim3((unsigned)((g.NQB + 255) / 256), (unsigned)coverage_row_slabs(g)), dim3(256), 0, st, pacc,
                     t.qb_off, t.sc_off, t.qb_seq, g.NQB, groups, slab, part);
  SB_LAUNCH_CHECK("coverage_partial_kernel");
  hipLaunchKernelGGL(coverage_reduce_kernel, dim3((unsigned)((g.NQB + 255) / 256)), dim3(256), 0, st, part, t.qb_off, t.qb_seq, g.NQB, g.Hs,
                     coverage_out);
  SB_LAUNCH_CHECK("coverage_reduce_kernel");
  return SB_OK;
}

int sb_perf_predict(const sb_perf_table* t, double length, double budget, double* latency_out) {
  int rc = check_table(t);
  if (rc != SB_OK) return rc;
  if (!latency_out) { set_error("null latency_out"); return SB_ERR_INVALID_ARG; }
  *latency_out = predict(t, length, budget);
  return SB_OK;
}

int sb_perf_align(const sb_perf_table* t, double length, double target_latency, int32_t max_budget, int32_t* budget_out) {
  int rc = check_table(t);
  if (rc != SB_OK) return rc;
  if (!budget_out || max_budget < 1) { set_error("bad budget_out or max_budget"); return SB_ERR_INVALID_ARG; }
  *budget_out = align(t, length, target_latency, max_budget);
  return SB_OK;
}

int sb_dst_tune(const sb_problem* p, const float* coverage_host, const sb_perf_table* perf, int anchor, double threshold_p,
                int32_t* topk_final_out, int32_t* topk_anchor_out, double* t_anchor_out) {
  Geo g;
  int rc = make_geo(p, &g);
  if (rc != SB_OK) return rc;
  if ((rc = check_table(perf)) != SB_OK) return rc;
  if (anchor != SB_ANCHOR_MIN && anchor != SB_ANCHOR_MEAN && anchor != SB_ANCHOR_MAX) { set_error("bad anchor %d", anchor); return SB_ERR_INVALID_ARG; }
  if (g.S > 0 && (!coverage_host || !topk_final_out)) { set_error("null coverage_host or topk_final_out"); return SB_ERR_INVALID_ARG; }
  std::vector<int> n(g.S), kb(g.S);
  std::vector<double> T;
  for (int s = 0; s < g.S; ++s) {
    const int64_t L = (int64_t)p->cu_seqlens_host[s + 1] - p->cu_seqlens_host[s];
    n[s] = (int)((L + g.B - 1) / g.B);
    const int cap = n[s] > 1 ? n[s] : 1;
    kb[s] = p->topk_host[s] < cap ? p->topk_host[s] : cap;
    if (n[s] > 0) T.push_back(predict(perf, (double)L, (double)kb[s]));
  }
  double Ta = 0.0;
  if (!T.empty()) {
    if (anchor == SB_ANCHOR_MEAN) {
      double sum = 0.0;
      for (double v : T) sum += v;
      Ta = sum / (double)T.size();
    } else {
      Ta = T[0];
      for (double v : T) Ta = anchor == SB_ANCHOR_MIN ? (v < Ta ? v : Ta) : (v > Ta ? v : Ta);
    }
  }
  if (t_anchor_out) *t_anchor_out = Ta;
  int64_t off = 0;
  for (int s = 0; s < g.S; ++s) {
    int kf = kb[s], ka = kb[s];
    if (n[s] > 0) {
      const int64_t L = (int64_t)p->cu_seqlens_host[s + 1] - p->cu_seqlens_host[s];
      const float* C = coverage_host + off;
      ka = align(perf, (double)L, Ta, n[s]);
      kf = ka;
      if ((double)C[kb[s] - 1] - (double)C[ka - 1] > threshold_p) {
        for (int k = 1; k <= n[s]; ++k)
          if ((double)C[kb[s] - 1] - (double)C[k - 1] <= threshold_p) { kf = k; break; }
      }
    }
    topk_final_out[s] = kf;
    if (topk_anchor_out) topk_anchor_out[s] = ka;
    off += n[s];
  }
  return SB_OK;
}

}  // extern "C"
