// Block-sparse attention forward (paper Eq. 2) on bf16 MFMA with fp32 online softmax.
//
// attn_fwd_head_kernel: a work item (sequence s, query head, query block i) of the longest-first work list is the job of one wavefront or
// of two (NW; see one_wavefront_per_item).  A wavefront owns all 64 query rows and walks 32-key strips of the selected key blocks, both of
// every block or, with two wavefronts, one each; the two then merge their partial results (reference, sum, unnormalised O) through LDS
// at the end.  It stages its own strips (asynchronous global->LDS loads into a private ring, two tiles ahead), so the loop has no barrier.
// Each K / V^T operand read from LDS feeds two MFMAs (one per 32-query half), which halves the LDS traffic per flop compared with a split
// by query rows.  S^T = K Q^T puts a query in a C-matrix column, so the softmax statistics are per lane and the probabilities convert to
// the B operand of O^T += V^T P^T without any cross-lane movement; V^T is read straight out of the row-major V strip with the transposing
// LDS read.
// What bounds it: at D = 128 a wavefront has its SIMD to itself, so what it waits for is idle time of the matrix cores, and it issues one
// instruction of any kind every four to five cycles (an exponential: nine), 6 beside each 32-cycle matrix instruction.  Hence a software
// pipeline over half tiles u (32 keys x 32 queries) of two stages of D/16 matrix instructions,
//   O(u-1), S(u+1)
// with the probabilities of u beside both; every matrix instruction is fenced with its share of the vector work, of the LDS reads and of
// the tile loads (two at a time), whose addresses are scalar work; no branch but the one in check().  Beyond that the chip lowers its
// clock under matrix load (a loop of these matrix instructions alone runs at 1.7 GHz of 2.4).  At D = 64 half as many matrix instructions
// go with the same vector work, which bounds it; two wavefronts share a SIMD.
// The fixed part of an item (6 us at D = 128: descriptor 0.7, indices 0.8, first strips and Q 2.0, output 2.7) counts half as much with
// one wavefront per item as with two.  Against a whole tile's softmax in a row on two wavefronts the forward of: the 32768-token batch,
// 32/8 heads: 2.02 -> 1.69 ms (with NW = 2: 1.74), one 131072-token sequence, top 32: 7.32 -> 6.2 (6.60), the 262144-token batch 20.9 ->
// 17.2 (18.5), 65536 tokens whose selection is a sink and a window 2.28 -> 1.79 (1.95); D = 64, 65536 tokens, 14/2 heads, blocks of 256:
// 1.59 -> 1.44 ms (there NW = 2).
#include <type_traits>

#include "sb_attn_common.h"

namespace sb {

constexpr int kFwdV = 3;  // V strips in a wavefront's ring: K even, K odd, then V of strip t in slot 2 + t % kFwdV.  Four rings fill a CU's LDS.
template <int D> constexpr int kFwdRing = (2 + kFwdV) * 32 * D * 2;

template <int D, bool OUT_F32, int NW, bool LOOP>
__device__ __attribute__((always_inline)) inline void fwd_head_item(const AttnParams& P, const WorkItem& item, int hh, char (&ring)[NW][kFwdRing<D>]) {
  constexpr int ROW_B = D * 2, STRIP_B = 32 * ROW_B, NOP = D / 16;
  constexpr float kLazy = 4.0f;
  using Loader = QuadLoader<D>;
  constexpr int LPS = Loader::LPS;
  const int tid = item_tid<LOOP>();
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int hs = item.hs, i = item.i, L = item.len;
  const int64_t seq0 = item.seq0;
  const int h = P.mode == SB_SELECT_PER_QHEAD ? hs : hs * P.G + hh;
  const int g = P.mode == SB_SELECT_PER_QHEAD ? hs / P.G : hs;

  StripWalk<D, NW> walk;
  walk.init(item, P.idx, P.Hkv, wave, lane);
  const int nstrips = walk.nstrips;
  // B operands of S^T = K Q^T: column = query 32b + lane%32, slots = d 16ks + 8hf + (0..7)
  bf16x8 qf[2][NOP];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    // (rows past the sequence's last repeat it and are not stored: a branch here would cost the loads' overlap)
    const bf16* qp = P.q + ((seq0 + min(i * 64 + 32 * b + l32, L - 1)) * P.Hq + h) * D + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < NOP; ++ks) qf[b][ks] = *(const bf16x8*)(qp + 16 * ks);
  }
  Loader loader;
  loader.init(P.Hkv, lane);
  // this wavefront's first strip of block 0
  const unsigned long long k0 = (unsigned long long)(P.k + ((seq0 + 32 * wave) * P.Hkv + g) * D);
  const unsigned long long v0 = (unsigned long long)(P.v + ((seq0 + 32 * wave) * P.Hkv + g) * D);
  const unsigned ring0 = lds_offset(&ring[wave][0]);
  unsigned long long off = walk.offset_of(0);  // of the newest strip requested
  unsigned bytes = walk.bytes_of(0);
  loader.issue(Loader::resource(k0 + off, bytes), ring0);
  loader.issue(Loader::resource(v0 + off, bytes), ring0 + 2 * STRIP_B);
  // the query operands must have landed before the loop, which waits for strips by count; here the wait is for the first strips as well
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int ks = 0; ks < NOP; ++ks) asm volatile("" : "+a"(qf[b][ks]));
  wait_vmcnt<0>();
  off = walk.offset_of(1);
  bytes = walk.bytes_of(1);
  loader.issue(Loader::resource(k0 + off, bytes), ring0 + STRIP_B);
  loader.issue(Loader::resource(v0 + off, bytes), ring0 + 3 * STRIP_B);

  // LDS byte addresses of this lane's operand reads: K rows in the first slot, V^T in the slot of the current tile
  unsigned row_a[NOP], tr_a[D / 32][2];
#pragma unroll
  for (int ks = 0; ks < NOP; ++ks) row_a[ks] = ring0 + l32 * ROW_B + 16 * ((2 * ks + hf) ^ chunk_swizzle<D>(l32));
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int r = 8 * half + 4 * hf + ((lane & 15) >> 2), d = 32 * dt + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      tr_a[dt][half] = ring0 + 2 * STRIP_B + r * ROW_B + 16 * ((d >> 3) ^ chunk_swizzle<D>(r)) + 2 * (d & 7);
    }
  auto ld_row = [&](int ks, unsigned off) __attribute__((always_inline)) {
    return *(const bf16x8 __attribute__((address_space(3)))*)(row_a[ks] + off);
  };
  // A operand x = kk * 4 + dt of O^T += V^T P^T: row = d (32dt + lane%32), slots = keys 16kk + 8(e/4) + 4hf + e%4
  auto ld_tr = [&](int x) __attribute__((always_inline)) {
    const int kk = x / (D / 32), dt = x % (D / 32);
    const unsigned o = kk * 16 * ROW_B;
    bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)(tr_a[dt][0] + o));
    bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)(tr_a[dt][1] + o));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  bf16x8 ka[NOP], vt[NOP];
  f32x16 sacc[2];
  bf16x8 pb[2][2];
  f32x16 oacc[D / 32][2];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) oacc[dt][0] = oacc[dt][1] = zero16();
  // m: reference of the exponent, neg_m = -m * scale * log2 e.  As long as a query has seen no score above -inf, m is -inf and neg_m the
  // largest number: a score of -inf then has probability 0, and the first finite one an infinite one, which fails the check below and
  // sets m there.
  constexpr float kNone = __FLT_MAX__;
  float m[2] = {-__builtin_inff(), -__builtin_inff()}, l[2] = {0.f, 0.f}, neg_m[2] = {kNone, kNone};
#pragma unroll
  for (int k = 0; k < NOP; ++k) { ka[k] = ld_row(k, 0); vt[k] = zero_bf16x8(); }
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): K_0 has been read
  off = walk.offset_of(2);
  bytes = walk.bytes_of(2);
  loader.issue(Loader::resource(k0 + off, bytes), ring0);

  // P = exp2(S c - m c) of a half tile in steps s = 0 .. 14, one beside each matrix instruction: about one exponential a step, its
  // argument a step before it and its conversion to bf16 a step after it, because an exponential's result is not ready for the next
  // instruction.  The half tile's row sum, of the probabilities as rounded, i.e. of the weights that O applies, comes last and in four
  // chains: a dot product waits for the one before it and for the matrix cores (one chain, a product a step: 834 ns a tile in a loop of
  // these instructions alone, like this 740; without any sum 700).
  float px[16], psum = 0.f;
  bf16x2 py[8];
  auto exp_step = [](int v) { return v < 9 ? v + 1 : v < 15 ? 10 + (v - 9) / 2 : 13; };
  auto p_step = [&](int b, int s) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (exp_step(v) == s) px[v] = fast_exp2(px[v]);
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (exp_step(v) == s + 1) px[v] = __builtin_fmaf(sacc[b][v], P.scale_log2e, neg_m[b]);
#pragma unroll
    for (int c = 0; c < 8; ++c)
      if (exp_step(2 * c + 1) + 1 == s) {
        py[c][0] = (bf16)px[2 * c];
        py[c][1] = (bf16)px[2 * c + 1];
        pb[b][c >> 2][(2 * c) & 7] = py[c][0];
        pb[b][c >> 2][(2 * c + 1) & 7] = py[c][1];
      }
    if (s == 14) {
      float part[4];
#pragma unroll
      for (int c = 0; c < 8; ++c) part[c & 3] = sum2(py[c], c < 4 ? 0.f : part[c & 3]);
      psum = (part[0] + part[1]) + (part[2] + part[3]);
    }
  };
  // The reference follows the true maximum lazily: only when a lane's 16 probabilities add up to more than 16 * 2^kLazy (so one of them
  // exceeds 2^kLazy, and one above 2^8 always does it), which costs one comparison per half tile where the maximum of the scores would
  // cost ten instructions.  The scores are still there: the reference moves, what has been summed with the old one is rescaled, and the
  // probabilities are computed again.
  // The score that becomes the reference has probability 1, which bf16 holds exactly.  Two wavefronts have a reference each, so that two
  // strips of a row have such a score where one wavefront has one: it adds what rounding took from the strip after the one that moved the
  // reference (`limit` is negative then, so that the branch is taken), 8 matrix instructions per query half and move: 0.7 us of an item,
  // 0.5 - 2 % of a launch.  Without it float32 outputs of rows of 1 to 27 tiles were 4 to 6 % further off than two wavefronts' (2-norm), with
  // it they are 4 to 7 % less.  (Scores of standard deviation 3 and 2^8 for kLazy: 4 % further off with two wavefronts, 9 to 21 % with one.)
  constexpr float kMost = 16.0f * 16.0f;  // 16 * 2^kLazy
  float limit[2] = {kMost, kMost};
  auto check = [&](int b) __attribute__((always_inline)) {
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(psum <= limit[b])) != 0, 0)) {
      int add_rest = __builtin_amdgcn_readfirstlane(limit[b] < 0.f);
      asm volatile("" : "+s"(add_rest));  // (from here on the old limit is not needed: else the loop would copy it from register to register)
      limit[b] = kMost;
      if (NW == 2 || __builtin_amdgcn_ballot_w64(!(psum <= kMost)) != 0) {
        float mx = max3(sacc[b][0], sacc[b][1], sacc[b][2]);
#pragma unroll
        for (int v = 3; v < 15; v += 2) mx = max3(mx, sacc[b][v], sacc[b][v + 1]);
        mx = max_across_halves(fmaxf(mx, sacc[b][15]));
        const bool first = m[b] == -__builtin_inff();  // nothing accumulated yet for this query: nothing to rescale
        const bool move = first | ((mx - m[b]) * P.scale_log2e > kLazy);
        const float m_new = move ? fmaxf(m[b], mx) : m[b];
        const float alpha = first ? 1.0f : fast_exp2((m[b] - m_new) * P.scale_log2e);
        neg_m[b] = m_new == -__builtin_inff() ? kNone : -m_new * P.scale_log2e;
        l[b] *= alpha;
        m[b] = m_new;
        if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
          for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) oacc[dt][b][v] = scale_acc(oacc[dt][b][v], alpha);
        }
#pragma unroll
        for (int v = 0; v < 15; ++v) p_step(b, v);
        if (NW == 1) limit[b] = -1.0f;
      }
      if (NW == 1 && add_rest) {
        // P = its upper 16 bits + the rest: both above 0, so that an infinite value in V stays infinite (0 * inf, or a rest below 0, would
        // make NaN of it).  The rest has 2^-23 P added, for a P that has no other.
        bf16x8 rest[2];
        float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const unsigned x0 = __float_as_uint(px[2 * c]), x1 = __float_as_uint(px[2 * c + 1]);
          const bf16x2 upper = __builtin_bit_cast(bf16x2, __builtin_amdgcn_perm(x1, x0, 0x07060302));
          bf16x2 lower;
          lower[0] = (bf16)__builtin_fmaf(px[2 * c], 1.0f + 0x1p-23f, -__uint_as_float(x0 & 0xffff0000u));
          lower[1] = (bf16)__builtin_fmaf(px[2 * c + 1], 1.0f + 0x1p-23f, -__uint_as_float(x1 & 0xffff0000u));
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            pb[b][c >> 2][(2 * c + e) & 7] = upper[e];
            rest[c >> 2][(2 * c + e) & 7] = lower[e];
          }
          part[c & 1] = sum2(upper, part[c & 1]);
          part[2 + (c & 1)] = sum2(lower, part[2 + (c & 1)]);
        }
        psum = (part[0] + part[1]) + (part[2] + part[3]);
        asm volatile("s_nop 1" : "+v"(rest[0]), "+v"(rest[1]));  // two wait states between a vector write and its use as an operand
#pragma unroll
        for (int k = 0; k < NOP; ++k) mfma32_sum(oacc[k % (D / 32)][b], vt[k], rest[k / (D / 32)]);
      }
      asm volatile("s_nop 1" ::: "memory");  // likewise
    }
    l[b] += psum;
  };

#define SB_FENCE() __builtin_amdgcn_sched_barrier(0)
  constexpr int PER = 8 / NOP;  // steps of the probabilities per matrix instruction
  unsigned vs0 = ring0 + 2 * STRIP_B, vs1 = vs0 + STRIP_B, vs2 = vs1 + STRIP_B;  // LDS slots of V_t, V_{t+1}, V_{t+2}
  // u = (strip t, query half B): stages O(u-1) and S(u+1) with the probabilities of u; PAR = t % 2.  DIAG: a strip of the diagonal tile,
  // LAST: the row's last strip, nothing follows it.  With NW = 1 the last strip is the diagonal tile's keys 32 .. 63, which query half 0
  // does not see: u = (last, 0) has no scores, no probabilities and no sum.
  auto half_tile = [&](auto diag_c, auto last_c, auto par_c, auto b_c, int t) __attribute__((always_inline)) {
    constexpr int B = decltype(b_c)::value, PAR = decltype(par_c)::value;
    constexpr bool DIAG = decltype(diag_c)::value, LAST = decltype(last_c)::value;
    constexpr bool SEEN = !(LAST && NW == 1 && B == 0);                       // u has visible keys
    constexpr bool PREV = !(LAST && NW == 1 && B == 1);                       // u - 1 has
    constexpr bool NEXT = LAST ? B == 0 : !(DIAG && NW == 1 && B == 1);       // u + 1 exists and has
    const int key0 = NW == 2 ? 32 * wave : LAST ? 32 : 0;
#pragma unroll
    for (int k = 0; k < NOP; ++k) asm volatile("" : "+a"(qf[B ^ 1][k]));
    // B = 0: V_{t+2} is requested, into the slot of V_{t-1}.  B = 1: K_{t+3}, into the slot of K_{t+1}, whose operands are in ka.
    i32x4 rsrc;
    unsigned slot = 0;
    if constexpr (!LAST) {
      if (B == 1) {
        off = walk.offset_of(t + 3);
        bytes = walk.bytes_of(t + 3);
      }
      rsrc = Loader::resource((B == 0 ? v0 : k0) + off, bytes);
      slot = B == 0 ? vs2 : ring0 + (PAR ^ 1) * STRIP_B;
    }
    if (B == 0) {
      // V_t has landed; K_{t+1}, V_{t+1} and K_{t+2} may still be on their way
      wait_vmcnt<3 * LPS>();
    }
    SB_FENCE();
#pragma unroll
    for (int k = 0; k < NOP; ++k) {  // O(u-1); with B = 0 every operand register is refilled from V_t
      if (PREV) mfma32_sum(oacc[k % (D / 32)][B ^ 1], vt[k], pb[B ^ 1][k / (D / 32)]);
      if (B == 0) vt[k] = ld_tr(k);
      if (B == 1 && !LAST) {
        if (k == NOP / 4) __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): K_{t+1} is in ka
        tr_a[k >> 1][k & 1] += vs1 - vs0;  // on to V of the next tile
        if (k == NOP - 1) {
          const unsigned vs = vs0;
          vs0 = vs1; vs1 = vs2; vs2 = vs;
        }
      }
      if (!PREV && k == 0) asm volatile("s_nop 7\n\ts_nop 7" : "+v"(sacc[B]));  // (no matrix instructions between S(u) and its first reader)
      if (DIAG && SEEN && k == 1) {  // causal mask inside the diagonal tile
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (key0 + c_row(v, hf) > 32 * B + l32) sacc[B][v] = -__builtin_inff();
      }
      if (SEEN && k > 0) {
#pragma unroll
        for (int a = 0; a < PER; ++a) p_step(B, PER * (k - 1) + a);
      }
      SB_FENCE();
      if constexpr (!LAST) {
        if (D == 128 && k == 3) loader.template issue2<0>(rsrc, slot);
        if constexpr (D == 128) { if (k == 6) loader.template issue2<2>(rsrc, slot); }
        if (D == 64 && k == 1) loader.template issue2<0>(rsrc, slot);
      }
      SB_FENCE();
    }
#pragma unroll
    for (int k = 0; k < NOP; ++k) {  // S(u+1); with B = 0 every operand register is refilled from K_{t+1}
      if (NEXT) {
        if (k == 0) mfma32_first(sacc[B ^ 1], ka[k], qf[B ^ 1][k]);
        else mfma32_more(sacc[B ^ 1], ka[k], qf[B ^ 1][k]);
      }
      if (B == 0 && !LAST) {
        // V_t is in vt (its reads must not keep those of K_{t+1} waiting one by one)
        if (k == NOP / 4) {
          wait_vmcnt<2 * LPS + LPS / 2>();  // K_{t+1} has landed; V_{t+1}, K_{t+2} and half of V_{t+2} may still be on their way
          __builtin_amdgcn_s_waitcnt(0xC07F);
#pragma unroll
          for (int a = 0; a < NOP / 4; ++a) ka[a] = ld_row(a, (PAR ^ 1) * STRIP_B);
        }
        if (k >= NOP / 4) ka[k] = ld_row(k, (PAR ^ 1) * STRIP_B);
      }
      if (SEEN) {
#pragma unroll
        for (int a = 0; a < PER; ++a) p_step(B, PER * (NOP - 1 + k) + a);
        if (PER == 2 && k == NOP - 1) p_step(B, 14);
      }
      SB_FENCE();
      if constexpr (!LAST) {
        if constexpr (D == 128) {
          if (k == 3) loader.template issue2<4>(rsrc, slot);
          if (k == 6) loader.template issue2<6>(rsrc, slot);
        }
        if (D == 64 && k == 1) loader.template issue2<2>(rsrc, slot);
      }
      SB_FENCE();
    }
    if (SEEN) check(B);
    SB_FENCE();
  };
  using std::integral_constant;
  using std::false_type;
  using std::true_type;
  using I0 = integral_constant<int, 0>;
  using I1 = integral_constant<int, 1>;
  {
    // nothing precedes the first half tile: its O stage adds zeros
#pragma unroll
    for (int q = 0; q < 2; ++q) pb[1][q] = zero_bf16x8();
#pragma unroll
    for (int k = 0; k < NOP; ++k) {
      if (k == 0) mfma32_first(sacc[0], ka[k], qf[0][k]);
      else mfma32_more(sacc[0], ka[k], qf[0][k]);
    }
    int t = 0;
    for (; t + 2 < nstrips; t += 2) {
      walk.window(t, 4, lane);
      half_tile(false_type(), false_type(), I0(), I0(), t);
      half_tile(false_type(), false_type(), I0(), I1(), t);
      half_tile(false_type(), false_type(), I1(), I0(), t + 1);
      half_tile(false_type(), false_type(), I1(), I1(), t + 1);
    }
    if (NW == 1 || t + 2 == nstrips) {
      using Diag = integral_constant<bool, NW == 1>;
      half_tile(Diag(), false_type(), I0(), I0(), t);
      half_tile(Diag(), false_type(), I0(), I1(), t);
      ++t;
    }
    half_tile(true_type(), true_type(), I0(), I0(), t);
    half_tile(true_type(), true_type(), I0(), I1(), t);
#pragma unroll
    for (int k = 0; k < NOP; ++k) mfma32_sum(oacc[k % (D / 32)][1], vt[k], pb[1][k / (D / 32)]);
    // the compiler does not see these as matrix instructions: their results are read no sooner than this
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) asm volatile("s_nop 7\n\ts_nop 7" : "+a"(oacc[dt][0]), "+a"(oacc[dt][1]));
  }
#undef SB_FENCE
  wait_vmcnt<0>();  // the strips past the last tile
  l[0] += __shfl_xor(l[0], 32, 64);
  l[1] += __shfl_xor(l[1], 32, 64);
  if constexpr (NW == 1) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const float inv = 1.0f / l[b];
      const int64_t tq = seq0 + i * 64 + 32 * b;
      const int rows = min(32, L - i * 64 - 32 * b);
      store_rows<D, OUT_F32>(&ring[0][b * 2 * STRIP_B], P.o, (tq * P.Hq + h) * D, (int64_t)P.Hq * D, rows, lane,
                             [&](int dt, int v) __attribute__((always_inline)) { return oacc[dt][b][v] * inv; });
      // (a row without any score above -inf has no softmax: NaN, as the merge below makes of it)
      const float lse = l[b] > 0.f ? (m[b] * P.scale_log2e + __builtin_log2f(l[b])) * 0.69314718055994531f : __builtin_nanf("");
      if (hf == 0 && l32 < rows) P.lse[(int64_t)h * P.T + tq + l32] = lse;
    }
  } else {
    // ---- merge the two key halves: wavefront w finalises query half w and hands the other half over
    float* xbuf = (float*)&ring[wave][0];            // this wavefront's outgoing partial, [register][lane]
    const float* ybuf = (const float*)&ring[wave ^ 1][0];  // the partner's
    constexpr int NR = 16 * (D / 32);
    static_assert((NR + 2) * 64 * sizeof(float) <= 3 * STRIP_B, "partial and output rows share the ring");
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if (b != wave) {
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
          for (int v = 0; v < 16; ++v) xbuf[(16 * dt + v) * 64 + lane] = oacc[dt][b][v];
        xbuf[NR * 64 + lane] = m[b];
        xbuf[(NR + 1) * 64 + lane] = l[b];
      }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if (b == wave) {
        const float m2 = ybuf[NR * 64 + lane], l2 = ybuf[(NR + 1) * 64 + lane];
        const float mt = fmaxf(m[b], m2);  // finite for every existing query: its own key is never masked
        const float w1 = fast_exp2((m[b] - mt) * P.scale_log2e), w2 = fast_exp2((m2 - mt) * P.scale_log2e);
        const float lt = l[b] * w1 + l2 * w2;
        const float inv = 1.0f / lt;
        const float c1 = w1 * inv, c2 = w2 * inv;
        const int64_t tq = seq0 + i * 64 + 32 * b;
        const int rows = min(32, L - i * 64 - 32 * b);
        store_rows<D, OUT_F32>(&ring[wave][3 * STRIP_B], P.o, (tq * P.Hq + h) * D, (int64_t)P.Hq * D, rows, lane, [&](int dt, int v) __attribute__((always_inline)) {
          return oacc[dt][b][v] * c1 + ybuf[(16 * dt + v) * 64 + lane] * c2;
        });
        if (hf == 0 && l32 < rows) P.lse[(int64_t)h * P.T + tq + l32] = (mt * P.scale_log2e + __builtin_log2f(lt)) * 0.69314718055994531f;
      }
    }
  }
}

template <int D, bool OUT_F32, int NW, bool LOOP>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 64 ? 2 : 1))) void attn_fwd_head_kernel(AttnParams P, int heads) {
  __shared__ __attribute__((aligned(1024))) char ring[NW][kFwdRing<D>];
  BusyTimer timer;
  timer.start(P);
  for_items<D, NW, LOOP, false>(P, heads, (int*)&ring[NW - 1][kFwdRing<D> - 4],
                [&](const AttnParams& p, const WorkItem& item, int hh) __attribute__((always_inline)) { fwd_head_item<D, OUT_F32, NW, LOOP>(p, item, hh, ring); });
  timer.stop(P);
}

// ---------------------------------------------------------------------------------------------
// Forward kernel for per-KV-group selection at D = 128: the query heads of a KV group share a work item, so one
// workgroup takes 3 or 4 of them and they share the item's K/V tiles in LDS (whole tiles,
// double-buffered by asynchronous loads) instead of fetching them once per head.  Two wavefronts per
// query head; a wavefront owns 32 query rows and all 64 keys of every selected tile, as two 32-key
// halves with one online-softmax step each.  The register budget (256) lets two wavefronts share a
// SIMD, so one runs its exponentials while the other runs matrix instructions; one operand set
// rotates through both contractions (K rows, then V^T through the transposing read, each register
// refilled right after the MFMA that consumed it).
template <bool OUT_F32>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void attn_fwd_group_kernel(AttnParams P, int heads) {
  constexpr int D = 128;
  constexpr int TILE_B = 64 * D * 2, ROW_B = D * 2, NOP = D / 16;
  constexpr float kLazy = 8.0f;
  __shared__ __attribute__((aligned(1024))) bf16 tiles[2][2][64 * D];  // [buffer][K, V]
  constexpr int kJ = 256;
  __shared__ int jbuf[kJ];
  BusyTimer timer;
  timer.start(P);
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  int pos = claim_item(blockIdx.x, P.n_items, P.ticket ? P.ticket + kTicketInts * blockIdx.y : nullptr);
  if (pos < 0) return;
  asm volatile("" : "+v"(pos));  // (scalar loads make the compiler keep more in registers than there are: 16 of 256 spilled, with vector ones it takes 210)
  const WorkItem item = P.items[pos];
  const int hs = item.hs, i = item.i, L = item.len, e0 = item.e0, ntiles = item.ntiles;
  const int64_t seq0 = item.seq0;
  const int strip = wave & 1;
  const int hh = blockIdx.y * (nthr / 128) + (wave >> 1);  // query head of the group this wavefront works for
  const bool head_ok = hh < heads;
  const int h = hs * P.G + (head_ok ? hh : 0);  // per-KV-group mode: the item's selection head is the KV head
  const int g = hs;
  const int qloc = strip * 32 + l32;
  const bool qvalid = head_ok && i * 64 + qloc < L;
  const int64_t tq = seq0 + i * 64 + qloc;

  auto stage_indices = [&](int t0) {
    __syncthreads();
    for (int a = tid; a < kJ; a += nthr) jbuf[a] = t0 + a < ntiles ? P.idx[e0 + t0 + a] : 0;
    __syncthreads();
  };
  TileLoader<D> loader;  // a workgroup has six or eight wavefronts
  loader.init(P.Hkv, wave, lane);
  auto issue = [&](int t) {
    const int j = __builtin_amdgcn_readfirstlane(jbuf[t % kJ]);
    const int64_t kv0 = seq0 + (int64_t)j * 64;
    const int kvalid = min(64, L - j * 64);
    loader.issue(tiles[t & 1][0], P.k, kv0, kvalid, P.Hkv, g);
    loader.issue(tiles[t & 1][1], P.v, kv0, kvalid, P.Hkv, g);
  };

  // B operand of S^T = K Q^T: column = query lane%32 of the strip, slots = d 16ks + 8hf + (0..7)
  bf16x8 qf[NOP];
  {
    const bf16* qp = P.q + (tq * P.Hq + h) * D + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < NOP; ++ks) qf[ks] = qvalid ? *(const bf16x8*)(qp + 16 * ks) : zero_bf16x8();
  }
  stage_indices(0);
  // everything loaded so far must have landed before the tile loads start: from here on the only
  // vector-memory operations in flight are tile loads, which the loop waits for by count
#pragma unroll
  for (int ks = 0; ks < NOP; ++ks) asm volatile("" : "+v"(qf[ks]));
  issue(0);

  const unsigned tiles0 = lds_offset(&tiles[0][0][0]);
  unsigned row_a[NOP], tr_a[D / 32][2];
#pragma unroll
  for (int ks = 0; ks < NOP; ++ks) row_a[ks] = tiles0 + l32 * ROW_B + 16 * ((2 * ks + hf) ^ chunk_swizzle<D>(l32));
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int r = 8 * half + 4 * hf + ((lane & 15) >> 2), d = 32 * dt + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      tr_a[dt][half] = tiles0 + TILE_B + r * ROW_B + 16 * ((d >> 3) ^ chunk_swizzle<D>(r)) + 2 * (d & 7);
    }
  auto ld_row = [&](int ks, unsigned off) __attribute__((always_inline)) {
    return *(const bf16x8 __attribute__((address_space(3)))*)(row_a[ks] + off);
  };
  // A operand of O^T += V^T P^T: row = d (32dt + lane%32), slots = keys 16kk + 8(e/4) + 4hf + e%4 of this wavefront's rows
  auto ld_tr = [&](int kk, int dt, unsigned off) __attribute__((always_inline)) {
    const unsigned o = off + kk * 16 * ROW_B;
    bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)(tr_a[dt][0] + o));
    bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)(tr_a[dt][1] + o));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };

  f32x16 oacc[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) oacc[dt] = zero16();
  float m = -__builtin_inff(), neg_m = 0.f, l = 0.f;
  bf16x8 op[NOP];

  // The diagonal block is always the last tile of a row: it takes its own instantiation of the tile
  // body, so that the other tiles carry no mask selects.
  auto tile = [&](auto diag_c, auto buf_c, int t) __attribute__((always_inline)) {
    constexpr bool diag = decltype(diag_c)::value;
    constexpr unsigned BO = decltype(buf_c)::value * 2 * TILE_B;  // the tile's buffer, as an immediate offset of every LDS read
    const bool more = t + 1 < ntiles;
    if (more && (t + 1) % kJ == 0) stage_indices(t + 1);
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();  // tile t has landed for everyone; everyone is done with tile t-1
    if (more) issue(t + 1);
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {  // keys 32mt .. 32mt+31 of the tile
#pragma unroll
      for (int ks = 0; ks < NOP; ++ks) op[ks] = ld_row(ks, BO + mt * 32 * ROW_B);  // K rows
      __builtin_amdgcn_sched_barrier(0);
      f32x16 sacc = zero16();
#pragma unroll
      for (int ks = 0; ks < NOP; ++ks) {  // S^T = K Q^T, refilling every operand register with a V^T operand
        sacc = mfma32(op[ks], qf[ks], sacc);
        op[ks] = ld_tr(2 * mt + ks / (D / 32), ks % (D / 32), BO);
      }
#pragma unroll
      for (int i_ = 0; i_ < NOP; ++i_) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (diag) {  // causal mask inside the diagonal block (also removes keys past the end of the sequence)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (32 * mt + c_row(v, hf) > qloc) sacc[v] = -__builtin_inff();
      }
      // max3 below is inline asm, whose reads of the matrix instructions' results the compiler's hazard recogniser
      // does not see: a vector instruction may read a register written by an 8-pass matrix instruction only 12 wait
      // states after it.  (The masked tile goes through compiler-visible selects first.)  Without the wait a lane now
      // and then took a stale value into its running maximum: harmless for the result's accuracy (the softmax does
      // not depend on the reference point) but not bitwise repeatable.
      if (!diag) asm volatile("s_nop 7\n\ts_nop 3" : "+v"(sacc));
      // online softmax with a lazy running maximum, the reference moved in a branch that is rarely taken (see the kernel above; two
      // wavefronts share the SIMD's vector unit here, which is what bounds them: 32768-token batch, 32/8 heads, 1744 -> 1642 us)
      float mx = max3(sacc[0], sacc[1], sacc[2]);
#pragma unroll
      for (int v = 3; v < 15; v += 2) mx = max3(mx, sacc[v], sacc[v + 1]);
      mx = max3(mx, sacc[15], sacc[15]);
      if (__builtin_amdgcn_ballot_w64(!((mx - m) * P.scale_log2e <= kLazy)) != 0) {
        mx = max_across_halves(mx);
        const bool first = m == -__builtin_inff();  // nothing accumulated yet for this query
        const bool move = first | ((mx - m) * P.scale_log2e > kLazy);
        const float m_new = move ? fmaxf(m, mx) : m;
        const float m_use = m_new == -__builtin_inff() ? 0.f : m_new;  // no unmasked key seen yet: keep the exponent finite
        const float alpha = first ? 1.0f : fast_exp2((m - m_use) * P.scale_log2e);
        neg_m = -m_use * P.scale_log2e;
        m = m_new;
        if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
          l *= alpha;
#pragma unroll
          for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) oacc[dt][v] *= alpha;
        }
      }
      bf16x8 pb[2];
#pragma unroll
      for (int v = 0; v < 16; ++v) pb[v >> 3][v & 7] = (bf16)fast_exp2(__builtin_fmaf(sacc[v], P.scale_log2e, neg_m));
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {  // the row sum adds the probabilities as rounded to bf16, the weights the accumulation applies
        const bf16x8 x = pb[kk];
        l = sum2(__builtin_shufflevector(x, x, 0, 1), l);
        l = sum2(__builtin_shufflevector(x, x, 2, 3), l);
        l = sum2(__builtin_shufflevector(x, x, 4, 5), l);
        l = sum2(__builtin_shufflevector(x, x, 6, 7), l);
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt) oacc[dt] = mfma32(op[kk * (D / 32) + dt], pb[kk], oacc[dt]);
    }
  };
  {  // two tiles per iteration, so that the buffer of a tile is known at compile time
    using B0 = std::integral_constant<int, 0>;
    using B1 = std::integral_constant<int, 1>;
    int t = 0;
    for (; t + 2 < ntiles; t += 2) {
      tile(std::false_type(), B0(), t);
      tile(std::false_type(), B1(), t + 1);
    }
    if (t + 2 == ntiles) {
      tile(std::false_type(), B0(), t);
      tile(std::true_type(), B1(), t + 1);
    } else {
      tile(std::true_type(), B0(), t);
    }
  }

  l += __shfl_xor(l, 32, 64);  // the two lane halves hold different keys of the same query
  if (qvalid) {
    const float inv = 1.0f / l;  // l > 0 for every existing query: its own key is never masked
    const int64_t obase = (tq * P.Hq + h) * D;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int vg = 0; vg < 4; ++vg) {
        const int d0 = 32 * dt + 8 * vg + 4 * hf;
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = oacc[dt][4 * vg + e] * inv;
        if (OUT_F32) {
          *(float4*)((float*)P.o + obase + d0) = make_float4(x[0], x[1], x[2], x[3]);
        } else {
          bf16x4 y;
          y[0] = (bf16)x[0]; y[1] = (bf16)x[1]; y[2] = (bf16)x[2]; y[3] = (bf16)x[3];
          *(bf16x4*)((bf16*)P.o + obase + d0) = y;
        }
      }
    if (hf == 0) P.lse[(int64_t)h * P.T + tq] = (m * P.scale_log2e + __builtin_log2f(l)) * 0.69314718055994531f;
  }
  timer.stop(P);
}

// float -> bf16 (round to nearest even) copies used when the caller's tensors are float: up to four tensors, one after the other, as
// one launch (a launch costs a small problem 4 us; element counts are multiples of head_dim).  The launch ends at kConvertWgs
// workgroups, a quarter of the threads that one dimension of a launch may have; tensors with more elements than that are strided over.
constexpr int64_t kConvertWgs = 1 << 22;
__global__ __launch_bounds__(256) void f32_to_bf16_kernel(Conversions c, int64_t n4) {
  for (int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x; u < n4; u += (int64_t)gridDim.x * 256) {
    int64_t at = u;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (at < c.n4[t]) {
        const float4 x = ((const float4*)c.src[t])[at];
        bf16x4 y;
        y[0] = (bf16)x.x; y[1] = (bf16)x.y; y[2] = (bf16)x.z; y[3] = (bf16)x.w;
        ((bf16x4*)c.dst[t])[at] = y;
        break;
      }
      at -= c.n4[t];
    }
  }
}

int convert_f32_to_bf16(const Conversions& c, hipStream_t st) {
  const int64_t n4 = c.n4[0] + c.n4[1] + c.n4[2] + c.n4[3], wgs = (n4 + 255) / 256;
  hipLaunchKernelGGL(f32_to_bf16_kernel, dim3((unsigned)(wgs < kConvertWgs ? wgs : kConvertWgs)), dim3(256), 0, st, c, n4);
  SB_LAUNCH_CHECK("f32_to_bf16_kernel");
  return SB_OK;
}

template <int D>
static void launch_fwd_head(const Geo& g, const AttnParams& P, hipStream_t st, int heads) {
  const bool one = one_wavefront_per_item(g, (int64_t)g.Hq * g.NQB, D == 64 ? 24 : 16);
  const dim3 grid((unsigned)head_grid(P, heads, one ? 1 : 2));
  auto launch = [&](auto f32, auto nw, auto loop) {
    constexpr int NW = decltype(nw)::value;
    hipLaunchKernelGGL((attn_fwd_head_kernel<D, decltype(f32)::value, NW, decltype(loop)::value>), grid, dim3(64 * NW), 0, st, P, heads);
  };
  auto with_loop = [&](auto f32, auto nw) {
    if constexpr (D == 128) {
      if (P.deal == kDealDraw) return launch(f32, nw, std::true_type());
    }
    launch(f32, nw, std::false_type());
  };
  auto with_nw = [&](auto f32) {
    if (one) with_loop(f32, std::integral_constant<int, 1>()); else with_loop(f32, std::integral_constant<int, 2>());
  };
  if (P.out_f32) with_nw(std::true_type()); else with_nw(std::false_type());
}

}  // namespace sb

using namespace sb;

extern "C" int sb_sparse_attn_fwd(const sb_problem* p, const void* q, const void* k, const void* v,
                                  const int32_t* sel_rowptr, const int32_t* sel_idx, const void* plan, void* o,
                                  float* lse, void* ws, void* stream) {
  Geo gb;
  int rc = make_geo(p, &gb);
  if (rc != SB_OK) return rc;
  if (gb.S == 0 || gb.T == 0 || gb.NQB == 0) return SB_OK;
  const Geo g = tile_geo(gb);  // the kernels work on 64-row tiles; for larger selection blocks the plan holds the tile-level selection
  if (!q || !k || !v || !sel_rowptr || !sel_idx || !plan || !o || !lse || !ws) { set_error("null argument"); return SB_ERR_INVALID_ARG; }
  hipStream_t st = (hipStream_t)stream;
  PlanOffsets po = plan_offsets(gb);
  WsOffsets wo = fwd_ws_offsets(g);
  const char* pb = (const char*)plan;
  char* wb = (char*)ws;
  Tables t = make_tables(g, p, (void*)(pb + po.tables));
  AttnParams P{};
  if (g.dtype == SB_F32) {
    Conversions c{};
    c.add(q, wb + wo.qc, (int64_t)g.T * g.Hq * g.D);
    c.add(k, wb + wo.kc, (int64_t)g.T * g.Hkv * g.D);
    c.add(v, wb + wo.vc, (int64_t)g.T * g.Hkv * g.D);
    if ((rc = convert_f32_to_bf16(c, st)) != SB_OK) return rc;
    P.q = (const bf16*)(wb + wo.qc); P.k = (const bf16*)(wb + wo.kc); P.v = (const bf16*)(wb + wo.vc);
  } else {
    P.q = (const bf16*)q; P.k = (const bf16*)k; P.v = (const bf16*)v;
  }
  P.o = o; P.lse = lse;
  P.idx = gb.r == 1 ? sel_idx : (const int32_t*)(pb + po.t_idx);
  P.items = (const WorkItem*)(pb + po.items);
  P.cu = t.cu; P.qb_off = t.qb_off; P.qb_seq = t.qb_seq; P.bm_off = t.bm_off;
  P.NQB = g.NQB; P.T = g.T; P.Hq = g.Hq; P.Hkv = g.Hkv; P.G = g.G; P.Hs = g.Hs; P.mode = g.mode;
  P.scale = g.softmax_scale; P.scale_log2e = g.softmax_scale * 1.4426950408889634f;
  P.out_f32 = g.dtype == SB_F32;
  P.cu_busy = nullptr;
  if (g_instrument & 1) {
    if ((rc = fill_zero(wb + wo.cu_busy, sizeof(uint64_t) * SB_CU_SLOTS, st)) != SB_OK) return rc;
    P.cu_busy = (unsigned long long*)(wb + wo.cu_busy);
  }
  const int heads = g.mode == SB_SELECT_PER_QHEAD ? 1 : g.G;  // query heads that share a work item
  const int64_t n_items = (int64_t)g.Hs * g.NQB;
  if (n_items > 0x3fffffffll) { set_error("too many work items for one launch"); return SB_ERR_INVALID_ARG; }
  const int parts = (heads + 3) / 4, hpp = (heads + parts - 1) / parts;  // the group kernel takes `hpp` heads per workgroup
  P.n_items = (int)n_items; P.ticket = nullptr;
  const bool group = g.D == 128 && hpp >= 3 && parts * hpp == heads;
  P.deal = group ? kDealPosition : forward_deal(g, n_items, heads);
  const bool tickets = group ? use_tickets(n_items) && parts <= kTicketPlanes : P.deal != kDealPosition;
  KernelTimer kt(K_FWD, st);
  if (tickets) {
    P.ticket = (int*)(wb + wo.ticket);
    if ((rc = fill_zero(P.ticket, sizeof(int32_t) * kTicketInts * (group ? parts : 1), st)) != SB_OK) return rc;
  }
  // Heads that share K/V tiles in LDS gather a third of what the per-head kernel does: faster on long sequences (131072 tokens, top 32:
  // 4.58 against 4.69 ms, 262144 tokens 15.8 against 16.0; the 32768-token batch 1.78 against 1.76), but not with a head slot left idle,
  // and not at D = 64 (65536 tokens, 14/2 heads, blocks of 256: 1.49 against 1.37).
  if (group) {
    dim3 grid((unsigned)(tickets ? held_grid(n_items) : (n_items + 7) / 8 * 8), (unsigned)parts), block(128 * hpp);
    if (P.out_f32) hipLaunchKernelGGL((attn_fwd_group_kernel<true>), grid, block, 0, st, P, heads);
    else hipLaunchKernelGGL((attn_fwd_group_kernel<false>), grid, block, 0, st, P, heads);
  } else {
    if (head_ids(n_items, heads) > 0x7fffffffll) { set_error("too many work items for one launch"); return SB_ERR_INVALID_ARG; }
    if (g.D == 128) launch_fwd_head<128>(g, P, st, heads);
    else launch_fwd_head<64>(g, P, st, heads);
  }
  SB_LAUNCH_CHECK("attn_fwd_kernel");
  return SB_OK;
}
