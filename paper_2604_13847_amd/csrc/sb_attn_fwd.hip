// Block-sparse attention forward (paper Eq. 2) on bf16 MFMA with fp32 online softmax.
//
// One workgroup of two wavefronts per work item (sequence s, query head, query block i), taken from
// the longest-first work list.  The two wavefronts split every selected key block by KEYS: wavefront
// w owns keys 32w .. 32w+31 of each block and all 64 query rows, and runs an online softmax of its
// own over its half of the keys (running max, running sum and an unnormalised O per wavefront); the
// two partial results are merged once, at the end, through LDS.  Because a wavefront only ever
// touches its own key strips, it stages them itself (asynchronous global->LDS loads into a private
// ring of strips K0 V0 K1 V1 ..., three strips ahead) and the main loop has no barrier at all.
// Each K / V^T operand read from LDS feeds two MFMAs (one per 32-query half), which halves the LDS
// traffic per flop compared with a split by query rows.
// S^T = K Q^T puts a query in a C-matrix column, so the softmax statistics are per lane and the
// probabilities convert to the B operand of O^T += V^T P^T without any cross-lane movement; V^T is
// read straight out of the row-major V strip with the transposing LDS read.
// That is attn_fwd_kernel, for head_dim 64.  It is held to 256 registers, so that two wavefronts share a SIMD and one runs its
// exponentials (which outlast the matrix instructions there) under the other's matrix instructions: 2.14 -> 1.67 ms on 65536 tokens,
// 14/2 heads, selection blocks of 256, and 1.56 with the softmax's branch (matrix cores busy 28 -> 44 % of the cycles).
// Head_dim 128 takes the registers of a whole SIMD and has a kernel of its own, attn_fwd_head_kernel.
#include <type_traits>

#include "sb_attn_common.h"

namespace sb {

template <bool OUT_F32>
__global__ __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(2))) void attn_fwd_kernel(AttnParams P, int n_items, int heads) {
  constexpr int D = 64;
  constexpr int NS = 4;          // strips in a wavefront's ring
  constexpr int SLOT = 32 * D;   // elements per strip
  constexpr int LPS = StripLoader<D>::LPS;
  constexpr float kLazy = 8.0f;  // see the softmax below
  __shared__ __attribute__((aligned(1024))) bf16 ring[2][NS][SLOT];
  static_assert(sizeof(bf16) * NS * SLOT >= (16 * (D / 32) + 2) * 64 * sizeof(float), "merge buffer must fit in a ring");
  BusyTimer timer;
  timer.start(P);
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  // Workgroup id -> (position in the work list, query head of the group).  In per-KV-group mode the
  // `heads` query heads of an item take ids that are 8 apart, so they run on the same XCD (ids are
  // dealt round-robin to the 8 XCDs) and share its L2 for the K/V strips.
  int pos = (int)(blockIdx.x / (8u * heads)) * 8 + (int)(blockIdx.x & 7u);
  const int hh = (int)(blockIdx.x >> 3) % heads;
  pos = claim_item(pos, n_items, P.ticket ? P.ticket + hh : nullptr);
  if (pos < 0) return;
  const WorkItem item = uniform_item(P.items, pos);
  const int hs = item.hs, i = item.i, L = item.len, e0 = item.e0, ntiles = item.ntiles;
  const int64_t seq0 = item.seq0;
  const int h = P.mode == SB_SELECT_PER_QHEAD ? hs : hs * P.G + hh;
  const int g = P.mode == SB_SELECT_PER_QHEAD ? hs / P.G : hs;

  // query fragments of both 32-row halves: qf[b][ks] = Q[32b + lane%32][16ks + 8*(lane/32) .. +7]
  bf16x8 qf[2][D / 16];
  bool qvalid[2];
  int64_t tq[2];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int qloc = 32 * b + l32;
    qvalid[b] = i * 64 + qloc < L;
    tq[b] = seq0 + i * 64 + qloc;
    const bf16* qp = P.q + (tq[b] * P.Hq + h) * D + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) qf[b][ks] = qvalid[b] ? *(const bf16x8*)(qp + 16 * ks) : zero_bf16x8();
  }
  // The row's block indices live in one register across the wavefront (lane a holds entry jb0 + a),
  // refilled every ~64 tiles; a refill waits for all loads in flight, which is rare enough.  Requests
  // run at most two entries behind the newest one, so the window keeps two entries of slack.
  int jb0 = 0;
  int jreg = lane < ntiles ? P.idx[e0 + lane] : 0;
  auto refill = [&](int first) __attribute__((always_inline)) {
    jb0 = first;
    jreg = jb0 + lane < ntiles ? P.idx[e0 + jb0 + lane] : 0;
    // wait here, inside the caller's branch: otherwise the compiler puts a full wait at the join after
    // it, which would drain the strip loads in flight every time
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  };
  auto block_of = [&](int x) __attribute__((always_inline)) {
    if (x - jb0 >= 64) refill(x - 2);
    return __builtin_amdgcn_readlane(jreg, x - jb0);
  };
  // The wavefront's strips (rows 32*wave .. +31 of a selected block's K or V) are loaded in the order
  // in which the pipelined loop below consumes them:
  //   c = 0: K_0;   c = 2i+1: K_{i+1};   c = 2i+2: V_i;   c = 2*ntiles-1 (the last): V_{ntiles-1}
  // Strip c lives in ring slot c % NS and is issued as soon as strip c - NS has been read.
  StripLoader<D> loader;
  loader.init(P.Hkv, lane);
  const int nstrips = 2 * ntiles;
  const char* const k0 = (const char*)(P.k + ((seq0 + 32 * wave) * P.Hkv + g) * D);  // this wavefront's strip of block 0
  const char* const v0 = (const char*)(P.v + ((seq0 + 32 * wave) * P.Hkv + g) * D);
  const unsigned block_pitch = 64u * (unsigned)P.Hkv * D * 2;  // bytes from one key block to the next
  const unsigned ring0 = lds_offset(&ring[wave][0][0]);
  const int Lw = L - 32 * wave;  // rows of the sequence from this wavefront's strip of block 0 on
  auto issue_strip = [&](int slot, bool is_v, int tile) __attribute__((always_inline)) {
    const int j = block_of(tile);
    loader.issue(ring0 + slot * (SLOT * 2), (is_v ? v0 : k0) + (unsigned long long)(unsigned)j * block_pitch, Lw - j * 64);
  };
  int issued = -1;  // newest strip issued so far
  auto try_issue = [&](int c) __attribute__((always_inline)) {
    if (c >= nstrips) return;
    const bool is_v = c == nstrips - 1 || (c != 0 && (c & 1) == 0);
    const int tile = c == 0 ? 0 : c == nstrips - 1 ? ntiles - 1 : (c & 1) ? (c + 1) >> 1 : (c >> 1) - 1;
    issue_strip(c % NS, is_v, tile);
    issued = c;
  };
  // waits until strip c has landed (loads complete in order, so the newer ones may stay in flight)
  auto wait_strip = [&](int c) __attribute__((always_inline)) {
    const int younger = issued - c;
    if (younger >= 3) wait_vmcnt<3 * LPS>();
    else if (younger == 2) wait_vmcnt<2 * LPS>();
    else if (younger == 1) wait_vmcnt<LPS>();
    else wait_vmcnt<0>();
  };
  // LDS addresses of this lane's operand reads within slot 0 of the wavefront's ring; the slot is a
  // compile-time offset wherever the loop is unrolled
  unsigned k_addr[D / 16], v_addr[D / 32][2];
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) k_addr[ks] = ring0 + l32 * (D * 2) + 16 * ((2 * ks + hf) ^ chunk_swizzle<D>(l32));
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int r = 8 * half + 4 * hf + ((lane & 15) >> 2), d = 32 * dt + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      v_addr[dt][half] = ring0 + r * (D * 2) + 16 * ((d >> 3) ^ chunk_swizzle<D>(r)) + 2 * (d & 7);
    }
  bf16x8 ka[D / 16], va[D / 32][2];
  auto read_k = [&](int slot) __attribute__((always_inline)) {  // operands of S^T = K Q^T: K rows of this wavefront, all of d
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) ka[ks] = *(const bf16x8 __attribute__((address_space(3)))*)(k_addr[ks] + slot * (SLOT * 2));
  };
  // operands of O^T += V^T P^T through the transposing read: contraction slots of step kk are the
  // keys 16kk + 8*(e/4) + 4*(lane/32) + e%4 (rows 16 apart share the swizzle, so kk is a plain offset)
  auto read_v = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)(v_addr[dt][0] + slot * (SLOT * 2) + kk * 16 * (D * 2)));
        bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)(v_addr[dt][1] + slot * (SLOT * 2) + kk * 16 * (D * 2)));
        va[dt][kk] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      }
  };
  // the query fragments and indices must have landed before the strip loads start: from here on the
  // only vector-memory operations in flight are strip loads, which the loop waits for by count
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) asm volatile("" : "+v"(qf[b][ks]));
  asm volatile("" : "+v"(jreg));

  f32x16 oacc[D / 32][2];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) oacc[dt][0] = oacc[dt][1] = zero16();
  float m[2] = {-__builtin_inff(), -__builtin_inff()}, l[2] = {0.f, 0.f};
  f32x16 sa[2][2];  // raw scores of the current and the next tile (ping-pong)
  bf16x8 pb[2][2];
  float alpha[2];

  auto scores = [&](f32x16* dst) __attribute__((always_inline)) {  // dst = K Q^T for the strip whose operands are in ka
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      dst[b] = zero16();
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks) dst[b] = mfma32(ka[ks], qf[b][ks], dst[b]);
    }
  };
  auto rescale = [&]() __attribute__((always_inline)) {
    if (__builtin_amdgcn_ballot_w64((alpha[0] != 1.0f) | (alpha[1] != 1.0f)) != 0) {
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int v = 0; v < 16; ++v) oacc[dt][b][v] *= alpha[b];
    }
  };
  // online softmax on raw scores sc: p = exp2(scale*log2e * (s - m)) -> pb, running sums updated
  float neg_m[2];
  auto max_of = [&](const f32x16& x) __attribute__((always_inline)) {  // of this lane's keys
    float mx = max3(x[0], x[1], x[2]);
#pragma unroll
    for (int v = 3; v < 15; v += 2) mx = max3(mx, x[v], x[v + 1]);
    return fmaxf(mx, x[15]);
  };
  auto reference = [&](const float* mx_lane) __attribute__((always_inline)) {  // moves m, sets alpha
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const float mx = max_across_halves(mx_lane[b]);
      // Lazy running maximum: the reference m[b] used in the exponent follows the true maximum only
      // when that has grown by more than kLazy (in log2 units), so p stays below 2^kLazy and the
      // accumulated O needs rescaling only then.  The result is the same up to rounding (O and the
      // row sum carry the same factor), and the rescale branch becomes rare instead of the rule.
      const bool first = m[b] == -__builtin_inff();  // nothing accumulated yet for this query: nothing to rescale
      const bool move = first | ((mx - m[b]) * P.scale_log2e > kLazy);
      const float m_new = move ? fmaxf(m[b], mx) : m[b];
      // a wavefront may have seen no unmasked key yet for a query (its strip of the diagonal block can
      // be entirely above the diagonal): keep the exponent finite then
      const float m_use = m_new == -__builtin_inff() ? 0.f : m_new;
      alpha[b] = first ? 1.0f : fast_exp2((m[b] - m_use) * P.scale_log2e);
      neg_m[b] = -m_use * P.scale_log2e;
      l[b] *= alpha[b];
      m[b] = m_new;
    }
  };
  auto softmax = [&](const f32x16* sc) __attribute__((always_inline)) {
    const float mx[2] = {max_of(sc[0]), max_of(sc[1])};
    // Whether any lane's own maximum has grown that far is one comparison per lane, so everything else about the reference moves
    // into a branch that a row takes in its first tiles: the vector work, not the matrix work, bounds this head dimension
    // (1674 -> 1563 us on 65536 tokens, 14/2 heads, selection blocks of 256).
    if (__builtin_amdgcn_ballot_w64(!((mx[0] - m[0]) * P.scale_log2e <= kLazy) | !((mx[1] - m[1]) * P.scale_log2e <= kLazy)) != 0) {
      reference(mx);
      rescale();
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
      for (int v = 0; v < 16; ++v) pb[b][v >> 3][v & 7] = (bf16)fast_exp2(__builtin_fmaf(sc[b][v], P.scale_log2e, neg_m[b]));
      // the row sum adds up the probabilities as rounded to bf16, i.e. exactly the weights the
      // accumulation below applies, two per instruction
      float rs = l[b];
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
      {
        const bf16x8 x = pb[b][kk];
        rs = sum2(__builtin_shufflevector(x, x, 0, 1), rs);
        rs = sum2(__builtin_shufflevector(x, x, 2, 3), rs);
        rs = sum2(__builtin_shufflevector(x, x, 4, 5), rs);
        rs = sum2(__builtin_shufflevector(x, x, 6, 7), rs);
      }
      l[b] = rs;
    }
  };
  auto accumulate = [&]() __attribute__((always_inline)) {  // O^T += V^T P^T with the operands in va and pb
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int b = 0; b < 2; ++b) oacc[dt][b] = mfma32(va[dt][kk], pb[b][kk], oacc[dt][b]);
  };

  // ---- prologue: S_0, and the K operands of tile 1
#pragma unroll
  for (int c = 0; c < NS; ++c) try_issue(c);
  wait_strip(0);
  read_k(0);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  try_issue(NS);
  scores(sa[0]);
  if (ntiles > 1) {
    wait_strip(1);
    read_k(1);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    try_issue(NS + 1);
  }
  // ---- steady state: step t turns S_t into P_t while the MFMAs of S_{t+1} run, then accumulates
  // P_t V_t while the operands of S_{t+2} are fetched.  The loop is unrolled by two so that ring
  // slots and the score ping-pong are compile-time; steps far enough from the end of the row
  // (STEADY) know how many loads are in flight and that every strip they prefetch exists.
  auto step = [&](auto par_c, auto steady_c, int t) __attribute__((always_inline)) {
    constexpr int PAR = decltype(par_c)::value;  // t % 2
    constexpr bool STEADY = decltype(steady_c)::value;
    constexpr int SV = (2 * PAR + 2) % NS, SK = (2 * PAR + 3) % NS;  // slots of strips 2t+2 (V_t) and 2t+3 (K_{t+2})
    // max3 in the softmax is inline asm, whose reads of the matrix instructions' results the compiler's hazard recogniser does not
    // see: 12 wait states after an 8-pass instruction
    asm volatile("s_nop 7\n\ts_nop 3" : "+v"(sa[PAR][0]), "+v"(sa[PAR][1]));
    if (STEADY) wait_vmcnt<3 * LPS>(); else wait_strip(2 * t + 2);
    read_v(SV);
    scores(sa[PAR ^ 1]);
    softmax(sa[PAR]);
    // The probabilities of the first 16 keys are pinned above the rescale branch so that their
    // exponentials overlap the score MFMAs; those of the other 16 may sink below it and overlap the
    // first half of the accumulation MFMAs.
    asm volatile("" : "+v"(pb[0][0]), "+v"(pb[1][0]));
    if (STEADY) {
      wait_vmcnt<2 * LPS>();
      read_k(SK);
    } else if (t + 2 < ntiles) {
      wait_strip(2 * t + 3);
      read_k(SK);
    }
    __builtin_amdgcn_sched_barrier(0x47F);  // the LDS reads stay above the MFMAs: they must be done before their slot is refilled below
    accumulate();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slots about to be refilled have been read
    if (STEADY) {  // tiles t+2 and t+4 are not the row's last, so their blocks are complete; the window holds them
      loader.issue_full(ring0 + SV * (SLOT * 2), v0 + (unsigned long long)(unsigned)__builtin_amdgcn_readlane(jreg, t + 2 - jb0) * block_pitch);
      loader.issue_full(ring0 + SK * (SLOT * 2), k0 + (unsigned long long)(unsigned)__builtin_amdgcn_readlane(jreg, t + 4 - jb0) * block_pitch);
      issued = 2 * t + 3 + NS;
    } else {
      try_issue(2 * t + 2 + NS);
      try_issue(2 * t + 3 + NS);
    }
  };
  using std::integral_constant;
  int t = 0;
  for (; t + 6 < ntiles; t += 2) {  // both steps prefetch tiles <= t + 5, none of them the row's last (the only one that can be ragged)
    if (t + 5 - jb0 >= 64) refill(t + 2);
    step(integral_constant<int, 0>(), integral_constant<bool, true>(), t);
    step(integral_constant<int, 1>(), integral_constant<bool, true>(), t + 1);
  }
  for (; t + 1 < ntiles; t += 2) {
    step(integral_constant<int, 0>(), integral_constant<bool, false>(), t);
    if (t + 2 < ntiles) step(integral_constant<int, 1>(), integral_constant<bool, false>(), t + 1);
  }
  // ---- last tile: the diagonal block, causal mask inside it
  if ((ntiles - 1) & 1) {
    sa[0][0] = sa[1][0];
    sa[0][1] = sa[1][1];
  }
  wait_strip(nstrips - 1);
  read_v((nstrips - 1) % NS);
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (32 * wave + c_row(v, hf) > 32 * b + l32) sa[0][b][v] = -__builtin_inff();
  softmax(sa[0]);
  accumulate();

  // ---- merge the two key halves: wavefront w finalises query half w and hands the other half over
  l[0] += __shfl_xor(l[0], 32, 64);
  l[1] += __shfl_xor(l[1], 32, 64);
  float* xbuf = (float*)&ring[wave][0][0];            // this wavefront's outgoing partial, [register][lane]
  const float* ybuf = (const float*)&ring[wave ^ 1][0][0];  // the partner's
  constexpr int NR = 16 * (D / 32);
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
      if (qvalid[b]) {
        const int64_t obase = (tq[b] * P.Hq + h) * D;
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
          for (int vg = 0; vg < 4; ++vg) {
            const int d0 = 32 * dt + 8 * vg + 4 * hf;
            float x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = oacc[dt][b][4 * vg + e] * c1 + ybuf[(16 * dt + 4 * vg + e) * 64 + lane] * c2;
            if (OUT_F32) {
              *(float4*)((float*)P.o + obase + d0) = make_float4(x[0], x[1], x[2], x[3]);
            } else {
              bf16x4 y;
              y[0] = (bf16)x[0]; y[1] = (bf16)x[1]; y[2] = (bf16)x[2]; y[3] = (bf16)x[3];
              *(bf16x4*)((bf16*)P.o + obase + d0) = y;
            }
          }
        if (hf == 0) P.lse[(int64_t)h * P.T + tq[b]] = (mt * P.scale_log2e + __builtin_log2f(lt)) * 0.69314718055994531f;
      }
    }
  }
  timer.stop(P);
}

// ---------------------------------------------------------------------------------------------
// The same for D = 128 and one query head, by one wavefront (NW = 1: it walks both 32-key strips of every tile, nothing is merged) or
// two (as above; for problems of few items, see one_wavefront_per_item).
// What bounds it: a wavefront has its SIMD to itself, so what it waits for is idle time of the matrix cores, and it issues one
// instruction of any kind every four to five cycles (an exponential: nine), 6 beside each 32-cycle matrix instruction.  Hence a software
// pipeline over half tiles u (32 keys x 32 queries) of two stages of 8 matrix instructions,
//   O(u-1), S(u+1)
// with the probabilities of u beside both; every matrix instruction is fenced with its share of the vector work, of the LDS reads and of
// the tile loads (two at a time), whose addresses are scalar work; no branch but the one in check().  Beyond that the chip lowers its
// clock under matrix load (a loop of these matrix instructions alone runs at 1.7 GHz of 2.4), so what saves instructions saves time
// twice.  Per tile and SIMD, a third of the time is what the matrix instructions alone would take at 2.4 GHz.
// The fixed part of an item (6 us: descriptor 0.7, indices 0.8, first strips and Q 2.0, output 2.7) counts half as much with one
// wavefront per item as with two.  Against the kernel above at D = 128 (two wavefronts, a whole tile's softmax in a row) the forward of:
// the 32768-token batch, 32/8 heads: 2.05 -> 1.67 ms (with NW = 2: 1.74), one 131072-token sequence, top 32: 7.30 -> 6.24 (6.51), the
// 262144-token batch: 20.3 -> 18.0 (20.7), 65536 tokens whose selection is a sink and a window: 2.27 -> 1.75 (1.95).
template <bool OUT_F32, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(1))) void attn_fwd_head_kernel(AttnParams P, int n_items, int heads) {
  constexpr int D = 128, ROW_B = D * 2, STRIP_B = 32 * ROW_B, NOP = D / 16, NV = 3;
  constexpr float kLazy = 8.0f;
  using Loader = QuadLoader<D>;
  constexpr int LPS = Loader::LPS;
  // per wavefront: K even, K odd, then V of strip t in slot 2 + t % 3.  Four wavefronts' rings fill a CU's LDS.
  constexpr int RING_B = (2 + NV) * STRIP_B;
  __shared__ __attribute__((aligned(1024))) char ring[NW][RING_B];
  BusyTimer timer;
  timer.start(P);
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  // Workgroup id -> (position in the work list, query head of the group), see the kernel above
  int pos = (int)(blockIdx.x / (8u * heads)) * 8 + (int)(blockIdx.x & 7u);
  const int hh = (int)(blockIdx.x >> 3) % heads;
  pos = claim_item(pos, n_items, P.ticket ? P.ticket + hh : nullptr, NW == 2 ? (int*)&ring[NW - 1][RING_B - 4] : nullptr);
  if (pos < 0) return;
  const WorkItem item = uniform_item(P.items, pos);
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
  // m: reference of the exponent, neg_m = -m * scale * log2 e.  Before a query's first tile neg_m is +inf, so that the first sum of
  // probabilities fails the check below and m is set there.
  float m[2] = {-__builtin_inff(), -__builtin_inff()}, l[2] = {0.f, 0.f}, neg_m[2] = {__builtin_inff(), __builtin_inff()};
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
  // The reference follows the true maximum lazily: only when a lane's 16 probabilities add up to more than 2^12 (so one of them exceeds
  // 2^8), which costs one comparison per half tile where the maximum of the scores would cost ten instructions.  The scores are still
  // there: the reference moves, what has been summed with the old one is rescaled, and the probabilities are computed again.
  auto check = [&](int b) __attribute__((always_inline)) {
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(psum <= 4096.f)) != 0, 0)) {
      float mx = max3(sacc[b][0], sacc[b][1], sacc[b][2]);
#pragma unroll
      for (int v = 3; v < 15; v += 2) mx = max3(mx, sacc[b][v], sacc[b][v + 1]);
      mx = max_across_halves(fmaxf(mx, sacc[b][15]));
      const bool first = m[b] == -__builtin_inff();  // nothing accumulated yet for this query: nothing to rescale
      const bool move = first | ((mx - m[b]) * P.scale_log2e > kLazy);
      const float m_new = move ? fmaxf(m[b], mx) : m[b];
      // a wavefront may have seen no unmasked key yet for a query: keep the exponent finite then
      const float m_use = m_new == -__builtin_inff() ? 0.f : m_new;
      const float alpha = first ? 1.0f : fast_exp2((m[b] - m_use) * P.scale_log2e);
      neg_m[b] = -m_use * P.scale_log2e;
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
      asm volatile("s_nop 1" ::: "memory");  // two wait states between a vector write and its use as an operand
    }
    l[b] += psum;
  };

#define SB_FENCE() __builtin_amdgcn_sched_barrier(0)
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
        if (k == 2) __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): K_{t+1} is in ka
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
      if (SEEN && k > 0) p_step(B, k - 1);
      SB_FENCE();
      if constexpr (!LAST) {
        if (k == 3) loader.template issue2<0>(rsrc, slot);
        if (k == 6) loader.template issue2<2>(rsrc, slot);
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
        if (k == 2) {
          wait_vmcnt<2 * LPS + 4>();  // K_{t+1} has landed; V_{t+1}, K_{t+2} and half of V_{t+2} may still be on their way
          __builtin_amdgcn_s_waitcnt(0xC07F);
          ka[0] = ld_row(0, (PAR ^ 1) * STRIP_B);
          ka[1] = ld_row(1, (PAR ^ 1) * STRIP_B);
        }
        if (k >= 2) ka[k] = ld_row(k, (PAR ^ 1) * STRIP_B);
      }
      if (SEEN) p_step(B, 7 + k);
      SB_FENCE();
      if constexpr (!LAST) {
        if (k == 3) loader.template issue2<4>(rsrc, slot);
        if (k == 6) loader.template issue2<6>(rsrc, slot);
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
      if (hf == 0 && l32 < rows) P.lse[(int64_t)h * P.T + tq + l32] = (m[b] * P.scale_log2e + __builtin_log2f(l[b])) * 0.69314718055994531f;
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
  timer.stop(P);
}

// ---------------------------------------------------------------------------------------------
// Forward kernel for per-KV-group selection: the query heads of a KV group share a work item, so one
// workgroup takes 3 or 4 of them and they share the item's K/V tiles in LDS (whole tiles,
// double-buffered by asynchronous loads) instead of fetching them once per head.  Two wavefronts per
// query head; a wavefront owns 32 query rows and all 64 keys of every selected tile, as two 32-key
// halves with one online-softmax step each.  The register budget (256) lets two wavefronts share a
// SIMD, so one runs its exponentials while the other runs matrix instructions; one operand set
// rotates through both contractions (K rows, then V^T through the transposing read, each register
// refilled right after the MFMA that consumed it).
template <int D, bool OUT_F32>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void attn_fwd_group_kernel(AttnParams P, int heads) {
  constexpr int TILE_B = 64 * D * 2, ROW_B = D * 2, NOP = D / 16;
  constexpr float kLazy = 8.0f;
  __shared__ __attribute__((aligned(1024))) bf16 tiles[2][2][64 * D];  // [buffer][K, V]
  constexpr int kJ = 256;
  __shared__ int jbuf[kJ];
  BusyTimer timer;
  timer.start(P);
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int pos = claim_item(blockIdx.x, P.n_items, P.ticket ? P.ticket + blockIdx.y : nullptr);
  if (pos < 0) return;
  // (at D = 128 scalar descriptors make the compiler keep more in registers than there are: 1.70 -> 1.74 ms on the 32768-token batch)
  const WorkItem item = D == 64 ? uniform_item(P.items, pos) : P.items[pos];
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
  TileLoader<D, 4> loader;  // a workgroup has six or eight wavefronts: the first four share the tile loads
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
  P.rowptr = gb.r == 1 ? sel_rowptr : (const int32_t*)(pb + po.t_rowptr);
  P.idx = gb.r == 1 ? sel_idx : (const int32_t*)(pb + po.t_idx); P.work = (const int32_t*)(pb + po.work_fwd);
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
  const bool tickets = use_tickets(n_items) && heads <= kTicketSlots;
  P.n_items = (int)n_items; P.ticket = nullptr;
  KernelTimer kt(K_FWD, st);
  if (tickets) {
    P.ticket = (int*)(wb + wo.ticket);
    if ((rc = fill_zero(P.ticket, sizeof(int32_t) * kTicketSlots, st)) != SB_OK) return rc;
  }
  const int64_t n_slots = ticketed_grid(n_items, tickets);  // workgroups per head plane
  if (hpp >= 3 && parts * hpp == heads) {  // heads share K/V tiles in LDS; with a head slot left idle the per-head kernel is faster
    dim3 grid((unsigned)n_slots, (unsigned)parts), block(128 * hpp);
#define SB_FWD_LAUNCH(DD, FF) hipLaunchKernelGGL((attn_fwd_group_kernel<DD, FF>), grid, block, 0, st, P, heads)
    if (g.D == 128) {
      if (P.out_f32) SB_FWD_LAUNCH(128, true); else SB_FWD_LAUNCH(128, false);
    } else {
      if (P.out_f32) SB_FWD_LAUNCH(64, true); else SB_FWD_LAUNCH(64, false);
    }
#undef SB_FWD_LAUNCH
  } else {
    const int64_t n_wg = n_slots * heads;
    if (n_wg > 0x7fffffffll) { set_error("too many work items for one launch"); return SB_ERR_INVALID_ARG; }
    dim3 grid((unsigned)n_wg);
#define SB_FWD_LAUNCH(FF) hipLaunchKernelGGL((attn_fwd_kernel<FF>), grid, dim3(128), 0, st, P, (int)n_items, heads)
    if (g.D == 128) {
#define SB_FWD_HEAD_LAUNCH(FF, NW) hipLaunchKernelGGL((attn_fwd_head_kernel<FF, NW>), grid, dim3(64 * NW), 0, st, P, (int)n_items, heads)
      if (one_wavefront_per_item(g, (int64_t)g.Hq * g.NQB, 16)) {
        if (P.out_f32) SB_FWD_HEAD_LAUNCH(true, 1); else SB_FWD_HEAD_LAUNCH(false, 1);
      } else {
        if (P.out_f32) SB_FWD_HEAD_LAUNCH(true, 2); else SB_FWD_HEAD_LAUNCH(false, 2);
      }
#undef SB_FWD_HEAD_LAUNCH
    } else {
      if (P.out_f32) SB_FWD_LAUNCH(true); else SB_FWD_LAUNCH(false);
    }
#undef SB_FWD_LAUNCH
  }
  SB_LAUNCH_CHECK("attn_fwd_kernel");
  return SB_OK;
}
