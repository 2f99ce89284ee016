// Block-sparse attention backward (gradient of paper Eq. 2 with the selection held fixed).
//
//   Dr = rowsum(dO * O)                                    (prologue of the query-major kernel, which owns every row once)
//   P  = exp(scale * S - LSE),  dP = dO V^T,  dS = P * (dP - Dr)
//   dQ = scale * dS K          query-major kernel, same work items and tile walk as the forward
//   dK = scale * dS^T Q, dV = P^T dO   key-major kernel: one workgroup owns key block (s, g, j),
//        keeps its K/V strip in registers, walks the query blocks that kept j (transpose bitmap, last
//        query block first) for every query head of the KV group and accumulates in registers; each output
//        element is written once, in a fixed order, so the result is deterministic.
#include <type_traits>

#include "sb_attn_common.h"

namespace sb {

// ---------------------------------------------------------------------------------------------
// Query-major dQ kernel for few items at D = 64.  Same work items as the forward, one query head per workgroup of four wavefronts: the K and
// V tiles of the selected blocks are double-buffered in LDS as whole tiles by asynchronous loads and shared by the workgroup; a wavefront
// owns 32 query rows and one 32-key half of every tile (the two partial dQ of a row are added through LDS at the end); Q, dO, LSE and
// Dr of its rows stay in registers.  Every (token, query head) row belongs to exactly one workgroup of this kernel, so its prologue is also
// where Dr is computed (from the dO registers and one read of O) and left, with LSE * log2 e, for the key-major kernel.
// Transposed products put a query in a C-matrix column: S^T = K Q^T, dP^T = V dO^T, so LSE and Dr are per-lane scalars and dS^T converts to
// the B operand of dQ^T += K^T dS^T without cross-lane movement; K^T comes from the row-major K tile through the transposing LDS read.
// Four wavefronts get through the longest item sooner than the kernel below, which wins where the chip is full: 336 items of 1 - 42 tiles
// 30.6 against 32.8 us, 1504 of 1 - 16 tiles 47 against 49, but 6144 of 1 - 16 tiles 152 against 131.
template <bool OUT_F32>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void attn_bwd_dq_kernel(AttnParams P) {
  constexpr int D = 64;
  constexpr int TILE_B = 64 * D * 2, ROW_B = D * 2, NOP = D / 16;
  __shared__ __attribute__((aligned(1024))) bf16 tiles[2][2][64 * D];  // [buffer][K, V]
  constexpr int kJ = 256;
  __shared__ int jbuf[kJ];
  static_assert(sizeof(tiles) >= 2 * 16 * (D / 32) * 64 * sizeof(float), "partial dQ must fit in the tile buffers");
  BusyTimer timer;
  timer.start(P);
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int pos = (int)blockIdx.x < P.n_items ? (int)blockIdx.x : -1;  // (so few items are dealt by position)
  if (pos < 0) return;
  const WorkItem item = uniform_item(P.items, pos);
  const int hs = item.hs, i = item.i, L = item.len, e0 = item.e0, ntiles = item.ntiles;
  const int64_t seq0 = item.seq0;
  const int strip = wave & 1, kh = wave >> 1;
  const int h = P.mode == SB_SELECT_PER_QHEAD ? hs : hs * P.G + (int)blockIdx.y;
  const int g = h / P.G;
  const int qloc = strip * 32 + l32;
  const bool qvalid = i * 64 + qloc < L;
  const int64_t tq = seq0 + i * 64 + qloc;

  auto stage_indices = [&](int t0) {
    __syncthreads();
    for (int a = tid; a < kJ; a += 256) jbuf[a] = t0 + a < ntiles ? P.idx[e0 + t0 + a] : 0;
    __syncthreads();
  };
  TileLoader<D> loader;
  loader.init(P.Hkv, wave, lane);
  auto issue = [&](int t) {
    const int j = __builtin_amdgcn_readfirstlane(jbuf[t % kJ]);
    const int64_t kv0 = seq0 + (int64_t)j * 64;
    const int kvalid = min(64, L - j * 64);
    loader.issue(tiles[t & 1][0], P.k, kv0, kvalid, P.Hkv, g);
    loader.issue(tiles[t & 1][1], P.v, kv0, kvalid, P.Hkv, g);
  };

  // B operands: column = query lane%32 of the strip, slots = d 16ks + 8hf + (0..7)
  bf16x8 qf[NOP], dof[NOP];
  float lse2 = __builtin_inff(), dr = 0.f;  // rows that do not exist: P = exp2(x - inf) = 0
  {
    const bf16* qp = P.q + (tq * P.Hq + h) * D + 8 * hf;
    const bf16* dp = P.d_o + (tq * P.Hq + h) * D + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < NOP; ++ks) {
      qf[ks] = qvalid ? *(const bf16x8*)(qp + 16 * ks) : zero_bf16x8();
      dof[ks] = qvalid ? *(const bf16x8*)(dp + 16 * ks) : zero_bf16x8();
    }
    // Dr of the lane's query: its half of the head dimension here, the other half in lane ^ 32
    float part = 0.f;
    if (qvalid) {
      if (OUT_F32) {
        const float* op_ = (const float*)P.o + (tq * P.Hq + h) * D + 8 * hf;
#pragma unroll
        for (int ks = 0; ks < NOP; ++ks) {
          const float4 a = *(const float4*)(op_ + 16 * ks), b = *(const float4*)(op_ + 16 * ks + 4);
          part += (float)dof[ks][0] * a.x + (float)dof[ks][1] * a.y + (float)dof[ks][2] * a.z + (float)dof[ks][3] * a.w;
          part += (float)dof[ks][4] * b.x + (float)dof[ks][5] * b.y + (float)dof[ks][6] * b.z + (float)dof[ks][7] * b.w;
        }
      } else {
        const bf16* op_ = (const bf16*)P.o + (tq * P.Hq + h) * D + 8 * hf;
#pragma unroll
        for (int ks = 0; ks < NOP; ++ks) {
          const bf16x8 ov = *(const bf16x8*)(op_ + 16 * ks);
#pragma unroll
          for (int e = 0; e < 8; ++e) part += (float)dof[ks][e] * (float)ov[e];
        }
      }
      lse2 = P.lse[(int64_t)h * P.T + tq] * 1.4426950408889634f;
    }
    dr = part + __shfl_xor(part, 32, 64);
  }
  stage_indices(0);
  // everything loaded so far must have landed before the tile loads start (see the forward kernel)
#pragma unroll
  for (int ks = 0; ks < NOP; ++ks) asm volatile("" : "+v"(qf[ks]), "+v"(dof[ks]));
  asm volatile("" : "+v"(lse2), "+v"(dr));
  issue(0);

  // LDS byte addresses of this lane's operand reads inside buffer 0's K tile, key half kh; the buffer
  // and everything else is a compile-time offset
  const unsigned tiles0 = lds_offset(&tiles[0][0][0]);
  unsigned row_a[NOP], tr_a[D / 32][2];
#pragma unroll
  for (int ks = 0; ks < NOP; ++ks) row_a[ks] = tiles0 + (32 * kh + l32) * ROW_B + 16 * ((2 * ks + hf) ^ chunk_swizzle<D>(l32));
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int r = 8 * half + 4 * hf + ((lane & 15) >> 2), d = 32 * dt + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      tr_a[dt][half] = tiles0 + (32 * kh + r) * ROW_B + 16 * ((d >> 3) ^ chunk_swizzle<D>(r)) + 2 * (d & 7);
    }
  auto ld_row = [&](int ks, unsigned off) __attribute__((always_inline)) {
    return *(const bf16x8 __attribute__((address_space(3)))*)(row_a[ks] + off);
  };
  // A operand of dQ^T += K^T dS^T: row = d (32dt + lane%32), slots = keys 16kk + 8(e/4) + 4hf + e%4 of this wavefront's rows
  auto ld_tr = [&](int kk, int dt, unsigned off) __attribute__((always_inline)) {
    const unsigned o = off + kk * 16 * ROW_B;
    bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)(tr_a[dt][0] + o));
    bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)(tr_a[dt][1] + o));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };

  bf16x8 op[NOP];  // one rotating operand set: a register is refilled for the next contraction as soon as it has been consumed

  // A row that keeps only its own block sees few keys: its O is not an average, |O| is of the size of |v|, and the
  // rounding of the stored O (2^-9 relative) moves rowsum(dO * O) by up to ~0.1, which dS = P (dP - Dr) amplifies
  // where one key dominates the row.  For these items Dr is taken from the identity rowsum(dO * O) = sum_j P_j dP_j
  // instead, in fp32 from the one tile the row has, normalised by sum_j P_j (P carries the rounding of the stored LSE).
  if (ntiles == 1) {
    __shared__ float drx[4][64];
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    float num = 0.f, den = 0.f;
    f32x16 sacc = zero16(), dpacc = zero16();
#pragma unroll
    for (int ks = 0; ks < NOP; ++ks) op[ks] = ld_row(ks, 0);
#pragma unroll
    for (int ks = 0; ks < NOP; ++ks) sacc = mfma32(op[ks], qf[ks], sacc);
#pragma unroll
    for (int ks = 0; ks < NOP; ++ks) op[ks] = ld_row(ks, TILE_B);
#pragma unroll
    for (int ks = 0; ks < NOP; ++ks) dpacc = mfma32(op[ks], dof[ks], dpacc);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const bool masked = 32 * kh + c_row(v, hf) > qloc;  // the tile is the diagonal block
      const float pv = masked ? 0.f : fast_exp2(__builtin_fmaf(sacc[v], P.scale_log2e, -lse2));
      num = __builtin_fmaf(pv, dpacc[v], num);
      den += pv;
    }
    num += __shfl_xor(num, 32, 64);
    den += __shfl_xor(den, 32, 64);
    if (hf == 0) { drx[wave][l32] = num; drx[wave][32 + l32] = den; }
    __syncthreads();  // the other key half of the row is with wavefront wave ^ 2
    num += drx[wave ^ 2][l32];
    den += drx[wave ^ 2][32 + l32];
    if (den > 0.f) dr = num / den;
  }
  if (qvalid && kh == 0 && hf == 0) {
    P.drow[(int64_t)h * P.T + tq] = dr;
    P.lse2[(int64_t)h * P.T + tq] = lse2;
  }

  f32x16 dqacc[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) dqacc[dt] = zero16();

  // The diagonal block is always the last tile of a row: it takes its own instantiation of the tile
  // body, so that the other tiles carry no mask selects.
  auto tile = [&](auto diag_c, auto buf_c, int t) __attribute__((always_inline)) {
    constexpr bool diag = decltype(diag_c)::value;
    constexpr unsigned BO = decltype(buf_c)::value * 2 * TILE_B;  // the tile's buffer is an immediate offset of every LDS read
    const bool more = t + 1 < ntiles;
    if (more && (t + 1) % kJ == 0) stage_indices(t + 1);
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();  // tile t has landed for everyone; everyone is done with tile t-1
    if (more) issue(t + 1);
#pragma unroll
    for (int ks = 0; ks < NOP; ++ks) op[ks] = ld_row(ks, BO);  // K rows
    __builtin_amdgcn_sched_barrier(0);
    f32x16 sacc = zero16(), dpacc = zero16();
#pragma unroll
    for (int ks = 0; ks < NOP; ++ks) {  // S^T = K Q^T, refilling every operand register with the V row operand
      sacc = mfma32(op[ks], qf[ks], sacc);
      op[ks] = ld_row(ks, BO + TILE_B);
    }
#pragma unroll
    for (int i_ = 0; i_ < NOP; ++i_) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < NOP; ++ks) {  // dP^T = V dO^T, refilling with the K^T operands of the dQ step
      dpacc = mfma32(op[ks], dof[ks], dpacc);
      op[ks] = ld_tr(ks / (D / 32), ks % (D / 32), BO);
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
        if (32 * kh + c_row(v, hf) > qloc) sacc[v] = -__builtin_inff();
    }
    bf16x8 dsb[2];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float pv = fast_exp2(__builtin_fmaf(sacc[v], P.scale_log2e, -lse2));
      dsb[v >> 3][v & 7] = (bf16)(pv * (dpacc[v] - dr));
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt) dqacc[dt] = mfma32(op[q * (D / 32) + dt], dsb[q], dqacc[dt]);
    // the matrix instructions of the first 16 keys run under the pointwise work of the other 16
    __builtin_amdgcn_sched_group_barrier(0x002, 40, 0);
#pragma unroll
    for (int i_ = 0; i_ < D / 32; ++i_) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 40 / (D / 32), 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, D / 32, 0);
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
  {  // add the two key halves of every row: the kh = 1 wavefront hands its partial over
    float* xbuf = (float*)&tiles[0][0][0] + (size_t)strip * (16 * (D / 32) * 64);
    __syncthreads();  // everyone is done with the tile buffers
    if (kh == 1) {
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) xbuf[(16 * dt + v) * 64 + lane] = dqacc[dt][v];
    }
    __syncthreads();
    if (kh == 0) {
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) dqacc[dt][v] += xbuf[(16 * dt + v) * 64 + lane];
    }
  }
  if (qvalid && kh == 0) {
    const int64_t obase = (tq * P.Hq + h) * D;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int vg = 0; vg < 4; ++vg) {
        const int d0 = 32 * dt + 8 * vg + 4 * hf;
        float x0 = dqacc[dt][4 * vg] * P.scale, x1 = dqacc[dt][4 * vg + 1] * P.scale, x2 = dqacc[dt][4 * vg + 2] * P.scale,
              x3 = dqacc[dt][4 * vg + 3] * P.scale;
        if (OUT_F32) {
          *(float4*)((float*)P.dq + obase + d0) = make_float4(x0, x1, x2, x3);
        } else {
          bf16x4 y;
          y[0] = (bf16)x0; y[1] = (bf16)x1; y[2] = (bf16)x2; y[3] = (bf16)x3;
          *(bf16x4*)((bf16*)P.dq + obase + d0) = y;
        }
      }
  }
  timer.stop(P);
}

// ---------------------------------------------------------------------------------------------
// The same by one or two wavefronts as in the forward kernel (NW, StripWalk; see one_wavefront_per_item): a wavefront owns all 64 query rows and walks 32-key strips, so that an operand read from LDS feeds two matrix
// instructions (with 32 rows per wavefront LDS reads take as long as the matrix instructions); it stages its own strips of K and V, two
// of each, without any barrier in the loop.  At D = 128 it needs the registers of a whole SIMD, so the loop is a software pipeline over
// half tiles u (32 keys x 32 queries), stages of D/16 matrix instructions:
//   S(u), dP(u), dQ(u-1)
// with P(u) beside dP(u) and dQ(u-1), and dS(u) beside dQ(u-1) and the next S; every matrix instruction is fenced with its share of
// the vector work and LDS reads, and nothing waits for a result of the stage before.
// The item's descriptor comes by scalar loads and no load is behind a branch (rows and strips that do not exist are loaded as copies of
// the last row and as zeros), so that addresses and counts are scalar work and the loop is one block; one wait for all of LDS stands
// where nothing is due, instead of one before each use, and a strip's eight loads take 16 scalar instructions: 43 in the two-tile loop,
// 119 before.  What bounds it now is the clock that the chip keeps under load (1.6 GHz, matrix cores busy 61 %) and, on long
// sequences, the gathers.  With branches and half the item / without them / and one wavefront per item: the 32768-token batch, 32/8 heads
// 2.44 / 2.23 / 2.14 ms, one 131072-token sequence, top 32: 7.62 / 7.24 / 6.49, the 262144-token batch 23.3 / 22.3 / 20.5, 65536 tokens
// whose selection is a sink and a window 2.66 / 2.42 / 2.19.  Where the heads of a KV group share their selection, against one workgroup
// of all of them that shares the tiles in LDS (32 rows per wavefront): the 32768-token batch 2.37 -> 2.09 ms, the 131072-token sequence
// 6.45 -> 5.82, 65536 tokens with 28/4 heads 5.75 -> 4.54.  At D = 64 two wavefronts share a SIMD (one to five registers spilled before the
// loop); against the kernel above on 65536 tokens, 14/2 heads, blocks of 256: 1.98 -> 1.77 ms, per KV group 2.45 -> 1.75.
template <int D> constexpr int kDqRing = 4 * 32 * D * 2;  // a wavefront's K even, K odd, V even, V odd strips

template <int D, bool OUT_F32, int NW, bool LOOP>
__device__ __attribute__((always_inline)) inline void dq_head_item(const AttnParams& P, const WorkItem& item, int hh, char (&ring)[NW][kDqRing<D>]) {
  constexpr int ROW_B = D * 2, STRIP_B = 32 * ROW_B, NOP = D / 16;
  using Loader = QuadLoader<D>;
  constexpr int LPS = Loader::LPS;
  constexpr int KV = D == 64 ? NOP : 6;  // Q, dQ and the dO operands below this one live in accumulation registers, the other dO operands do not fit there
  constexpr int PER = 8 / NOP;           // registers of the vector work per matrix instruction
  const int tid = item_tid<LOOP>();
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int hs = item.hs, i = item.i, L = item.len, ntiles = item.ntiles;
  const int64_t seq0 = item.seq0;
  const int h = P.mode == SB_SELECT_PER_QHEAD ? hs : hs * P.G + hh;
  const int g = P.mode == SB_SELECT_PER_QHEAD ? hs / P.G : hs;

  StripWalk<D, NW> walk;
  walk.init(item, P.idx, P.Hkv, wave, lane);
  const int nstrips = walk.nstrips;
  // B operands: column = query 32b + lane%32, slots = d 16ks + 8hf + (0..7)
  // (rows past the sequence's last repeat it and are not stored: a branch here would cost the loads' overlap)
  bf16x8 qf[2][NOP], dof[2][NOP];
  float lse2[2], dr[2];
  bool qvalid[2];
  int64_t tq[2];
  typedef typename std::conditional<OUT_F32, float, bf16>::type out_t;
  typedef out_t out8 __attribute__((ext_vector_type(8)));
  out8 ov[2][NOP];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int qloc = 32 * b + l32;
    qvalid[b] = i * 64 + qloc < L;
    tq[b] = seq0 + min(i * 64 + qloc, L - 1);
    const int64_t row = (tq[b] * P.Hq + h) * D + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < NOP; ++ks) qf[b][ks] = *(const bf16x8*)(P.q + row + 16 * ks);
#pragma unroll
    for (int ks = 0; ks < NOP; ++ks) dof[b][ks] = *(const bf16x8*)(P.d_o + row + 16 * ks);
#pragma unroll
    for (int ks = 0; ks < NOP; ++ks) ov[b][ks] = *(const out8*)((const out_t*)P.o + row + 16 * ks);
    lse2[b] = P.lse[(int64_t)h * P.T + tq[b]];
  }
  Loader loader;
  loader.init(P.Hkv, lane);
  // this wavefront's first strip of block 0
  const unsigned long long k0 = (unsigned long long)(P.k + ((seq0 + 32 * wave) * P.Hkv + g) * D);
  const unsigned long long v0 = (unsigned long long)(P.v + ((seq0 + 32 * wave) * P.Hkv + g) * D);
  const unsigned ring0 = lds_offset(&ring[wave][0]);
  unsigned long long off = walk.offset_of(0);  // of the newest strip requested
  unsigned bytes = walk.bytes_of(0);
  loader.issue(Loader::resource(v0 + off, bytes), ring0 + 2 * STRIP_B);
  loader.issue(Loader::resource(k0 + off, bytes), ring0);
  // the rows' operands must have landed before the loop, which waits for strips by count; here the wait is for the first strips as well
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    lse2[b] *= 1.4426950408889634f;
    float part = 0.f;  // Dr: the lane's half of the head dimension, the other half is in lane ^ 32
#pragma unroll
    for (int ks = 0; ks < NOP; ++ks)
#pragma unroll
      for (int e = 0; e < 8; ++e) part += (float)dof[b][ks][e] * (float)ov[b][ks][e];
    dr[b] = part + __shfl_xor(part, 32, 64);
  }
#pragma unroll
  for (int b = 0; b < 2; ++b) {
#pragma unroll
    for (int ks = 0; ks < NOP; ++ks) {
      asm volatile("" : "+a"(qf[b][ks]));
      if (ks < KV) asm volatile("" : "+a"(dof[b][ks]));
      else asm volatile("" : "+v"(dof[b][ks]));
    }
    asm volatile("" : "+v"(lse2[b]), "+v"(dr[b]));
  }
  wait_vmcnt<0>();
  off = walk.offset_of(1);
  bytes = walk.bytes_of(1);
  loader.issue(Loader::resource(v0 + off, bytes), ring0 + 3 * STRIP_B);
  loader.issue(Loader::resource(k0 + off, bytes), ring0 + STRIP_B);

  // LDS byte addresses of this lane's operand reads in the wavefront's first slot
  unsigned row_a[NOP], tr_a[D / 32][2];
#pragma unroll
  for (int ks = 0; ks < NOP; ++ks) row_a[ks] = ring0 + l32 * ROW_B + 16 * ((2 * ks + hf) ^ chunk_swizzle<D>(l32));
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int r = 8 * half + 4 * hf + ((lane & 15) >> 2), d = 32 * dt + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      tr_a[dt][half] = ring0 + r * ROW_B + 16 * ((d >> 3) ^ chunk_swizzle<D>(r)) + 2 * (d & 7);
    }
  auto ld_row = [&](int ks, unsigned off) __attribute__((always_inline)) {
    return *(const bf16x8 __attribute__((address_space(3)))*)(row_a[ks] + off);
  };
  // A operand x = kk * 4 + dt of dQ^T += K^T dS^T: row = d (32dt + lane%32), slots = keys 16kk + 8(e/4) + 4hf + e%4
  auto ld_tr = [&](int x, unsigned off) __attribute__((always_inline)) {
    const int kk = x / (D / 32), dt = x % (D / 32);
    const unsigned o = off + kk * 16 * ROW_B;
    bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)(tr_a[dt][0] + o));
    bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)(tr_a[dt][1] + o));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  bf16x8 ka[NOP], va[NOP], kt[NOP];
  f32x16 sacc[2], dpacc;
  bf16x8 dsb[2][2];
  f32x16 dqacc[D / 32][2];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) dqacc[dt][0] = dqacc[dt][1] = zero16();
#pragma unroll
  for (int k = 0; k < NOP; ++k) kt[k] = zero_bf16x8();
#pragma unroll
  for (int k = 0; k < NOP; ++k) { ka[k] = ld_row(k, 0); va[k] = ld_row(k, 2 * STRIP_B); }

  // P = exp2(S c - lse2) of register v of query half b, in place; in a strip of the diagonal tile (first key: key0) 0 above the diagonal
  auto prob = [&](auto diag_c, int key0, int b, int v) __attribute__((always_inline)) {
    float pv = fast_exp2(__builtin_fmaf(sacc[b][v], P.scale_log2e, -lse2[b]));
    if (decltype(diag_c)::value && key0 + c_row(v, hf) > 32 * b + l32) pv = 0.f;
    sacc[b][v] = pv;
  };
  float ds_even;
  auto dscore = [&](int b, int v) __attribute__((always_inline)) {  // dS = P (dP - Dr), to bf16 in pairs
    const float x = sacc[b][v] * (dpacc[v] - dr[b]);
    if ((v & 1) == 0) { ds_even = x; return; }
    dsb[b][v >> 3][(v & 7) - 1] = (bf16)ds_even;
    dsb[b][v >> 3][v & 7] = (bf16)x;
  };
  // Dr of a row that keeps only its own block comes from sum_j P_j dP_j / sum_j P_j, as in the kernel above
  if (ntiles == 1) {
    __shared__ float drx[NW][2][64];  // [wavefront][query half][sums, normalisers]
    float num[2] = {0.f, 0.f}, den[2] = {0.f, 0.f};
    if (NW == 1) wait_vmcnt<0>();
#pragma unroll
    for (int strip = 0; strip < 3 - NW; ++strip) {  // this wavefront's strips of the row's only tile
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        f32x16 s_ = zero16(), dp = zero16();
#pragma unroll
        for (int k = 0; k < NOP; ++k) s_ = mfma32(strip == 0 ? ka[k] : ld_row(k, STRIP_B), qf[b][k], s_);
#pragma unroll
        for (int k = 0; k < NOP; ++k) dp = mfma32(strip == 0 ? va[k] : ld_row(k, 3 * STRIP_B), dof[b][k], dp);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const bool masked = 32 * (wave + strip) + c_row(v, hf) > 32 * b + l32;
          const float pv = masked ? 0.f : fast_exp2(__builtin_fmaf(s_[v], P.scale_log2e, -lse2[b]));
          num[b] = __builtin_fmaf(pv, dp[v], num[b]);
          den[b] += pv;
        }
      }
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      num[b] += __shfl_xor(num[b], 32, 64);
      den[b] += __shfl_xor(den[b], 32, 64);
      if (NW == 2 && hf == 0) { drx[wave][b][l32] = num[b]; drx[wave][b][32 + l32] = den[b]; }
    }
    if constexpr (NW == 2) {
      __syncthreads();
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        num[b] += drx[wave ^ 1][b][l32];
        den[b] += drx[wave ^ 1][b][32 + l32];
      }
    }
#pragma unroll
    for (int b = 0; b < 2; ++b)
      if (den[b] > 0.f) dr[b] = num[b] / den[b];
  }

#define SB_FENCE() __builtin_amdgcn_sched_barrier(0)
  // half tile u = (strip t, query half B); PAR = t % 2, known at compile time but for the last strip with NW = 2.  DIAG, LAST, and what the
  // last strip's query half 0 does not see with NW = 1: as in the forward kernel.
  auto half_tile = [&](auto diag_c, auto last_c, auto PAR, auto b_c, int t) __attribute__((always_inline)) {
    constexpr int B = decltype(b_c)::value;
    constexpr bool LAST = decltype(last_c)::value;
    constexpr bool SEEN = !(LAST && NW == 1 && B == 0);  // u has visible keys
    constexpr bool PREV = !(LAST && NW == 1 && B == 1);  // u - 1 has
    const int key0 = NW == 2 ? 32 * wave : LAST ? 32 : 0;
#pragma unroll
    for (int k = 0; k < NOP; ++k) {
      asm volatile("" : "+a"(qf[B][k]));
      if (k < KV) asm volatile("" : "+a"(dof[B][k]));
      else asm volatile("" : "+v"(dof[B][k]));
    }
    // strips t + 2 follow: V with B = 0, into the slot of V_t, whose operands are in va; K with B = 1, into the slot of K_t, likewise in kt
    i32x4 rsrc;
    unsigned slot = 0;
    if constexpr (!LAST) {
      if (B == 0) {
        off = walk.offset_of(t + 2);
        bytes = walk.bytes_of(t + 2);
      }
      rsrc = Loader::resource((B == 0 ? v0 : k0) + off, bytes);
      slot = ring0 + ((B == 0 ? 2 : 0) + PAR) * STRIP_B;
    }
    SB_FENCE();
    // One wait for all of LDS where nothing is due soon, instead of one before each use.  B = 0: K_t and V_t are in ka and va, and slot
    // V_t is free.
    if (B == 0) __builtin_amdgcn_s_waitcnt(0xC07F);
    SB_FENCE();
#pragma unroll
    for (int k = 0; k < NOP; ++k) {
      if (SEEN) {
        if (k == 0) mfma32_first(sacc[B], ka[k], qf[B][k]);
        else mfma32_more(sacc[B], ka[k], qf[B][k]);
      }
      if (PREV) {  // (before the row's first half tile: zeros)
#pragma unroll
        for (int a = 0; a < PER; ++a) dscore(B ^ 1, 8 + PER * k + a);
      }
      if (B == 1 && !LAST) {
        if (k == 1) {
          __builtin_amdgcn_s_waitcnt(0xC07F);  // K_t is in kt, its slot is free
          wait_vmcnt<LPS>();                   // strips t + 1 have landed (V_{t+2} may still be on its way)
          ka[0] = ld_row(0, (PAR ^ 1) * STRIP_B);
        }
        if (k >= 1) ka[k] = ld_row(k, (PAR ^ 1) * STRIP_B);
      }
      SB_FENCE();
      if constexpr (!LAST) {
        if (k == 2) loader.template issue2<0>(rsrc, slot);
        if constexpr (D == 128) { if (k == 5) loader.template issue2<2>(rsrc, slot); }
      }
      SB_FENCE();
    }
#pragma unroll
    for (int k = 0; k < NOP; ++k) {
      if (SEEN) {
        if (k == 0) mfma32_first(dpacc, va[k], dof[B][k]);
        else if (k < KV) mfma32_more(dpacc, va[k], dof[B][k]);
        else mfma32_more_v(dpacc, va[k], dof[B][k]);
      }
      if (B == 1 && !LAST) va[k] = ld_row(k, (2 + (PAR ^ 1)) * STRIP_B);
      // (two matrix instructions after the last of S before its first reader, see mfma32_first: of the two at D = 64 the compiler would put
      // the reader ahead of the second)
      if (D == 64 && k == NOP / 4) SB_FENCE();
      if (SEEN && k >= NOP / 4) {  // 0 .. 5
#pragma unroll
        for (int a = 0; a < PER; ++a) prob(diag_c, key0, B, PER * (k - NOP / 4) + a);
      }
      SB_FENCE();
      if constexpr (!LAST) {
        if constexpr (D == 128) {
          if (k == 1) loader.template issue2<4>(rsrc, slot);
          if (k == 5) loader.template issue2<6>(rsrc, slot);
        } else {
          if (k == 1) loader.template issue2<2>(rsrc, slot);
        }
      }
      SB_FENCE();
    }
    if (!PREV) asm volatile("s_nop 7\n\ts_nop 7" : "+v"(dpacc));  // (no matrix instructions between dP(u) and its first reader)
#pragma unroll
    for (int k = 0; k < NOP; ++k) {
      if (PREV) mfma32_sum(dqacc[k % (D / 32)][B ^ 1], kt[k], dsb[B ^ 1][k / (D / 32)]);
      if (B == 0) kt[k] = ld_tr(k, PAR * STRIP_B);
      if (SEEN) {
        constexpr int P128[9] = {6, 8, 10, 11, 12, 13, 14, 15, 16}, P64[5] = {6, 9, 12, 14, 16};
#pragma unroll
        for (int v = D == 64 ? P64[k % 4] : P128[k]; v < (D == 64 ? P64[k % 4 + 1] : P128[k + 1]); ++v) prob(diag_c, key0, B, v);
        if (k >= NOP / 2) {  // (two matrix instructions after the last of dP at the least)
#pragma unroll
          for (int v = 0; v < 2 * PER; ++v) dscore(B, 2 * PER * (k - NOP / 2) + v);
        }
      }
      SB_FENCE();
    }
    // (the conversions stay where they are: the compiler would carry the floats over the loop's edge and convert them one by one)
    asm volatile("" : "+v"(dsb[B][0]), "+v"(dsb[B ^ 1][1]));
  };
  using std::integral_constant;
  using std::false_type;
  using std::true_type;
  using I0 = integral_constant<int, 0>;
  using I1 = integral_constant<int, 1>;
  {
    // nothing precedes the first half tile: its dQ stage adds zeros
    sacc[1] = zero16();
    dpacc = zero16();
#pragma unroll
    for (int q = 0; q < 2; ++q) dsb[1][q] = zero_bf16x8();
    int t = 0;
    for (; t + 2 < nstrips; t += 2) {
      walk.window(t, 3, lane);
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
    if constexpr (NW == 1) {
      half_tile(true_type(), true_type(), I1(), I0(), t);
      half_tile(true_type(), true_type(), I1(), I1(), t);
    } else {
      half_tile(true_type(), true_type(), t & 1, I0(), t);
      half_tile(true_type(), true_type(), t & 1, I1(), t);
    }
#pragma unroll
    for (int v = 8; v < 16; ++v) dscore(1, v);
    asm volatile("s_nop 3" : "+v"(dsb[1][0]), "+v"(dsb[1][1]));  // two wait states between a vector write and its use as an operand
#pragma unroll
    for (int k = 0; k < NOP; ++k) mfma32_sum(dqacc[k % (D / 32)][1], kt[k], dsb[1][k / (D / 32)]);
    // the compiler does not see these as matrix instructions: their results are read no sooner than this
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) asm volatile("s_nop 7\n\ts_nop 7" : "+a"(dqacc[dt][0]), "+a"(dqacc[dt][1]));
  }
#undef SB_FENCE
  wait_vmcnt<0>();  // the strips past the last tile
  // with two wavefronts the two key halves are added: wavefront w finishes query half w and hands the other half over
  float* xbuf = (float*)&ring[wave][0];
  const float* ybuf = (const float*)&ring[NW == 2 ? wave ^ 1 : 0][0];
  if constexpr (NW == 2) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
      if (b != wave) {
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
          for (int v = 0; v < 16; ++v) xbuf[(16 * dt + v) * 64 + lane] = dqacc[dt][b][v];
      }
    __syncthreads();
  }
#pragma unroll
  for (int b = 0; b < 2; ++b)
    if (NW == 1 || b == wave) {
      if (qvalid[b] && hf == 0) {
        P.drow[(int64_t)h * P.T + tq[b]] = dr[b];
        P.lse2[(int64_t)h * P.T + tq[b]] = lse2[b];
      }
      const int64_t first = seq0 + i * 64 + 32 * b;
      store_rows<D, OUT_F32>(&ring[wave][(NW == 1 ? 2 * b : 2) * STRIP_B], P.dq, (first * P.Hq + h) * D, (int64_t)P.Hq * D, min(32, L - i * 64 - 32 * b), lane,
                             [&](int dt, int v) __attribute__((always_inline)) {
                               return (NW == 1 ? dqacc[dt][b][v] : dqacc[dt][b][v] + ybuf[(16 * dt + v) * 64 + lane]) * P.scale;
                             });
    }
}

template <int D, bool OUT_F32, int NW, bool LOOP>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 64 ? 2 : 1))) void attn_bwd_dq_head_kernel(AttnParams P, int heads) {
  __shared__ __attribute__((aligned(1024))) char ring[NW][kDqRing<D>];
  BusyTimer timer;
  timer.start(P);
  for_items<D, NW, LOOP, !LOOP>(P, heads, (int*)&ring[NW - 1][kDqRing<D> - 4],
                [&](const AttnParams& p, const WorkItem& item, int hh) __attribute__((always_inline)) { dq_head_item<D, OUT_F32, NW, LOOP>(p, item, hh, ring); });
  timer.stop(P);
}

// ---------------------------------------------------------------------------------------------
// Key-major dK/dV kernel: 2 wavefronts, each owns 32 keys of key block (s, g, j) and keeps their
// K and V rows in registers for the whole launch.  The Q and dO tiles (plus the rows' log-sum-exp
// in base 2 and Dr) of the query blocks that kept j are double-buffered in LDS by asynchronous
// loads; both are read row-wise (S = Q K^T, dP = dO V^T) and through the transposing LDS read
// (dV += P^T dO, dK += dS^T Q).
// The column's tiles are visited query block by query block, from the sequence's last query block
// down to the diagonal, all query heads of the KV group at one query block before the next:
// concurrent columns of one KV head (same XCD) start at the same query block, advance at a similar
// pace and so ask for the same Q/dO tiles at about the same time and meet them in that XCD's L2.
// What bounds it: one wavefront per SIMD (it needs more than 256 registers), so every wait is idle time of the matrix cores, and
// under matrix load the chip runs at 1.5 - 1.75 GHz of its 2.4.  Hence the software pipeline over half tiles (32 queries) below:
// every matrix instruction carries the same share of vector work and LDS reads, fenced step by step, results are used two
// stages after they were started, and the tile loads are issued two at a time between matrix instructions instead of 17 in a
// row.  The scores are kept out of the accumulation registers (mfma32_first).  32768-token batch, 32/8 heads, D = 128:
// 3.66 -> 3.24 ms (matrix cores busy 48 -> 57 % of the cycles), the 262144-token batch, whose gathers come through the fabric at
// 6 TB/s: 36.7 -> 34.9 ms.  A scalar instruction takes as long to issue as a vector one here: with a half tile's two resources put
// together once from the tile's addresses, instead of before every pair of loads (50 scalar instructions a tile, before: 110), 3.25 ->
// 3.06 and 35.8 -> 34.3 ms.  A tile that is not one of a pair of unmasked ones takes the masked form, its mask
// moved out of the way where there is nothing to mask: with a form for each the code was a quarter longer and 16 vector and 176 scalar
// registers were spilled around the loop, now 39 scalar ones (2039 tokens in short sequences 31.9 -> 30.9 us, long columns the same).
// One wait per half stage for its LDS operands, instead of one before each matrix instruction: the same time.
// D = 64 needs half the registers: there two wavefronts share a SIMD instead, with a shorter pipeline that fits 256 of them, and the
// shorter tile list (8 bitmap words per chunk) lets four workgroups share a CU's LDS.  Matrix cores busy 34 -> 48 % with half tiles computed
// from start to end, at a clock that the chip lowers from 1.86 to 1.62 GHz for it; with the pipeline 65536 tokens, 14/2 heads, selection
// blocks of 256: 2.92 -> 2.69 ms.
template <int D, bool OUT_F32>
__global__ __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(D == 64 ? 2 : 1))) void attn_bwd_dkv_kernel(AttnParams P) {
  constexpr int TILE_B = 64 * D * 2;  // bytes of one Q or dO tile
  constexpr int BUF_B = 2 * TILE_B;   // bytes of one buffer (Q tile, dO tile)
  constexpr int ROW_B = D * 2;
  __shared__ __attribute__((aligned(1024))) bf16 tiles[2][2][64 * D];  // [buffer][Q, dO]
  __shared__ __attribute__((aligned(256))) float rowstat[4][2][64];    // [buffer, half][LSE * log2(e), Dr]: 32 rows each, the other 32 unused
  constexpr int kCW = D == 64 ? 8 : 16;  // bitmap words (32 query blocks each) handled per chunk
  __shared__ uint32_t bm_s[8][kCW];  // bitmap words of up to 8 selection heads
  __shared__ uint16_t tl_s[kCW * 32 * 8];  // the chunk's tiles in processing order
  __shared__ int ntl_s;
  // workgroups 0 .. sub_slots-1: the sub-parts; then one per item, for those that are walked as a whole
  int at = (int)blockIdx.x - P.sub_slots;
  if (P.ticket) {  // the list's second half by ticket (only where there are no sub-parts)
    const int n_items = P.counters[3] * P.Hkv, lead = key_lead(n_items);
    if (at >= n_items + (int)key_extra(n_items)) return;
    if (at >= lead) {
      __shared__ int sh_claim;
      if (threadIdx.x == 0) sh_claim = draw_item(at & 7, lead, n_items, P.ticket);
      __syncthreads();
      at = __builtin_amdgcn_readfirstlane(sh_claim);
      if (at < 0) return;
    }
  }
  const ColItem item = at < 0 ? P.sub_items[blockIdx.x].item : P.bwd_items[at];
  if (item.col < 0) return;  // the lists are padded to their largest possible length
  int nsub = 1, run0 = 0, run1 = item.weight;  // workgroups that walk the item; this one's run of its tiles in walk order
  if (at < 0) {
    const int sub = P.sub_items[blockIdx.x].sub;
    nsub = (item.weight + P.sub_weight - 1) / P.sub_weight;
    run0 = (int)((int64_t)item.weight * sub / nsub);
    run1 = (int)((int64_t)item.weight * (sub + 1) / nsub);
  } else if (P.sub_slots > 0 && P.sub_base[at] >= 0) {
    return;
  }
  BusyTimer timer;
  timer.start(P);
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  // item.col: g * NQB + global block index
  const int wlo = item.wrange & 0xffff, whi = item.wrange >> 16;  // bitmap words of the column this item covers
  const int g = (int)((unsigned)item.col / (unsigned)P.NQB);
  const int qbj = item.col - g * (int)P.NQB;
  const int s = P.qb_seq[qbj];
  const int j = qbj - P.qb_off[s];
  const int n = P.qb_off[s + 1] - P.qb_off[s];
  const int64_t seq0 = P.cu[s];
  const int L = P.cu[s + 1] - P.cu[s];
  const int kloc = wave * 32 + l32;
  const bool kvalid = j * 64 + kloc < L;
  const int64_t tk = seq0 + j * 64 + kloc;

  bf16x8 kf[D / 16], vf[D / 16];
  {
    const bf16* kp = P.k + (tk * P.Hkv + g) * D + 8 * hf;
    const bf16* vp = P.v + (tk * P.Hkv + g) * D + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
      kf[ks] = kvalid ? *(const bf16x8*)(kp + 16 * ks) : zero_bf16x8();
      vf[ks] = kvalid ? *(const bf16x8*)(vp + 16 * ks) : zero_bf16x8();
    }
  }
  f32x16 dkacc[D / 32], dvacc[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) { dkacc[dt] = zero16(); dvacc[dt] = zero16(); }

  // LDS byte addresses of this lane's operand reads inside buffer 0 (the buffer and everything else is an
  // offset: rows 16 apart share the swizzle)
  unsigned row_a[D / 16], tr_a[D / 32][2];
  const unsigned stat_a = lds_offset(&rowstat[0][0][0]) + 16 * hf;
  {
    const unsigned tiles0 = lds_offset(&tiles[0][0][0]);
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) row_a[ks] = tiles0 + l32 * ROW_B + 16 * ((2 * ks + hf) ^ chunk_swizzle<D>(l32));
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int r = 8 * half + 4 * hf + ((lane & 15) >> 2), d = 32 * dt + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
        tr_a[dt][half] = tiles0 + r * ROW_B + 16 * ((d >> 3) ^ chunk_swizzle<D>(r)) + 2 * (d & 7);
      }
  }
  auto lds16 = [](unsigned a) __attribute__((always_inline)) { return *(const bf16x8 __attribute__((address_space(3)))*)a; };
  auto lds_f4 = [](unsigned a) __attribute__((always_inline)) { return *(const f32x4 __attribute__((address_space(3)))*)a; };
  constexpr int NOP = D / 16;  // operands (and matrix instructions) per pipeline stage
  // A operand ks of S = Q K^T / dP = dO V^T: rows lane%32 of the half tile at byte offset `off`, d 16ks + 8hf + (0..7)
  auto ld_row = [&](int ks, unsigned off) __attribute__((always_inline)) { return lds16(row_a[ks] + off); };
  // B operand x = kk * D/32 + dt of dV += P^T dO / dK += dS^T Q: contraction slots = queries 16kk + 8(e/4) + 4hf + e%4 of the
  // half tile at byte offset `off`, column = d (32dt + lane%32), through the transposing read
  auto ld_tr = [&](int x, unsigned off) __attribute__((always_inline)) {
    const int kk = x / (D / 32), dt = x % (D / 32);
    const unsigned o = off + kk * 16 * ROW_B;
    bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)(tr_a[dt][0] + o));
    bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)(tr_a[dt][1] + o));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };

  // A half tile is 32 query rows: wavefront 0 loads its Q rows, wavefront 1 its dO rows, and each 32 of the rows' statistics
  // (wavefront 0 the LSE, wavefront 1 Dr).  Rows past the end of the sequence arrive as zeros: their P is 1 and their dS 0,
  // and both meet zero rows of dO and Q.
  using Loader = QuadLoader<D>;
  Loader loader;
  loader.init(P.Hq, lane);
  constexpr int kLoadsPerHalf = Loader::LPS + 1;  // asynchronous loads one wavefront issues per half tile
  const unsigned pitch = (unsigned)P.Hq * D * 2;
  const unsigned long long src0 = (unsigned long long)((wave == 0 ? P.q : P.d_o) + (seq0 * P.Hq + (int64_t)g * P.G) * D);
  const unsigned long long stat0 = (unsigned long long)((wave == 0 ? P.lse2 : P.drow) + (int64_t)g * P.G * P.T + seq0);
  const unsigned dst0 = lds_offset(tiles[0][wave]), sdst0 = lds_offset(rowstat[0][wave]);
  const int lane4 = 4 * lane;
  // Only the sequence's last query block, n - 1, can lack rows: bytes that exist of rows 32 half .. +31 and of their statistics.
  const int last_rows = L - (n - 1) * 64;
  const unsigned full_bytes = 31u * pitch + D * 2;
  const unsigned last_bytes[2] = {(unsigned)(min(last_rows, 32) - 1) * pitch + D * 2, last_rows > 32 ? (unsigned)(last_rows - 33) * pitch + D * 2 : 0u};
  const unsigned last_stat[2] = {4u * min(last_rows, 32), 4u * max(last_rows - 32, 0)};
  // where query block i, head sel of the group come from (wave-uniform), and of a half tile: where from and where to
  struct Tile { unsigned long long rows, stat; bool last; };
  auto tile_of = [&](int i, int sel) __attribute__((always_inline)) {
    Tile x;
    x.rows = src0 + (unsigned long long)(unsigned)i * (64u * pitch) + (unsigned)sel * (unsigned)(D * 2);
    x.stat = stat0 + (unsigned long long)(unsigned)sel * (4u * (unsigned)P.T) + (unsigned)i * 256u;
    x.last = i == n - 1;
    return x;
  };
  struct Half { i32x4 rows, stat; unsigned slot, stat_slot; };
  auto half_of = [&](int buf, int half, Tile x) __attribute__((always_inline)) {
    return Half{Loader::resource(x.rows + half * (32u * pitch), x.last ? last_bytes[half] : full_bytes),
                Loader::resource(x.stat + half * 128u, x.last ? last_stat[half] : 128u), dst0 + buf * BUF_B + half * 32 * ROW_B, sdst0 + (2 * buf + half) * 512};
  };
  auto issue_half = [&](Half x) __attribute__((always_inline)) {
    load_floats(x.stat_slot, x.stat, lane4);
    loader.issue(x.rows, x.slot);
  };

  constexpr int PH = D == 64 ? 1 : 2;      // half tiles of dP and of P as operands that are kept
  f32x16 sacc[2], dpacc[PH];  // [half]: scores, then (in place) probabilities; dP
  bf16x8 pa[PH][2], dsa[2];   // P [half][16 queries] and dS [16 queries] as operands
  bf16x8 op[NOP];  // one rotating operand set: a register is refilled for the next stage right after the matrix instruction that used it
  f32x4 st_l[2], st_d[2];    // LSE and Dr of the rows 8vg + 4hf + (0..3) of a half tile, vg even / odd
  auto ld_stat = [&](unsigned so, int vg) __attribute__((always_inline)) { return lds_f4(stat_a + so + 32 * vg); };
  // P = exp2(S c - lse2) of register v of a half tile (query row 32 half + 8(v/4) + 4hf + v%4), in place, and to bf16 in pairs;
  // once the last row of a group of four has been used, the statistics two groups on are fetched in its place
  auto prob = [&](auto diag_c, int key, int half, int v, unsigned so) __attribute__((always_inline)) {
    float pv = fast_exp2(__builtin_fmaf(sacc[half][v], P.scale_log2e, -st_l[(v >> 2) & 1][v & 3]));
    if (decltype(diag_c)::value && key > 32 * half + c_row(v, hf)) pv = 0.f;  // causal mask inside the diagonal tile
    sacc[half][v] = pv;
    if (v & 1) {
      pa[half % PH][v >> 3][(v & 7) - 1] = (bf16)sacc[half][v - 1];
      pa[half % PH][v >> 3][v & 7] = (bf16)pv;
    }
    if ((v & 3) == 3 && v < 8) st_l[(v >> 2) & 1] = ld_stat(so, (v >> 2) + 2);
  };
  auto dscore = [&](int half, int v, unsigned so) __attribute__((always_inline)) {  // dS = P (dP - Dr), likewise
    f32x16& dp = dpacc[half % PH];
    dp[v] = sacc[half][v] * (dp[v] - st_d[(v >> 2) & 1][v & 3]);
    if (v & 1) {
      dsa[v >> 3][(v & 7) - 1] = (bf16)dp[v - 1];
      dsa[v >> 3][v & 7] = (bf16)dp[v];
    }
    if ((v & 3) == 3 && v < 8) st_d[(v >> 2) & 1] = ld_stat(so + 256, (v >> 2) + 2);
  };

  const int words = (n + 31) >> 5;
  const bool per_qhead = P.mode == SB_SELECT_PER_QHEAD;
  const int nsel = per_qhead ? P.G : 1;      // bitmap columns (selection heads) of this KV head
  const int hpe = per_qhead ? 1 : P.G;       // query heads each set bit stands for
  int walked = 0;                            // tiles of the item before the current chunk
  for (int sel0 = 0; sel0 < nsel; sel0 += 8) {                  // selection heads in groups of 8
    const int ns8 = min(8, nsel - sel0);
    for (int wend = whi, w0; wend > wlo; wend = w0) {  // chunks of up to kCW bitmap words, last first
      w0 = max(wlo, wend - kCW);
      const int wn = wend - w0;
      // ---- the chunk's tile list: entry = (query block - 32 w0) * 8 + head, ordered by query block, then head.
      // The list is walked backwards (last query block first): every column of a sequence then starts at
      // the same query block and, selecting at a similar density, stays close to its neighbours.
      __syncthreads();
      for (int a = tid; a < ns8 * kCW; a += 128) {
        const int sel = a / kCW, w = a % kCW;
        const int hs = per_qhead ? g * P.G + sel0 + sel : g;
        bm_s[sel][w] = w < wn ? P.bitmap[(int64_t)P.Hs * P.bm_off[s] + ((int64_t)hs * n + j) * words + w0 + w] : 0u;
      }
      __syncthreads();
      if (tid < 64) {  // lane w counts the tiles of word w, a wavefront scan turns counts into list positions
        int cnt = 0;
        if (tid < kCW)
          for (int sel = 0; sel < ns8; ++sel) cnt += __builtin_popcount(bm_s[sel][tid]) * hpe;
        int incl = cnt;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const int up = __shfl_up(incl, off, 64);
          if (tid >= off) incl += up;
        }
        if (tid == 63) ntl_s = incl;
        int pos = incl - cnt;
        if (tid < kCW && cnt > 0) {
          uint32_t any = 0;
          for (int sel = 0; sel < ns8; ++sel) any |= bm_s[sel][tid];
          while (any) {
            const int b = __builtin_ctz(any);
            any &= any - 1;
            if (per_qhead) {
              for (int sel = 0; sel < ns8; ++sel)
                if ((bm_s[sel][tid] >> b) & 1u) tl_s[pos++] = (uint16_t)((32 * tid + b) * 8 + sel);
            } else {
              for (int hh = 0; hh < hpe; ++hh) tl_s[pos++] = (uint16_t)((32 * tid + b) * 8 + hh);
            }
          }
        }
      }
      __syncthreads();
      const int nall = __builtin_amdgcn_readfirstlane(ntl_s);
      // the part of the chunk's tiles that lies in this workgroup's run
      const int lo = max(run0 - walked, 0), ntl = min(run1 - walked, nall) - lo;
      walked += nall;
      if (ntl <= 0) continue;
      // the diagonal tiles (query block j itself) are the first of the list, i.e. the last to be processed: count them
      int nd = 0;
      if (j >= 32 * w0 && j < 32 * (w0 + wn)) {
        for (int sel = 0; sel < ns8; ++sel) nd += (int)((bm_s[sel][(j >> 5) - w0] >> (j & 31)) & 1u) * hpe;
        nd = __builtin_amdgcn_readfirstlane(nd);
        nd = max(lo + ntl - max(lo, nall - nd), 0);
      }
      const uint16_t* const list = tl_s + (nall - 1 - lo);  // tile t of the run is list[-t]
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks) {
        if constexpr (D == 64) asm volatile("" : "+v"(kf[ks]), "+v"(vf[ks]));
        else asm volatile("" : "+a"(kf[ks]), "+a"(vf[ks]));
      }
      auto tile_from = [&](int e) __attribute__((always_inline)) { return tile_of(32 * w0 + (e >> 3), sel0 + (e & 7)); };
      auto entry = [&](int t) __attribute__((always_inline)) { return tile_from(__builtin_amdgcn_readfirstlane((int)list[-t])); };
      using H0 = std::integral_constant<int, 0>;
      using H1 = std::integral_constant<int, 1>;
      const int nn = ntl - nd;  // tiles without a mask
      if constexpr (D == 64) {
        // ---- D = 64: two wavefronts share a SIMD in 256 registers, which leaves no room for the longer pipeline below.  The stages
        //   S(u), dK(u-1), dP(u), dV(u)
        // of four matrix instructions need only the scores of two half tiles at a time: dS(u-1) goes beside S(u) and the start of
        // dK(u-1), P(u) beside the rest, dP(u) and the start of dV(u); every matrix instruction is fenced with its share, as below.  The
        // other wavefront of the SIMD fills what is left.  Half tile u-1 has been read when stage dV(u) begins: after a barrier its
        // buffer takes the loads of half tile u+3.
        Tile newest = entry(0);  // the newest tile that loads have been issued for
        issue_half(half_of(0, 0, newest));
        issue_half(half_of(0, 1, newest));
        newest = entry(min(1, ntl - 1));
        issue_half(half_of(1, 0, newest));
        wait_vmcnt<2 * kLoadsPerHalf>();
        __builtin_amdgcn_s_barrier();
#pragma unroll
        for (int k = 0; k < NOP; ++k) op[k] = ld_row(k, 0);
        auto half_tile = [&](auto first_c, auto last_c, auto diag_c, auto half_c, int buf, int t) __attribute__((always_inline)) {
          constexpr bool FIRST = decltype(first_c)::value, LAST = decltype(last_c)::value;
          constexpr int HALF = decltype(half_c)::value, PREV = 1 - HALF;
          const unsigned CO = buf * BUF_B + HALF * 32 * ROW_B;                                // half tile u
          const unsigned PO = (HALF ? buf : 1 - buf) * BUF_B + PREV * 32 * ROW_B;              // u - 1
          const unsigned NO = (HALF ? 1 - buf : buf) * BUF_B + PREV * 32 * ROW_B;              // u + 1
          const unsigned SO = (2 * buf + HALF) * 512, PSO = (HALF ? 2 * buf : 2 * (1 - buf) + 1) * 512;
          const int key = t < nn ? -1 : kloc;  // (no row lies before it: nothing is masked)
          int e2 = 0;
#define SB_FENCE() __builtin_amdgcn_sched_barrier(0)
          SB_FENCE();
          if (!LAST && HALF == 1) e2 = (int)list[-min(t + 2, ntl - 1)];
#pragma unroll
          for (int k = 0; k < NOP; ++k) {
            if (!LAST) sacc[HALF] = mfma32(op[k], kf[k], k == 0 ? zero16() : sacc[HALF]);
            if (!FIRST) {
              op[k] = ld_tr(k, PO);
#pragma unroll
              for (int e = 0; e < 3; ++e) dscore(PREV, 3 * k + e, PSO);
            } else {
              op[k] = ld_row(k, CO + TILE_B);
            }
            SB_FENCE();
          }
          if (!LAST) { st_l[0] = ld_stat(SO, 0); st_l[1] = ld_stat(SO, 1); }
          SB_FENCE();
#pragma unroll
          for (int k = 0; k < NOP; ++k) {
            if (!FIRST) {
              dkacc[k % (D / 32)] = mfma32(dsa[k / (D / 32)], op[k], dkacc[k % (D / 32)]);
              if (!LAST) op[k] = ld_row(k, CO + TILE_B);
              if (k == 0)
#pragma unroll
                for (int v = 12; v < 16; ++v) dscore(PREV, v, PSO);
            }
            if (!LAST && k > 0) { prob(diag_c, key, HALF, 2 * k - 2, SO); prob(diag_c, key, HALF, 2 * k - 1, SO); }
            SB_FENCE();
          }
          if constexpr (!LAST) {
#pragma unroll
            for (int k = 0; k < NOP; ++k) {
              dpacc[0] = mfma32(op[k], vf[k], k == 0 ? zero16() : dpacc[0]);
              op[k] = ld_tr(k, CO + TILE_B);
              prob(diag_c, key, HALF, 6 + 2 * k, SO);
              prob(diag_c, key, HALF, 7 + 2 * k, SO);
              SB_FENCE();
            }
            if (HALF == 1) newest = tile_from(__builtin_amdgcn_readfirstlane(e2));
            const Half nxt = half_of(HALF == 0 ? 1 - buf : buf, PREV, newest);
            // half tile u - 1 has been read by this wavefront and its part of u + 1 has landed
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
            wait_vmcnt<kLoadsPerHalf>();
            __builtin_amdgcn_s_barrier();
            st_d[0] = ld_stat(SO + 256, 0);
            st_d[1] = ld_stat(SO + 256, 1);
            load_floats(nxt.stat_slot, nxt.stat, lane4);
            SB_FENCE();
#pragma unroll
            for (int k = 0; k < NOP; ++k) {
              dvacc[k % (D / 32)] = mfma32(pa[0][k / (D / 32)], op[k], dvacc[k % (D / 32)]);
              op[k] = ld_row(k, NO);  // (after the last half tile of the chunk this reads a stale buffer and is not used)
              if (k == 0) { prob(diag_c, key, HALF, 14, SO); prob(diag_c, key, HALF, 15, SO); }
              SB_FENCE();
              if (k == 0) loader.template issue2<0>(nxt.rows, nxt.slot);
              if (k == 2) loader.template issue2<2>(nxt.rows, nxt.slot);
              SB_FENCE();
            }
          }
#undef SB_FENCE
        };
        {
          using std::true_type;
          using std::false_type;
          auto tile = [&](auto first_c, auto diag_c, int buf, int t) __attribute__((always_inline)) {
            half_tile(first_c, false_type(), diag_c, H0(), buf, t);
            half_tile(false_type(), false_type(), diag_c, H1(), buf, t);
          };
          // (the masked form for what is not a pair of unmasked tiles, as at D = 128: with a form for each 66 vector registers were spilled,
          // and a column of 16 tiles took 23.9 us, now 18.0; computed from start to end 21.0)
          int t = 1;
          tile(true_type(), true_type(), 0, 0);
          for (; t + 2 <= nn; t += 2) {
            tile(false_type(), false_type(), 1, t);
            tile(false_type(), false_type(), 0, t + 1);
          }
          for (; t < ntl; ++t) tile(false_type(), true_type(), t & 1, t);
          half_tile(false_type(), true_type(), false_type(), H0(), ntl & 1, ntl);
          wait_vmcnt<0>();  // the loads past the last tile
        }
      } else {
        // ---- software pipeline over half tiles u = 0, 1, ...: four stages of NOP matrix instructions each,
        //   S(u), dP(u), dV(u-1), dK(u-1)
        // with P(u) spread under the last two and dS(u-1) under the first two, so that every matrix instruction has the same
        // share of vector work beside it and nothing waits for a result of the stage before.  The operands of a stage are
        // fetched from LDS while the previous one computes.  Half tile u-1 has been read when stage dK(u-1) begins: after a
        // barrier its buffer takes the loads of half tile u+3, two at a time.
        Tile newest = entry(0);  // the newest tile that loads have been issued for
        issue_half(half_of(0, 0, newest));
        issue_half(half_of(0, 1, newest));
        newest = entry(min(1, ntl - 1));
        Half nxt = half_of(1, 0, newest);
        issue_half(nxt);
        wait_vmcnt<2 * kLoadsPerHalf>();
        __builtin_amdgcn_s_barrier();
#pragma unroll
        for (int ks = 0; ks < NOP; ++ks) op[ks] = ld_row(ks, 0);
        // one half tile: HALF of tile t, whose buffer is `buf`.  FIRST: nothing precedes it; LAST: there is no half tile u any
        // more, only dV and dK of u-1 are left.  Loads are issued past the chunk's last tile too (its last tile once more, never
        // read), so that their number in flight is the same everywhere.
        auto half_tile = [&](auto first_c, auto last_c, auto diag_c, auto half_c, int buf, int t) __attribute__((always_inline)) {
          constexpr bool FIRST = decltype(first_c)::value, LAST = decltype(last_c)::value;
          constexpr int HALF = decltype(half_c)::value, PREV = 1 - HALF, LPS = Loader::LPS;
          const unsigned CO = buf * BUF_B + HALF * 32 * ROW_B;                               // half tile u
          const unsigned PO = (HALF ? buf : 1 - buf) * BUF_B + PREV * 32 * ROW_B;             // u - 1
          const unsigned NO = (HALF ? 1 - buf : buf) * BUF_B + PREV * 32 * ROW_B;             // u + 1
          const unsigned SO = (2 * buf + HALF) * 512, PSO = (HALF ? 2 * buf : 2 * (1 - buf) + 1) * 512;
          const int key = t < nn ? -1 : kloc;  // (no row lies before it: nothing is masked)
          int e2 = 0;
          constexpr int EPS = 8 / NOP;  // rows (accumulator registers) of the pointwise work per matrix instruction
          // Every step is fenced: one matrix instruction, the refill of its operand, its share of the vector work.
#define SB_FENCE() __builtin_amdgcn_sched_barrier(0)
          SB_FENCE();
          if (!LAST && HALF == 1) e2 = (int)list[-min(t + 2, ntl - 1)];
#pragma unroll
          for (int k = 0; k < NOP; ++k) {
            if (!LAST) {
              if (k == 0) mfma32_first(sacc[HALF], op[k], kf[k]);
              else mfma32_more(sacc[HALF], op[k], kf[k]);
              op[k] = ld_row(k, CO + TILE_B);
            }
            if (!FIRST)
#pragma unroll
              for (int e = 0; e < EPS; ++e) dscore(PREV, EPS * k + e, PSO);
            SB_FENCE();
          }
          if constexpr (!FIRST && !LAST && LPS > 4) loader.template issue2<LPS - 4>(nxt.rows, nxt.slot);
          if (!LAST) { st_l[0] = ld_stat(SO, 0); st_l[1] = ld_stat(SO, 1); }
          SB_FENCE();
#pragma unroll
          for (int k = 0; k < NOP; ++k) {
            if (!LAST) {
              if (k == 0) mfma32_first(dpacc[HALF], op[k], vf[k]);
              else mfma32_more(dpacc[HALF], op[k], vf[k]);
            }
            if (!FIRST) {
              op[k] = ld_tr(k, PO + TILE_B);
#pragma unroll
              for (int e = 0; e < EPS; ++e) dscore(PREV, 8 + EPS * k + e, PSO);
            }
            SB_FENCE();
          }
          if constexpr (!FIRST && !LAST) loader.template issue2<LPS - 2>(nxt.rows, nxt.slot);
          SB_FENCE();
#pragma unroll
          for (int k = 0; k < NOP; ++k) {
            if (!FIRST) {
              dvacc[k % (D / 32)] = mfma32(pa[PREV][k / (D / 32)], op[k], dvacc[k % (D / 32)]);
              op[k] = ld_tr(k, PO);
            }
            if (!LAST)
#pragma unroll
              for (int e = 0; e < EPS; ++e) prob(diag_c, key, HALF, EPS * k + e, SO);
            if (!LAST && k == NOP / 2) {  // scalar work for the loads below, while matrix instructions run
              if (HALF == 1) newest = tile_from(__builtin_amdgcn_readfirstlane(e2));
              nxt = half_of(HALF == 0 ? 1 - buf : buf, PREV, newest);
            }
            SB_FENCE();
          }
          if (!LAST) {
            // half tile u - 1 has been read by this wavefront and its part of u + 1 has landed
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
            wait_vmcnt<kLoadsPerHalf>();
            __builtin_amdgcn_s_barrier();
            st_d[0] = ld_stat(SO + 256, 0);
            st_d[1] = ld_stat(SO + 256, 1);
            load_floats(nxt.stat_slot, nxt.stat, lane4);
            SB_FENCE();
          }
#pragma unroll
          for (int k = 0; k < NOP; ++k) {
            if (!FIRST) dkacc[k % (D / 32)] = mfma32(dsa[k / (D / 32)], op[k], dkacc[k % (D / 32)]);
            if (!LAST) {
              op[k] = ld_row(k, NO);  // (after the last half tile of the chunk this reads a stale buffer and is not used)
#pragma unroll
              for (int e = 0; e < EPS; ++e) prob(diag_c, key, HALF, 8 + EPS * k + e, SO);
            }
            SB_FENCE();
            if constexpr (!LAST) {
              if (k == 0) loader.template issue2<0>(nxt.rows, nxt.slot);
              if constexpr (LPS > 4) { if (k == NOP / 2) loader.template issue2<2>(nxt.rows, nxt.slot); }
              SB_FENCE();
            }
          }
#undef SB_FENCE
        };
        {
          using std::true_type;
          using std::false_type;
          auto tile = [&](auto first_c, auto diag_c, int buf, int t) __attribute__((always_inline)) {
            half_tile(first_c, false_type(), diag_c, H0(), buf, t);
            half_tile(false_type(), false_type(), diag_c, H1(), buf, t);
          };
          int t = 1;
          tile(true_type(), true_type(), 0, 0);
          for (; t + 2 <= nn; t += 2) {
            tile(false_type(), false_type(), 1, t);
            tile(false_type(), false_type(), 0, t + 1);
          }
          for (; t < ntl; ++t) tile(false_type(), true_type(), t & 1, t);
          half_tile(false_type(), true_type(), false_type(), H0(), ntl & 1, ntl);
          wait_vmcnt<0>();  // the loads past the last tile
        }
      }
    }
  }
  // C layout: column = d (32dt + l32), register v = key row c_row(v, hf) of this wavefront's strip
  if (item.slot >= 0 || nsub > 1) {  // a part of a split column, or of an item: leave the fp32 partial sums for the reduction
    float* part = nsub > 1 ? P.sub_partials + (size_t)blockIdx.x * (2 * 64 * D) : P.partials + (size_t)item.slot * (2 * 64 * D);
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int kr = wave * 32 + c_row(v, hf);
        part[kr * D + 32 * dt + l32] = dkacc[dt][v];
        part[(64 + kr) * D + 32 * dt + l32] = dvacc[dt][v];
      }
    timer.stop(P);
    return;
  }
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int kr = wave * 32 + c_row(v, hf);
      if (j * 64 + kr < L) {
        const int64_t off = ((seq0 + j * 64 + kr) * P.Hkv + g) * D + 32 * dt + l32;
        if (OUT_F32) {
          ((float*)P.dk)[off] = dkacc[dt][v] * P.scale;
          ((float*)P.dv)[off] = dvacc[dt][v];
        } else {
          ((bf16*)P.dk)[off] = (bf16)(dkacc[dt][v] * P.scale);
          ((bf16*)P.dv)[off] = (bf16)dvacc[dt][v];
        }
      }
    }
  timer.stop(P);
}

// dK/dV of the columns that more than one workgroup walked: the fp32 partial sums added in walk order (last query blocks first),
// then the scale and the rounding of the other columns.  Workgroups (x, y): x < extra: split column x; otherwise item x - extra,
// if it is a whole column walked in sub-parts.  y: 16 rows of the key block.
template <int D, bool OUT_F32>
__global__ __launch_bounds__(256) void attn_bwd_dkv_reduce_kernel(AttnParams P, int extra) {
  const int x = blockIdx.x;
  int64_t col;
  int slot0 = 0, np = 1, at = 0;
  if (x < extra) {
    if (x >= P.counters[1]) return;
    col = P.split_cols[3 * x];
    slot0 = P.split_cols[3 * x + 1];
    np = P.split_cols[3 * x + 2];
  } else {
    at = x - extra;
    const ColItem item = P.bwd_items[at];
    if (item.col < 0 || item.slot >= 0 || P.sub_base[at] < 0) return;
    col = item.col;
  }
  const int g = (int)(col / P.NQB);
  const int qbj = (int)(col - (int64_t)g * P.NQB);
  const int s = P.qb_seq[qbj];
  const int j = qbj - P.qb_off[s];
  const int64_t seq0 = P.cu[s];
  const int rows = min(64, P.cu[s + 1] - P.cu[s] - j * 64);
  constexpr int S = 2 * 64 * D;
  for (int u = threadIdx.x; u < 16 * D / 4; u += 256) {
    const int e = blockIdx.y * 16 * D + 4 * u;
    if (e >= rows * D) return;
    f32x4 dk = {0.f, 0.f, 0.f, 0.f}, dv = dk;
    // n partial sums, `stride` floats apart, in order; four of them in flight (one after the other a column of eleven waited eleven times:
    // 2039 tokens, 16/2 heads: 10.2 -> 7.5 us)
    auto add = [&](const float* part, int n, size_t stride) {
      int u = 0;
      for (; u + 4 <= n; u += 4) {
        f32x4 x[4], y[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          x[c] = *(const f32x4*)(part + (u + c) * stride + e);
          y[c] = *(const f32x4*)(part + (u + c) * stride + 64 * D + e);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) { dk += x[c]; dv += y[c]; }
      }
      for (; u < n; ++u) {
        dk += *(const f32x4*)(part + u * stride + e);
        dv += *(const f32x4*)(part + u * stride + 64 * D + e);
      }
    };
    if (P.sub_slots == 0) {
      add(P.partials + (size_t)slot0 * S, np, S);
    } else {
      for (int p = 0; p < np; ++p) {
        const int it = x < extra ? P.part_item[slot0 + p] : at;
        const int sub0 = P.sub_base[it];
        if (sub0 >= 0) add(P.sub_partials + ((size_t)sub0 * P.Hkv + g) * S, (P.bwd_items[it].weight + P.sub_weight - 1) / P.sub_weight, (size_t)P.Hkv * S);
        else add(P.partials + (size_t)(slot0 + p) * S, 1, S);
      }
    }
    const int kr = e / D, d = e % D;
    const int64_t off = ((seq0 + j * 64 + kr) * P.Hkv + g) * D + d;
    dk *= P.scale;
    if (OUT_F32) {
      *(f32x4*)((float*)P.dk + off) = dk;
      *(f32x4*)((float*)P.dv + off) = dv;
    } else {
      bf16x4 a, b;
#pragma unroll
      for (int c = 0; c < 4; ++c) { a[c] = (bf16)dk[c]; b[c] = (bf16)dv[c]; }
      *(bf16x4*)((bf16*)P.dk + off) = a;
      *(bf16x4*)((bf16*)P.dv + off) = b;
    }
  }
}

constexpr int64_t kDqFewItems = 2048;  // (items, query heads) below which D = 64 takes attn_bwd_dq_kernel: fewer than kTicketMinItems
static_assert(kDqFewItems <= kTicketMinItems, "attn_bwd_dq_kernel deals its items by position");

template <int D, bool F32>
static int launch_bwd(const Geo& g, const AttnParams& P, hipStream_t st) {
  // query-major dQ: one workgroup per (item, query head)
  const int heads = g.mode == SB_SELECT_PER_QHEAD ? 1 : g.G;
  const int64_t items = (int64_t)g.Hq * g.NQB;
  KernelTimer kt(K_BWD_DQ, st);
  if (D == 64 && items < kDqFewItems) {
    hipLaunchKernelGGL((attn_bwd_dq_kernel<F32>), dim3((unsigned)((P.n_items + 7) / 8 * 8), (unsigned)heads), dim3(256), 0, st, P);
  } else {
    if (head_ids(P.n_items, heads) > 0x7fffffffll) { set_error("too many work items for one launch"); return SB_ERR_INVALID_ARG; }
    const bool one = one_wavefront_per_item(g, items, 24);
    const dim3 grid((unsigned)head_grid(P, heads, one ? 1 : 2));
    auto launch = [&](auto nw, auto loop) {
      constexpr int NW = decltype(nw)::value;
      hipLaunchKernelGGL((attn_bwd_dq_head_kernel<D, F32, NW, decltype(loop)::value>), grid, dim3(64 * NW), 0, st, P, heads);
    };
    auto with_loop = [&](auto nw) {
      if constexpr (D == 128) {
        if (P.deal == kDealDraw) return launch(nw, std::true_type());
      }
      launch(nw, std::false_type());
    };
    if (one) with_loop(std::integral_constant<int, 1>()); else with_loop(std::integral_constant<int, 2>());
  }
  SB_LAUNCH_CHECK("attn_bwd_dq_kernel");
  return SB_OK;
}

template <int D, bool F32>
static int launch_dkv(const Geo& g, const AttnParams& P, hipStream_t st) {
  const int64_t extra = split_extra_max(g);
  const int64_t n_items = (int64_t)g.Hkv * (g.NQB + extra);
  if (P.sub_slots + n_items > 0x7fffffffll) { set_error("too many key-major items for one launch"); return SB_ERR_INVALID_ARG; }
  dim3 grid((unsigned)(P.sub_slots + n_items + (P.ticket ? key_extra(n_items) : 0))), block(128);
  KernelTimer kt(K_BWD_DKV, st);
  hipLaunchKernelGGL((attn_bwd_dkv_kernel<D, F32>), grid, block, 0, st, P);
  SB_LAUNCH_CHECK("attn_bwd_dkv_kernel");
  const int64_t reduced = extra + (P.sub_slots > 0 ? n_items : 0);
  if (reduced > 0) {  // at most that many columns are cut; workgroups beyond the actual count return at once
    hipLaunchKernelGGL((attn_bwd_dkv_reduce_kernel<D, F32>), dim3((unsigned)reduced, 4), dim3(256), 0, st, P, (int)extra);
    SB_LAUNCH_CHECK("attn_bwd_dkv_reduce_kernel");
  }
  return SB_OK;
}

}  // namespace sb

using namespace sb;

extern "C" int sb_sparse_attn_bwd(const sb_problem* p, const void* q, const void* k, const void* v, const void* o,
                                  const float* lse, const void* d_o, const int32_t* sel_rowptr, const int32_t* sel_idx,
                                  const void* plan, void* dq, void* dk, void* dv, void* ws, void* stream) {
  Geo gb;
  int rc = make_geo(p, &gb);
  if (rc != SB_OK) return rc;
  if (gb.S == 0 || gb.T == 0 || gb.NQB == 0) return SB_OK;
  const Geo g = tile_geo(gb);  // the kernels work on 64-row tiles; for larger selection blocks the plan holds the tile-level selection
  if (!q || !k || !v || !o || !lse || !d_o || !sel_rowptr || !sel_idx || !plan || !dq || !dk || !dv || !ws) {
    set_error("null argument");
    return SB_ERR_INVALID_ARG;
  }
  hipStream_t st = (hipStream_t)stream;
  PlanOffsets po = plan_offsets(gb);
  WsOffsets wo = bwd_ws_offsets(g);
  const char* pb = (const char*)plan;
  char* wb = (char*)ws;
  Tables t = make_tables(g, p, (void*)(pb + po.tables));
  AttnParams P{};
  const bool f32 = g.dtype == SB_F32;
  if (f32) {
    KernelTimer kt(K_BWD_PREP, st);  // float32 inputs only: the conversions to the kernels' operand type
    Conversions c{};
    c.add(q, wb + wo.qc, (int64_t)g.T * g.Hq * g.D);
    c.add(k, wb + wo.kc, (int64_t)g.T * g.Hkv * g.D);
    c.add(v, wb + wo.vc, (int64_t)g.T * g.Hkv * g.D);
    c.add(d_o, wb + wo.doc, (int64_t)g.T * g.Hq * g.D);
    if ((rc = convert_f32_to_bf16(c, st)) != SB_OK) return rc;
    P.q = (const bf16*)(wb + wo.qc); P.k = (const bf16*)(wb + wo.kc); P.v = (const bf16*)(wb + wo.vc);
    P.d_o = (const bf16*)(wb + wo.doc);
  } else {
    P.q = (const bf16*)q; P.k = (const bf16*)k; P.v = (const bf16*)v; P.d_o = (const bf16*)d_o;
  }
  float* drow = (float*)(wb + wo.drow);
  float* lse2 = (float*)(wb + wo.lse2);
  P.o = (void*)o; P.lse = (float*)lse; P.drow = drow; P.lse2 = lse2; P.dq = dq; P.dk = dk; P.dv = dv;
  P.idx = gb.r == 1 ? sel_idx : (const int32_t*)(pb + po.t_idx);
  P.items = (const WorkItem*)(pb + po.items);
  P.bitmap = (const uint32_t*)(pb + po.bitmap);
  P.bwd_items = (const ColItem*)(pb + po.bwd_items);
  P.split_cols = (const int32_t*)(pb + po.split_cols);
  P.counters = (const int32_t*)(pb + po.counters);
  P.partials = (float*)(wb + wo.partials);
  P.sub_base = (const int32_t*)(pb + po.sub_base);
  P.part_item = (const int32_t*)(pb + po.part_item);
  P.sub_partials = P.partials + 2 * (size_t)split_extra_max(g) * (2 * 64 * g.D);
  P.sub_items = (const SubItem*)(pb + po.sub_items);
  P.sub_slots = g.Hkv * sub_slots_max(g);
  P.sub_weight = sub_weight(g);
  P.cu = t.cu; P.qb_off = t.qb_off; P.qb_seq = t.qb_seq; P.bm_off = t.bm_off;
  P.NQB = g.NQB; P.T = g.T; P.Hq = g.Hq; P.Hkv = g.Hkv; P.G = g.G; P.Hs = g.Hs; P.mode = g.mode;
  P.scale = g.softmax_scale; P.scale_log2e = g.softmax_scale * 1.4426950408889634f;
  P.out_f32 = f32;
  P.cu_busy = nullptr;
  if (g_instrument & 1) {
    if ((rc = fill_zero(wb + wo.cu_busy, sizeof(uint64_t) * SB_CU_SLOTS, st)) != SB_OK) return rc;
    P.cu_busy = (unsigned long long*)(wb + wo.cu_busy);
  }
  const int heads = g.mode == SB_SELECT_PER_QHEAD ? 1 : g.G;
  const int64_t n_items = (int64_t)g.Hs * g.NQB;
  if (n_items > 0x3fffffffll) { set_error("too many work items for one launch"); return SB_ERR_INVALID_ARG; }
  P.n_items = (int)n_items;
  P.ticket = nullptr;
  AttnParams Pq = P;
  Pq.deal = dq_deal(g, n_items, heads);
  if (Pq.deal != kDealPosition) {
    Pq.ticket = (int*)(wb + wo.ticket);
    // (the sub-parts of small problems are dealt by position)
    if (P.sub_slots == 0 && use_key_tickets(g, (int64_t)g.Hkv * (g.NQB + split_extra_max(g)))) P.ticket = Pq.ticket + kTicketInts;
    if ((rc = fill_zero(Pq.ticket, sizeof(int32_t) * kTicketInts * 2, st)) != SB_OK) return rc;
  }
  if (g.D == 128) {
    rc = f32 ? launch_bwd<128, true>(g, Pq, st) : launch_bwd<128, false>(g, Pq, st);
    if (rc != SB_OK) return rc;
    rc = f32 ? launch_dkv<128, true>(g, P, st) : launch_dkv<128, false>(g, P, st);
  } else {
    rc = f32 ? launch_bwd<64, true>(g, Pq, st) : launch_bwd<64, false>(g, Pq, st);
    if (rc != SB_OK) return rc;
    rc = f32 ? launch_dkv<64, true>(g, P, st) : launch_dkv<64, false>(g, P, st);
  }
  return rc;
}
