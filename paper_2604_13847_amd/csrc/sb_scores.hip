// Routing scores (paper section 2.2, MoBA indexer): mean-pool the blocks of K and Q, then
// score = score_scale * <pooled Q block i, pooled K block j> for past blocks j < i.
// Pooling is HBM-bound (K and Q are read once); the score tiles run on the fp32 matrix cores and
// write the score matrix once.
#include "sb_geom.h"
#include "sb_internal.h"
#include "sb_score_tile.h"

namespace sb {

__device__ inline float bf16_bits_to_float(uint32_t b) { return __uint_as_float(b << 16); }

// Mean over the valid tokens of one block, for 8 (bf16) or 4 (float) adjacent columns per thread: 16-byte loads, eight
// rows in flight per thread.  grid = (NQB, column groups of Q, then column groups of K); X is [T][H*D]; out is [NQB][H*D] float.
// Q and K share a launch: the second one cost a small batch 4 us, and the K part alone fills only a fifth of the chip.
template <bool F32>
__global__ __launch_bounds__(256) void pool_kernel(const void* __restrict__ Q, const void* __restrict__ K, int qcols, int kcols, int qgroups,
                                                   GeomArgs ga, float* __restrict__ qbar, float* __restrict__ kbar) {
  constexpr int CPT = F32 ? 4 : 8;  // columns per thread
  const bool is_q = (int)blockIdx.y < qgroups;
  const void* __restrict__ X = is_q ? Q : K;
  float* __restrict__ out = is_q ? qbar : kbar;
  const int cols = is_q ? qcols : kcols;
  const int qb = blockIdx.x;
  const int c0 = (((int)blockIdx.y - (is_q ? 0 : qgroups)) * 256 + threadIdx.x) * CPT;
  const BatchGeom bg(ga);
  const int s = bg.seq_of(qb);
  const int j = qb - bg.get(s).qb0;
  if (c0 >= cols) return;
  const int L = ga.cu[s + 1] - ga.cu[s];
  const int first = j * ga.B, last = min((j + 1) * ga.B, L);
  const int64_t row0 = (int64_t)ga.cu[s] + first;
  float a[CPT];
#pragma unroll
  for (int e = 0; e < CPT; ++e) a[e] = 0.f;
  if (F32) {
    const float* p = (const float*)X + row0 * cols + c0;
#pragma unroll 8
    for (int r = 0; r < last - first; ++r) {
      float4 v = *(const float4*)(p + (int64_t)r * cols);
      a[0] += v.x; a[1] += v.y; a[2] += v.z; a[3] += v.w;
    }
  } else {
    const uint16_t* p = (const uint16_t*)X + row0 * cols + c0;
#pragma unroll 8
    for (int r = 0; r < last - first; ++r) {
      const uint4 v = *(const uint4*)(p + (int64_t)r * cols);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        a[2 * e] += bf16_bits_to_float(w[e] & 0xffffu);
        a[2 * e + 1] += bf16_bits_to_float(w[e] >> 16);
      }
    }
  }
  const float inv = 1.0f / (float)(last - first);
  float* o = out + (int64_t)qb * cols + c0;
#pragma unroll
  for (int e = 0; e < CPT; e += 4) *(float4*)(o + e) = make_float4(a[e] * inv, a[e + 1] * inv, a[e + 2] * inv, a[e + 3] * inv);
}

// Score tiles on the fp32 matrix cores (the selection is taken on fp32 scores, so the operands stay
// fp32).  One workgroup per (64 query blocks of one sequence, chunk of up to 2^kScChunkLog * 64 key
// blocks, selection head): each of the four wavefronts keeps 16 query rows in registers, straight from memory; the pooled key
// tiles are staged in LDS one after the other, and a wavefront computes the four 16 x 16 tiles of its rows in every 64 x 64 score
// tile, transposed, so that a lane holds four columns of a row and stores 16 bytes at once.  Tiles right of the diagonal are
// -infinity without being computed, and the last chunk of a row tile also fills every column to
// its right with -infinity, so that the whole n x n matrix is defined.  Splitting the columns over
// workgroups keeps the longest workgroup short however long the sequence is.
// What bounds it: the matrix takes 0.11 ms to write and 0.11 ms of the fp32 matrix cores (131072 tokens, 32 heads: 537 MB), and a
// workgroup waits between two barriers per tile, so it needs others beside it: with the query tile in LDS too two of them fitted a CU,
// without it four, at 128 registers, eight of them spilled (addresses, read back once a key tile): 0.306 -> 0.229 ms.
// A key tile takes a workgroup 2 us, so where four to a workgroup make fewer workgroups than the chip runs at once, each gets one
// (18889 tokens, 32/8 heads: 27 -> 21 us, 26565 tokens in several sequences, 16/2 heads: 22 -> 17); otherwise four, which share the query rows.
constexpr int kScChunkLog = 2;
constexpr int64_t kScFewWgs = 512;

// workgroups of a sequence with nt row tiles, 2^lg key tiles each: sum over it < nt of (it / 2^lg + 1)
__host__ __device__ inline int64_t score_items(int64_t nt, int lg) {
  const int64_t q = nt >> lg, r = nt & ((1 << lg) - 1);
  return ((q * (q + 1) / 2) << lg) + r * (q + 1);
}

template <int D, int lg>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void score_kernel(
    const float* __restrict__ qbar, const float* __restrict__ kbar, GeomArgs ga, int Hq, int Hkv, int Hs, int G, int mode, float scale,
    float* __restrict__ scores) {
  constexpr int chunk = 1 << lg;
  constexpr int LD = D + 4;  // padded row length (floats) of the LDS tile
  __shared__ float ks[64 * LD];
  const int tid = threadIdx.x;
  // (sequence, row tile, column chunk) of this workgroup
  const BatchGeom bg(ga);
  int64_t x = blockIdx.x;
  const int s = bg.locate(x, [](int n) { return score_items((n + 63) >> 6, lg); });
  if (s >= ga.S) return;
  // row tile `it` starts at item score_items(it), with it / chunk + 1 chunks: about sqrt(2 chunk x), then corrected
  int it = (int)sqrtf(2.f * chunk * (float)x);
  while (it > 0 && score_items(it, lg) > x) --it;
  while (score_items(it + 1, lg) <= x) ++it;
  const int jc = (int)(x - score_items(it, lg));
  const int hs = blockIdx.y;
  const SeqGeom sg = bg.get(s);
  const int n = sg.n;
  const int64_t qb0 = sg.qb0;
  float* out = scores + (int64_t)Hs * sg.sc_off + (int64_t)hs * n * n;
  const int i0 = it * 64;
  const int rows = min(64, n - i0);
  const int heads = mode == SB_SELECT_PER_QHEAD ? 1 : G;
  const int h0 = mode == SB_SELECT_PER_QHEAD ? hs : hs * G;
  const int g = h0 / G;
  const int wave = tid >> 6, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
  const float ninf = -__builtin_inff();
  // This lane's quarter of query row 16 * wave + l16, summed over the group's heads in per-KV-group mode.  Rows past the end repeat the
  // last one; their results are dropped.
  float a[D / 4];
#pragma unroll
  for (int t = 0; t < D / 4; ++t) a[t] = 0.f;
  for (int hh = 0; hh < heads; ++hh) add_quarter<D>(a, qbar + ((qb0 + min(i0 + 16 * wave + l16, n - 1)) * Hq + h0 + hh) * D, kq);
  // columns j .. j+3 of row i; where the row ends in between, those that exist
  auto store4 = [&](int i, int j, f32x4s x) __attribute__((always_inline)) {
    typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // (a row starts at any multiple of four bytes)
    float* o = out + (int64_t)i * n + j;
    if (j + 4 <= n) {
      *(f32x4u*)o = x;
    } else {
#pragma unroll
      for (int v = 0; v < 3; ++v)
        if (j + v < n) o[v] = x[v];
    }
  };
  // A key tile is fetched into registers one tile ahead (its loads are in flight while the tile before it is being
  // multiplied) and written to LDS between the two barriers.
  constexpr int PF = 64 * (D / 4) / 256;  // float4 per thread and key tile
  float4 pf[PF];
  auto fetch = [&](int jt) __attribute__((always_inline)) {
    const int j0 = jt * 64, colsv = min(64, n - j0);
#pragma unroll
    for (int x = 0; x < PF; ++x) {
      const int u = tid + 256 * x, r = u / (D / 4), cc = (u % (D / 4)) * 4;
      pf[x] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (r < colsv) pf[x] = *(const float4*)(kbar + ((qb0 + j0 + r) * Hkv + g) * D + cc);
    }
  };
  auto computed = [&](int jt) { return jt * 64 < n && jt <= it; };  // key tiles that are multiplied (a prefix of the chunk)
  if (computed(jc * chunk)) fetch(jc * chunk);
  for (int c = 0; c < chunk; ++c) {
    const int jt = jc * chunk + c, j0 = jt * 64;
    if (j0 >= n) break;
    if (jt > it) {  // entirely in the future of these rows
      for (int u = tid; u < rows * 16; u += 256) store4(i0 + (u >> 4), j0 + 4 * (u & 15), f32x4s{ninf, ninf, ninf, ninf});
      continue;
    }
    __syncthreads();  // the previous key tile has been consumed
#pragma unroll
    for (int x = 0; x < PF; ++x) {
      const int u = tid + 256 * x, r = u / (D / 4), cc = (u % (D / 4)) * 4;
      *(float4*)(ks + r * LD + cc) = pf[x];
    }
    if (c + 1 < chunk && computed(jt + 1)) fetch(jt + 1);
    __syncthreads();
#pragma unroll
    for (int c4 = 0; c4 < 4; ++c4) {
      const int i = i0 + 16 * wave + l16, j = j0 + 16 * c4 + 4 * kq;  // this lane's row, first of its four columns
      const bool future = j0 + 16 * c4 > i0 + 16 * wave + 15;  // the whole 16 x 16 tile lies right of the diagonal
      f32x4s acc = {0.f, 0.f, 0.f, 0.f};
      if (!future) {
        float b[D / 4];
        load_quarter<D>(b, ks + (16 * c4 + l16) * LD, kq);
        acc = score_tile16<D>(b, a);  // (transposed: the lane gets four columns of a row, not four rows of a column)
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[v] = j + v < i ? scale * acc[v] : ninf;
      if (i < n) store4(i, j, acc);
    }
  }
  if (jc == it >> lg) {  // last chunk of this row tile: every column to its right is in the future
    const int jstart = (jc + 1) * chunk * 64;
    for (int r = wave; r < rows; r += 4)
      for (int j = jstart + 4 * lane; j < n; j += 256) store4(i0 + r, j, f32x4s{ninf, ninf, ninf, ninf});
  }
}

// Mean-pools Q and K into the workspace behind the geometry tables.
int launch_pool(const Geo& g, const GeomArgs& ga, const void* q, const void* k, float* kbar_out, void* ws, hipStream_t st, float** qbar_p,
                float** kbar_p) {
  char* b = (char*)ws + align_up(table_offsets(g).bytes);
  float* qbar = (float*)b;
  float* kbar = (float*)(b + align_up(sizeof(float) * (size_t)g.NQB * g.Hq * g.D));
  const int qcols = g.Hq * g.D, kcols = g.Hkv * g.D;
  const int per_wg = 256 * (g.dtype == SB_F32 ? 4 : 8);  // columns per workgroup (head_dim is a multiple of 8)
  const int qgroups = (qcols + per_wg - 1) / per_wg, kgroups = (kcols + per_wg - 1) / per_wg;
  dim3 grid((unsigned)g.NQB, (unsigned)(qgroups + kgroups));
  {
    KernelTimer kt(K_POOL, st);
    if (g.dtype == SB_F32)
      hipLaunchKernelGGL(pool_kernel<true>, grid, dim3(256), 0, st, q, k, qcols, kcols, qgroups, ga, qbar, kbar);
    else
      hipLaunchKernelGGL(pool_kernel<false>, grid, dim3(256), 0, st, q, k, qcols, kcols, qgroups, ga, qbar, kbar);
  }
  SB_LAUNCH_CHECK("pool_kernel");
  if (kbar_out)
    SB_CHECK_HIP(hipMemcpyAsync(kbar_out, kbar, sizeof(float) * (size_t)g.NQB * g.Hkv * g.D, hipMemcpyDeviceToDevice, st));
  *qbar_p = qbar;
  *kbar_p = kbar;
  return SB_OK;
}

}  // namespace sb

using namespace sb;

extern "C" int sb_block_scores(const sb_problem* p, const void* q, const void* k, float* kbar_out, float* scores_out,
                               void* ws, void* stream) {
  Geo g;
  int rc = make_geo(p, &g);
  if (rc != SB_OK) return rc;
  if (g.S == 0 || g.T == 0 || g.NQB == 0) return SB_OK;
  if (!q || !k || !scores_out || !ws) { set_error("null q, k, scores_out or ws"); return SB_ERR_INVALID_ARG; }
  if ((rc = check_device_arrays(p)) != SB_OK) return rc;
  hipStream_t st = (hipStream_t)stream;
  if (g.S > kLaneSeqs && (rc = launch_geom(g, p, ws, st)) != SB_OK) return rc;
  const GeomArgs ga = make_geom_args(g, p, make_tables(g, p, ws));
  float *qbar = nullptr, *kbar = nullptr;
  if ((rc = launch_pool(g, ga, q, k, kbar_out, ws, st, &qbar, &kbar)) != SB_OK) return rc;
  auto count = [&](int lg) {  // (sequence, row tile, column chunk) triples
    int64_t items = 0;
    for (int s = 0; s < g.S; ++s) {
      const int64_t L = (int64_t)p->cu_seqlens_host[s + 1] - p->cu_seqlens_host[s];
      const int64_t n = (L + g.B - 1) / g.B;
      items += score_items((n + 63) / 64, lg);
    }
    return items;
  };
  int lg = kScChunkLog;
  int64_t items = count(lg);
  if (items * g.Hs < kScFewWgs) items = count(lg = 0);
  if (items > 0x7fffffffll) { set_error("too many score tiles for one launch"); return SB_ERR_INVALID_ARG; }
  dim3 gs((unsigned)items, (unsigned)g.Hs);
  KernelTimer kt(K_SCORE, st);
#define SB_SCORE_LAUNCH(DD, LG) \
  hipLaunchKernelGGL((score_kernel<DD, LG>), gs, dim3(256), 0, st, qbar, kbar, ga, g.Hq, g.Hkv, g.Hs, g.G, g.mode, g.score_scale, scores_out)
  if (g.D == 128) {
    if (lg == 0) SB_SCORE_LAUNCH(128, 0); else SB_SCORE_LAUNCH(128, kScChunkLog);
  } else {
    if (lg == 0) SB_SCORE_LAUNCH(64, 0); else SB_SCORE_LAUNCH(64, kScChunkLog);
  }
#undef SB_SCORE_LAUNCH
  SB_LAUNCH_CHECK("score_kernel");
  return SB_OK;
}
