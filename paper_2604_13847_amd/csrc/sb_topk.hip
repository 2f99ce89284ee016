// Top-K block selection (paper section 2.2): per row (sequence, selection head, query block i)
// keep the diagonal block plus the best c-1 past blocks under the total order
// (score descending, block index ascending; -0 == +0; NaN below everything).
// One wavefront per row: order-preserving 32-bit keys in registers or LDS, a 4-pass radix select for the
// threshold key, then an index-ordered compaction, so the result is a pure function of the scores.
#include <mutex>

#include "sb_geom.h"
#include "sb_internal.h"
#include "sb_score_tile.h"

namespace sb {

// Rows of up to 64 E past blocks (at most kRegKeys) with their keys in registers.
constexpr int kRegKeys = 2048;
template <int E>
__device__ __forceinline__ void select_in_registers(const float* row, int* hist, int lane, int m, int need, int i, int32_t* __restrict__ out) {
  // A buffer that ends with the past blocks: no branch and no address of its own for any of the loads.  The whole offset is the lane's, a
  // register per 4 KB and an immediate: the bounds check leaves the scalar offset out.
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)row, 0, 4 * m, 0x20000);
  uint32_t keys[E], largest = 0;
#pragma unroll
  for (int r0 = 0; r0 < E; r0 += 16) {
    int at = 4 * lane + 256 * r0;
    asm volatile("" : "+v"(at));  // (or the offsets are worked out from what the walks below need, a register each)
#pragma unroll
    for (int r = r0; r < r0 + 16 && r < E; ++r) keys[r] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, at + 256 * (r - r0), 0, 0);
  }
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const uint32_t key = order_key(__uint_as_float(keys[r]));
    keys[r] = lane < m - 64 * r ? key : 0u;
    largest = max(largest, keys[r]);
  }
  select_row([&](auto f) __attribute__((always_inline)) { walk_registers<E>(keys, lane, m, f); }, hist, lane, m, need, i, out, largest);
}

// One wavefront per row (several rows per workgroup, no workgroup barrier anywhere): keys in registers, or for batches with longer rows
// (REGS = false) in the wavefront's own LDS region, which also holds a 256-bin histogram.
// What bounds it: instruction issue, and latencies where LDS leaves few wavefronts on a CU: with 9 KB a wavefront for rows of 2048 keys four a
// SIMD, each walk over the keys an LDS read and a wait a step; in 69 registers seven, and no reads: 131072 tokens, 32 heads 0.180 -> 0.109 ms.
// Rows of up to 256 keys gain little (the 32768-token batch 23.1 -> 21.1 us).
template <bool REGS>
__global__ __launch_bounds__(256) void topk_kernel(const float* __restrict__ scores, GeomArgs ga, int64_t NQB, int Hs, int64_t nnz_unit,
                                                   int region_words, int32_t* __restrict__ rowptr, int32_t* __restrict__ idx) {
  extern __shared__ uint32_t smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t row_id = (int64_t)blockIdx.x * (blockDim.x >> 6) + wave;  // hs * NQB + query block
  if (row_id >= (int64_t)Hs * NQB) return;
  uint32_t* keys = smem + (size_t)wave * region_words;
  int* hist = (int*)(keys + region_words - 256);
  const int hs = (int)(row_id / NQB);
  const int qb = (int)(row_id - (int64_t)hs * NQB);
  const BatchGeom bg(ga);
  const SeqGeom sg = bg.get(bg.seq_of(qb));
  const int i = qb - sg.qb0, n = sg.n, k = sg.k;
  const int c = min(k, i + 1);
  const int64_t start = (int64_t)hs * nnz_unit + sg.row_base + sel_rows_before(i, k);
  if (lane == 0) {
    rowptr[row_id] = (int32_t)start;
    if (row_id == (int64_t)Hs * NQB - 1) rowptr[(int64_t)Hs * NQB] = (int32_t)(start + c);
  }
  int32_t* out = idx + start;
  const int need = c - 1, m = i;  // choose `need` of the m past blocks
  if (need == m) {                // everything is kept (also covers need == 0 with i == 0)
    for (int j = lane; j <= i; j += 64) out[j] = j;
    return;
  }
  if (need == 0) {
    if (lane == 0) out[0] = i;
    return;
  }
  const float* row = scores + (int64_t)Hs * sg.sc_off + ((int64_t)hs * n + i) * n;
  if constexpr (REGS) {
    if (m <= 256) select_in_registers<4>(row, hist, lane, m, need, i, out);
    else if (m <= 512) select_in_registers<8>(row, hist, lane, m, need, i, out);
    else if (m <= 1024) select_in_registers<16>(row, hist, lane, m, need, i, out);
    else select_in_registers<32>(row, hist, lane, m, need, i, out);
    return;
  }
  uint32_t largest = 0;
  for (int j0 = lane; j0 < m; j0 += 64 * 8) {  // eight independent loads in flight per lane: the row comes from HBM
    float x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = j0 + 64 * u < m ? row[j0 + 64 * u] : 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (j0 + 64 * u < m) {
        const uint32_t key = order_key(x[u]);
        largest = max(largest, key);
        keys[j0 + 64 * u] = key;
      }
  }
  wave_lds_fence();
  select_row([&](auto f) __attribute__((always_inline)) { walk_keys(keys, lane, m, f); }, hist, lane, m, need, i, out, largest);
}

// Scores and selection in one kernel: the scores of a row never leave the compute unit.  One
// workgroup of 16 wavefronts owns R consecutive query blocks of the packed batch and one selection
// head.  For each sequence that these blocks touch, every wavefront computes 16 x 16 score tiles
// (the rows' pooled queries in registers, pooled keys straight from memory: they are small and stay
// in L2), the tiles of all these sequences dealt to the wavefronts in turn, and leaves the order keys of the past blocks in LDS, row by row;
// after one barrier wavefront
// w selects for row w exactly as topk_kernel does.  R (16, or fewer for very long sequences) is what
// fits in LDS: R rows of `stride` keys plus one histogram per wavefront.  SCORES: the matrix is written as well, as score_kernel writes it.
constexpr int kFusedWaves = 16;

template <int D, bool SCORES>
__global__ __launch_bounds__(64 * kFusedWaves) void score_select_kernel(
    const float* __restrict__ qbar, const float* __restrict__ kbar, GeomArgs ga, int64_t NQB, int Hq, int Hkv, int Hs, int G, int mode,
    float scale, int64_t nnz_unit, int R, int stride, float* __restrict__ scores, int32_t* __restrict__ rowptr, int32_t* __restrict__ idx) {
  extern __shared__ uint32_t smem[];
  uint32_t* keys = smem;                            // [R][stride]
  int* hist = (int*)(smem + (size_t)R * stride);    // [kFusedWaves][256]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, kq = lane >> 4;
  const BatchGeom bg(ga);
  // Workgroup ids run over the selection heads first and workgroups go to the eight XCDs in turn: head index
  // (x % 8) * (Hs / 8) + x / 8 gives every XCD a contiguous range of heads, i.e. few KV heads, whose pooled keys
  // (n * D floats each) then stay in that XCD's L2.
  const int hx = blockIdx.x % Hs;
  const int64_t gy = blockIdx.x / Hs, ngroups = gridDim.x / Hs;
  const int hs = (Hs & 7) == 0 ? (hx & 7) * (Hs >> 3) + (hx >> 3) : hx;
  const int heads = mode == SB_SELECT_PER_QHEAD ? 1 : G;
  const int h0 = mode == SB_SELECT_PER_QHEAD ? hs : hs * G;
  const int g = h0 / G;
  // rows late in a sequence have the most past blocks: hand out the last groups of blocks first
  const int64_t b0 = (ngroups - 1 - gy) * R, b1 = min(NQB, b0 + R);
  int dealt = 0;  // 16 x 16 tiles so far: the wavefronts take them in turn, whichever sequence they are of
  for (int64_t ba = b0; ba < b1;) {
    const SeqGeom sg = bg.get(bg.seq_of((int)ba));
    const int64_t qb0 = sg.qb0;
    const int n = sg.n;
    const int ia = (int)(ba - qb0), ib = (int)min((int64_t)n, ia + (b1 - ba));  // rows [ia, ib) of sequence s
    const int nrows = ib - ia, r0 = (int)(ba - b0);
    const int k = sg.k;
    // a row needs its scores only if it keeps some but not all of its past blocks: 2 <= k <= i
    const bool choose = k >= 2 && ib - 1 >= k;
    if (SCORES || choose) {
      const int ntiles = (ib - 1 + 15) / 16;  // block j is in the past of some row of the segment iff j < ib - 1
      int ct = (wave - dealt) & (kFusedWaves - 1);
      dealt += ntiles;
      if (ct < ntiles) {
        float a[D / 4];
#pragma unroll
        for (int t = 0; t < D / 4; ++t) a[t] = 0.f;
        const int ra = min(ia + l16, ib - 1);  // rows past the segment repeat its last row; their results are dropped
        for (int hh = 0; hh < heads; ++hh) add_quarter<D>(a, qbar + ((qb0 + ra) * Hq + h0 + hh) * D, kq);
        for (; ct < ntiles; ct += kFusedWaves) {
          const int j = ct * 16 + l16;
          float b[D / 4];
          load_quarter<D>(b, kbar + ((qb0 + min(j, n - 1)) * Hkv + g) * D, kq);
          const f32x4s acc = score_tile16<D>(a, b);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int r = 4 * kq + v;
            if (r < nrows && j < ia + r) {
              if (choose) keys[(size_t)(r0 + r) * stride + j] = order_key(scale * acc[v]);
              if (SCORES) scores[(int64_t)Hs * sg.sc_off + ((int64_t)hs * n + ia + r) * n + j] = scale * acc[v];
            }
          }
        }
      }
    }
    ba += nrows;
  }
  __syncthreads();
  if (b0 + wave >= b1) return;
  // wavefront w: row b0 + w
  const int qb = (int)b0 + wave;
  const SeqGeom sg = bg.get(bg.seq_of(qb));
  const int n = sg.n, i = qb - sg.qb0, k = sg.k;
  const int c = min(k, i + 1);
  const int64_t row_id = (int64_t)hs * NQB + qb;
  const int64_t start = (int64_t)hs * nnz_unit + sg.row_base + sel_rows_before(i, k);
  if (lane == 0) {
    rowptr[row_id] = (int32_t)start;
    if (row_id == (int64_t)Hs * NQB - 1) rowptr[(int64_t)Hs * NQB] = (int32_t)(start + c);
  }
  if (SCORES) {  // the blocks that are not in the row's past
    float* row = scores + (int64_t)Hs * sg.sc_off + ((int64_t)hs * n + i) * n;
    for (int j = i + lane; j < n; j += 64) row[j] = -__builtin_inff();
  }
  int32_t* out = idx + start;
  const int need = c - 1, m = i;
  if (need == m) {
    for (int j = lane; j <= i; j += 64) out[j] = j;
  } else if (need == 0) {
    if (lane == 0) out[0] = i;
  } else {
    uint32_t largest = 0;
    auto walk = [&](auto f) __attribute__((always_inline)) { walk_keys(keys + (size_t)wave * stride, lane, m, f); };
    walk([&](int, uint32_t key, bool) { largest = max(largest, key); });
    select_row(walk, hist + 256 * wave, lane, m, need, i, out, largest);
  }
}

}  // namespace sb

using namespace sb;

constexpr size_t kLdsUnasked = 48 * 1024;  // dynamic LDS that a kernel may have without its limit being raised

// launches the selection on tables that are already in device memory
static int select_launch(const Geo& g, const GeomArgs& ga, const float* scores, int32_t* sel_rowptr_out, int32_t* sel_idx_out,
                         hipStream_t st) {
  // every wavefront owns 256 histogram bins and, where keys are not in registers, a region of n_max keys (rounded up to 64); as many rows
  // per workgroup (at most four) as fit in 64 KiB
  const bool regs = g.n_max <= kRegKeys + 1;
  const int region_words = (regs ? 0 : (int)((g.n_max + 63) / 64 * 64)) + 256;
  int W = (int)(65536 / (sizeof(uint32_t) * (size_t)region_words));
  W = W < 1 ? 1 : (W > 4 ? 4 : W);
  const size_t smem = sizeof(uint32_t) * (size_t)region_words * W;
  if (smem > kLdsUnasked) {  // raise the kernel's dynamic LDS limit; once per device, whichever thread comes first
    static std::mutex mu;
    static bool attr_set[kMaxDevices] = {};
    int dev = 0;
    SB_CHECK_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) { set_error("device ordinal %d out of range", dev); return SB_ERR_UNSUPPORTED; }
    std::lock_guard<std::mutex> lock(mu);
    if (!attr_set[dev]) {
      SB_CHECK_HIP(hipFuncSetAttribute((const void*)topk_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)(sizeof(uint32_t) * (SB_MAX_BLOCKS_PER_SEQ + 256))));
      attr_set[dev] = true;
    }
  }
  const int64_t rows = (int64_t)g.Hs * g.NQB;
  dim3 grid((unsigned)((rows + W - 1) / W));
  KernelTimer kt(K_TOPK, st);
  hipLaunchKernelGGL(regs ? topk_kernel<true> : topk_kernel<false>, grid, dim3(64 * W), smem, st, scores, ga, g.NQB, g.Hs, g.nnz_unit, region_words, sel_rowptr_out,
                     sel_idx_out);
  SB_LAUNCH_CHECK("topk_kernel");
  return SB_OK;
}

// the geometry tables, where the kernels read them
static int need_tables(const Geo& g, const sb_problem* p, void* ws, hipStream_t st) {
  return g.S > kLaneSeqs ? launch_geom(g, p, ws, st) : SB_OK;
}

extern "C" int sb_select_topk(const sb_problem* p, const float* scores, int32_t* sel_rowptr_out, int32_t* sel_idx_out,
                              void* ws, void* stream) {
  Geo g;
  int rc = make_geo(p, &g);
  if (rc != SB_OK) return rc;
  if (!sel_rowptr_out) { set_error("null sel_rowptr_out"); return SB_ERR_INVALID_ARG; }
  hipStream_t st = (hipStream_t)stream;
  if (g.S == 0 || g.T == 0 || g.NQB == 0) {
    return fill_zero(sel_rowptr_out, sizeof(int32_t), st);
  }
  if (!scores || !sel_idx_out || !ws) { set_error("null scores, sel_idx_out or ws"); return SB_ERR_INVALID_ARG; }
  if ((rc = check_device_arrays(p)) != SB_OK) return rc;
  if ((rc = need_tables(g, p, ws, st)) != SB_OK) return rc;
  return select_launch(g, make_geom_args(g, p, make_tables(g, p, ws)), scores, sel_rowptr_out, sel_idx_out, st);
}

// LDS layout of the kernel that scores and selects.  A row of keys is padded to a stride of 4 mod 16 words, so that the four query rows a
// store instruction touches fall into different banks.
static int fused_stride(const Geo& g) { return (g.n_max + 63) / 64 * 64 + 4; }
static size_t fused_lds(const Geo& g, int R) { return sizeof(uint32_t) * ((size_t)R * fused_stride(g) + 256 * (size_t)kFusedWaves); }

// launches the kernel that scores and selects; qbar/kbar are the pooled arrays, `scores` may be null
static int score_select_launch(const Geo& g, const GeomArgs& ga, const float* qbar, const float* kbar, float* scores, int32_t* sel_rowptr_out,
                               int32_t* sel_idx_out, hipStream_t st) {
  const int stride = fused_stride(g);
  int R = kFusedWaves;
  if (fused_lds(g, R) > kLdsUnasked) {
    static std::mutex mu;
    static int lds_of_device[kMaxDevices] = {};  // LDS a workgroup may use, once the kernels' limit has been raised to it
    int dev = 0;
    SB_CHECK_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) { set_error("device ordinal %d out of range", dev); return SB_ERR_UNSUPPORTED; }
    int cap = 0;
    {
      std::lock_guard<std::mutex> lock(mu);
      if (!lds_of_device[dev]) {
        int per_block = 0;
        SB_CHECK_HIP(hipDeviceGetAttribute(&per_block, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
        SB_CHECK_HIP(hipFuncSetAttribute((const void*)score_select_kernel<128, false>, hipFuncAttributeMaxDynamicSharedMemorySize, per_block));
        SB_CHECK_HIP(hipFuncSetAttribute((const void*)score_select_kernel<64, false>, hipFuncAttributeMaxDynamicSharedMemorySize, per_block));
        lds_of_device[dev] = per_block;
      }
      cap = lds_of_device[dev];
    }
    while (R > 1 && fused_lds(g, R) > (size_t)cap) R >>= 1;
    if (fused_lds(g, R) > (size_t)cap) {
      set_error("a sequence of %d blocks does not fit the fused selection (%zu bytes of LDS, %d available): pass scores_out", g.n_max,
                fused_lds(g, R), cap);
      return SB_ERR_UNSUPPORTED;
    }
  }
  const size_t smem = fused_lds(g, R);
  const int64_t groups = (g.NQB + R - 1) / R;
  if (groups * g.Hs > 0x7fffffffll) { set_error("too many rows for one launch of the fused selection: pass scores_out"); return SB_ERR_UNSUPPORTED; }
  KernelTimer kt(K_SCORE_SELECT, st);
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)(groups * g.Hs)), dim3(64 * kFusedWaves), smem, st, qbar, kbar, ga, g.NQB, g.Hq, g.Hkv, g.Hs, g.G,
                       g.mode, g.score_scale, g.nnz_unit, R, stride, scores, sel_rowptr_out, sel_idx_out);
  };
  if (g.D == 128) launch(scores ? score_select_kernel<128, true> : score_select_kernel<128, false>);
  else launch(scores ? score_select_kernel<64, true> : score_select_kernel<64, false>);
  SB_LAUNCH_CHECK("score_select_kernel");
  return SB_OK;
}

// Where the caller wants the score matrix too, one kernel or two?  One saves a launch and reads no scores, but gathers the pooled keys
// for 16 rows at a time where score_kernel takes 64: up to one round of its workgroups, and no more LDS than it has without asking (so that
// a first call makes no runtime call that it did not make before).  Two kernels / one, with the pooling: 1000 tokens,
// one head 15.1 / 12.9 us, 8192 tokens, 32/8 heads (256 workgroups) 34.1 / 24.8, four sequences of 2048 tokens 30.0 / 24.5.  At 512
// workgroups the two are level (the two kernels of then took 55 us, of which score_kernel has since lost a fifth, one takes 52).  With the
// sequences of a workgroup's rows one after the other, a barrier each, 2039 tokens in short sequences took 19.9 us in place of 12.6; their
// tiles dealt to all wavefronts: 10.5.
constexpr int64_t kFusedWgs = 256;
static bool score_and_select_at_once(const Geo& g) {
  return (g.NQB + kFusedWaves - 1) / kFusedWaves * g.Hs <= kFusedWgs && fused_lds(g, kFusedWaves) <= kLdsUnasked;
}

extern "C" int sb_score_select(const sb_problem* p, const void* q, const void* k, float* kbar_out, float* scores_out,
                               int32_t* sel_rowptr_out, int32_t* sel_idx_out, void* ws, void* stream) {
  Geo g;
  int rc = make_geo(p, &g);
  if (rc != SB_OK) return rc;
  if (!sel_rowptr_out) { set_error("null sel_rowptr_out"); return SB_ERR_INVALID_ARG; }
  hipStream_t st = (hipStream_t)stream;
  if (g.S == 0 || g.T == 0 || g.NQB == 0) {
    return fill_zero(sel_rowptr_out, sizeof(int32_t), st);
  }
  if (!sel_idx_out) { set_error("null sel_idx_out"); return SB_ERR_INVALID_ARG; }
  if (!q || !k || !ws) { set_error("null q, k or ws"); return SB_ERR_INVALID_ARG; }
  if ((rc = check_device_arrays(p)) != SB_OK) return rc;
  const GeomArgs ga = make_geom_args(g, p, make_tables(g, p, ws));
  if (scores_out && !score_and_select_at_once(g)) {  // write the score matrix, then select from it
    rc = sb_block_scores(p, q, k, kbar_out, scores_out, ws, stream);  // leaves the geometry tables, where they are needed, at the start of ws
    if (rc != SB_OK) return rc;
    return select_launch(g, ga, scores_out, sel_rowptr_out, sel_idx_out, st);
  }
  if ((rc = need_tables(g, p, ws, st)) != SB_OK) return rc;
  float *qbar = nullptr, *kbar = nullptr;
  if ((rc = launch_pool(g, ga, q, k, kbar_out, ws, st, &qbar, &kbar)) != SB_OK) return rc;
  return score_select_launch(g, ga, qbar, kbar, scores_out, sel_rowptr_out, sel_idx_out, st);
}

// ---------------------------------------------------------------------------------------------
// sb_select_topk for callers that cannot allocate: the geometry tables that `ws` holds in sb_select_topk live in a
// file-scope device array instead.  In host code the array's name is only a stand-in; its device address is looked up
// once per device (each GPU has its own copy at its own address) and that pointer is what the kernels receive.
static __device__ __align__(256) unsigned char scratch[SB_STATIC_SELECT_WS_BYTES];

static int static_scratch_ptr(void** out) {
  static std::mutex mu;
  static void* ptr_of_device[kMaxDevices] = {};
  int dev = 0;
  SB_CHECK_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) { set_error("device ordinal %d out of range", dev); return SB_ERR_UNSUPPORTED; }
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr_of_device[dev]) {
    void* ptr = nullptr;
    SB_CHECK_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) { set_error("hipGetSymbolAddress returned a null pointer"); return SB_ERR_HIP; }
    ptr_of_device[dev] = ptr;
  }
  *out = ptr_of_device[dev];
  return SB_OK;
}

extern "C" int sb_select_topk_static(const sb_problem* p, const float* scores, int32_t* sel_rowptr_out, int32_t* sel_idx_out,
                                     void* stream) {
  Geo g;
  int rc = make_geo(p, &g);
  if (rc != SB_OK) return rc;
  if (!sel_rowptr_out) { set_error("null sel_rowptr_out"); return SB_ERR_INVALID_ARG; }
  hipStream_t st = (hipStream_t)stream;
  if (g.S == 0 || g.T == 0 || g.NQB == 0) return fill_zero(sel_rowptr_out, sizeof(int32_t), st);
  if (!scores || !sel_idx_out) { set_error("null scores or sel_idx_out"); return SB_ERR_INVALID_ARG; }
  const size_t need = align_up(table_offsets(g).bytes);
  if (need > (size_t)SB_STATIC_SELECT_WS_BYTES) {
    set_error("problem needs %zu bytes of geometry tables, the built-in scratch holds %d (use sb_select_topk)", need,
              (int)SB_STATIC_SELECT_WS_BYTES);
    return SB_ERR_WORKSPACE_TOO_SMALL;
  }
  if ((rc = check_device_arrays(p)) != SB_OK) return rc;
  void* ws = nullptr;
  if ((rc = static_scratch_ptr(&ws)) != SB_OK) return rc;
  // (from kLaneSeqs + 1 sequences on:) every table entry the selection reads is rewritten by this call: nothing has to start at zero
  if ((rc = need_tables(g, p, ws, st)) != SB_OK) return rc;
  return select_launch(g, make_geom_args(g, p, make_tables(g, p, ws)), scores, sel_rowptr_out, sel_idx_out, st);
}
