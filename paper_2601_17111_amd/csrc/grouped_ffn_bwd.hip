// Backward of step 4 of the LLEP hot path (the grouped SwiGLU expert GEMMs):
// input gradients of the range's rows and per-expert weight gradients with
// the gradient return of spilled chunks (Sec. 1 and Sec. 4: LLEP stays exact
// in training, the spilled chunks' weight gradients go back to the expert's
// native device and are added there). The GEMMs are gemm.h's kernel with its
// backward epilogues.
#include "gemm.h"

namespace llep {

// ---------------------------------------------------------------------------
// Backward of the grouped SwiGLU FFN (bf16), for the groups of one device or
// of all devices. Given d out for the groups' rows (from the combine's
// backward):
//   1. g, u = X [Wg | Wu] (row-major by x_perm row), unless the training
//      forward kept them
//   2. d act = d out Wd^T; epilogue: d g, d u and act = silu(g) u
//   3. dX = [d g | d u] [Wg | Wu]^T               (x_perm rows)
//   4. weight gradients, in fp32 per expert: the rows of an expert's groups
//      are laid end to end in gradient-return order (the group on the
//      expert's native device first, then the other devices in increasing
//      order; each group padded with zero rows to a multiple of 32), and
//      dWg | dWu = X^T [d g | d u], dWd = act^T d out contract over that
//      segment, so an expert's gradient sums its native partial and then the
//      returned partials, in a fixed order.
// ---------------------------------------------------------------------------

struct BwdLayout {
  size_t tiles_off, wge_off, kbase_off, chunk_off;
  size_t gu_off, dgu_off, xt_off, dot_off, actt_off, dgut_off, total;
  int64_t max_groups, max_mtiles, prow_max, kmax;
};

static size_t round256(size_t v) { return (v + 255) / 256 * 256; }

static BwdLayout bwd_layout(int64_t R, int32_t E, int32_t P, int32_t D, int32_t F) {
  BwdLayout L;
  L.max_groups = 2 * int64_t(E) + P;
  L.max_mtiles = R / kTileM + L.max_groups + 1;
  L.prow_max = R + 16 * L.max_groups;
  L.kmax = (R + 32 * L.max_groups + 31) / 32 * 32;
  size_t o = 256;  // counters: n_mtiles, n_wg, k-slices in use, work counter, long n_wg,
                   // copy counter
  L.tiles_off = o;  o = round256(o + size_t(L.max_mtiles) * 16);
  L.wge_off = o;    o = round256(o + size_t(E) * 16);
  L.kbase_off = o;  o = round256(o + size_t(L.max_groups) * 4);
  L.chunk_off = o;  o = round256(o + size_t(L.kmax / 32) * 4);
  L.gu_off = o;     o = round256(o + size_t(R) * 2 * F * 2);  // by x_perm row
  L.dgu_off = o;    o = round256(o + size_t(L.prow_max) * 2 * F * 2);
  L.xt_off = o;     o = round256(o + size_t(D) * L.kmax * 2);
  L.dot_off = o;    o = round256(o + size_t(D) * L.kmax * 2);
  L.actt_off = o;   o = round256(o + size_t(F) * L.kmax * 2);
  L.dgut_off = o;   o = round256(o + size_t(2 * F) * L.kmax * 2);
  L.total = o;
  return L;
}

// float32 path: [d g | d u] (gate / up interleaved per 32 like the packed
// [Wg | Wu]) and the activation, per x_perm row
static size_t f32_bwd_bytes(int64_t R, int32_t F) {
  return 256 + round256(size_t(R) * 3 * F * 4);
}

bool ffn_backward_rows_ok(int64_t R, int32_t E, int32_t P) {
  // a DMA lane's byte offset reaches 16 blocks of kmax / 32 KB each
  return bwd_layout(R, E, P, 64, 64).kmax * 512 <= int64_t(INT32_MAX);
}

size_t ffn_backward_workspace_bytes(int64_t R, int32_t E, int32_t P, int32_t D, int32_t F,
                                    llep_dtype dtype) {
  if (dtype == LLEP_F32) return f32_bwd_bytes(R, F);
  return bwd_layout(R, E, P, D, F).total;
}

// One workgroup. For the groups [lo, hi) of the range: each group's first
// weight-gradient row (kbase[group], a multiple of 32) in gradient-return
// order, the owner group of every 32-row chunk, and the
// experts present with their segment (first 32-row slice, slices), longest
// segment first (ties: lower expert id), and how many of them have at least
// long_slices slices (those tiles are handed out before the input-gradient
// tiles, the shorter ones after them). Zeroes the work counters of the
// multi-problem launch and of the d act launch's copies.
__global__ __launch_bounds__(1024) void wgrad_table_kernel(
    const int32_t *__restrict__ groups, const int32_t *__restrict__ group_begin, int32_t device,
    int32_t P, int32_t E, int32_t M, int32_t *__restrict__ kbase,
    int32_t *__restrict__ chunk_group, int4 *__restrict__ wg_experts, int32_t *__restrict__ n_wg,
    int32_t long_slices, int32_t *__restrict__ n_wg_long, int32_t *__restrict__ kslices,
    int32_t *__restrict__ queue, int32_t *__restrict__ copy_counter) {
  __shared__ int32_t se[kMaxChunks], skey[kMaxChunks], ssl[kMaxChunks], skb[kMaxChunks];
  __shared__ int32_t esl[LLEP_MAX_EXPERTS];
  const int tid = threadIdx.x;
  const int lo = device < 0 ? group_begin[0] : group_begin[device];
  const int hi = device < 0 ? group_begin[P] : group_begin[device + 1];
  const int G = min(hi - lo, kMaxChunks);
  for (int i = tid; i < G; i += blockDim.x) {
    const int32_t *gr = groups + 4 * (lo + i);
    const int d = gr[0], e = gr[1], n = gr[3];
    se[i] = e;
    skey[i] = d == e / M ? -1 : d;  // native device first
    ssl[i] = (n + 31) / 32;
  }
  __syncthreads();
  // (the loops over groups and experts below are unrolled so that their
  // LDS reads, which do not depend on one another, are in flight together)
  for (int i = tid; i < G; i += blockDim.x) {
    int32_t kb = 0;
#pragma unroll 8
    for (int j = 0; j < G; ++j)
      if (se[j] < se[i] || (se[j] == se[i] && skey[j] < skey[i])) kb += ssl[j];
    kbase[lo + i] = kb * 32;
    skb[i] = kb;
  }
  for (int e = tid; e < E; e += blockDim.x) {
    int32_t sl = 0;
#pragma unroll 8
    for (int j = 0; j < G; ++j) sl += se[j] == e ? ssl[j] : 0;
    esl[e] = sl;
  }
  __syncthreads();
  // owner group of every 32-row slice: one wave per group, its lanes
  // striding over the group's slices
  for (int i = tid / kWave; i < G; i += blockDim.x / kWave)
    for (int c = skb[i] + tid % kWave; c < skb[i] + ssl[i]; c += kWave) chunk_group[c] = lo + i;
  for (int e = tid; e < E; e += blockDim.x) {
    const int32_t sl = esl[e];
    if (sl == 0) continue;
    int32_t idx = 0, start = 0;
#pragma unroll 8
    for (int f = 0; f < E; ++f) idx += esl[f] > sl || (esl[f] == sl && f < e);
#pragma unroll 8
    for (int j = 0; j < G; ++j) start += se[j] < e ? ssl[j] : 0;
    wg_experts[idx] = make_int4(e, start, sl, 0);
  }
  // counts over the experts and groups: one wave, lanes striding, then a
  // wave sum
  if (tid < kWave) {
    int32_t n = 0, nl = 0, tot = 0;
    for (int e = tid; e < E; e += kWave) {
      n += esl[e] > 0;
      nl += esl[e] > 0 && esl[e] >= long_slices;
    }
    for (int j = tid; j < G; j += kWave) tot += ssl[j];
    for (int off = kWave / 2; off > 0; off >>= 1) {
      n += __shfl_xor(n, off);
      nl += __shfl_xor(nl, off);
      tot += __shfl_xor(tot, off);
    }
    if (tid == 0) {
      *n_wg = n;
      *n_wg_long = nl;
      *kslices = tot;
      *queue = 0;
      *copy_counter = 0;
    }
  }
}

// The other weight-gradient operands: C columns of the range's rows
// (row-major by x_perm row, ld elements) copied into the weight-gradient
// layout, blocks of 16 columns x 32 rows over [C][kmax], row kbase[g] + r of
// the layout = row r of group g (zero for the padding r >= n_g). Item i of a
// source is its 32-row slice c = i / (C / 64) and its 64-column group
// i % (C / 64); the two sources (X, d out) follow one another.
struct WgradCopy {
  const uint16_t *src[2];
  uint16_t *dst[2];
  int64_t ld;
  int32_t C;  // a multiple of 64
  int64_t kmax;
  const int32_t *groups, *kbase, *chunk_group, *kslices;
  int32_t *counter;  // items taken; zeroed by the table kernel
};

constexpr int kCopyBatch = 8;             // items per counter claim
constexpr int kCopyTileBytes = 64 * 32 * 2;  // LDS staging tile of one wave

// One wavefront copies items taken kCopyBatch at a time from w.counter until
// none is left, with no barrier: each wave stages through its own LDS tile
// (`tile`, kCopyTileBytes) of 64 columns x 32 rows, column-major, the four
// 8-row chunks of column col in slots chunk ^ ((col / 8) % 4) so that a
// write instruction spreads over the banks. The loads of a batch are all
// issued before its first item is staged.
__device__ __forceinline__ void wgrad_copy_items(const WgradCopy &w, uint16_t *tile) {
  const int lane = threadIdx.x & 63;
  const int cgroups = w.C / 64;
  const int per_src = __builtin_amdgcn_readfirstlane(*w.kslices) * cgroups;
  const int n_items = 2 * per_src;
  // load layout: lane l holds row 8 q + l / 8 of the slice, columns
  // 8 (l % 8) .. + 7 of the item's 64 (each load instruction covers 8 whole
  // rows of 128 bytes)
  const int a = lane & 7, b = lane >> 3;
  const bool odd = b & 1;
  for (;;) {
    int b0 = 0;
    if (lane == 0) b0 = atomicAdd(w.counter, kCopyBatch);
    b0 = __builtin_amdgcn_readfirstlane(b0);
    if (b0 >= n_items) break;
    i32x4 v[kCopyBatch][4];
#pragma unroll
    for (int j = 0; j < kCopyBatch; ++j) {
      const int i = min(b0 + j, n_items - 1);  // past the end: the last item again (not stored)
      const int s = i >= per_src, rem = i - s * per_src;
      const int c = rem / cgroups, cc = rem - c * cgroups;
      const int gi = w.chunk_group[c];
      const int n = w.groups[4 * gi + 3];
      const int r0 = c * 32 - w.kbase[gi];
      const uint16_t *src = w.src[s] + int64_t(w.groups[4 * gi + 2]) * w.ld + cc * 64 + a * 8;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = r0 + 8 * q + b;
        v[j][q] = i32x4{0, 0, 0, 0};
        if (row < n) v[j][q] = *reinterpret_cast<const i32x4 *>(src + int64_t(row) * w.ld);
      }
    }
#pragma unroll
    for (int j = 0; j < kCopyBatch; ++j) {
      const int i = b0 + j;
      if (i >= n_items) break;
      const int s = i >= per_src, rem = i - s * per_src;
      const int c = rem / cgroups, cc = rem - c * cgroups;
      // the previous item's reads of the tile are done before it is rewritten
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      // Lanes l and l ^ 8 hold rows r and r ^ 1 of the same columns: each
      // writes one 32-bit word of two rows, the even-row lane for the even
      // column of a pair, the odd-row lane for the odd one.
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t mine = uint32_t(v[j][q][e]);
          const uint32_t other = uint32_t(__shfl_xor(int(mine), 8));
          const uint32_t word = odd ? ((other >> 16) | (mine & 0xffff0000u))
                                    : ((mine & 0xffffu) | (other << 16));
          const int col = 8 * a + 2 * e + int(odd);
          *reinterpret_cast<uint32_t *>(tile + col * 32 + ((q ^ (a & 3)) << 3) + (b & 6)) = word;
        }
      }
      // the tile is written before any lane reads it back
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      // block bb: columns 16 bb .. 16 bb + 15; lane l column l / 4, rows
      // 8 (l % 4) .. + 7
      uint16_t *dst = w.dst[s] + int64_t(c) * 512 + (lane >> 2) * 32 + (lane & 3) * 8;
#pragma unroll
      for (int bb = 0; bb < 4; ++bb) {
        const int col = bb * 16 + (lane >> 2);
        *reinterpret_cast<i32x4 *>(dst + int64_t(cc * 4 + bb) * (w.kmax / 32) * 512) =
            *reinterpret_cast<const i32x4 *>(tile + col * 32 + (((lane & 3) ^ ((col >> 3) & 3)) << 3));
      }
    }
  }
}

// Step 2 of the backward (d act GEMM with the SwiGLU backward epilogue) and
// the copies of X and d out into the weight-gradient layout in one launch:
// the GEMM deals its tiles in rounds, so the workgroups without a tile in the
// last, partly filled round start on the copies while the others finish
// their tiles, and everyone takes copy items once its tiles are done.
template <int BN, int WAVES_M, int WAVES_N>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N)
__attribute__((amdgpu_waves_per_eu(WAVES_M * WAVES_N / 4, WAVES_M * WAVES_N / 4)))
void dact_kernel(GemmArgs g, WgradCopy w) {
  static_assert(WAVES_M * WAVES_N * kCopyTileBytes <= ring_bytes<BN>(), "copy tiles fit the ring");
  __shared__ __attribute__((aligned(1024))) char smem[ring_bytes<BN>()];
  __shared__ int32_t s_next;
  {
    LaunchSched<256, BN, false> sched(g, &s_next);
    TileCoord t;
    if (sched.first(t)) gemm_tiles<BN, WAVES_M, WAVES_N, kEpiSwigluBwd, false, true>(g, smem, t, sched);
  }
  // every wave is done with the ring (its last epilogue's staging reads)
  // before the copies reuse it
  __syncthreads();
  wgrad_copy_items(w, reinterpret_cast<uint16_t *>(smem + (threadIdx.x >> 6) * kCopyTileBytes));
}

// ---------------------------------------------------------------------------
// Zeros for the weight gradients of the experts without a group in the range
// (the GEMMs write every element of the others). Bound by the stores to HBM;
// every workgroup finds the absent experts from the group table itself (a few
// loads) and takes 16 KB pieces of their three matrices in turn, so a few
// absent experts still spread over the chip. Zeroing every expert first and
// then writing it again took 453 us of a gpt-oss-20b backward of 2048 tokens
// and 340 us of a qwen3-30b-a3b one of 8192 (3.2 and 2.4 GB); with every
// expert present this launch takes 5 us.
// ---------------------------------------------------------------------------

constexpr int kZeroThreads = 256, kZeroGrid = 2048;
constexpr int kZeroPiece = 4096;  // floats; divides D * F (multiples of 64 each)

__global__ __launch_bounds__(kZeroThreads) void zero_absent_kernel(
    const int32_t *__restrict__ groups, const int32_t *__restrict__ group_begin, int32_t cap,
    int32_t device, int32_t P, int32_t E, int64_t per, float *__restrict__ dwg,
    float *__restrict__ dwu, float *__restrict__ dwd) {
  __shared__ int32_t present[LLEP_MAX_EXPERTS], absent[LLEP_MAX_EXPERTS];
  __shared__ int32_t n_absent;
  const int tid = threadIdx.x;
  const int lo = device < 0 ? group_begin[0] : group_begin[device];
  const int hi = min(cap, device < 0 ? group_begin[P] : group_begin[device + 1]);
  for (int e = tid; e < E; e += kZeroThreads) present[e] = 0;
  if (tid == 0) n_absent = 0;
  __syncthreads();
  for (int g = lo + tid; g < hi; g += kZeroThreads) {
    const int e = groups[4 * g + 1];
    if (e >= 0 && e < E) present[e] = 1;
  }
  __syncthreads();
  if (tid < kWave) {  // in expert order, so that every workgroup has the same list
    int n = 0;
    for (int e0 = 0; e0 < E; e0 += kWave) {
      const bool out = e0 + tid < E && !present[e0 + tid];
      const uint64_t m = __ballot(out);
      if (out) absent[n + __popcll(m & lanemask_lt())] = e0 + tid;
      n += __popcll(m);
    }
    if (tid == 0) n_absent = n;
  }
  __syncthreads();
  const int64_t pieces = per / kZeroPiece, total = 3 * pieces * n_absent;
  for (int64_t i = blockIdx.x; i < total; i += gridDim.x) {
    const int64_t m = i / pieces;  // (expert, matrix)
    float *dst = (m % 3 == 0 ? dwg : m % 3 == 1 ? dwu : dwd) + absent[m / 3] * per +
                 (i % pieces) * kZeroPiece + tid * 4;
#pragma unroll
    for (int k = 0; k < kZeroPiece; k += 4 * kZeroThreads)
      *reinterpret_cast<f32x4 *>(dst + k) = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
}

hipError_t launch_zero_absent(const FfnBwdArgs &a, hipStream_t stream) {
  hipLaunchKernelGGL(zero_absent_kernel, dim3(kZeroGrid), dim3(kZeroThreads), 0, stream, a.groups,
                     a.group_begin, 2 * a.E + a.P, a.device, a.P, a.E, int64_t(a.D) * a.F,
                     a.dw_gate, a.dw_up, a.dw_down);
  return hipGetLastError();
}

hipError_t launch_grouped_ffn_backward(const FfnBwdArgs &a, hipStream_t stream) {
  if (a.dtype == LLEP_F32) {
    float *dgu = reinterpret_cast<float *>(static_cast<char *>(a.ws) + 256);
    return launch_ffn_f32_backward(a, dgu, dgu + size_t(a.R) * 2 * a.F, stream);
  }
  const BwdLayout L = bwd_layout(a.R, a.E, a.P, a.D, a.F);
  char *ws = static_cast<char *>(a.ws);
  int32_t *n_mtiles = reinterpret_cast<int32_t *>(ws);
  int32_t *n_wg = n_mtiles + 1;
  int32_t *kslices = n_mtiles + 2;
  int32_t *queue = n_mtiles + 3;
  int32_t *n_wg_long = n_mtiles + 4;
  int32_t *copy_counter = n_mtiles + 5;
  int4 *tiles = reinterpret_cast<int4 *>(ws + L.tiles_off);
  int4 *wge = reinterpret_cast<int4 *>(ws + L.wge_off);
  int32_t *kbase = reinterpret_cast<int32_t *>(ws + L.kbase_off);
  int32_t *chunk = reinterpret_cast<int32_t *>(ws + L.chunk_off);
  uint16_t *gu = reinterpret_cast<uint16_t *>(ws + L.gu_off);
  uint16_t *dgu = reinterpret_cast<uint16_t *>(ws + L.dgu_off);
  uint16_t *xt = reinterpret_cast<uint16_t *>(ws + L.xt_off);
  uint16_t *dot = reinterpret_cast<uint16_t *>(ws + L.dot_off);
  uint16_t *actt = reinterpret_cast<uint16_t *>(ws + L.actt_off);
  uint16_t *dgut = reinterpret_cast<uint16_t *>(ws + L.dgut_off);
  const int grid = (cu_count() + 7) / 8 * 8;
  const int D = a.D, F = a.F;
  hipError_t err;
#define LLEP_CHECK_LAUNCH()            \
  do {                                 \
    err = hipGetLastError();           \
    if (err != hipSuccess) return err; \
  } while (0)
  err = launch_tile_table(a.groups, a.group_begin, 2 * a.E + a.P, a.device, a.P, tiles, n_mtiles,
                          stream);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(wgrad_table_kernel, dim3(1), dim3(1024), 0, stream, a.groups, a.group_begin,
                     a.device, a.P, a.E, a.E / a.P, kbase, chunk, wge, n_wg, 2 * F / kSK,
                     n_wg_long, kslices, queue, copy_counter);
  LLEP_CHECK_LAUNCH();
  constexpr int NT = 64 * kWavesM * kWavesN;
  constexpr int NT192 = 64 * kWavesM192 * kWavesN192;
  const bool d192 = D % 256 != 0 && D % 192 == 0;
  const bool f192 = F % 256 != 0 && F % 192 == 0;
  // 1. g, u = X [Wg | Wu] (interleaved per 32), row-major by x_perm row,
  // unless the forward saved them
  GemmArgs g = {};
  g.A = static_cast<const uint16_t *>(a.x_perm);
  g.lda = D;
  g.B = static_cast<const uint16_t *>(a.w_gate_up);
  g.b_expert_stride = int64_t(2) * F * D;
  g.b_blk_stride = int64_t(D / kSK) * 1024;
  g.C = gu;
  g.ldc = 2 * F;
  g.groups = a.groups;
  g.tiles = tiles;
  g.n_mtiles = n_mtiles;
  g.N = 2 * F;
  g.Kdim = D;
  if (!a.gate_up) {
    hipLaunchKernelGGL((gemm256_kernel<256, kWavesM, kWavesN, kEpiPlain, false, false>),
                       dim3(grid), dim3(NT), 0, stream, g);
    LLEP_CHECK_LAUNCH();
  }
  // 2. d act = d out Wd^T; the epilogue writes [d g | d u] blocked (for dX)
  // and [d g | d u], act transposed into the weight-gradient layout; in the
  // same launch, the other weight-gradient operands X and d out, with the
  // rows of each expert laid end to end along k (gradient-return order)
  GemmArgs g2 = g;
  g2.A = static_cast<const uint16_t *>(a.d_out_perm);
  g2.lda = D;
  g2.B = static_cast<const uint16_t *>(a.w_down_t);
  g2.b_expert_stride = int64_t(F) * D;
  g2.b_blk_stride = int64_t(D / kSK) * 1024;
  g2.C = dgu;
  g2.ldc = F;
  g2.N = F;
  g2.Kdim = D;
  g2.GU = a.gate_up ? static_cast<const uint16_t *>(a.gate_up) : gu;
  g2.dgu_t = dgut;
  g2.act_t = actt;
  g2.kbase = kbase;
  g2.kmax = L.kmax;
  WgradCopy wc = {};
  wc.src[0] = static_cast<const uint16_t *>(a.x_perm);
  wc.src[1] = static_cast<const uint16_t *>(a.d_out_perm);
  wc.dst[0] = xt;
  wc.dst[1] = dot;
  wc.ld = D;
  wc.C = D;
  wc.kmax = L.kmax;
  wc.groups = a.groups;
  wc.kbase = kbase;
  wc.chunk_group = chunk;
  wc.kslices = kslices;
  wc.counter = copy_counter;
  if (f192)
    hipLaunchKernelGGL((dact_kernel<192, kWavesM192, kWavesN192>), dim3(grid), dim3(NT192), 0,
                       stream, g2, wc);
  else
    hipLaunchKernelGGL((dact_kernel<256, kWavesM, kWavesN>), dim3(grid), dim3(NT), 0, stream, g2,
                       wc);
  LLEP_CHECK_LAUNCH();
  // 3. one launch: dX = [d g | d u] [Wg | Wu]^T into the x_perm rows, and
  // the weight gradients X^T [d g | d u] (de-interleaved into dWg, dWu) and
  // act^T d out, per expert over its k-segment
  GemmArgs g3 = g;
  g3.A = dgu;
  g3.lda = 2 * F;
  g3.a_blk_stride = int64_t(2 * F / kSK) * 1024;
  g3.B = static_cast<const uint16_t *>(a.w_gate_up_t);
  g3.b_expert_stride = int64_t(2) * F * D;
  g3.b_blk_stride = int64_t(2 * F / kSK) * 1024;
  g3.C = static_cast<uint16_t *>(a.dx_perm);
  g3.ldc = D;
  g3.N = D;
  g3.Kdim = 2 * F;
  const int64_t wblk = (L.kmax / 32) * 1024;
  g3.wp[0] = WgProblem{xt, dgut, wblk, a.dw_gate, a.dw_up, int64_t(D) * F, D, 2 * F, 1};
  g3.wp[1] = WgProblem{actt, dot, wblk, a.dw_down, nullptr, int64_t(F) * D, F, D, 0};
  g3.wg_experts = wge;
  g3.n_wg = n_wg;
  g3.n_wg_long = n_wg_long;
  g3.queue = queue;
  // 256 x 192 tiles: the 256 x 256 ring fills the LDS and leaves no room for
  // the work counter's broadcast slot
  hipLaunchKernelGGL((gemm256_kernel<192, kWavesM192, kWavesN192, kEpiBwdMulti, true, false>),
                     dim3(grid), dim3(NT192), 0, stream, g3);
  LLEP_CHECK_LAUNCH();
#undef LLEP_CHECK_LAUNCH
  return hipSuccess;
}

}  // namespace llep
