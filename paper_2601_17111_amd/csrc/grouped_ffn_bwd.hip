// Backward of step 4 of the LLEP hot path (the grouped SwiGLU expert GEMMs):
// input gradients of the range's rows and per-expert weight gradients with
// the gradient return of spilled chunks (Sec. 1 and Sec. 4: LLEP stays exact
// in training, the spilled chunks' weight gradients go back to the expert's
// native device and are added there). The GEMMs are gemm.h's kernel and
// wgrad.h's weight-gradient tiles.
#include "gemm.h"
#include "wgrad.h"

namespace llep {

// ---------------------------------------------------------------------------
// Backward of the grouped SwiGLU FFN (bf16), for the groups of one device or
// of all devices. Given d out for the groups' rows (from the combine's
// backward):
//   1. g, u = X [Wg | Wu] (row-major by x_perm row), unless the training
//      forward kept them
//   2. d act = d out Wd^T; epilogue: d g, d u and act = silu(g) u
//   3. dX = [d g | d u] [Wg | Wu]^T               (x_perm rows)
//   4. weight gradients, in fp32 per expert: dWg | dWu = X^T [d g | d u] and
//      dWd = act^T d out, contracted over the rows of the expert's groups in
//      gradient-return order (the group on the expert's native device first,
//      then the other devices in increasing order), so an expert's gradient
//      sums its native partial and then the returned partials, in a fixed
//      order.
// ---------------------------------------------------------------------------

struct BwdLayout {
  size_t tiles_off, wge_off, wgg_off, gu_off, dgu_off, act_off, total;
  int64_t max_groups, max_mtiles, prow_max;
};

static size_t round256(size_t v) { return (v + 255) / 256 * 256; }

static BwdLayout bwd_layout(int64_t R, int32_t E, int32_t P, int32_t F) {
  BwdLayout L;
  L.max_groups = 2 * int64_t(E) + P;
  L.max_mtiles = R / kTileM + L.max_groups + 1;
  // a weight-gradient slice reads two 16-row blocks, also where its group
  // ends in the first: one block more than the padded rows
  L.prow_max = R + 16 * L.max_groups + 16;
  size_t o = 256;  // counters: n_mtiles, n_wg, work counter, long n_wg
  L.tiles_off = o;  o = round256(o + size_t(L.max_mtiles) * 16);
  L.wge_off = o;    o = round256(o + size_t(E) * 16);
  L.wgg_off = o;    o = round256(o + size_t(L.max_groups) * 16);
  L.gu_off = o;     o = round256(o + size_t(R) * 2 * F * 2);  // by x_perm row
  L.dgu_off = o;    o = round256(o + size_t(L.prow_max) * 2 * F * 2);
  L.act_off = o;    o = round256(o + size_t(L.prow_max) * F * 2);
  L.total = o;
  return L;
}

// float32 path: [d g | d u] (gate / up interleaved per 32 like the packed
// [Wg | Wu]) and the activation, per x_perm row
static size_t f32_bwd_bytes(int64_t R, int32_t F) {
  return 256 + round256(size_t(R) * 3 * F * 4);
}

bool ffn_backward_rows_ok(int64_t R, int32_t E, int32_t P) {
  // A limit of the interface: the rows, with every group that a plan can have
  // padded to 32, are fewer than 2^22. (No operand needs it: wgrad.h takes a
  // group from a 64-bit base, and what it accepts is not changed.)
  const int64_t max_groups = 2 * int64_t(E) + P;
  return (R + 32 * max_groups + 31) / 32 * 32 < (int64_t(1) << 22);
}

size_t ffn_backward_workspace_bytes(int64_t R, int32_t E, int32_t P, int32_t D, int32_t F,
                                    llep_dtype dtype) {
  if (dtype == LLEP_F32) return f32_bwd_bytes(R, F);
  return bwd_layout(R, E, P, F).total;
}

// Two workgroups, one table each (as two launches 4.5 us more: a small training
// step 346.9 -> 342.4 us).
// Workgroup 1: the tile list of gemm.h's launches, one entry (group, m-tile,
// padded first row of the group) per kTileM rows of each group of the range.
// Workgroup 0: for the groups [lo, hi) of the range that have rows, sorted by
// expert and within an expert in gradient-return order: their first x_perm row, first
// 16-row block of padded rows, and rows; and the experts present with their
// first group and 32-row slices (each group's rounded up), most slices first
// (ties: lower expert id), and how many of them have at least long_slices
// slices (those tiles are handed out before the input-gradient tiles, the
// shorter ones after them). Zeroes the work counter of the multi-problem
// launch. Bound by latency: one scan over the groups (padded rows) and one
// over the experts (groups), and for an expert with several groups a count
// over the groups (qwen3-30b-a3b, 8192 tokens: 42 us with counts over all
// groups for every group).
constexpr int kTableThreads = 1024;

// exclusive sum over the workgroup's threads; *total: the sum
__device__ __forceinline__ int32_t block_scan(int32_t v, int32_t *wsum, int32_t *total) {
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  int32_t incl = v;
  for (int off = 1; off < kWave; off <<= 1) {
    const int32_t u = __shfl_up(incl, off);
    if (lane >= off) incl += u;
  }
  if (lane == kWave - 1) wsum[wave] = incl;
  __syncthreads();
  int32_t before = 0, sum = 0;
#pragma unroll
  for (int w = 0; w < kTableThreads / kWave; ++w) {
    const int32_t x = wsum[w];
    before += w < wave ? x : 0;
    sum += x;
  }
  *total = sum;
  __syncthreads();
  return before + incl - v;
}

__global__ __launch_bounds__(kTableThreads) void bwd_table_kernel(
    const int32_t *__restrict__ groups, const int32_t *__restrict__ group_begin, int32_t cap,
    int32_t device, int32_t P, int32_t E, int32_t M, int4 *__restrict__ wg_groups,
    int4 *__restrict__ wg_experts, int32_t *__restrict__ n_wg, int32_t long_slices,
    int32_t *__restrict__ n_wg_long, int32_t *__restrict__ queue, int4 *__restrict__ tiles,
    int32_t *__restrict__ n_mtiles) {
  constexpr int kPer = 2;  // adjacent groups per thread
  static_assert(kPer * kTableThreads >= kMaxChunks && LLEP_MAX_EXPERTS <= kTableThreads, "threads");
  __shared__ int32_t ge[kMaxChunks];                 // (expert << 1) | native
  __shared__ int32_t count[LLEP_MAX_EXPERTS], slices[LLEP_MAX_EXPERTS];
  __shared__ int32_t wsum[kTableThreads / kWave];
  __shared__ int32_t n_all, n_long;
  const int tid = threadIdx.x;
  const int lo = device < 0 ? group_begin[0] : group_begin[device];
  const int hi = min(cap, device < 0 ? group_begin[P] : group_begin[device + 1]);
  const int G = min(max(hi - lo, 0), kMaxChunks);
  int e[kPer], nat[kPer], row[kPer], n[kPer];
  int32_t pad = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int i = kPer * tid + j;
    const int32_t *p = groups + 4 * min(lo + i, cap - 1);
    e[j] = p[1];
    nat[j] = p[0] == e[j] / M;
    row[j] = p[2];
    n[j] = i < G ? p[3] : 0;
    pad += (n[j] + 15) / 16;
  }
  for (int x = tid; x < E; x += kTableThreads) count[x] = slices[x] = 0;
  if (tid == 0) n_all = n_long = 0;
  int32_t total;
  int32_t block = block_scan(pad, wsum, &total);  // (its barriers order the clearing)
  if (blockIdx.x == 1) {
    int32_t mt[kPer], sum = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) sum += mt[j] = (n[j] + kTileM - 1) / kTileM;
    int32_t at = block_scan(sum, wsum, &total);
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      for (int k = 0; k < mt[j]; ++k) tiles[at + k] = make_int4(lo + kPer * tid + j, k, 16 * block, 0);
      at += mt[j];
      block += (n[j] + 15) / 16;
    }
    if (tid == 0) *n_mtiles = total;
    return;
  }
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int i = kPer * tid + j;
    if (i >= G) continue;
    ge[i] = n[j] > 0 ? (e[j] << 1) | nat[j] : -1;  // (-1: no expert's)
    if (n[j] == 0) continue;
    atomicAdd(&count[e[j]], 1);
    atomicAdd(&slices[e[j]], (n[j] + 31) / 32);
  }
  __syncthreads();
  const int32_t own = tid < E ? count[tid] : 0, sl = tid < E ? slices[tid] : 0;
  const int32_t first = block_scan(own, wsum, &total);
  if (tid < E) {
    // position among the experts by slices
    if (sl > 0) {
      int32_t at = 0;
#pragma unroll 8
      for (int f = 0; f < E; ++f) at += slices[f] > sl || (slices[f] == sl && f < tid);
      wg_experts[at] = make_int4(tid, first, sl, 0);
      atomicAdd(&n_all, 1);
      if (sl >= long_slices) atomicAdd(&n_long, 1);
    }
    count[tid] = (first << 1) | (own > 1);  // (read by its own thread above)
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int i = kPer * tid + j;
    if (i >= G || n[j] == 0) continue;
    const int32_t c = count[e[j]];
    int32_t at = c >> 1;
    if ((c & 1) && !nat[j]) {
      // the native group, then the groups of smaller devices (the table is
      // device-major, so they come before this one)
#pragma unroll 4
      for (int g = 0; g < G; ++g) at += ge[g] >> 1 == e[j] && (g < i || (ge[g] & 1));
    }
    wg_groups[at] = make_int4(row[j], block, n[j], 0);
    block += (n[j] + 15) / 16;
  }
  if (tid == 0) {
    *n_wg = n_all;
    *n_wg_long = n_long;
    *queue = 0;
  }
}

// Step 3: the weight-gradient tiles (wgrad.h) and the input-gradient tiles
// (gemm.h) from one work counter, longest first, so that the last ones to
// start are short and the workgroups finish together: the weight-gradient
// tiles of the experts whose contraction is at least as long as an
// input-gradient tile's, then the input-gradient tiles, then the other
// weight-gradient tiles. A workgroup's first tile is its slot (each XCD a
// contiguous block of the order); it asks for the next one while it works.
struct BwdQueue {
  int n_long, n_wgt, n_main, n_mt, n_nt, per0, per1, G;
  int32_t *counter, *s_next;
  int u;  // the tile taken last

  __device__ __forceinline__ bool is_wg(int v) const {
    return v < n_long || (v >= n_long + n_main && v < n_wgt + n_main);
  }
  __device__ __forceinline__ void ask() const {
    if (threadIdx.x == 0) *s_next = atomicAdd(counter, 1) + G;
  }
  __device__ __forceinline__ void take() { u = __builtin_amdgcn_readfirstlane(*s_next); }
};

struct WgSched {
  const WgArgs &w;
  BwdQueue &q;
  __device__ __forceinline__ void decode(WgTile &t) const {
    wg_decode(w, q.u < q.n_long ? q.u : q.u - q.n_main, q.per0, q.per1, t);
  }
  __device__ __forceinline__ void request() const { q.ask(); }
  __device__ __forceinline__ bool next(WgTile &t) {
    q.take();
    if (!q.is_wg(q.u)) return false;
    decode(t);
    return true;
  }
};

struct DxSched {
  static constexpr bool kOpaqueLane = true;  // two loops: registers are short
  static constexpr bool kCoherentC = false;  // C is read only by later launches
  const GemmArgs &g;
  BwdQueue &q;
  __device__ __forceinline__ bool decode(TileCoord &t) const {
    return decode_tile<256, 192>(g, q.u - q.n_long, q.n_mt, q.n_nt, t);
  }
  __device__ __forceinline__ void request() const { q.ask(); }
  __device__ __forceinline__ bool next(TileCoord &t) {
    q.take();
    return !q.is_wg(q.u) && q.u < q.n_wgt + q.n_main && decode(t);
  }
  __device__ __forceinline__ void done(const TileCoord &, bool) const {}
};

__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void bwd_multi_kernel(GemmArgs g, WgArgs w, int32_t *counter) {
  __shared__ __attribute__((aligned(1024))) char smem[ring_bytes<192>()];
  __shared__ int32_t s_next;
  BwdQueue q;
  q.n_mt = __builtin_amdgcn_readfirstlane(*g.n_mtiles);
  q.n_nt = (g.N + 191) / 192;
  q.n_main = q.n_mt * q.n_nt;
  q.per0 = ((w.p[0].M + 255) / 256) * ((w.p[0].N + 191) / 192);
  q.per1 = ((w.p[1].M + 255) / 256) * ((w.p[1].N + 191) / 192);
  q.n_wgt = __builtin_amdgcn_readfirstlane(*w.n_experts) * (q.per0 + q.per1);
  q.n_long = __builtin_amdgcn_readfirstlane(*w.n_long) * (q.per0 + q.per1);
  q.G = gridDim.x;  // a multiple of 8
  q.counter = counter;
  q.s_next = &s_next;
  q.u = (blockIdx.x % 8) * (q.G / 8) + blockIdx.x / 8;
  while (q.u < q.n_wgt + q.n_main) {
    if (q.is_wg(q.u)) {
      WgSched s{w, q};
      WgTile t;
      s.decode(t);
      wgrad_tiles(w, smem, t, s);
    } else {
      DxSched s{g, q};
      TileCoord t;
      if (!s.decode(t)) break;
      gemm_tiles<192, kWavesM192, kWavesN192, kEpiPlain, true, false>(g, smem, t, s);
    }
    // the last epilogue's staging reads are done before the ring fills again
    wait_and_sync<63>();
  }
}

// ---------------------------------------------------------------------------
// Zeros for the weight gradients of the experts without rows in the range
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
    if (e >= 0 && e < E && groups[4 * g + 3] > 0) present[e] = 1;
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
  const BwdLayout L = bwd_layout(a.R, a.E, a.P, a.F);
  char *ws = static_cast<char *>(a.ws);
  int32_t *n_mtiles = reinterpret_cast<int32_t *>(ws);
  int32_t *n_wg = n_mtiles + 1;
  int32_t *queue = n_mtiles + 2;
  int32_t *n_wg_long = n_mtiles + 3;
  int4 *tiles = reinterpret_cast<int4 *>(ws + L.tiles_off);
  int4 *wge = reinterpret_cast<int4 *>(ws + L.wge_off);
  int4 *wgg = reinterpret_cast<int4 *>(ws + L.wgg_off);
  uint16_t *gu = reinterpret_cast<uint16_t *>(ws + L.gu_off);
  uint16_t *dgu = reinterpret_cast<uint16_t *>(ws + L.dgu_off);
  uint16_t *act = reinterpret_cast<uint16_t *>(ws + L.act_off);
  const int grid = (cu_count() + 7) / 8 * 8;
  const int D = a.D, F = a.F;
  hipError_t err;
#define LLEP_CHECK_LAUNCH()            \
  do {                                 \
    err = hipGetLastError();           \
    if (err != hipSuccess) return err; \
  } while (0)
  hipLaunchKernelGGL(bwd_table_kernel, dim3(2), dim3(kTableThreads), 0, stream, a.groups,
                     a.group_begin, 2 * a.E + a.P, a.device, a.P, a.E, a.E / a.P, wgg, wge, n_wg,
                     2 * F / kSK, n_wg_long, queue, tiles, n_mtiles);
  LLEP_CHECK_LAUNCH();
  constexpr int NT = 64 * kWavesM * kWavesN;
  constexpr int NT192 = 64 * kWavesM192 * kWavesN192;
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
  // 2. d act = d out Wd^T; the epilogue writes [d g | d u] and act blocked
  // over padded rows
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
  g2.act = act;
  if (f192)
    hipLaunchKernelGGL((gemm256_kernel<192, kWavesM192, kWavesN192, kEpiSwigluBwd, false, true>),
                       dim3(grid), dim3(NT192), 0, stream, g2);
  else
    hipLaunchKernelGGL((gemm256_kernel<256, kWavesM, kWavesN, kEpiSwigluBwd, false, true>),
                       dim3(grid), dim3(NT), 0, stream, g2);
  LLEP_CHECK_LAUNCH();
  // 3. one launch: dX = [d g | d u] [Wg | Wu]^T into the x_perm rows, and
  // the weight gradients X^T [d g | d u] (de-interleaved into dWg, dWu) and
  // act^T d out, per expert over its rows
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
  WgArgs w = {};
  w.p[0] = WgProblem{static_cast<const uint16_t *>(a.x_perm), dgu, a.dw_gate, a.dw_up, D, 2 * F};
  w.p[1] = WgProblem{static_cast<const uint16_t *>(a.d_out_perm), act, a.dw_down, nullptr, D, F};
  w.experts = wge;
  w.groups = wgg;
  w.n_experts = n_wg;
  w.n_long = n_wg_long;
  hipLaunchKernelGGL(bwd_multi_kernel, dim3(grid), dim3(NT192), 0, stream, g3, w, queue);
  LLEP_CHECK_LAUNCH();
#undef LLEP_CHECK_LAUNCH
  return hipSuccess;
}

}  // namespace llep
