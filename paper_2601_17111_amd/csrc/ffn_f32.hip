// The float32 grouped SwiGLU FFN, forward and backward (reference precision:
// float32 operands, products and sums, no intermediate rounding), on the
// float32 matrix instruction.
//
// The layers run in float32 are small, so these kernels are bound by latency:
// what counts is few launches, few serial steps and enough workgroups. A
// workgroup (four wavefronts) takes a tile of 64 rows of one group x 128
// columns, each wave 32 x 64; slices 32 deep go through registers into LDS,
// the next one loading while the current one is multiplied. Every workgroup
// finds its tile in the group table itself. Each accumulator is kept as two
// sums (even and odd pairs of k), which halves the length of the chains of
// additions and lets two instructions overlap.
//
// Against one thread per output element: a training step of the tiny-fp32
// layer (T = 256, D = 64, F = 128) 187 -> 81 us, drawn steps of up to 768
// tokens and D, F of 64-512 233-1364 -> 56-129 us; the error against 64 bits
// falls by a quarter (shorter chains).
#include <algorithm>

#include "common.h"
#include "gemm.h"
#include "kernels.h"

namespace llep {

namespace {

constexpr int kThreads = 256;
constexpr int kRows = 64, kCols = 128, kDeep = 32;  // tile
constexpr int kLd = kDeep + 4;  // LDS row, floats: 16-byte aligned, spread over the banks
constexpr int kWgCols = 64;     // weight-gradient tile: 64 x 64, 32 rows of the groups deep

enum F32Epi : int { kPlain = 0, kSwiglu = 1, kSwigluBwd = 2 };

struct F32Gemm {
  const float *A;
  int64_t lda;
  const float *B;  // packed, N rows of K per expert
  int32_t N, K;
  float *C;        // plain: [row][N]; SwiGLU: act [row][N / 2]; backward: [d g | d u] [row][2 N]
  float *C2;       // SwiGLU: g and u [row][N], or null; backward: act [row][N]
  const float *GU; // backward: g and u [row][2 N] (may be C)
};

struct F32Range {
  const int32_t *groups, *group_begin;
  int32_t cap, device, P;
};

struct Tile {
  int e, row, rows;  // expert, first x_perm row, valid rows
};

// Tile m of the range's groups in pieces of 64 rows. One whole wave; false
// past the last.
__device__ __forceinline__ bool find_tile(const F32Range &r, int m, Tile &t) {
  const int lo = r.device < 0 ? r.group_begin[0] : r.group_begin[r.device];
  const int hi = min(r.cap, r.device < 0 ? r.group_begin[r.P] : r.group_begin[r.device + 1]);
  const int lane = lane_id();
  int base = 0;
  for (int g0 = lo; g0 < hi; g0 += kWave) {
    const int32_t *p = r.groups + 4 * min(g0 + lane, hi - 1);
    const int e = p[1], row = p[2], n = g0 + lane < hi ? p[3] : 0;
    const int own = (n + kRows - 1) / kRows;
    int incl = own;
    for (int off = 1; off < kWave; off <<= 1) {
      const int v = __shfl_up(incl, off);
      if (lane >= off) incl += v;
    }
    const uint64_t past = __ballot(base + incl > m);
    if (past) {
      const int l = __builtin_ctzll(past);
      const int at = (m - base - (__shfl(incl, l) - __shfl(own, l))) * kRows;
      t.e = __shfl(e, l);
      t.row = __shfl(row, l) + at;
      t.rows = min(kRows, __shfl(n, l) - at);
      return true;
    }
    base += __shfl(incl, kWave - 1);
  }
  return false;
}

struct F32Smem {
  float a[kRows][kLd];
  float b[kCols][kLd];
};

// One tile of C = A B^T: rows [t.row, + t.rows), columns [n0, + 128).
template <int kEpi>
__device__ __forceinline__ void f32_tile(const F32Gemm &g, const Tile &t, int n0, F32Smem &s) {
  const int tid = threadIdx.x, lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int wr = wave >> 1, wc = wave & 1, h = lane >> 5;
  const int cols = min(kCols, g.N - n0);  // a multiple of 64
  // loads of a slice: float4 i of the tile; A rows past the valid ones re-read
  // the last, B blocks past the last column re-read the last block
  constexpr int kA4 = kRows * kDeep / 4 / kThreads, kB4 = kCols * kDeep / 4 / kThreads;
  f32x4 va[kA4], vb[kB4];
  const float *Be = g.B + int64_t(t.e) * g.N * g.K;
  auto load = [&](int k0) {
#pragma unroll
    for (int i = 0; i < kA4; ++i) {
      const int u = i * kThreads + tid, r = min(u / (kDeep / 4), t.rows - 1), k = u % (kDeep / 4) * 4;
      va[i] = *reinterpret_cast<const f32x4 *>(g.A + int64_t(t.row + r) * g.lda + k0 + k);
    }
#pragma unroll
    for (int i = 0; i < kB4; ++i) {
      const int u = i * kThreads + tid, c = min(u / (kDeep / 4), cols - 1), k = u % (kDeep / 4) * 4;
      vb[i] = *reinterpret_cast<const f32x4 *>(Be + packed_index(n0 + c, k0 + k, g.K));
    }
  };
  f32x16 acc[2][2];
#pragma unroll
  for (int v = 0; v < 2; ++v)
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[v][p][q] = 0.0f;
  load(0);
  for (int k0 = 0; k0 < g.K; k0 += kDeep) {
    __syncthreads();  // the previous slice is read
#pragma unroll
    for (int i = 0; i < kA4; ++i) {
      const int u = i * kThreads + tid;
      *reinterpret_cast<f32x4 *>(&s.a[u / (kDeep / 4)][u % (kDeep / 4) * 4]) = va[i];
    }
#pragma unroll
    for (int i = 0; i < kB4; ++i) {
      const int u = i * kThreads + tid;
      *reinterpret_cast<f32x4 *>(&s.b[u / (kDeep / 4)][u % (kDeep / 4) * 4]) = vb[i];
    }
    __syncthreads();
    if (k0 + kDeep < g.K) load(k0 + kDeep);
    // lane half h holds k = 8 j + 4 h + i of a group of 8: product i takes the
    // two k of both halves
#pragma unroll
    for (int j = 0; j < kDeep / 8; ++j) {
      const f32x4 a = *reinterpret_cast<const f32x4 *>(&s.a[wr * 32 + (lane & 31)][8 * j + 4 * h]);
      f32x4 b[2];
#pragma unroll
      for (int v = 0; v < 2; ++v)
        b[v] = *reinterpret_cast<const f32x4 *>(&s.b[wc * 64 + v * 32 + (lane & 31)][8 * j + 4 * h]);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 2; ++v)
          acc[v][i & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[v][i], a[i], acc[v][i & 1], 0, 0, 0);
    }
  }
  // lane l holds row l % 32 and, in slots 4 q .. 4 q + 3, columns 8 q + 4 h + 0..3
  const int row = wr * 32 + (lane & 31);
  if (row >= t.rows || wc * 64 >= cols) return;
  const int64_t xr = t.row + row;
  auto four = [&](int v, int q) {
    f32x4 x;
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = acc[v][0][4 * q + e] + acc[v][1][4 * q + e];
    return x;
  };
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int c = n0 + wc * 64 + 8 * q + 4 * h;  // column of block 0; block 1 is 32 further
    const f32x4 x0 = four(0, q), x1 = four(1, q);
    if constexpr (kEpi == kPlain) {
      *reinterpret_cast<f32x4 *>(g.C + xr * g.N + c) = x0;
      *reinterpret_cast<f32x4 *>(g.C + xr * g.N + c + 32) = x1;
    } else if constexpr (kEpi == kSwiglu) {
      // block 0: gate columns, block 1: the matching up columns
      if (g.C2) {
        *reinterpret_cast<f32x4 *>(g.C2 + xr * g.N + c) = x0;
        *reinterpret_cast<f32x4 *>(g.C2 + xr * g.N + c + 32) = x1;
      }
      f32x4 y;
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = x0[e] / (1.0f + expf(-x0[e])) * x1[e];
      const int f = (n0 + wc * 64) / 2 + 8 * q + 4 * h;
      *reinterpret_cast<f32x4 *>(g.C + xr * (g.N / 2) + f) = y;
    } else {
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const f32x4 da = v ? x1 : x0;
        const int f = c + 32 * v;
        const int64_t at = xr * 2 * g.N + 64 * (f / 32) + f % 32;
        const f32x4 gv = *reinterpret_cast<const f32x4 *>(g.GU + at);
        const f32x4 uv = *reinterpret_cast<const f32x4 *>(g.GU + at + 32);
        f32x4 dg, du, ac;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float sg = 1.0f / (1.0f + expf(-gv[e]));
          dg[e] = da[e] * uv[e] * (sg * (1.0f + gv[e] * (1.0f - sg)));
          du[e] = da[e] * gv[e] * sg;
          ac[e] = gv[e] * sg * uv[e];
        }
        *reinterpret_cast<f32x4 *>(g.C + at) = dg;
        *reinterpret_cast<f32x4 *>(g.C + at + 32) = du;
        *reinterpret_cast<f32x4 *>(g.C2 + xr * g.N + f) = ac;
      }
    }
  }
}

// grid: column tiles x an upper bound of the row tiles
template <int kEpi>
__global__ __launch_bounds__(kThreads) void f32_gemm_kernel(F32Gemm g, F32Range r) {
  __shared__ __attribute__((aligned(16))) F32Smem s;
  Tile t;
  // (every wave finds the same tile)
  for (int m = blockIdx.y; find_tile(r, m, t); m += gridDim.y)
    f32_tile<kEpi>(g, t, blockIdx.x * kCols, s);
}

// Weight gradients: tile (m0, n0) of expert e's A^T B, contracted over the
// rows of the expert's groups of the range in gradient-return order (the
// group on its native device e / M first, then by device), rows in order.
struct F32Wgrad {
  const float *A, *B;  // row-major by x_perm row
  int32_t M, N;        // columns of A and B
  float *C, *C2;       // [E][M][N]; gate/up (C2 set): gate into C, up into C2, [E][M][N / 2]
};

struct WgSmem {
  float a[kDeep][kWgCols + 4];
  float b[kDeep][kWgCols + 4];
};

__device__ __forceinline__ void f32_wgrad_tile(const F32Wgrad &g, const F32Range &r, int e, int nat,
                                               int m0, int n0, WgSmem &s) {
  const int tid = threadIdx.x, lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int wr = wave >> 1, wc = wave & 1, h = lane >> 5;
  const int lo = r.device < 0 ? r.group_begin[0] : r.group_begin[r.device];
  const int hi = min(r.cap, r.device < 0 ? r.group_begin[r.P] : r.group_begin[r.device + 1]);
  f32x16 acc[2];
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[p][q] = 0.0f;
  bool any = false;
  // every thread: 2 float4 of A and of B per slice of 32 rows
  constexpr int kPer = kDeep * kWgCols / 4 / kThreads;
  auto rows_of = [&](int row, int n) {
    f32x4 va[kPer], vb[kPer];
    auto load = [&](int k0) {
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        const int u = i * kThreads + tid, k = u / (kWgCols / 4), c = u % (kWgCols / 4) * 4;
        va[i] = vb[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if (k0 + k < n) {
          const int64_t xr = row + k0 + k;
          va[i] = *reinterpret_cast<const f32x4 *>(g.A + xr * g.M + m0 + c);
          vb[i] = *reinterpret_cast<const f32x4 *>(g.B + xr * g.N + n0 + c);
        }
      }
    };
    load(0);
    for (int k0 = 0; k0 < n; k0 += kDeep) {
      __syncthreads();
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        const int u = i * kThreads + tid, k = u / (kWgCols / 4), c = u % (kWgCols / 4) * 4;
        *reinterpret_cast<f32x4 *>(&s.a[k][c]) = va[i];
        *reinterpret_cast<f32x4 *>(&s.b[k][c]) = vb[i];
      }
      __syncthreads();
      if (k0 + kDeep < n) load(k0 + kDeep);
      // (rows past the end of the group add zero products: not multiplied)
      const int deep = min(kDeep, n - k0);
#pragma unroll 8
      for (int j = 0; j < (deep + 1) / 2; ++j)
        acc[j & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(
            s.b[2 * j + h][wc * 32 + (lane & 31)], s.a[2 * j + h][wr * 32 + (lane & 31)],
            acc[j & 1], 0, 0, 0);
    }
  };
  for (int pass = 0; pass < 2; ++pass)
    for (int g0 = lo; g0 < hi; g0 += kWave) {
      const int32_t *p = r.groups + 4 * min(g0 + lane, hi - 1);
      const int d = p[0], ge = p[1], row = p[2], n = p[3];
      uint64_t mine = __ballot(g0 + lane < hi && n > 0 && ge == e && (d == nat) == (pass == 0));
      while (mine) {
        const int l = __builtin_ctzll(mine);
        mine &= mine - 1;
        any = true;
        rows_of(__shfl(row, l), __shfl(n, l));
      }
    }
  if (!any) return;  // experts without rows in the range are not written
  const int row = m0 + wr * 32 + (lane & 31), col0 = n0 + wc * 32;
  float *C = g.C;
  int ld = g.N, col = col0;
  if (g.C2) {  // gate / up interleaved per 32 columns
    C = col0 & 32 ? g.C2 : g.C;
    ld = g.N / 2;
    col = col0 / 64 * 32;
  }
  float *dst = C + (int64_t(e) * g.M + row) * ld + col + 4 * h;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    f32x4 x;
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = acc[0][4 * q + i] + acc[1][4 * q + i];
    *reinterpret_cast<f32x4 *>(dst + 8 * q) = x;
  }
}

// The input gradient's tiles, then both weight gradients' of every expert.
__global__ __launch_bounds__(kThreads) void f32_bwd_kernel(F32Gemm dx, int32_t dx_tiles,
                                                           F32Wgrad w0, F32Wgrad w1, F32Range r,
                                                           int32_t M) {
  __shared__ __attribute__((aligned(16))) char mem[std::max(sizeof(F32Smem), sizeof(WgSmem))];
  int u = blockIdx.x;
  const int dx_cols = (dx.N + kCols - 1) / kCols;
  if (u < dx_tiles * dx_cols) {
    Tile t;
    if (!find_tile(r, u / dx_cols, t)) return;
    f32_tile<kPlain>(dx, t, u % dx_cols * kCols, *reinterpret_cast<F32Smem *>(mem));
    return;
  }
  u -= dx_tiles * dx_cols;
  const int n0 = w0.N / kWgCols, n1 = w1.N / kWgCols;
  const int per0 = w0.M / kWgCols * n0, per1 = w1.M / kWgCols * n1;
  const int e = u / (per0 + per1), i = u % (per0 + per1);
  WgSmem &s = *reinterpret_cast<WgSmem *>(mem);
  if (i < per0)
    f32_wgrad_tile(w0, r, e, e / M, i / n0 * kWgCols, i % n0 * kWgCols, s);
  else
    f32_wgrad_tile(w1, r, e, e / M, (i - per0) / n1 * kWgCols, (i - per0) % n1 * kWgCols, s);
}

}  // namespace

// an upper bound of the pieces of 64 rows of a range's groups
static int row_tiles(int64_t R, int32_t E, int32_t P) {
  return int(R / kRows + std::min<int64_t>(R, 2 * int64_t(E) + P));
}

template <int kEpi>
static hipError_t gemm(const F32Gemm &g, const F32Range &r, int tiles, hipStream_t stream) {
  if (tiles == 0) return hipSuccess;
  hipLaunchKernelGGL(f32_gemm_kernel<kEpi>,
                     dim3((g.N + kCols - 1) / kCols, std::min(tiles, 32768)), dim3(kThreads), 0,
                     stream, g, r);
  return hipGetLastError();
}

hipError_t launch_ffn_f32(const FfnArgs &a, void *act, hipStream_t stream) {
  const F32Range r = {a.groups, a.group_begin, 2 * a.E + a.P, a.device, a.P};
  const int tiles = row_tiles(a.R, a.E, a.P);
  float *h = static_cast<float *>(act);
  const F32Gemm up = {static_cast<const float *>(a.x_perm), a.D,
                      static_cast<const float *>(a.w_gate_up), 2 * a.F, a.D, h,
                      static_cast<float *>(a.gate_up_out), nullptr};
  const hipError_t err = gemm<kSwiglu>(up, r, tiles, stream);
  if (err != hipSuccess) return err;
  const F32Gemm down = {h, a.F, static_cast<const float *>(a.w_down), a.D, a.F,
                        static_cast<float *>(a.out_perm), nullptr, nullptr};
  return gemm<kPlain>(down, r, tiles, stream);
}

// dgu: [R][2F], act: [R][F] of the workspace
hipError_t launch_ffn_f32_backward(const FfnBwdArgs &a, float *dgu, float *act,
                                   hipStream_t stream) {
  const F32Range r = {a.groups, a.group_begin, 2 * a.E + a.P, a.device, a.P};
  const int tiles = row_tiles(a.R, a.E, a.P);
  const float *x = static_cast<const float *>(a.x_perm);
  const float *dout = static_cast<const float *>(a.d_out_perm);
  hipError_t err;
  if (!a.gate_up) {  // g and u again, where their gradients go afterwards
    const F32Gemm gu = {x, a.D, static_cast<const float *>(a.w_gate_up), 2 * a.F, a.D, dgu,
                        nullptr, nullptr};
    if ((err = gemm<kPlain>(gu, r, tiles, stream)) != hipSuccess) return err;
  }
  const F32Gemm da = {dout, a.D, static_cast<const float *>(a.w_down_t), a.F, a.D, dgu, act,
                      a.gate_up ? static_cast<const float *>(a.gate_up) : dgu};
  if ((err = gemm<kSwigluBwd>(da, r, tiles, stream)) != hipSuccess) return err;
  const F32Gemm dx = {dgu, 2 * int64_t(a.F), static_cast<const float *>(a.w_gate_up_t), a.D,
                      2 * a.F, static_cast<float *>(a.dx_perm), nullptr, nullptr};
  const F32Wgrad w0 = {x, dgu, a.D, 2 * a.F, a.dw_gate, a.dw_up};
  const F32Wgrad w1 = {act, dout, a.F, a.D, a.dw_down, nullptr};
  const int64_t per = 3 * (int64_t(a.D) / kWgCols) * (a.F / kWgCols);
  const int64_t blocks = int64_t(tiles) * ((a.D + kCols - 1) / kCols) + a.E * per;
  hipLaunchKernelGGL(f32_bwd_kernel, dim3(uint32_t(blocks)), dim3(kThreads), 0, stream, dx, tiles,
                     w0, w1, r, a.E / a.P);
  return hipGetLastError();
}

}  // namespace llep
