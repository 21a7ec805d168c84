// Weight-gradient tiles of the backward: per expert, A^T B contracted over the
// rows of the expert's groups, both operands read as the other steps leave
// them, with the contraction index (the row) outermost:
//   A   row-major by x_perm row (X, or d out): its columns are the tile's 256
//       output rows;
//   B   in 16 x 32 blocks over padded rows ([d g | d u], or the activation):
//       its columns are the tile's 192 output columns.
// The transposition happens on the way from the LDS to the matrix cores:
// ds_read_b64_tr_b16 hands each lane four values of one column from four
// rows. (Copying X and d out, and writing [d g | d u] and the activation a
// second time, transposed, took 250 us of the d act launch of a qwen3-30b-a3b
// step of 8192 tokens: 1.9 GB.)
//
// The pipeline is gemm.h's: k-slices of 32 rows through a ring of kStages LDS
// stages by DMA, issued by half the waves, with the fragment reads and the DMA
// between the MFMAs. A slice never spans two groups; a group's last slice may
// have fewer than 32 rows, and the rows past them (re-reads of the group's
// last row of A, whatever follows in B) are overwritten with zeros in the LDS
// before they are multiplied.
#pragma once

#include "gemm.h"

namespace llep {

// A weight-gradient problem. gate_up: C[m][n] with the columns of C (gate) and
// C2 (up) interleaved per 32, each [E][M][N / 2]; otherwise C[n][m],
// [E][N][M].
struct WgProblem {
  const uint16_t *A;  // row-major, lda = M
  const uint16_t *B;  // blocked, N columns
  float *C, *C2;
  int32_t M, N;
};

struct WgArgs {
  WgProblem p[2];            // 0: gate/up, 1: down
  const int4 *experts;       // (expert, first entry of `groups`, k-slices, 0), longest first
  const int4 *groups;        // (first x_perm row, first 16-row block of B, rows, 0) by expert
                             // in gradient-return order
  const int32_t *n_experts;  // with k-slices
  const int32_t *n_long;     // the first of them whose tiles are at least as long as a main tile
};

// Wave-uniform load of a table entry through the scalar cache (the tables were
// written by an earlier launch), so that it does not queue behind the DMA.
__device__ __forceinline__ int4 load_entry(const int4 *p) {
  typedef __attribute__((address_space(4))) const i32x4 *cptr;
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint64_t u =
      (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(v >> 32)))) << 32) |
      uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(v)));
  const i32x4 v4 = *reinterpret_cast<cptr>(u);
  return make_int4(v4.x, v4.y, v4.z, v4.w);
}

struct WgTile {
  int prob, e, m0, n0, mv, nv;  // problem, expert, first row / column, valid rows / columns
  int group, nk;                // first entry of WgArgs::groups, k-slices
};

// Tile u of the experts' tiles: expert-major, then problem, m-tile, n-tile.
__device__ __forceinline__ void wg_decode(const WgArgs &g, int u, int per0, int per1, WgTile &t) {
  const int i = u / (per0 + per1);
  int rem = u - i * (per0 + per1);
  t.prob = rem >= per0;
  rem -= t.prob ? per0 : 0;
  const int M = t.prob ? g.p[1].M : g.p[0].M, N = t.prob ? g.p[1].N : g.p[0].N;
  const int n_nt = (N + 191) / 192;
  const int4 we = load_entry(g.experts + i);
  t.e = we.x;
  t.group = we.y;
  t.nk = we.z;
  t.m0 = rem / n_nt * 256;
  t.n0 = rem % n_nt * 192;
  t.mv = min(256, M - t.m0);
  t.nv = min(192, N - t.n0);
}

typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 *lds_i16x4_ptr;

// Two transposed reads `step` bytes apart (four rows): a lane's eight k of one
// column.
__device__ __forceinline__ bf16x8 read_tr(const char *p, int step) {
  const i16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_ptr)(p));
  const i16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_ptr)(p + step));
  const __attribute__((ext_vector_type(8))) short v = {a[0], a[1], a[2], a[3],
                                                       b[0], b[1], b[2], b[3]};
  return __builtin_bit_cast(bf16x8, v);
}

// The tile loop of one workgroup, as gemm_tiles: 8 waves, 4 x 2, each 64 x 96.
template <class Sched>
__device__ __forceinline__ void wgrad_tiles(const WgArgs &g, char *smem, WgTile t, Sched &sched) {
  constexpr int NW = 8, NWD = 4, TM = 2, TN = 3;
  constexpr uint32_t A_STAGE = 32 * 512, B_STAGE = 12 * 1024, STAGE = A_STAGE + B_STAGE;
  constexpr int A_PER = 16 / NWD, B_PER = 12 / NWD, PER = A_PER + B_PER;
  static_assert(kStages * STAGE == ring_bytes<192>() && kSK == 32 && kAhead == 4, "ring");
  // (opaque, so that what is derived from it holds no register in the other
  // tile loop of the launch)
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1, h = lane >> 5;
  const uint32_t s0 = lds_addr(smem);

  // ---- requests: the slice asked for next (DMA waves) --------------------
  const char *Ab, *Bb;           // the slice's first row of A, block of B
  int q_group, q_left, q_limit;  // table entry, rows left in the group, offA's row limit
  int lda;                       // bytes per row of A
  int64_t b_row;                 // bytes per 16-row block of B
  int32_t offA[A_PER], offB[B_PER];
  const char *A0, *B0;
  int mv;
  // rows of A past the group's last re-read it
  auto set_off = [&](int limit) {
    int ln = lane;
    asm volatile("" : "+v"(ln));  // not hoisted out of the tile loop
#pragma unroll
    for (int j = 0; j < A_PER; ++j) {
      // KB wave + NWD j of the stage: two rows of 32 16-byte chunks; chunk
      // slot s of row r holds logical chunk s ^ 4 (r % 4)
      const int r = 2 * (wave + NWD * j) + (ln >> 5);
      const int c = min((ln & 31) ^ ((r & 3) << 2), (mv >> 3) - 1);
      offA[j] = min(r, limit - 1) * lda + c * 16;
    }
    q_limit = limit;
  };
  auto next_group = [&]() {
    const int4 e = load_entry(g.groups + q_group);
    ++q_group;
    Ab = A0 + int64_t(e.x) * lda;
    Bb = B0 + int64_t(e.y) * b_row;
    q_left = e.z;
  };
  auto setup = [&](const WgTile &c) {
    const bool down = c.prob != 0;
    const int M = down ? g.p[1].M : g.p[0].M, N = down ? g.p[1].N : g.p[0].N;
    lda = 2 * M;
    b_row = int64_t(N >> 5) * 1024;
    mv = c.mv;
    A0 = reinterpret_cast<const char *>(down ? g.p[1].A : g.p[0].A) + c.m0 * 2;
    B0 = reinterpret_cast<const char *>(down ? g.p[1].B : g.p[0].B) + (c.n0 >> 5) * 1024;
    int ln = lane;
    asm volatile("" : "+v"(ln));
#pragma unroll
    for (int j = 0; j < B_PER; ++j) {
      const int b = wave + NWD * j;  // block b / 2 of the tile's columns, b % 2 of the slice's rows
      offB[j] = int32_t((b & 1) * b_row) + min(b >> 1, (c.nv >> 5) - 1) * 1024 + ln * 16;
    }
    q_group = c.group;
    next_group();
    set_off(min(32, q_left));
  };
  // before the slice's first DMA / after its last
  auto open = [&]() {
    if (q_left <= 0) next_group();
    const int limit = min(32, q_left);
    if (limit != q_limit) set_off(limit);
  };
  auto close = [&]() {
    Ab += 32 * int64_t(lda);
    Bb += 2 * b_row;
    q_left -= 32;
  };
  auto dma = [&](int d, int st) {
    const uint32_t base = s0 + st * STAGE;
    if (d < A_PER)
      dma16(Ab, offA[d], base + (wave + NWD * d) * 1024);
    else
      dma16(Bb, offB[d - A_PER], base + A_STAGE + (wave + NWD * (d - A_PER)) * 1024);
  };
  auto issue = [&](int st) {
    if (wave >= NWD) return;
    open();
#pragma unroll
    for (int d = 0; d < PER; ++d) dma(d, st);
    close();
  };

  // ---- slices read: rows of the next one to become readable (all waves) ---
  int r_group, r_left;
  auto slice_rows = [&]() {
    if (r_left <= 0) {
      r_left = load_entry(g.groups + r_group).z;
      ++r_group;
    }
    const int n = min(32, r_left);
    r_left -= 32;
    return n;
  };
  // After the barrier that makes the slice in stage st readable: zeros in the
  // rows past its last, then another barrier.
  auto fix = [&](int st) {
    const int n = slice_rows();
    if (n == 32) return;
    char *a = smem + st * STAGE, *b = a + A_STAGE;
    const i32x4 z = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int u = int(threadIdx.x) + 512 * k;
      if ((u >> 5) >= n) *reinterpret_cast<i32x4 *>(a + u * 16) = z;
      if (u < 768 && ((u >> 6) & 1) * 16 + ((u & 63) >> 2) >= n)
        *reinterpret_cast<i32x4 *>(b + u * 16) = z;
    }
    asm volatile("" ::: "memory");
    wait_cnt<63, 0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  // ---- fragments ------------------------------------------------------------
  // In a group of 16 lanes, lane i reads four columns 4 (i % 4) .. of row
  // i / 4 and receives column i of the four rows. Lane group (h, half): rows
  // 8 h + 4 t .. + 3 (t = 0, 1: the two reads), columns 16 half .. + 15.
  const int r4 = (lane & 15) >> 2, c4 = lane & 3, half = (lane >> 4) & 1;
  int aoff[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i)
    aoff[i] = (8 * h + r4) * 512 + (((wm * 8 + i * 4 + 2 * half + (c4 >> 1)) ^ (r4 << 2)) << 4) +
              (c4 & 1) * 8;
  const int boff = int(A_STAGE) + wn * TN * 2048 + (8 * h + r4) * 64 + half * 32 + c4 * 8;
  auto read_a = [&](int st, int ks, int i) {
    return read_tr(smem + st * STAGE + aoff[i] + ks * 16 * 512, 4 * 512);
  };
  auto read_b = [&](int st, int ks, int j) {
    return read_tr(smem + st * STAGE + boff + (j * 2 + ks) * 1024, 4 * 64);
  };
  auto read_frags = [&](int st, int ks, bf16x8 (&fa)[TM], bf16x8 (&fb)[TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[i] = read_a(st, ks, i);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[j] = read_b(st, ks, j);
  };
  auto mfma_step = [&](f32x16 (&acc)[TM][TN], const bf16x8 (&fa)[TM], const bf16x8 (&fb)[TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
  };
  // one k-step of MFMAs with the next step's fragment reads and the DMA
  // [dma_lo, dma_hi) of the slice being requested spread between them
  constexpr int NM = TM * TN, NR = TM + TN, D0 = PER / 2;
  auto step = [&](auto dma_wave, f32x16 (&acc)[TM][TN], const bf16x8 (&fa)[TM],
                  const bf16x8 (&fb)[TN], bf16x8 (&na)[TM], bf16x8 (&nb)[TN], int st_next,
                  int ks_next, int dma_lo, int dma_hi, int st_dma) {
    const int NS = NR + (dma_hi - dma_lo);
#pragma unroll
    for (int s = 0; s < NM; ++s) {
      acc[s / TN][s % TN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          fb[s % TN], fa[s / TN], acc[s / TN][s % TN], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < NR + PER; ++q) {
        if (q < NS && q * NM >= s * NS && q * NM < (s + 1) * NS) {
          if (q < TM)
            na[q] = read_a(st_next, ks_next, q);
          else if (q < NR)
            nb[q - TM] = read_b(st_next, ks_next, q - TM);
          else if constexpr (decltype(dma_wave)::value)
            dma(dma_lo + q - NR, st_dma);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };
  auto next_stage = [](int st) { return st + 1 == kStages ? 0 : st + 1; };

  setup(t);
#pragma unroll
  for (int k = 0; k < kAhead; ++k)
    if (k < t.nk) issue(k);

  for (;;) {
    const int nk = t.nk;
    sched.request();
    r_group = t.group;
    r_left = 0;
    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.0f;
    // (waves whose blocks lie past the last row or column meet the same
    // barriers without reads or MFMAs)
    const int active =
        __builtin_amdgcn_readfirstlane(int(t.mv > wm * TM * 32 && t.nv > wn * TN * 32));
    if (nk >= kAhead)
      wait_and_sync<(kAhead - 1) * PER>();
    else
      wait_and_sync<0>();
    fix(0);
    int st = 0, st_req = kAhead % kStages, kt = 0;
    if (active) {
      bf16x8 fa0[TM], fb0[TN], fa1[TM], fb1[TN];
      read_frags(0, 0, fa0, fb0);
      auto steady = [&](auto dma_wave) {
        for (; kt < nk - kAhead; ++kt) {
          if constexpr (decltype(dma_wave)::value) open();
          step(dma_wave, acc, fa0, fb0, fa1, fb1, st, 1, 0, D0, st_req);
          wait_and_sync<(kAhead - 2) * PER + D0>();
          st = next_stage(st);
          fix(st);
          step(dma_wave, acc, fa1, fb1, fa0, fb0, st, 0, D0, PER, st_req);
          if constexpr (decltype(dma_wave)::value) close();
          st_req = next_stage(st_req);
        }
      };
      if (wave < NWD)
        steady(std::true_type{});
      else
        steady(std::false_type{});
      for (; kt < nk - 1; ++kt) {
        read_frags(st, 1, fa1, fb1);
        mfma_step(acc, fa0, fb0);
        const int left = nk - 2 - kt;
        if (left >= 2)
          wait_and_sync<2 * PER>();
        else if (left == 1)
          wait_and_sync<PER>();
        else
          wait_and_sync<0>();
        st = next_stage(st);
        fix(st);
        read_frags(st, 0, fa0, fb0);
        mfma_step(acc, fa1, fb1);
      }
      read_frags(st, 1, fa1, fb1);
      mfma_step(acc, fa0, fb0);
      mfma_step(acc, fa1, fb1);
    } else {
      for (; kt < nk - kAhead; ++kt) {
        issue(st_req);
        st_req = next_stage(st_req);
        wait_and_sync<(kAhead - 1) * PER>();
        st = next_stage(st);
        fix(st);
      }
      for (; kt < nk - 1; ++kt) {
        const int left = nk - 2 - kt;
        if (left >= 2)
          wait_and_sync<2 * PER>();
        else if (left == 1)
          wait_and_sync<PER>();
        else
          wait_and_sync<0>();
        st = next_stage(st);
        fix(st);
      }
    }
    __syncthreads();  // every wave is done with the ring
    const WgTile c = t;
    const bool more = sched.next(t);
    if (more) {
      setup(t);
#pragma unroll
      for (int k = 0; k < kAhead - 1; ++k)
        if (k < t.nk) issue(k);
    }

    // Epilogue: a 32 x 32 accumulator block has lane l at row m = l % 32 and
    // slots 4 q + e at column n = 8 q + 4 h + e. Each block is staged in the
    // wave's part of the last two stages so that the stores are whole 128-byte
    // row pieces: rows m for the gate/up problem, rows n for the down problem
    // (whose gradient is [n][m]). Non-temporal: nothing in the call reads the
    // gradients back.
    constexpr uint32_t STAGING = 2 * STAGE / NW;
    constexpr int RS = 32 * 4 + 16;
    static_assert(32 * RS <= STAGING, "staging");
    char *stg = smem + (kStages - 2) * STAGE + wave * STAGING;
    const int rr = lane >> 3, rc = (lane & 7) * 4;
    const bool down = c.prob != 0;
    float *C = down ? g.p[1].C : g.p[0].C;
    float *C2 = g.p[0].C2;
    const int M = down ? g.p[1].M : g.p[0].M, N = down ? g.p[1].N : g.p[0].N;
    const int64_t base = int64_t(c.e) * (down ? int64_t(M) * N : int64_t(M) * (N >> 1));
    const int ld = down ? M : N >> 1;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = wm * TM * 32 + i * 32;
      if (m >= c.mv) break;  // (M and N are multiples of 64: blocks are whole)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int n = wn * TN * 32 + j * 32;
        if (n >= c.nv) continue;
        const int mg = c.m0 + m, ng = c.n0 + n;
        float *dst;
        if (down) {
          dst = C + base + int64_t(ng) * ld + mg;
#pragma unroll
          for (int q = 0; q < 16; ++q)
            *reinterpret_cast<float *>(stg + (8 * (q >> 2) + 4 * h + (q & 3)) * RS + (lane & 31) * 4) =
                acc[i][j][q];
        } else {
          dst = ((ng & 32) ? C2 : C) + base + int64_t(mg) * ld + 32 * (ng >> 6);
#pragma unroll
          for (int q = 0; q < 4; ++q)
            *reinterpret_cast<f32x4 *>(stg + (lane & 31) * RS + (8 * q + 4 * h) * 4) =
                f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2],
                      acc[i][j][4 * q + 3]};
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int r = 8 * k + rr;
          const f32x4 v = *reinterpret_cast<const f32x4 *>(stg + r * RS + rc * 4);
          __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(dst + int64_t(r) * ld + rc));
        }
      }
    }
    if (!more) break;
    // the staging reads are done before slice kAhead - 1 lands there
    wait_and_sync<63>();
    if (kAhead - 1 < t.nk) issue(kAhead - 1);
  }
}

}  // namespace llep
