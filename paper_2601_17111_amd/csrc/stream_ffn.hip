// Step 4 for calls of few rows (decode, short prompts): the grouped SwiGLU
// expert GEMMs as a stream of the weights.
//
// With a few rows per expert the work is reading each expert's weights once,
// and the 256 x 256 tiles of gemm.h leave most of the chip without a tile (a
// token of a 32-expert layer has K = 4 experts, 92 gate/up tiles for 256 CUs,
// and one CU takes 80 us for its 1.5 MB of weights). Here a wavefront's unit
// of work is 32 packed weight rows (16 gate and 16 up columns, or 32 output
// columns) for one piece of at most 256 of its expert's rows:
//   - pieces of at most 16 rows: every wavefront works alone, with its own
//     ring of k-slices in the LDS and no barrier;
//   - larger pieces: the four wavefronts of a workgroup take four neighbouring
//     units and share the slices of the rows.
// Operands move to the LDS by DMA, and the slices of the next unit are asked
// for while the last ones of the current unit are in use, so that requests
// stay in flight from unit to unit.
//
// Every output element is the same sum as in gemm.h: the same
// v_mfma_f32_32x32x16_bf16 with the weights as first operand, over the same k
// order, and the same epilogue arithmetic, so the results do not depend on
// which of the two kernels ran.
//
// Bound by HBM while an expert has up to about 64 rows: 64 experts of D = F =
// 2880 with 8, 32, 64 and 128 rows each read their weights at 6.4, 6.0, 5.4
// and 4.2 TB/s (gemm.h: 5.8, 5.5, 5.3 and 4.4). Forward of one call, gemm.h ->
// here: gpt-oss-20b, 1 token 116 -> 44 us, 37 tokens 310 -> 253 us, with 90%
// of the pairs on one expert 202 -> 138 us; qwen3-30b-a3b, 1 token 79 -> 26
// us, 37 tokens 206 -> 183 us; deepseek-v3, 16 tokens with 95% on one expert
// 212 -> 145 us; 16 experts of 1024 x 768, 1 token 63 -> 20 us. With larger
// groups the 256 x 256 tiles do more work per byte from the L2 and win
// (use_stream_ffn).
#include <algorithm>

#include "gemm.h"

namespace llep {

constexpr int kStreamWaves = 4;
constexpr int kStreamThreads = kStreamWaves * kWave;
constexpr int kStreamLds = 144 * 1024;  // bytes of the rings
// Rows of a piece at most: 256, so that the weights are read once per 256
// rows, but 64 while all units of such pieces fit one round of the
// workgroups, where more of them at work count for more (16 experts of 1024 x
// 768, 148 rows of which 133 on one expert: 45 -> 31 us).
constexpr int kPieceRows = 256, kPieceRowsFew = 64;
constexpr int kMaxPieces = LLEP_MAX_EXPERTS + kStreamRows / kPieceRowsFew;
// Classes of pieces by rows: more than 128, 65-128, 33-64, 17-32, at most 16
// (16, 8, 4, 2 or 1 blocks of 16 rows).
constexpr int kClasses = 5;
constexpr int kCountBits = 12;

struct StreamArgs {
  const uint16_t *A;     // gate/up: x_perm, row-major; down: activation, blocked
  int64_t a_stride;      // bytes per row (gate/up) or per 16-row block (down)
  const uint16_t *B;     // packed weights
  int64_t b_expert_stride, b_blk_stride;  // elements; bytes per 16-row block
  uint16_t *C;           // gate/up: activation, blocked; down: out_perm, row-major
  uint16_t *gu_save;     // gate/up, training: g and u, row-major; or null
  const int32_t *groups, *group_begin;
  int32_t cap, device, P;
  int32_t N, nk;         // columns of C and 32-deep k-slices of the contraction (even)
};

// The rows of the range by expert: the rows of an expert's groups (a hot
// expert's pairs are spread over the devices) end to end, cut into pieces, so
// that its weights are read once per 256 rows however the plan spread them.
// In the activation an expert's rows start on a 16-row block.
struct StreamTable {
  uint16_t row[kStreamRows];   // x_perm rows, expert after expert
  int32_t list[kMaxPieces];    // pieces by class; see pack_piece
  uint16_t first[kMaxPieces];  // a piece's first place in `row`
  uint64_t wcount[kStreamWaves];
  int32_t wsize[kStreamWaves];
};
// used while the table is built, in the rings' memory
struct StreamBuild {
  int32_t expert[LLEP_MAX_EXPERTS];  // (groups << 16) | rows, then the first place
  int32_t group[kMaxChunks];         // (expert << 16) | rows
  i32x4 large[kStreamRows / 17 + 1];  // groups of more than 16 rows: place, row, rows
  int32_t n_large;
};
static_assert(kStreamRows < (1 << 15) && LLEP_MAX_EXPERTS <= (1 << 9) &&
              kStreamRows / 16 + LLEP_MAX_EXPERTS <= (1 << 10), "packed fields");
static_assert(sizeof(StreamBuild) <= kStreamLds, "built in the rings' memory");

// expert, rows (1-256), first 16-row block of the activation, and whether it
// is its expert's only piece
__device__ __forceinline__ int pack_piece(int e, int rows, int block, bool once) {
  return e | ((rows - 1) << 9) | (block << 17) | (int(once) << 27);
}

// class of a piece of n < 256 rows (-1: none)
__device__ __forceinline__ int class_of(int n) {
  return n == 0 ? -1 : n > 128 ? 0 : n > 64 ? 1 : n > 32 ? 2 : n > 16 ? 3 : 4;
}

// Every workgroup builds the table for itself (a separate launch would cost
// 5 us): rows per expert, one scan over the experts of rows, blocks and the
// pieces of each class, and each group's place among its expert's rows.
// shared_units: units of a shared piece. first[c]: where class c starts in the
// list.
__device__ __forceinline__ void build_table(const StreamArgs &a, StreamTable &t, StreamBuild &s,
                                            int shared_units, int (&first)[kClasses + 1]) {
  constexpr int kPer = (kMaxChunks + kStreamThreads - 1) / kStreamThreads;
  constexpr int kPerE = LLEP_MAX_EXPERTS / kStreamThreads;
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int lo = a.device < 0 ? a.group_begin[0] : a.group_begin[a.device];
  const int hi = min(a.cap, a.device < 0 ? a.group_begin[a.P] : a.group_begin[a.device + 1]);
  int32_t ge[kPer], gr[kPer], gn[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int32_t *p = a.groups + 4 * min(tid + kStreamThreads * j, a.cap - 1);
    ge[j] = p[1] & (LLEP_MAX_EXPERTS - 1);
    gr[j] = p[2];
    gn[j] = p[3];
  }
  for (int e = tid; e < LLEP_MAX_EXPERTS; e += kStreamThreads) s.expert[e] = 0;
  if (tid == 0) s.n_large = 0;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int g = tid + kStreamThreads * j;
    if (g < lo || g >= hi) gn[j] = 0;
    if (g < lo || g >= hi) continue;
    s.group[g] = (ge[j] << 16) | gn[j];
    if (gn[j] > 0) atomicAdd(&s.expert[ge[j]], (1 << 16) | gn[j]);
  }
  __syncthreads();
  // rows of the group's expert in the groups before it (an expert has one
  // group per device, most experts one in all)
  int before[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    before[j] = 0;
    if (gn[j] == 0 || s.expert[ge[j]] < (2 << 16)) continue;
#pragma unroll 4
    for (int g = lo; g < tid + kStreamThreads * j; ++g)
      before[j] += s.group[g] >> 16 == ge[j] ? s.group[g] & 0xffff : 0;
  }
  int n[kPerE];
#pragma unroll
  for (int j = 0; j < kPerE; ++j) n[j] = s.expert[kPerE * tid + j] & 0xffff;
  // one 64-bit word holds the counts of all classes (12 bits each), one
  // 32-bit word the blocks and the rows
  static_assert(kMaxPieces < (1 << kCountBits) && kClasses * kCountBits <= 64, "counts");
  auto count = [](uint64_t v, int c) { return int(v >> (kCountBits * c)) & ((1 << kCountBits) - 1); };
  int at[kClasses];  // this thread's places in the lists
  int base;          // and its experts' first block and row
  int piece = kPieceRows;
  for (;;) {
    const int whole_class = piece == kPieceRows ? 0 : 2;
    uint64_t own = 0;
    int size = 0;
#pragma unroll
    for (int j = 0; j < kPerE; ++j) {
      const int cls = class_of(n[j] % piece);
      own += (uint64_t(n[j] / piece) << (kCountBits * whole_class)) +
             (cls >= 0 ? uint64_t(1) << (kCountBits * cls) : 0);
      size += ((n[j] + 15) / 16 << 16) | n[j];
    }
    uint64_t incl = own;
    int isize = size;
    for (int off = 1; off < kWave; off <<= 1) {
      const uint64_t v = (uint64_t(uint32_t(__shfl_up(int(incl >> 32), off))) << 32) |
                         uint32_t(__shfl_up(int(incl), off));
      const int z = __shfl_up(isize, off);
      if (lane >= off) {
        incl += v;
        isize += z;
      }
    }
    if (lane == kWave - 1) {
      t.wcount[wave] = incl;
      t.wsize[wave] = isize;
    }
    __syncthreads();
    uint64_t ahead = incl - own, total = 0;
    int rows = 0;
    base = isize - size;
#pragma unroll
    for (int w = 0; w < kStreamWaves; ++w) {
      const uint64_t v = t.wcount[w];
      const int z = t.wsize[w];
      ahead += w < wave ? v : 0;
      base += w < wave ? z : 0;
      total += v;
      rows += z & 0xffff;
    }
    first[0] = 0;
#pragma unroll
    for (int c = 0; c < kClasses; ++c) {
      at[c] = first[c] + count(ahead, c);
      first[c + 1] = __builtin_amdgcn_readfirstlane(first[c] + count(total, c));
    }
    // (an upper bound of the pieces of 64 rows; no more pieces than experts:
    // nothing to cut)
    const int few = (first[kClasses] + rows / kPieceRowsFew) * shared_units;
    if (piece == kPieceRowsFew || few > int(gridDim.x) || count(total, 0) + count(total, 1) == 0)
      break;
    piece = kPieceRowsFew;
    __syncthreads();  // the sums are read before they are rewritten
  }
#pragma unroll
  for (int j = 0; j < kPerE; ++j) {
    const int e = kPerE * tid + j, whole = n[j] / piece, rem = n[j] % piece;
    const int block = base >> 16, place = base & 0xffff;
    auto put = [&](int &i, int k, int rows) {
      t.list[i] = pack_piece(e, rows, block + k * (piece / 16), n[j] <= piece);
      t.first[i] = uint16_t(place + k * piece);
      ++i;
    };
    s.expert[e] = place;
    for (int k = 0; k < whole; ++k) put(piece == kPieceRows ? at[0] : at[2], k, piece);
    const int cls = class_of(rem);
#pragma unroll
    for (int c = 0; c < kClasses; ++c)
      if (cls == c) put(at[c], whole, rem);
    base += ((n[j] + 15) / 16 << 16) | n[j];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    if (gn[j] == 0) continue;
    const int place = s.expert[ge[j]] + before[j];
    if (gn[j] > 16) {
      s.large[atomicAdd(&s.n_large, 1)] = i32x4{place, gr[j], gn[j], 0};
    } else {
      for (int i = 0; i < gn[j]; ++i) t.row[place + i] = uint16_t(gr[j] + i);
    }
  }
  __syncthreads();
  for (int i = wave; i < s.n_large; i += kStreamWaves) {
    const i32x4 g = s.large[i];
    for (int r = lane; r < g.z; r += kWave) t.row[g.x + r] = uint16_t(g.y + r);
  }
  __syncthreads();
}

// The `count` units u0, u0 + step, ... of one class: kA 16-row blocks of A and
// kD 32-deep k-slices per ring stage. kShare 1: units of this wave alone, in
// its own ring. kShare 4: of the workgroup, each of four neighbouring column
// units; the waves stand kRows x (4 / kRows) over the unit's rows and columns
// (two by two from 65 rows on: fewer fragment reads from the LDS per MFMA).
template <int kPhase, int kA, int kD, int kShare, int kRows>
__device__ __forceinline__ void stream_units(const StreamArgs &a, const StreamTable &t,
                                             int class_at, char *ring, int u0, int step,
                                             int count) {
  constexpr int kB = 2;  // 16-row blocks of the weights per wave and slice
  constexpr int kAPer = kD * kA / kShare;  // DMA instructions per stage and wave, 1 KB each
  constexpr int kPer = kD * kB + kAPer;
  constexpr int kMT = kA < 2 ? 1 : kA / 2 / kRows;  // 32-row blocks of a wave's accumulators
  constexpr int kU = kRows;                         // and its column units
  constexpr int kStage = kPer * kShare * 1024;
  constexpr int kRingBytes = kStreamLds / kStreamWaves * kShare;
  constexpr int kRing = kRingBytes / kStage;  // stages
  static_assert(kD * kA % kShare == 0 && kRing >= 3 && (kRing - 1) * kPer < 64, "ring");
  // two slices of a row-major A are 128 contiguous bytes per row: whole lines
  static_assert(kPhase != 0 || kD == 2, "the layout of x_perm's rows below");
  if (count <= 0) return;
  const int32_t *list = t.list + class_at;
  const uint16_t *first = t.first + class_at;
  const int lane = lane_id();
  const int h = lane >> 5;
  const int wave = kShare == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int row_w = kRows == 1 ? 0 : wave / (kShare / kRows) * 32 * kMT;  // the wave's first row
  const int col_w = kRows == 1 ? wave : wave % (kShare / kRows) * kU;     // and column unit
  const int n_col = a.N / (kPhase == 0 ? 16 : 32);
  const int n_unit = (n_col + kShare - 1) / kShare;  // units per piece
  const int nk = a.nk / kD, total = count * nk;  // stages per unit, in all

  const uint32_t ring0 = lds_addr(ring);
  const int kc_load = (lane & 3) ^ ((lane >> 4) & 3);
  const int32_t blk_lane = (lane >> 2) * 64 + kc_load * 16;
  const int32_t b_next = int32_t((kPhase == 0 ? 2 : 1) * a.b_blk_stride);

  // a unit's place: piece and unit of the piece; the piece's expert, first
  // block of the activation, first place in t.row, and rows
  struct Unit {
    int piece, col, e, block, place, rows;
    bool once;  // the only piece of its expert
  };
  auto load_piece = [&](Unit &u) {
    const int p = __builtin_amdgcn_readfirstlane(list[u.piece]);
    u.e = p & 511;
    u.rows = ((p >> 9) & 255) + 1;
    u.block = (p >> 17) & 1023;
    u.once = p >> 27;
    u.place = __builtin_amdgcn_readfirstlane(first[u.piece]);
  };
  auto advance = [&](Unit &u) {
    u.col += step;
    if (u.col < n_unit) return;
    do {
      u.col -= n_unit;
      ++u.piece;
    } while (u.col >= n_unit);
    load_piece(u);
  };

  // requests: the unit and stage asked for next
  Unit q;
  q.piece = u0 / n_unit;
  q.col = u0 - q.piece * n_unit;
  load_piece(q);
  const char *Ab, *Bb;
  int32_t offA[kAPer];
  auto setup = [&]() {
    const int col = min(kShare * q.col + wave, n_col - 1);  // past the last column: not stored
    const int nb = kPhase == 0 ? 4 * (col >> 1) + (col & 1) : 2 * col;
    Bb = reinterpret_cast<const char *>(a.B) + int64_t(q.e) * a.b_expert_stride * 2 +
         nb * a.b_blk_stride;
    Ab = reinterpret_cast<const char *>(a.A) + (kPhase == 0 ? 0 : q.block * a.a_stride);
    const int32_t stride = int32_t(a.a_stride);
    // byte offset of piece row r in x_perm (all rows: below 2^30 bytes); rows
    // (blocks) past the valid ones re-read the last
    auto row_off = [&](int r) { return int(t.row[q.place + min(r, q.rows - 1)]) * stride; };
    static_assert(int64_t(kStreamRows) * LLEP_MAX_FFN_DIM * 2 <= (1 << 30), "row offsets");
#pragma unroll
    for (int j = 0; j < kAPer; ++j) {
      const int ja = wave * kAPer + j;  // KB of the stage's A
      if (kPhase == 0) {  // 8 rows of 128 bytes; chunk swizzled by (row / 2) % 8
        const int r = 8 * ja + (lane >> 3);
        offA[j] = row_off(r) + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
      } else {  // slice ja / kA, a block of 16 rows x 64 bytes
        offA[j] = min(ja % kA, (q.rows - 1) >> 4) * stride + blk_lane + ja / kA * 1024;
      }
    }
  };
  setup();
  int q_k = 0, issued = 0;
  uint32_t q_stage = ring0;
  // a stage in LDS: A (gate/up: rows of 128 bytes; down: per slice kA blocks of
  // 16 rows x 64 bytes), then per wave and slice kB blocks of the weights
  auto request = [&]() {
    // The weights first: they come from memory, the rows mostly from the L2.
    // Weights that no other piece reads pass by the caches (non-temporal):
    // 7-12% of the call on the layers measured below.
    const uint32_t b_st = q_stage + (kD * kA + wave * kD * kB) * 1024;
    if (q.once) {
#pragma unroll
      for (int i = 0; i < kD * kB; ++i)
        dma16<true>(Bb + i / kB * 1024, i % kB * b_next + blk_lane, b_st + i * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < kD * kB; ++i)
        dma16(Bb + i / kB * 1024, i % kB * b_next + blk_lane, b_st + i * 1024);
    }
#pragma unroll
    for (int j = 0; j < kAPer; ++j) dma16(Ab, offA[j], q_stage + (wave * kAPer + j) * 1024);
    Bb += kD * 1024;
    Ab += kD * (kPhase == 0 ? 64 : 1024);
    q_stage = q_stage == ring0 + (kRing - 1) * kStage ? ring0 : q_stage + kStage;
    ++issued;
    if (++q_k == nk && issued < total) {
      q_k = 0;
      advance(q);
      setup();
    }
  };
  for (int i = 0; i < kRing - 1 && i < total; ++i) request();

  Unit c;
  c.piece = u0 / n_unit;
  c.col = u0 - c.piece * n_unit;
  load_piece(c);
  int done = 0;
  const char *stage = ring;
  for (int u = 1;; ++u) {
    f32x16 acc[kMT][kU];
#pragma unroll
    for (int m = 0; m < kMT; ++m)
#pragma unroll
      for (int v = 0; v < kU; ++v)
#pragma unroll
        for (int s = 0; s < 16; ++s) acc[m][v][s] = 0.0f;
    for (int k = 0; k < nk; ++k) {
      // Stage `done` has landed once at most the later ones asked for are in
      // flight (requests complete in order; stores of an epilogue in between
      // only make this wait longer), and the reads of the stage before it are
      // done, so that one can be asked for again; with a shared ring, both
      // hold for every wave after the barrier.
      asm volatile("" ::: "memory");
      if (issued - done == kRing - 1)
        wait_cnt<(kRing - 2) * kPer, 0>();
      else
        wait_cnt<0, 0>();
      if (kShare > 1) __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      if (issued < total) request();
      ++done;
      const uint16_t *a_s = reinterpret_cast<const uint16_t *>(stage);
      const uint16_t *b_s = a_s + (kD * kA + col_w * kD * kB) * 512;
      bf16x8 fa[2 * kD][kMT], fb[2 * kD][kU];
#pragma unroll
      for (int s = 0; s < 2 * kD; ++s) {
        const int kc = (s & 1) * 2 + h;
#pragma unroll
        for (int v = 0; v < kU; ++v)
          fb[s][v] = *reinterpret_cast<const bf16x8 *>(
              &b_s[(v * kD + (s >> 1)) * kB * 512 + lds_swz32(lane & 31, kc)]);
#pragma unroll
        for (int m = 0; m < kMT; ++m) {
          const int r = kA == 1 ? lane & 15 : row_w + m * 32 + (lane & 31);
          fa[s][m] = *reinterpret_cast<const bf16x8 *>(
              kPhase == 0 ? &a_s[r * 64 + (((2 * s + h) ^ ((r >> 1) & 7)) << 3)]
                          : &a_s[(s >> 1) * kA * 512 + lds_swz32(r, kc)]);
        }
      }
#pragma unroll
      for (int s = 0; s < 2 * kD; ++s)
#pragma unroll
        for (int m = 0; m < kMT; ++m)
#pragma unroll
          for (int v = 0; v < kU; ++v)
            acc[m][v] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[s][v], fa[s][m], acc[m][v], 0, 0, 0);
      stage = stage == ring + (kRing - 1) * kStage ? ring : stage + kStage;
    }
    // Lane l holds row l % 32 of each 32-row block and, in slots 4 g + e, the
    // column 8 g + 4 (l / 32) + e of the unit's 32 weight rows. After the
    // half-wave swaps a lane has eight consecutive columns.
#pragma unroll
    for (int mv = 0; mv < kMT * kU; ++mv) {
      const int m = mv / kU, v = mv % kU;
      const int col = kShare * c.col + col_w + v;
      const int row = row_w + m * 32 + (lane & 31);  // of the piece
      const int xrow = t.row[c.place + min(row, c.rows - 1)];  // its row in x_perm
      const bool ok = row < c.rows && col < n_col;
      auto eight = [&](const float *f) {
        uint32_t a0 = pack_bf16x2(f[0], f[1]), a1 = pack_bf16x2(f[2], f[3]);
        uint32_t a2 = pack_bf16x2(f[4], f[5]), a3 = pack_bf16x2(f[6], f[7]);
        swap_halves(a0, a2);
        swap_halves(a1, a3);
        return make_uint4(a0, a1, a2, a3);
      };
      float lo[8], hi[8];
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        lo[s] = acc[m][v][s];
        hi[s] = acc[m][v][8 + s];
      }
      if (kPhase == 0) {
        // slots 0-7: 16 gate columns, slots 8-15: the matching up columns
        const int f = 16 * col;
        if (a.gu_save) {
          uint16_t *gr = a.gu_save + int64_t(xrow) * 2 * a.N + 64 * (f >> 5) + (f & 31) + 8 * h;
          const uint4 g8 = eight(lo), u8 = eight(hi);
          if (ok) {
            *reinterpret_cast<uint4 *>(gr) = g8;
            *reinterpret_cast<uint4 *>(gr + 32) = u8;
          }
        }
        float hv[8];
#pragma unroll
        for (int s = 0; s < 8; ++s)
          hv[s] = lo[s] * __builtin_amdgcn_rcpf(1.0f + __expf(-lo[s])) * hi[s];
        const uint4 h8 = eight(hv);
        if (ok)
          *reinterpret_cast<uint4 *>(a.C + (int64_t(c.block + (row >> 4)) * (a.N >> 5) + (f >> 5)) * 512 +
                                     (row & 15) * 32 + (f & 31) + 8 * h) = h8;
      } else {
        uint16_t *cr = a.C + int64_t(xrow) * a.N + 32 * col + 8 * h;
        const uint4 l8 = eight(lo), h8 = eight(hi);
        if (ok) {
          *reinterpret_cast<uint4 *>(cr) = l8;
          *reinterpret_cast<uint4 *>(cr + 16) = h8;
        }
      }
    }
    if (u == count) break;
    advance(c);
  }
}

template <int kPhase>
__global__ __launch_bounds__(kStreamThreads)
__attribute__((amdgpu_waves_per_eu(1, 1))) void stream_ffn_kernel(StreamArgs a) {
  __shared__ __attribute__((aligned(1024))) char rings[kStreamLds];
  __shared__ StreamTable t;
  int first[kClasses + 1];
  const int n_col = a.N / (kPhase == 0 ? 16 : 32);
  build_table(a, t, *reinterpret_cast<StreamBuild *>(rings), (n_col + 3) / 4, first);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  // Every XCD takes an eighth of each class's units (workgroups are dealt
  // round-robin over the XCDs). Its shared units go to its workgroups in turn,
  // so that the ones at work together share a piece's rows in the L2 (dealt
  // over all XCDs, the rows came from behind the L2s: 15% more time with 256
  // rows per expert). Its lone units are split so that the workgroups end
  // together by the estimated times below (a lone unit: 4). No counter, which
  // would have to be cleared first.
  constexpr int kCost[kClasses] = {48, 28, 20, 18, 4};
  constexpr int kLone = kClasses - 1;
  static_assert(int64_t(kMaxPieces) * (LLEP_MAX_FFN_DIM / 16) * 64 < INT32_MAX, "units");
  const int xcd = blockIdx.x % 8, me = blockIdx.x / 8, per = gridDim.x / 8;
  int u0[kClasses], k[kClasses];  // first unit and units of this workgroup
  const int lane = lane_id();
  int mine = 0;  // time of the shared units of workgroup `lane` of the XCD
  int all = 0;   // of all units of the XCD
  int turn = 0;
#pragma unroll
  for (int c = 0; c < kLone; ++c) {
    const int n = (first[c + 1] - first[c]) * ((n_col + 3) / 4);
    const int x0 = n * xcd / 8, cnt = n * (xcd + 1) / 8 - x0;
    auto place = [&](int j) { return j >= turn ? j - turn : j - turn + per; };
    auto units = [&](int j) { return place(j) < cnt ? (cnt - 1 - place(j)) / per + 1 : 0; };
    u0[c] = x0 + place(me);
    k[c] = units(me);
    mine += units(lane) * kCost[c];
    all += cnt * kCost[c];
    turn = (turn + cnt) % per;
  }
  {
    const int n = (first[kClasses] - first[kLone]) * n_col;
    const int x0 = n * xcd / 8, cnt = n * (xcd + 1) / 8 - x0;
    int a0 = cnt * me / per, a1 = cnt * (me + 1) / per;
    if (all > 0 && cnt > 0) {
      // in proportion to what a workgroup's shared units leave of the mean
      int room = lane < per ? max(0, (all + cnt * kCost[kLone]) / per - mine) : 0;
      if (__ballot(room > 0) == 0) room = lane < per;
      int incl = room;
      for (int off = 1; off < kWave; off <<= 1) {
        const int v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
      }
      const int sum = __shfl(incl, kWave - 1);
      const int at1 = __shfl(incl, me), at0 = at1 - __shfl(room, me);
      // exact at both ends (products below 2^53)
      a0 = int(double(cnt) * at0 / sum);
      a1 = int(double(cnt) * at1 / sum);
    }
    const int w0 = (a1 - a0) * wave / kStreamWaves, w1 = (a1 - a0) * (wave + 1) / kStreamWaves;
    u0[kLone] = x0 + a0 + w0;
    k[kLone] = w1 - w0;
  }
#pragma unroll
  for (int c = 0; c < kClasses; ++c) {
    u0[c] = __builtin_amdgcn_readfirstlane(u0[c]);
    k[c] = __builtin_amdgcn_readfirstlane(k[c]);
  }
  stream_units<kPhase, 16, 2, 4, 2>(a, t, first[0], rings, u0[0], per, k[0]);
  __syncthreads();  // every wave is done with the ring before the next class fills it
  stream_units<kPhase, 8, 2, 4, 2>(a, t, first[1], rings, u0[1], per, k[1]);
  __syncthreads();
  stream_units<kPhase, 4, 2, 4, 1>(a, t, first[2], rings, u0[2], per, k[2]);
  __syncthreads();
  stream_units<kPhase, 2, 2, 4, 1>(a, t, first[3], rings, u0[3], per, k[3]);
  __syncthreads();
  stream_units<kPhase, 1, 2, 1, 1>(a, t, first[4], rings + wave * (kStreamLds / kStreamWaves),
                                u0[4], 1, k[4]);
}

// Where the weight stream runs. Times are of the tiles / the stream in us, with
// uniform, Zipf(1.2) and hot routings (50-95% of the rows on one to four
// experts) on 1 and 8 devices; the routing is not known here.
//
// Every group: the tiles take 60-100 us from end to end however few there are,
// and then work at the higher rate on a hot expert's rows.
// - Up to 24 rows per expert on average and 1024 rows the stream wins or is
//   even (2880 x 2880: 32 experts, 768 rows, uniform 308 / 260, Zipf 311 / 283;
//   64 experts, 896 rows, Zipf on one device 519 / 512; 128 experts, 1024 rows,
//   80% on four 851 / 815). At the line up to 5% are lost with 95% of the rows
//   on one expert, and on some routings of 7168 x 2048 layers, both on one
//   device (128 experts of 2880 x 2880, 1024 rows, 95%: 342 / 356; 64 of 7168 x
//   2048, 896 rows, Zipf: 877 / 913).
//   Beyond it every skewed routing loses: 64 of 7168 x 2048 with 1536 rows 926 /
//   967 (Zipf) and 661 / 757 (95%), 128 of 2880 x 2880 with 3072 rows 1132 /
//   1146 and 781 / 854, for 2-7% that a uniform one gains.
// - While the whole call is short it wins whatever the rows per expert, down to
//   a single one: up to D F R = 5 10^9 (16 experts of 1024 x 768, R = 4096:
//   92-94 / 56-65; one expert of 2880 x 2880, R = 602: 133 / 107; 64 of 2048 x
//   768, R = 3178, 90% on one: 162 / 145), with more than 64 experts up to 4
//   10^9 (128 of 2048 x 768, Zipf: R = 2176 216 / 217, R = 3072 229 / 234).
//
// One device of several: its range is a part of the rows and experts, so the
// tiles have still less to fill the chip with (the device of most rows of 8, 64
// experts of 2880 x 2880, 1536 rows, 80% on one expert: 161 / 96). Up to the
// rows per expert or the size of above the stream is kept while the rows that
// the device can hold, the plan's capacity or for standard expert parallelism
// all of them, have D F rows <= 2 10^10 (all rows of 128 experts of 2880 x 2880
// on 8 devices, standard plan, Zipf: 2048 rows 233 / 230, 3072 rows 252 / 256
// and 259 / 292 with 95% on one expert).
bool use_stream_ffn(const FfnArgs &a) {
  if (a.R > kStreamRows) return false;
  const bool few = a.R <= int64_t(24) * a.E;
  const int64_t weight = int64_t(a.D) * a.F, work = weight * a.R;
  if (a.device >= 0 && a.P > 1)
    return (few || work <= int64_t(5000000000)) && weight * a.device_rows <= int64_t(20000000000);
  return (few && a.R <= 1024) || work <= (a.E <= 64 ? int64_t(5000000000) : int64_t(4000000000));
}

hipError_t launch_stream_ffn(const FfnArgs &a, void *act, hipStream_t stream) {
  // one workgroup per CU, a multiple of 8 (XCDs), at most 64 per XCD
  const int grid = std::min(512, (cu_count() + 7) / 8 * 8);
  StreamArgs s = {};
  s.A = static_cast<const uint16_t *>(a.x_perm);
  s.a_stride = int64_t(a.D) * 2;
  s.B = static_cast<const uint16_t *>(a.w_gate_up);
  s.b_expert_stride = int64_t(2) * a.F * a.D;
  s.b_blk_stride = int64_t(a.D / kSK) * 1024;
  s.C = static_cast<uint16_t *>(act);
  s.gu_save = static_cast<uint16_t *>(a.gate_up_out);
  s.groups = a.groups;
  s.group_begin = a.group_begin;
  s.cap = 2 * a.E + a.P;
  s.device = a.device;
  s.P = a.P;
  s.N = a.F;
  s.nk = a.D / kSK;
  hipLaunchKernelGGL(stream_ffn_kernel<0>, dim3(grid), dim3(kStreamThreads), 0, stream, s);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  s.A = static_cast<const uint16_t *>(act);
  s.a_stride = int64_t(a.F / kSK) * 1024;
  s.B = static_cast<const uint16_t *>(a.w_down);
  s.b_expert_stride = int64_t(a.D) * a.F;
  s.b_blk_stride = int64_t(a.F / kSK) * 1024;
  s.C = static_cast<uint16_t *>(a.out_perm);
  s.gu_save = nullptr;
  s.N = a.D;
  s.nk = a.F / kSK;
  hipLaunchKernelGGL(stream_ffn_kernel<1>, dim3(grid), dim3(kStreamThreads), 0, stream, s);
  return hipGetLastError();
}

}  // namespace llep
