// Attention block around the WERSA core (Section 3.1 steps 1-2: Q' = X W^Q, K' = X W^K,
// V' = X W^V, split into heads; Algorithm 1's closing line: merged heads times W_out) and its
// backward.  The projections are plain dense contractions over hidden = H*d: one bf16 MFMA
// GEMM kernel (float32 accumulation) in three operand forms,
//   NN  C[M][N] = A[M][K] B[K][N]              (forward: activations times weights as they are stored; the three
//       projections in one launch)
//   NT  C[M][N] = sum_s A_s[M][K] B_s[N][K]^T   (both operands contiguous along K; up to three
//       (A, B) pairs summed, which gives dX = dQ' W^Q^T + dK' W^K^T + dV' W^V^T in one pass; many tokens: NN
//       on transposed copies of the weights)
//   TN  C[M][N] = A[K][M]^T B[K][N]            (both operands contiguous across K: the weight
//       gradients X^T dQ' ...; split over K into float32 partials, reduced in fixed order)
// Heads are never transposed: the core reads and writes (B, n, H*d) through its strides.
#include "wersa_internal.h"

namespace wersa {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr int BK = 32;                       // k per stage
constexpr int kStages = 4;                   // LDS stages: one computed on, one landed or landing, two requested
constexpr int kGemmWaves = 4;                // 2 x 2 waves of WT x WT, WT = 128 or 64
constexpr int kBigTile = 256, kSmallTile = 128;   // workgroup tiles (2 WT)
constexpr int kMaxSrc = 3;
constexpr int kMaxSplit = 32;

// One product, or several in one launch.  batch products C[i] = A[i] B[i] of equal shape (the three
// projections, their three weight gradients), or batch = 1 and C[0] = sum of `count` products.
struct GemmJob {
  const bf16_t *a[kMaxSrc];
  const bf16_t *b[kMaxSrc];
  void *c[kMaxSrc];
  int count, batch;
};

// A value the compiler cannot follow: what is derived from it is computed where it is used, not kept in registers.
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

__device__ __forceinline__ bf16_t to_bf16(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }

// 16 bytes per lane from base + voff (bytes) to LDS at lds (bytes, wave-uniform) + 16 * lane, without passing
// through registers.  Written as a statement because the compiler waits for every such load before the next
// LDS read, whatever it reads; the caller counts them (vmcnt) instead.  It has no register outputs.
__device__ __forceinline__ void lds_dma16(uint32_t lds, uint32_t voff, const bf16_t *base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base)
               : "memory", "m0");
}

// Operand forms: TA = false: A [M][K] (lda), its LDS stage [row][32 k] in 64-byte rows; TA = true: A [K][M],
// stage [32 k][row]; TB alike for B [N][K] / [K][N].  Stages are unpadded (a direct load to LDS writes 64
// consecutive 16-byte pieces), so bank conflicts are avoided by permuting the pieces of a row:
//   [row][k]: piece c of row r at slot c ^ ((r / 4) % 4): any 16 rows read one piece each without conflict;
//   [k][row]: piece c of row k at slot c ^ (4 (k % 4)): the 4 k-rows x 64 bytes of a half-wave's transposing
//   read cover all 64 banks.
// OUT_F32: float32 output, one partial per (product, split), else bf16 output.  M, N multiples of 2 WT, every
// K range a multiple of 32.  DMA = false stages through registers: operands whose base is not 16-byte aligned.
//
// What bounds it: per matrix instruction (32 cycles) a wave of WT = 128 reads 0.5 KB of LDS, so a compute unit
// reads 64 B/clk and writes 32 of about 128; with two waves of 128 x 64 per SIMD (the form before) it was 96 + 32,
// the whole LDS bandwidth.  One wave per SIMD hides nothing by itself, so nothing may stall: operands of the next
// 16 k are read between the matrix instructions of the current ones, across the stage boundary too (a stage is
// known to have landed one step before it is needed), and global loads have two steps (2048 cycles) to land.  Reads and
// requests are spread over the 16 instructions of a half, one or the other after most of them: all reads in the first half
// of them and all requests in the second met the peak rates of LDS and of the load path.  The clock falls as the matrix
// units get busier: per tile of 256 x 256 x 2048 (65.5 thousand cycles of matrix instructions) NN takes 91.1 thousand cycles at 1665 MHz, and
// took 95.4 at 1720 before, TN 8 % fewer at a clock 5 % lower.  TN, its matrix cores 85 % busy, is limited by power; NN and NT leave them idle
// for 28 and 32 % of the cycles, why is not shown (requests of operands contiguous along k are half lines: TN has none, NN one, NT two).  A
// fifth stage, or one workgroup per tile, is slower.
//
// A workgroup of WT = 128 takes several tiles, one after the other (one per compute unit in flight).  The stages of its tiles are one
// sequence, so the first stages of the next tile are on their way while the last products and the stores of this one are made;
// the tile leaves through the stage that was computed on last.  bf16 output without column sums: the operands of the matrix
// instruction are exchanged, and B's rows or columns taken with bits 2 and 3 of their number exchanged, so that a lane holds 16-byte
// pieces of its own row of C (32 LDS writes per wave and tile of 128 x 128 instead of 256 two-byte ones).
// Measured against one tile per workgroup and rows on registers (131072 tokens, hidden 2048, 25 training steps of each in turn on one card,
// us per product): NN with column sums 953 -> 921, without 957 -> 858; NT one product 1016 -> 964, sum of three 915 -> 890; TN
// 846 -> 822.  1.1 TFLOP takes 580 us at the 1.9 PFLOP/s that a bare loop of the instruction sustains.
//
// Logical tiles are dealt to the eight XCDs in contiguous runs (workgroup w runs on XCD w % 8); a run goes down
// kGroupM row panels before it takes the next column panel, so that the 32 workgroups of an XCD at a time share
// 4 panels of A and 8 of B in its L2.
//
// colsum (bf16 output form of product 0, may be nullptr): float32 [M / 128][N], the column sums of 128 output rows
// from the float32 accumulators; the block uses them as the pooled-query partial sums of Q' = X W^Q (Section 3.1
// step 4) instead of a separate pass over Q'.  colmax (with colsum): float32 [M / 128][N / 64], the largest
// |accumulator| of 128 rows x 64 columns; the core derives the fp16 operand scale of a (batch, head) slice from them.
constexpr int kGroupM = 4;

template <int WT, bool TA, bool TB, bool OUT_F32, bool DMA, bool COLSUM>
__global__ __launch_bounds__(64 * kGemmWaves, WT == 128 ? 1 : 2) void gemm_bf16_kernel(
    GemmJob job, int lda, int ldb, int ldc, int M, int N, int K, int k_chunk, int splits, float *colsum, float *colmax) {
  constexpr int T = 2 * WT;              // workgroup tile, rows and columns
  constexpr int TI = WT / 32;            // 32 x 32 tiles per wave in each direction
  constexpr int OPB = T * BK * 2;        // bytes of one operand's stage
  constexpr int SB = 2 * OPB;            // bytes of a stage
  constexpr int G = OPB / 1024 / kGemmWaves;   // 1 KB loads per wave, operand and stage
  constexpr int RB = T * 2;              // bytes of a row of a [k][row] stage
  constexpr bool ROWS = !OUT_F32 && !COLSUM;   // accumulators with rows of C on lanes
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  typedef __attribute__((address_space(3))) unsigned char lds_byte;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte *)smem_raw;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31,
            h = lane >> 5;
  const int tm = M / T, tn = N / T * job.batch, tiles = tm * tn, total = tiles * splits;
  const int per = (total + 7) / 8, end = min(per, total - (int)(blockIdx.x % 8) * per);   // of this XCD's run of tiles
  struct Place {
    int m0, n0, which, split, k_begin, k_end;   // which: product of the batch
  };
  auto place = [&](int li) {   // tile li of the run
    const int lt = (blockIdx.x % 8) * per + li, split = lt / tiles, tile = lt % tiles;
    const int grp = tile / (kGroupM * tn), rest = tile - grp * kGroupM * tn, rows = min(kGroupM, tm - grp * kGroupM);
    const int nb = rest / rows, mt = grp * kGroupM + rest % rows, which = nb / (N / T);
    return Place{mt * T, (nb - which * (N / T)) * T, which, split, split * k_chunk, min(K, split * k_chunk + k_chunk)};
  };
  const int stride = gridDim.x / 8;
  if ((int)(blockIdx.x / 8) >= end) return;
  const int wm = (wave >> 1) * WT, wn = (wave & 1) * WT;

  // Source offsets of this lane's piece in the wave's G loads of each operand (bytes from the stage's corner).
  uint32_t va[G], vb[G];
#pragma unroll
  for (int u = 0; u < G; ++u) {
    const int ins = wave * G + u;
    auto off = [&](bool kmajor, int ld) -> uint32_t {
      if (!kmajor) {
        const int r = 16 * ins + (lane >> 2), c = (lane & 3) ^ ((lane >> 4) & 3);
        return (uint32_t)(r * ld * 2 + c * 16);
      }
      constexpr int PR = RB / 16, KR = 64 / PR;   // pieces per k row, k rows per load
      const int k = KR * ins + lane / PR, c = (lane % PR) ^ ((k & 3) << 2);
      return (uint32_t)(k * ld * 2 + c * 16);
    };
    va[u] = off(TA, lda);
    vb[u] = off(TB, ldb);
  }
  // The next stage to request; requests run ahead of the products, over the end of a tile into the next one.
  int li_next = blockIdx.x / 8;
  Place rq = place(li_next);
  int src = rq.which, left = (rq.k_end - rq.k_begin) / BK;   // stages of this source to request, this one counted
  auto corner = [&](const bf16_t *p, bool kmajor, int ld, int o0) {
    return p + (kmajor ? (int64_t)rq.k_begin * ld + o0 : (int64_t)o0 * ld + rq.k_begin);
  };
  const bf16_t *pa = corner(job.a[src], TA, lda, rq.m0), *pb = corner(job.b[src], TB, ldb, rq.n0);
  const int64_t da = TA ? (int64_t)BK * lda : BK, db = TB ? (int64_t)BK * ldb : BK;
  auto next_source = [&]() {   // pa and pb already point to the next stage of this source
    if (__builtin_expect(--left > 0, 1)) return;
    if (src - rq.which + 1 < job.count) {
      ++src;
    } else if (li_next + stride < end) {
      li_next += stride;
      rq = place(li_next);
      src = rq.which;
    }   // after the last stage of the last tile the last source is requested again, and never read
    left = (rq.k_end - rq.k_begin) / BK;
    pa = corner(job.a[src], TA, lda, rq.m0);
    pb = corner(job.b[src], TB, ldb, rq.n0);
  };
  typedef u16x8 u16x8_any __attribute__((aligned(2)));
  auto request = [&](int stage, int u, bool is_b) {
    const uint32_t at = (uint32_t)(stage * SB + (is_b ? OPB : 0) + (wave * G + u) * 1024);
    if (DMA) {
      lds_dma16(lds0 + at, is_b ? vb[u] : va[u], is_b ? pb : pa);
    } else {
      const u16x8 piece = *reinterpret_cast<const u16x8_any *>(reinterpret_cast<const unsigned char *>(is_b ? pb : pa) +
                                                               (is_b ? vb[u] : va[u]));
      *reinterpret_cast<u16x8 *>(smem_raw + at + 16 * lane) = piece;
    }
  };

  // Operand i of 16 k: A rows wm + 32 i .., or B columns wn + 32 i ...  [row][k]: one 16-byte read at row l32, k = 8 h.
  // [k][row]: the transposing read of gfx950 (ds_read_b64_tr_b16): within each group of 16 lanes, lane i passes the
  // address of four consecutive 16-bit values, taken as row i / 4, columns 4 (i % 4) .. + 3 of a 4 x 16 block, and
  // receives column i of that block.  (Lane mapping checked on the GPU with an index-valued LDS array.)
  typedef __attribute__((address_space(3))) s16x4 *lds_s16x4_ptr;
  typedef __attribute__((address_space(3))) bf16x8 *lds_bf16x8_ptr;
  const int i16 = lane & 15, g16 = (lane >> 4) & 1;
  // swap: lane l32 takes row or column l32 with bits 2 and 3 exchanged.
  auto lane_off = [&](bool kmajor, int w0, int i, bool swap) -> uint32_t {   // of operand i at ks = 0
    if (!kmajor) {
      const int r = swap ? (l32 & 19) | (l32 & 4) << 1 | (l32 & 8) >> 1 : l32;
      return (uint32_t)((w0 + 32 * i + r) * 64 + (h ^ ((r >> 2) & 3)) * 16);
    }
    const int four = swap ? (i16 & 1) << 1 | (i16 & 2) >> 1 : i16 & 3;
    const int piece = (w0 / 8 + 4 * i + 2 * g16 + (four >> 1)) ^ ((i16 >> 2) << 2);
    return (uint32_t)((8 * h + (i16 >> 2)) * RB + piece * 16 + (four & 1) * 8);
  };
  uint32_t oa[TI], ob[TI];
#pragma unroll
  for (int i = 0; i < TI; ++i) {
    oa[i] = lds0 + lane_off(TA, wm, i, false);
    ob[i] = lds0 + OPB + lane_off(TB, wn, i, ROWS);
  }
  auto operand = [&](bool kmajor, uint32_t base, int ks) -> bf16x8 {
    if (!kmajor) return *(lds_bf16x8_ptr)(ks ? base ^ 32u : base);   // piece 2 ks + h, permuted
    const uint32_t p = base + (uint32_t)(16 * ks * RB);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 4 * RB));
    s16x8 r;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      r[q] = lo[q];
      r[4 + q] = hi[q];
    }
    return __builtin_bit_cast(bf16x8, r);
  };

  f32x16 acc[TI][TI];
  // A wave's own loads up to the last `2 G` have landed; then every wave's.  (Its reads of the stage that is requested next went
  // into matrix instructions that are issued.)  Loads and stores are counted in order: the two steps after a tile's stores let
  // as many more operations be under way.
  constexpr int STORES = OUT_F32 ? TI * TI * 16 : TI * WT / 16, LATER = 2 * G + STORES < 63 ? 2 * G + STORES : 63;
  auto arrive = [&](bool stored) {
    if (!DMA) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // pieces written through registers
    if (stored)
      asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(LATER) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * G) : "memory");
  };
#pragma unroll
  for (int s = 0; s < kStages - 1; ++s) {
#pragma unroll
    for (int u = 0; u < G; ++u) {
      request(s, u, false);
      request(s, u, true);
    }
    pa += da;
    pb += db;
    next_source();
  }
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(4 * G) : "memory");
  bf16x8 a0[TI], b0[TI], a1[TI], b1[TI];
  // Sixteen (four) matrix instructions on one set of operands with the reads of the next set and the requests of a later
  // stage between them.
  auto half = [&](auto first, const bf16x8 *a, const bf16x8 *b, bf16x8 *an, bf16x8 *bn, uint32_t stage, int ks, int into, bool req_b) {
    constexpr int MM = TI * TI;
#pragma unroll
    for (int x = 0; x < MM; ++x) {
      const int i = x / TI, j = x % TI;
      const f32x16 c = decltype(first)::value ? f32x16{} : acc[i][j];
      acc[i][j] = ROWS ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], a[i], c, 0, 0, 0)
                       : __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], c, 0, 0, 0);
      if (MM == 16 ? (x & 1) == 0 : true) {   // A 0, B 0 .. TI - 1, A 1 ..: the order in which the next half takes them
        const int e = MM == 16 ? x / 2 : x;
        if (e == 0 || e > TI) an[e ? e - TI : 0] = operand(TA, oa[e ? e - TI : 0] + stage, ks);
        else bn[e - 1] = operand(TB, ob[e - 1] + stage, ks);
      }
      if (MM == 16 ? (x & 3) == 1 : x >= 2) {
        const int u = MM == 16 ? x / 4 : x - 2;
        if (u < G) request(into, u, req_b);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  int slot = 0;   // of the current stage
  auto step = [&](auto first, bool stored) {
    const int cur = slot, nxt = (slot + 1) % kStages, into = (slot + kStages - 1) % kStages;
    arrive(stored);   // the next stage has landed; every wave is done with the stage before, which `into` overwrites
    half(first, a0, b0, a1, b1, (uint32_t)(cur * SB), 1, into, false);
    pa += da;
    half(std::false_type{}, a1, b1, a0, b0, (uint32_t)(nxt * SB), 0, into, true);
    pb += db;
    slot = nxt;
    next_source();
  };
  for (int li = blockIdx.x / 8; li < end; li += stride) {
    const bool later = li != (int)(blockIdx.x / 8);
    const Place at = place(li);
    const int m0 = at.m0, n0 = at.n0, which = at.which;
    const int steps = (at.k_end - at.k_begin) / BK * job.count;
    // The last step of the tile before has read these operands too; a second time here costs less than their registers while
    // the tile is written.
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      a0[i] = operand(TA, oa[i] + slot * SB, 0);
      b0[i] = operand(TB, ob[i] + slot * SB, 0);
    }
    step(std::true_type{}, later);
    for (int s = 1; s < steps; ++s) step(std::false_type{}, later && s == 1);
    unsigned char *const free_stage = smem_raw + (slot + kStages - 1) % kStages * SB;   // the next request into it is after the next barrier

    if (OUT_F32) {
      // acc[i][j][r]: row wm + 32 i + 8 (r / 4) + 4 h + (r % 4), column wn + 32 j + l32.
      const int lane = opaque(threadIdx.x & 63), l32 = lane & 31, h = lane >> 5;
      float *C = splits == 1 ? reinterpret_cast<float *>(job.c[which])
                             : reinterpret_cast<float *>(job.c[0]) + ((int64_t)which * splits + at.split) * M * ldc;
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TI; ++j) {
          if (WT == 128) asm volatile("" : "+a"(acc[i][j]));   // stays where the products leave it until here
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int row = m0 + wm + 32 * i + 8 * (r >> 2) + 4 * h + (r & 3);
            C[(int64_t)row * ldc + n0 + wn + 32 * j + l32] = acc[i][j][r];
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      continue;
    }
    const int lane = opaque(threadIdx.x & 63), l32 = lane & 31, h = lane >> 5;   // addresses of this part are not kept over the products
    bf16_t *C = reinterpret_cast<bf16_t *>(job.c[which]);
    asm volatile("s_barrier" ::: "memory");   // every wave is done with the free stage
    // Column sums: per column one chain over a lane's 64 of the 128 rows.  WT = 128 adds while the rows are written (for every
    // product: the sums cost less than a second reading of the accumulators); with WT = 64 rows 64 .. 127 are another wave's,
    // which goes on from where the first one stopped, so that the sums have the same bits with either tile.
    float sum[TI], mx[TI];
#pragma unroll
    for (int j = 0; j < TI; ++j) sum[j] = mx[j] = 0.f;
    auto add = [&](int j, float v) {
      sum[j] += v;
      mx[j] = fmaxf(mx[j], fabsf(v));
    };
    if (COLSUM && WT == 64 && which == 0) {
      auto add_rows = [&]() {
#pragma unroll
        for (int j = 0; j < TI; ++j)
#pragma unroll
          for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) add(j, acc[i][j][r]);
      };
      float *carry = reinterpret_cast<float *>(free_stage) + (wave & 1) * (2 * TI * 64) + lane;
      if (wave < 2) {
        add_rows();
#pragma unroll
        for (int j = 0; j < TI; ++j) {
          carry[64 * j] = sum[j];
          carry[64 * (TI + j)] = mx[j];
        }
      }
      __syncthreads();
      if (wave >= 2) {
#pragma unroll
        for (int j = 0; j < TI; ++j) {
          sum[j] = carry[64 * j];
          mx[j] = carry[64 * (TI + j)];
        }
        add_rows();
      }
      __syncthreads();
    }
    // bf16 through a wave-private tile of 32 rows x WT columns: rows as whole lines.  Piece c (16 bytes) of row r at slot
    // c ^ f(r), where f separates the rows that one write covers.
    constexpr int PPR = WT / 8, RPS = 64 / PPR;   // pieces per row, rows per store
    unsigned char *tl = free_stage + wave * (32 * WT * 2);
    auto at_piece = [&](int r, int c) {
      const int f = ROWS ? (WT == 128 ? r & 15 : r >> 1 & 7) : (WT == 128 ? (r & 1) << 2 | (r & 4) << 1 : r & 4);
      return r * (WT * 2) + (c ^ f) * 16;
    };
    auto put = [&](int i) {
#pragma unroll
      for (int j = 0; j < TI; ++j) {
        if (WT == 128) asm volatile("" : "+a"(acc[i][j]));   // stays where the products leave it until here
        if (ROWS) {   // acc[i][j][r]: row wm + 32 i + l32, column wn + 32 j + 16 (r / 8) + 8 h + (r % 8)
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            u16x8 piece;
#pragma unroll
            for (int e = 0; e < 8; ++e) piece[e] = to_bf16(acc[i][j][8 * g + e]);
            *reinterpret_cast<u16x8 *>(tl + at_piece(l32, 4 * j + 2 * g + h)) = piece;
          }
        } else {
          // acc[i][j][r]: row wm + 32 i + 8 (r / 4) + 4 h + (r % 4), column wn + 32 j + l32.  Of rows r and r + 1 an even lane takes
          // row r of its column and the next, an odd lane row r + 1 of its column and the one before.
#pragma unroll
          for (int r = 0; r < 16; r += 2) {
            if (COLSUM && WT == 128) {
              add(j, acc[i][j][r]);
              add(j, acc[i][j][r + 1]);
            }
            typedef __bf16 pair __attribute__((ext_vector_type(2)));
            const uint32_t own = __builtin_bit_cast(uint32_t, pair{(__bf16)acc[i][j][r], (__bf16)acc[i][j][r + 1]});
            const uint32_t other = (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xB1, 0xF, 0xF, true);   // lane ^ 1
            const uint32_t word = __builtin_amdgcn_perm(other, own, lane & 1 ? 0x03020706u : 0x05040100u);
            const int row = 8 * (r >> 2) + 4 * h + (r & 3) + (lane & 1);
            *reinterpret_cast<uint32_t *>(tl + at_piece(row, 4 * j + (l32 >> 3)) + (l32 & 6) * 2) = word;
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    put(0);
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      u16x8 piece[32 / RPS];
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int u = 0; u < 32 / RPS; ++u)
        piece[u] = *reinterpret_cast<const u16x8 *>(tl + at_piece(RPS * u + lane / PPR, lane % PPR));
      __builtin_amdgcn_wave_barrier();
      if (i + 1 < TI) put(i + 1);
#pragma unroll
      for (int u = 0; u < 32 / RPS; ++u)
        *reinterpret_cast<u16x8 *>(C + (int64_t)(m0 + wm + 32 * i + RPS * u + lane / PPR) * ldc + n0 + wn + lane % PPR * 8) = piece[u];
    }
    if (COLSUM && which == 0) {
#pragma unroll
      for (int j = 0; j < TI; ++j)
        sum[j] += __shfl_xor(sum[j], 32, 64);   // the two half-waves hold the two halves of every 8-row group
      if (WT == 128 || wave >= 2) {
        const int64_t blk = (m0 + wm) >> 7;
        static_assert(kPooledMaxCols == 64, "two column tiles per maximum");
#pragma unroll
        for (int j = 0; j < TI; ++j) {
          if (h == 0) colsum[blk * N + n0 + wn + 32 * j + l32] = sum[j];
          if (colmax && (j & 1)) {
            float v = fmaxf(mx[j - 1], mx[j]);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
            if (lane == 0) colmax[blk * (N / 64) + (n0 + wn) / 64 + j / 2] = v;
          }
        }
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no load may land in LDS that is no longer this workgroup's
}

// out[e] = sum over splits of part[split][e], fixed order; blockIdx.y: product of the batch.
__global__ void splitk_reduce_kernel(const float *part, int splits, int64_t count, float *out0, float *out1, float *out2) {
  const int64_t e = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (e >= count) return;
  part += (int64_t)blockIdx.y * splits * count;
  float *out = blockIdx.y == 0 ? out0 : (blockIdx.y == 1 ? out1 : out2);
  float4 acc = *reinterpret_cast<const float4 *>(part + e);
  for (int s = 1; s < splits; ++s) {
    const float4 v = *reinterpret_cast<const float4 *>(part + (int64_t)s * count + e);
    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
  }
  *reinterpret_cast<float4 *>(out + e) = acc;
}

// out[i] = w[i]^T for up to three hidden x hidden matrices (blockIdx.z), one 64 x 64 tile per workgroup; w's base may be any.
struct TransposeJob {
  const bf16_t *w[kMaxSrc];
  bf16_t *out[kMaxSrc];
};
__global__ __launch_bounds__(256) void transpose_kernel(TransposeJob job, int hidden) {
  constexpr int LS = 64 + 2;   // (rows 33 words apart: a column's values are in different banks)
  __shared__ bf16_t tile[64 * LS];
  typedef u16x8 u16x8_any __attribute__((aligned(2)));
  typedef uint32_t u32_any __attribute__((aligned(4)));
  const bf16_t *w = job.w[blockIdx.z];
  bf16_t *out = job.out[blockIdx.z];
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int e = threadIdx.x + 256 * u, r = e >> 3, c = (e & 7) * 8;
    const u16x8 v = *reinterpret_cast<const u16x8_any *>(w + (int64_t)(r0 + r) * hidden + c0 + c);
#pragma unroll
    for (int q = 0; q < 8; q += 2) *reinterpret_cast<u32_any *>(&tile[r * LS + c + q]) = (uint32_t)v[q] | (uint32_t)v[q + 1] << 16;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int e = threadIdx.x + 256 * u, c = e >> 3, r = (e & 7) * 8;
    u16x8 v;
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = tile[(r + q) * LS + c];
    *reinterpret_cast<u16x8 *>(out + (int64_t)(c0 + c) * hidden + r0 + r) = v;
  }
}

// A grid of large tiles is one workgroup per compute unit, each takes several tiles.  Large tiles from one per compute unit on; fewer leave units idle.  Block inference, all products in large tiles against
// this rule: 2048 tokens, hidden 512 (48 and 16 large tiles) 68.7 -> 53.2 us; 4096 tokens, hidden 1024 (192 and 64)
// 115.9 -> 106.8; 8192 tokens (384, large either way, and 128) 161.8 -> 156.2; 16384 tokens (all large) 251.9, 251.8.
constexpr int kBigTileMin = 256, kComputeUnits = 256;

template <int WT, bool TA, bool TB, bool OUT_F32, bool DMA, bool COLSUM>
hipError_t launch_gemm_tile(const char *name, const GemmJob &job, int ld, int M, int N, int K, int k_chunk, int splits,
                            hipStream_t st, float *colsum, float *colmax) {
  constexpr size_t stage = (size_t)2 * (2 * WT) * BK * sizeof(bf16_t);
  constexpr size_t smem = kStages * stage;
  static_assert(stage >= (size_t)kGemmWaves * 32 * WT * sizeof(bf16_t), "the tiles on their way out fit into a stage");
  auto kern = &gemm_bf16_kernel<WT, TA, TB, OUT_F32, DMA, COLSUM>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  const int total = (M / (2 * WT)) * (N / (2 * WT)) * job.batch * splits;
  const int grid = min(((total + 7) / 8) * 8, WT == 128 ? kComputeUnits : INT_MAX);
  WERSA_STAGE(name, st, kern<<<grid, 64 * kGemmWaves, smem, st>>>(job, ld, ld, ld, M, N, K, k_chunk, splits, colsum, colmax));
  return hipSuccess;
}

template <bool TA, bool TB, bool OUT_F32, bool COLSUM = false>
hipError_t launch_gemm(const char *name, const GemmJob &job, int ld, int M, int N, int K, int k_chunk, int splits,
                       hipStream_t st, float *colsum = nullptr, float *colmax = nullptr) {
  bool aligned = true;   // direct loads to LDS take 16-byte aligned sources
  for (int i = 0; i < job.count * job.batch; ++i)
    aligned = aligned && ((uintptr_t)job.a[i] | (uintptr_t)job.b[i]) % 16 == 0;
  const int64_t big = (int64_t)(M / kBigTile) * (N / kBigTile) * job.batch * splits;
  if (!aligned)
    return launch_gemm_tile<64, TA, TB, OUT_F32, false, COLSUM>(name, job, ld, M, N, K, k_chunk, splits, st, colsum, colmax);
  if (big >= kBigTileMin)
    return launch_gemm_tile<128, TA, TB, OUT_F32, true, COLSUM>(name, job, ld, M, N, K, k_chunk, splits, st, colsum, colmax);
  return launch_gemm_tile<64, TA, TB, OUT_F32, true, COLSUM>(name, job, ld, M, N, K, k_chunk, splits, st, colsum, colmax);
}

constexpr int kMinChunk = 256;   // tokens

size_t up256(size_t x) { return (x + 255) / 256 * 256; }
struct BlockPlan {
  int64_t tokens, hidden, act;   // act = tokens * hidden elements
  int splits, k_chunk;           // split of the token axis for the weight gradients
  int wgrads;                    // weight gradients of Q, K, V per launch: 3 or 1
  bool transpose;                // the backward's products with a weight's transpose take a transposed copy
  wersa_desc core;
};

BlockPlan block_plan(const wersa_desc &c) {
  BlockPlan p{};
  p.tokens = (int64_t)c.B * c.n;
  p.hidden = (int64_t)c.H * c.d;
  p.act = p.tokens * p.hidden;
  // Weight gradients: 1024 workgroups of the large tile per product, at least 256 tokens each.  (512 make the float32 chain
  // over the tokens of a split twice as long; 131072 tokens, hidden 2048: 826 us per product and 26 for the sum of the partials
  // instead of 856 and 45.)
  const int64_t tiles = (p.hidden / kBigTile) * (p.hidden / kBigTile);
  int64_t z = 1024 / tiles;
  if (z > kMaxSplit) z = kMaxSplit;
  if (z > p.tokens / kMinChunk) z = p.tokens / kMinChunk;
  if (z < 1) z = 1;
  const int64_t steps = (p.tokens / BK + z - 1) / z;
  p.k_chunk = (int)(steps * BK);
  p.splits = (int)((p.tokens + p.k_chunk - 1) / p.k_chunk);
  // Three in one launch while their partials stay below 512 MiB (hidden 1024: 402 MB).  At hidden 2048 one product fills the chip
  // four times over and three launches with a third of the partials (805 -> 268 MB) take the same time (856 us each, 131072 tokens).
  p.wgrads = (int64_t)kMaxSrc * p.splits * p.hidden * p.hidden * 4 <= (int64_t)512 << 20 ? 3 : 1;
  p.core = c;
  p.core.stride_n = p.hidden;
  p.core.stride_h = c.d;
  p.core.stride_b = (int64_t)c.n * p.hidden;
  // With a transposed copy of the weight the second operand's requests are whole lines (see gemm_bf16_kernel): dA 964 -> 828 us, dX 859 -> 831 per
  // product at 131072 tokens, hidden 2048; the copies take 4 us each.  us per training step without and with them: hidden 512, 16384 tokens 369, 371,
  // 32768 523, 521, 131072 1588, 1571; 1024, 16384 799, 810, 32768 1285, 1271, 131072 4064, 4002; 2048, 8192 1320, 1322, 16384 2115, 2098, 32768
  // 3721, 3672, 131072 13196, 12952.
  // The copies lie in the core's workspace, before and after its own use of it.
  p.transpose = p.tokens >= 32768 && wersa_workspace_bytes(&p.core, 1) >= 3 * up256((size_t)p.hidden * p.hidden * 2);
  return p;
}

// Byte layouts. saved: Q' | K' | V' | A (bf16, (B, n, hidden)) | the core's saved buffer.
struct BlockSaved { size_t qp, kp, vp, a, core, total; };
struct BlockWs { size_t qsums, qmax, dA, dQp, dKp, dVp, part, core, total; };

BlockSaved block_saved(const BlockPlan &p) {
  BlockSaved s{};
  size_t off = 0;
  const size_t act = up256((size_t)p.act * 2);
  s.qp = off; off += act;
  s.kp = off; off += act;
  s.vp = off; off += act;
  s.a = off;  off += act;
  s.core = off; off += up256(wersa_saved_bytes(&p.core));
  s.total = off;
  return s;
}

BlockWs block_ws(const BlockPlan &p, int bwd) {
  BlockWs w{};
  size_t off = 0;
  if (!bwd) {
    w.qsums = off; off += up256((size_t)(p.tokens / 128) * p.hidden * 4);   // column sums of Q' per 128 rows
    w.qmax = off;  off += up256((size_t)(p.tokens / 128) * (p.hidden / kPooledMaxCols) * 4);   // and the largest |Q'| per 64 columns
  } else {
    const size_t act = up256((size_t)p.act * 2);
    w.dA = off;  off += act;
    w.dQp = off; off += act;
    w.dKp = off; off += act;
    w.dVp = off; off += act;
    w.part = off; off += p.splits == 1 ? 0 : up256((size_t)p.wgrads * p.splits * p.hidden * p.hidden * 4);   // (one: no partials)
  }
  w.core = off; off += up256(wersa_workspace_bytes(&p.core, bwd));
  w.total = off;
  return w;
}

// The caller's stride fields are ignored (the block lays its tensors out itself): the sizes are
// checked first, then the core descriptor the block builds from them goes through the core's
// own validation.
wersa_status validate_block(const wersa_desc *c) {
  if (!c) return WERSA_ERR_INVALID_ARG;
  if (c->B < 1 || c->H < 1 || c->n < 1 || c->d < 1 || c->m < 1 || c->L < 0) return WERSA_ERR_INVALID_ARG;
  if (c->dtype != WERSA_F32 && c->dtype != WERSA_BF16) return WERSA_ERR_INVALID_ARG;
  if (c->dtype != WERSA_BF16) return WERSA_ERR_UNSUPPORTED;
  const int64_t hidden = (int64_t)c->H * c->d, tokens = (int64_t)c->B * c->n;
  if (hidden % kBigTile != 0 || tokens % kBigTile != 0 || hidden > 16384) return WERSA_ERR_UNSUPPORTED;
  const BlockPlan p = block_plan(*c);
  return validate_desc(&p.core);
}

bool misaligned(const void *p, size_t a) { return ((uintptr_t)p % a) != 0; }

}  // namespace
}  // namespace wersa

using namespace wersa;

extern "C" {

size_t wersa_block_workspace_bytes(const wersa_desc *desc, int for_backward) {
  if (validate_block(desc) != WERSA_OK) return 0;
  return block_ws(block_plan(*desc), for_backward).total;
}

size_t wersa_block_saved_bytes(const wersa_desc *desc) {
  if (validate_block(desc) != WERSA_OK) return 0;
  return block_saved(block_plan(*desc)).total;
}

int64_t wersa_block_saved_offset(const wersa_desc *desc, int which) {
  if (validate_block(desc) != WERSA_OK) return -1;
  const BlockSaved s = block_saved(block_plan(*desc));
  switch (which) {
    case 0: return (int64_t)s.qp;
    case 1: return (int64_t)s.kp;
    case 2: return (int64_t)s.vp;
    case 3: return (int64_t)s.a;
    case 4: return (int64_t)s.core;
    default: return -1;
  }
}

int64_t wersa_block_workspace_offset(const wersa_desc *desc, int which) {
  if (validate_block(desc) != WERSA_OK) return -1;
  const BlockWs w = block_ws(block_plan(*desc), 1);
  switch (which) {
    case 0: return (int64_t)w.dA;
    case 1: return (int64_t)w.dQp;
    case 2: return (int64_t)w.dKp;
    case 3: return (int64_t)w.dVp;
    default: return -1;
  }
}

wersa_status wersa_block_forward(const wersa_desc *desc, const void *x, const void *wq, const void *wk,
                                 const void *wv, const void *wo, const void *omega_rf,
                                 const float *sigma, const float *gate_w, const float *gate_b,
                                 const float *scale_w, void *y, void *saved, void *workspace,
                                 size_t workspace_bytes, void *hip_stream) {
  const wersa_status vs = validate_block(desc);
  if (vs != WERSA_OK) return vs;
  if (!x || !wq || !wk || !wv || !wo || !omega_rf || !sigma || !gate_w || !gate_b || !scale_w || !y || !saved)
    return WERSA_ERR_INVALID_ARG;
  const BlockPlan p = block_plan(*desc);
  const BlockWs w = block_ws(p, 0);
  const BlockSaved sv = block_saved(p);
  if (!workspace || workspace_bytes < w.total || misaligned(workspace, 256) || misaligned(saved, 256))
    return WERSA_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)hip_stream;
  unsigned char *ws = (unsigned char *)workspace, *sb = (unsigned char *)saved;
  const int hid = (int)p.hidden, M = (int)p.tokens;
  bf16_t *proj[3] = {(bf16_t *)(sb + sv.qp), (bf16_t *)(sb + sv.kp), (bf16_t *)(sb + sv.vp)};
  {
    GemmJob job{};
    const void *w3[3] = {wq, wk, wv};
    for (int i = 0; i < 3; ++i) {
      job.a[i] = (const bf16_t *)x;
      job.b[i] = (const bf16_t *)w3[i];
      job.c[i] = proj[i];
    }
    job.count = 1;
    job.batch = 3;
    if (launch_gemm<false, true, false, true>("wersa_gemm_nn", job, hid, M, hid, hid, hid, 1, st, (float *)(ws + w.qsums),
                                        (float *)(ws + w.qmax)) != hipSuccess)
      return WERSA_ERR_LAUNCH;
  }
  bf16_t *A = (bf16_t *)(sb + sv.a);
  // The pooled query comes out of the W^Q GEMM's epilogue (the core takes it when it can).
  const PooledSums pooled{(const float *)(ws + w.qsums), p.hidden, (const float *)(ws + w.qmax)};
  const wersa_status cs = forward_checked(&p.core, proj[0], proj[1], proj[2], omega_rf, sigma, gate_w, gate_b,
                                          scale_w, A, sb + sv.core, ws + w.core,
                                          wersa_workspace_bytes(&p.core, 0), hip_stream, &pooled);
  if (cs != WERSA_OK) return cs;
  GemmJob job{};
  job.a[0] = A;
  job.b[0] = (const bf16_t *)wo;
  job.c[0] = y;
  job.count = job.batch = 1;
  if (launch_gemm<false, true, false>("wersa_gemm_nn", job, hid, M, hid, hid, hid, 1, st) != hipSuccess)
    return WERSA_ERR_LAUNCH;
  return hipGetLastError() == hipSuccess ? WERSA_OK : WERSA_ERR_LAUNCH;
}

wersa_status wersa_block_backward(const wersa_desc *desc, const void *x, const void *wq, const void *wk,
                                  const void *wv, const void *wo, const void *omega_rf,
                                  const float *sigma, const float *gate_w, const float *gate_b,
                                  const float *scale_w, const void *dy, const void *saved, void *dx,
                                  float *dwq, float *dwk, float *dwv, float *dwo, float *dgate_w,
                                  float *dgate_b, float *dscale_w, float *dsigma, void *workspace,
                                  size_t workspace_bytes, void *hip_stream) {
  const wersa_status vs = validate_block(desc);
  if (vs != WERSA_OK) return vs;
  if (!x || !wq || !wk || !wv || !wo || !omega_rf || !sigma || !gate_w || !gate_b || !scale_w || !dy ||
      !saved || !dx || !dwq || !dwk || !dwv || !dwo)
    return WERSA_ERR_INVALID_ARG;
  const BlockPlan p = block_plan(*desc);
  const BlockWs w = block_ws(p, 1);
  const BlockSaved sv = block_saved(p);
  if (!workspace || workspace_bytes < w.total || misaligned(workspace, 256) || misaligned(saved, 256))
    return WERSA_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)hip_stream;
  unsigned char *ws = (unsigned char *)workspace;
  const unsigned char *sb = (const unsigned char *)saved;
  const int hid = (int)p.hidden, M = (int)p.tokens;
  const bf16_t *Qp = (const bf16_t *)(sb + sv.qp), *Kp = (const bf16_t *)(sb + sv.kp),
               *Vp = (const bf16_t *)(sb + sv.vp), *A = (const bf16_t *)(sb + sv.a);
  bf16_t *dA = (bf16_t *)(ws + w.dA), *dQp = (bf16_t *)(ws + w.dQp), *dKp = (bf16_t *)(ws + w.dKp),
         *dVp = (bf16_t *)(ws + w.dVp);
  float *part = (float *)(ws + w.part);
  const int64_t wcount = (int64_t)hid * hid;

  auto weight_grads = [&](const bf16_t *left, int batch, const bf16_t *const *right, float *const *out) -> bool {
    GemmJob job{};
    for (int i = 0; i < batch; ++i) {
      job.a[i] = left;
      job.b[i] = right[i];
      job.c[i] = p.splits == 1 ? out[i] : part;
    }
    job.count = 1;
    job.batch = batch;
    if (launch_gemm<true, true, true>("wersa_gemm_tn", job, hid, hid, hid, M, p.k_chunk, p.splits, st) != hipSuccess)
      return false;
    if (p.splits > 1)
      WERSA_STAGE("wersa_splitk_reduce", st,
                  splitk_reduce_kernel<<<dim3((unsigned)((wcount / 4 + 255) / 256), batch), 256, 0, st>>>(
                      part, p.splits, wcount, out[0], batch > 1 ? out[1] : nullptr, batch > 2 ? out[2] : nullptr));
    return true;
  };

  // Products with a weight's transpose: `count` weights, as they are or transposed into the core's workspace.
  auto transposed = [&](int count, const void *const *w_as_stored, const bf16_t **out) {
    TransposeJob job{};
    for (int i = 0; i < count; ++i) {
      job.w[i] = (const bf16_t *)w_as_stored[i];
      job.out[i] = (bf16_t *)(ws + w.core + i * up256((size_t)wcount * 2));
      out[i] = p.transpose ? job.out[i] : job.w[i];
    }
    if (p.transpose) WERSA_STAGE("wersa_transpose", st, transpose_kernel<<<dim3(hid / 64, hid / 64, count), 256, 0, st>>>(job, hid));
  };
  auto times_transpose = [&](GemmJob &job) {
    return (p.transpose ? launch_gemm<false, true, false>("wersa_gemm_nn", job, hid, M, hid, hid, hid, 1, st)
                        : launch_gemm<false, false, false>("wersa_gemm_nt", job, hid, M, hid, hid, hid, 1, st)) == hipSuccess;
  };
  {  // dA = dY W_out^T
    GemmJob job{};
    job.a[0] = (const bf16_t *)dy;
    const void *const stored[1] = {wo};
    transposed(1, stored, job.b);
    job.c[0] = dA;
    job.count = job.batch = 1;
    if (!times_transpose(job)) return WERSA_ERR_LAUNCH;
  }
  {
    const bf16_t *const right[1] = {(const bf16_t *)dy};
    float *const outs[1] = {dwo};
    if (!weight_grads(A, 1, right, outs)) return WERSA_ERR_LAUNCH;
  }
  const wersa_status cs =
      wersa_backward(&p.core, Qp, Kp, Vp, omega_rf, sigma, gate_w, gate_b, scale_w, A, dA, sb + sv.core, dQp, dKp,
                     dVp, dgate_w, dgate_b, dscale_w, dsigma, ws + w.core, wersa_workspace_bytes(&p.core, 1),
                     hip_stream);
  if (cs != WERSA_OK) return cs;
  {  // dX = dQ' W^Q^T + dK' W^K^T + dV' W^V^T
    GemmJob job{};
    job.a[0] = dQp;
    job.a[1] = dKp;
    job.a[2] = dVp;
    const void *const stored[3] = {wq, wk, wv};
    transposed(3, stored, job.b);
    job.c[0] = dx;
    job.count = 3;
    job.batch = 1;
    if (!times_transpose(job)) return WERSA_ERR_LAUNCH;
  }
  const bf16_t *const right[3] = {dQp, dKp, dVp};
  float *const outs[3] = {dwq, dwk, dwv};
  for (int i = 0; i < 3; i += p.wgrads)
    if (!weight_grads((const bf16_t *)x, p.wgrads, right + i, outs + i)) return WERSA_ERR_LAUNCH;
  return hipGetLastError() == hipSuccess ? WERSA_OK : WERSA_ERR_LAUNCH;
}

}  // extern "C"
