// Split path: float32 arithmetic on the bf16 matrix cores, the n x m feature matrices in registers
// (Section 3.1 steps 3-8 and their derivatives; every dtype, head dimensions up to 128, any m).
//
// Every float32 operand of a contraction is written as a sum of three bf16 values,
//   x = x0 + x1 + x2,  x0 = bf16(x), x1 = bf16(x - x0), x2 = bf16(x - x0 - x1)   (24 significant bits),
// and a product of two such operands is the six bf16 products x0 y0, x0 y1, x1 y0, x0 y2, x1 y1, x2 y0
// accumulated in float32; what is left out (x1 y2, x2 y1, x2 y2) is at most 2^-24 of |x y|, a rounding error of the
// float32 product itself.  A bf16 tensor is one exact term, so products with it take three.  The bf16
// matrix rate is 16 times the float32 one, so even six products leave a factor of 2.7.
//
// What bounds it: per 32 x 32 tile of a feature matrix the matrix cores spend 32 cycles per product and 16 of the
// contraction's length (and where they form the residuals, two sparse ones), the vector units 5.5 instructions per
// element on the split and two on ReLU or mask; two waves per SIMD let one run under the other.  From d 64 on the matrix cores
// alone.  Scratch: grad_kernel with dV at d 64 88 bytes per lane (accumulators and operands fill the 256 registers).
//
// Measured against the generic kernels, which write every n x m feature matrix to memory: float32 training step, 128
// slices of 4000 tokens, d 32, m 1024: 13990 -> 2350 us; bf16 training step, 8 slices of 131072 tokens, d 16, m 1024:
// 26290 -> 2100 us; float32 inference, one slice of 1024 tokens, d 64, m 64: 118 -> 30 us.
//
// Layout: every operand is kept in the order in which a wave loads it ("operand tile": 32 vectors x 16
// k-values of bf16; lane (l32, h) holds vector l32, k = 8 h .. 8 h + 7, 16 bytes; 1 KiB).  Where k runs
// over the rows of an accumulator tile (features, or tokens), the k-slots stand for the rows in the
// order in which the accumulator registers hold them: slot (h, q) of half a is row 16 a + 8 (q / 4)
// + 4 h + q % 4.  The tensors of n x d (a small share of the time: m / 16 feature tiles are formed per
// row) are filtered, split and packed by streaming kernels; rows past n and columns past d are zeros.
#include "wersa_internal.h"

#include <initializer_list>
#include <type_traits>

// v_mul_legacy_f32 as the compiler's intrinsic (not as inline assembly: the wait states after a matrix instruction are
// the compiler's to insert).
extern "C" __device__ float amdgcn_mul_legacy(float, float) __asm("llvm.amdgcn.fmul.legacy");

namespace wersa {
namespace {

#include "wersa_small_kernels.inc"
#include "wersa_filter.inc"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

constexpr int kTile = 512;   // bf16 values of one operand tile

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.f;
  return z;
}
// x[lane] + x[lane ^ 32] in every lane
__device__ __forceinline__ float xor32_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Split of eight floats.
__device__ __forceinline__ void split8(const float *v, bf16x8 *t) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    f32x2 x;
    x[0] = v[2 * j];
    x[1] = v[2 * j + 1];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const bf16x2 p = __builtin_convertvector(x, bf16x2);
      t[i][2 * j] = p[0];
      t[i][2 * j + 1] = p[1];
      x[0] -= (float)p[0];
      x[1] -= (float)p[1];
    }
  }
}
// Split of an accumulator tile into operands (t[a][i]: half a, term i).  The vector units take 5.5 instructions per
// element for it, most of them for the two residuals x - x0 and x - x0 - x1.  LV of these come from the matrix
// cores instead: x - bf16(x) is the accumulator plus the product of a negated identity matrix, its columns in the order of the
// k-slots, with the packed term.  One entry per row is sparse enough for the 2:4 instruction, which takes all 32 rows of the term
// at once, and it is exact (one non-zero product per element; every value of 131072 with exponents from -125 to 124 equal to
// the subtraction's).  Measured (one SIMD, four waves): a matrix instruction takes 32 cycles of its
// own pipe and keeps the vector units from issuing for about 15, a vector instruction takes 4; a pair dot
// product (v_dot2c_f32_bf16, which would do a residual in one instruction) does not run beside matrix
// instructions at all.  A loop of split and products, two waves per SIMD, ns per 32 x 32 tile with both residuals from the vector
// units / from two dense 32 x 32 x 16 products each / four 4 x 4 x 4 / one sparse one: 24 products 477 / 447 / 439 / 395,
// 8 products 241 / 207 / 226 / 193.
struct NegIdentity {
  bf16x8 a;    // the stored two of every four entries: lane (row, half of the 32 k-slots)
  int index;   // which two, 2 bits each
  __device__ __forceinline__ explicit NegIdentity(int lane) {
    // Row r of the tile is in k-slot 16 (r / 16) + 8 (r / 4 % 2) + 4 (r / 8 % 2) + r % 4; a lane stores two entries, their places
    // ascending, of each of its four groups of four slots.
    const int r = lane & 31, place = r & 3, entry = 4 * (r >> 2 & 1) + 2 * (r >> 3 & 1) + (place == 3);
#pragma unroll
    for (int q = 0; q < 8; ++q) a[q] = (__bf16)(lane >> 5 == r >> 4 && q == entry ? -1.f : 0.f);
    index = (place == 3 ? 0xC : 0xC | place) * 0x1111;
  }
};
// Calls use(a, terms) for both halves.
template <int LV, typename F>
__device__ __forceinline__ void with_split(f32x16 x, const NegIdentity &ni, F use) {
  if (LV == 0) {   // one half at a time: fewer registers
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      float v[8];
      bf16x8 t[3];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = x[8 * a + q];
      split8(v, t);
      use(a, t);
    }
    return;
  }
  bf16x8 t[2][3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        f32x2 f;
        f[0] = x[8 * a + 2 * j];
        f[1] = x[8 * a + 2 * j + 1];
        const bf16x2 p = __builtin_convertvector(f, bf16x2);
        t[a][i][2 * j] = p[0];
        t[a][i][2 * j + 1] = p[1];
        if (i < 2 && i >= LV) {
          x[8 * a + 2 * j] -= (float)p[0];
          x[8 * a + 2 * j + 1] -= (float)p[1];
        }
      }
    if (i < LV) {
      const bf16x16 term = __builtin_shufflevector(t[0][i], t[1][i], 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
      x = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(ni.a, term, x, ni.index, 0, 0);
    }
  }
  use(0, t[0]);
  use(1, t[1]);
}
// Residuals left to the matrix cores, by what is idle: with head dimension 16, and 32 with one-term operands, the contractions are
// too short to fill them.  Training step, both residuals as two dense products each -> one sparse product each, the same bits: 8 slices of
// 131072 tokens, d 16, m 1024, bf16 2286 -> 2150 us; 32 of 16384, d 32, m 512, bf16 1042 -> 1018; d 16, float32 1054 -> 1025.  The vector units'
// residuals against one and two sparse ones with d 32 and three terms: contraction 333, 329, 331 us, key side's gradient 747, 729, 730, apply
// 344, 358, 371 (registers); with d 64 and 128 equal.
// spare: a kernel with registers for one of them at head dimension 32 with three terms.
constexpr int mfma_residuals(int DH, int PT, bool spare = false) {
  return DH == 16 || (DH == 32 && PT == 1) ? 2 : (DH == 32 && spare ? 1 : 0);
}
__device__ __forceinline__ void split1(float x, __bf16 *t) {
  t[0] = (__bf16)x;
  const float r = x - (float)t[0];
  t[1] = (__bf16)r;
  t[2] = (__bf16)(r - (float)t[1]);
}

// acc + the product of a three-term operand with one of NB terms, smallest products first.
// SWAP: the NB-term operand is the first one of the instruction (its vectors are the result's rows).
template <int NB, bool SWAP>
__device__ __forceinline__ f32x16 mfma_terms(f32x16 acc, const bf16x8 *x, const bf16x8 *y) {
  auto go = [&](int i, int j) { acc = SWAP ? mfma(y[j], x[i], acc) : mfma(x[i], y[j], acc); };
  if (NB == 3) {
    go(0, 2);
    go(1, 1);
    go(2, 0);
    go(0, 1);
    go(1, 0);
    go(0, 0);
  } else {
    go(2, 0);
    go(1, 0);
    go(0, 0);
  }
  return acc;
}
// acc + lo += the product of a three-term operand with one of NB terms, smallest products first.  acc takes the product of the
// leading terms, lo the others (lo may be acc).
template <int NB>
__device__ __forceinline__ void add_terms(f32x16 &acc, f32x16 &lo, const bf16x8 *x, const bf16x8 *y) {
  if (NB == 3) {
    lo = mfma(x[0], y[2], lo);
    lo = mfma(x[1], y[1], lo);
  }
  lo = mfma(x[2], y[0], lo);
  if (NB == 3) lo = mfma(x[0], y[1], lo);
  lo = mfma(x[1], y[0], lo);
  acc = mfma(x[0], y[0], acc);
}
__device__ __forceinline__ bf16x8 lds_operand(const bf16_t *tile, int lane) {
  return *reinterpret_cast<const bf16x8 *>(tile + lane * 8);
}
// All loads from memory have arrived.  Before a loop that requests its next stage first and works on operands loaded
// before it: the compiler would otherwise wait, in the loop, for those and with them for the stage just requested.
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }
__device__ __forceinline__ void store_operand(bf16_t *tile, int lane, bf16x8 v) {
  *reinterpret_cast<bf16x8 *>(tile + lane * 8) = v;
}

// 1 where x > 0, else 0 (also for NaN), exact for every float: one multiplication with output clamp.  With
// additions and plain moves it runs at twice the rate of the other vector instructions (measured: 2 cycles against 4).
__device__ __forceinline__ float positive(float x) { return __builtin_amdgcn_fmed3f(x * __builtin_inff(), 0.f, 1.f); }
// max(x, 0), 0 for NaN of either sign as fmaxf gives.  One instruction: fmaxf is two (it quiets a NaN first), and so is
// the median where the compiler sees that its bound is infinity.
__device__ __forceinline__ float relu(float x) {
  float bound = __builtin_inff();
  asm("" : "+s"(bound));
  return __builtin_amdgcn_fmed3f(x, 0.f, bound);
}
// x where mask is 1, 0 where it is 0, also for NaN and infinities (0 times anything is 0 in this instruction).
__device__ __forceinline__ float masked(float x, float mask) { return amdgcn_mul_legacy(x, mask); }

// ------------------------------------------------------------------------------------
// The ReLU's decisions as bits.  A gradient kernel needs of the projection only which elements were positive, and the kernel that has the
// projection in hand anyway (the contraction on the query side, the one of dV at head dimension 128 on the key side) writes it down:
// one 16-bit word per lane and 32 x 32 tile, n m / 8 bytes per slice, bits[slice][token tile][feature tile][64].  That is a third of
// the gradient kernel's products, its operands in LDS and the rows of X in registers less.
// A lane has 16 elements of a tile, with features on registers its token l32 and the features f with f / 4 % 2 = h, with tokens on registers
// the other way round; with r the register's number, word bit 8 (r % 2) + r / 2 % 2 + 2 (r / 4 % 2) + 4 (r / 8) is its element.
// Word bits 3, 0, 1, 2 and lane bits 0, 1, 3, 4 thus are bits 0, 1, 3, 4 of token and feature, or of feature and token: to go from one
// form to the other they change places, and lane bits 2 and 5 too (by where a lane's word is stored).  In memory: tokens on word bits,
// bit 2 of the token on bit 2 of the place.
// ------------------------------------------------------------------------------------
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ int decision_bit(int r) { return 8 * (r & 1) + (r >> 1 & 1) + 2 * (r >> 2 & 1) + 4 * (r >> 3); }
// Of the leading terms of the two halves of a tile after the ReLU, two instructions per pair (a positive value that is no zero in bf16
// counts as one: above 2^-134).
__device__ __forceinline__ uint32_t decisions(const bf16x8 (&lead)[2]) {
  u16x2 one = {1, 1};
  asm("" : "+s"(one));   // (of min(x, 1) the compiler makes two comparisons and two selections)
  uint32_t w = 0;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int j = 0; j < 4; ++j) {   // elements 2 j, 2 j + 1 of half a: bits 4 a + j % 2 + 2 (j / 2) of the two halves of the word
      bf16x2 e;
      e[0] = lead[a][2 * j];
      e[1] = lead[a][2 * j + 1];
      const uint32_t b = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, e), one));
      w |= b << (4 * a + j);
    }
  return __builtin_amdgcn_perm(w, w, 0x0C0C0200);
}
// Exchanges word bits 3, 0, 1, 2 with lane bits 0, 1, 3, 4, in both halves of the word.
struct TransposeDecisions {
  uint32_t sel, mask[3], rot[3];
  __device__ __forceinline__ explicit TransposeDecisions(int lane) {
    sel = lane & 1 ? 0x03070105u : 0x06020400u;
    const uint32_t m[3] = {0x55555555u, 0x33333333u, 0x0F0F0F0Fu};
    const int bit[3] = {2, 8, 16};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      mask[i] = lane & bit[i] ? ~m[i] : m[i];
      rot[i] = lane & bit[i] ? 1u << i : 32u - (1u << i);
    }
  }
  __device__ __forceinline__ uint32_t operator()(uint32_t w) const {
    // bytes 0 and 2: word bit 3 clear.  An even lane keeps them and takes the other's as its bytes 1 and 3.
    const uint32_t t = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xB1, 0xF, 0xF, false);   // lane ^ 1
    w = __builtin_amdgcn_perm(t, w, sel);
    auto merge = [&](uint32_t other, int i) { w = (w & mask[i]) | (__builtin_amdgcn_alignbit(other, other, rot[i]) & ~mask[i]); };
    merge((uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x4E, 0xF, 0xF, false), 0);    // lane ^ 2
    merge((uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x128, 0xF, 0xF, false), 1);   // lane ^ 8
    const auto r = __builtin_amdgcn_permlane16_swap(w, w, false, false);                  // lane ^ 16: the row that is not this lane's
    merge(mask[2] & 1 ? r[1] : r[0], 2);
    return w;
  }
};
// x where the word's bit of register r is set, 0 where it is not (also for NaN and infinities); half: which half of the word.
__device__ __forceinline__ float masked(float x, uint32_t word, int r, int half) {
  return __uint_as_float(__float_as_uint(x) & (uint32_t)__builtin_amdgcn_sbfe((int)word, 16 * half + decision_bit(r), 1));
}

// Product of the 16 values of an accumulator tile that a lane holds with 16 weights.  D and z are sums of these, D of eight
// at a time: one chain over all features or tokens is four times as far from the exact sum at 4096 features.
__device__ __forceinline__ float dot16(const f32x16 &x, const f32x4 (&w)[4]) {
  float acc = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc = fmaf(x[i], w[i >> 2][i & 3], acc);
  return acc;
}

// Eight consecutive elements as float; vec: the tensor's rows are 16-byte aligned.
__device__ __forceinline__ void load8(const float *p, bool vec, float *v) {
  if (vec) {
    const f32x4 a = reinterpret_cast<const f32x4 *>(p)[0], b = reinterpret_cast<const f32x4 *>(p)[1];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[q] = a[q];
      v[4 + q] = b[q];
    }
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = p[q];
  }
}
__device__ __forceinline__ void load8(const bf16_t *p, bool vec, float *v) {
  if (vec) {
    const u16x8 a = *reinterpret_cast<const u16x8 *>(p);
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = bf16_to_f32(a[q]);
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = bf16_to_f32(p[q]);
  }
}

// Sizes of one problem.
struct Dims {
  int n, d, m;
  int nt;    // 32-row tiles of tokens per slice (even: whole 64-row blocks)
  int mt;    // 32-feature tiles
};

// ------------------------------------------------------------------------------------
// Column sums of Q (and, for L > 6, of K) per chunk of rows; the first workgroups (om.blocks) carry the per-call constants and pack Omega.
// Grid (om.blocks + chunks * slices, 1, tensors): every workgroup has something to do.  (With the packing ones beside the chunks of every slice, idle but
// for slice 0, a multiple of eight to a slice put all chunks on the same few of the eight dies: 800 slices of 4720 tokens, d 64, m 48, float32, three
// chunks and five others, 269 us, 202 now; 893 of 1163, d 48, m 176 104, 58.)  Far fewer than 2^24 workgroups in what fits the card.
// ------------------------------------------------------------------------------------
// What no kernel writes of `saved` (the ends of sections that are rounded up, the feature tile past the last one, the coefficients of
// levels that are not there) is cleared by the first launch, so that two calls on the same inputs leave the same bytes, whatever was in the
// memory before: by one more of its packing workgroups, and a slice's coefficients by the workgroup of its first chunk.
// (A loop for every section would wait for the stores of the one before: 25 slices of 275 tokens, d 48, m 144, bf16 9.4 us, 7.1.)
struct Gaps {
  float *end[12];   // less than 64 values each
  int len[12];
  float *tile[2];
  int tile_len[2];
  float *coef;
};
Gaps gaps_of(const wersa_desc &c, const SavedLayout &sv, float *saved, int64_t tileA, int64_t tileB, const SplitSizes &z) {
  Gaps g{};
  int i = 0;
  const int64_t sl = (int64_t)c.B * c.H;
  auto end = [&](int64_t off, int64_t used) {   // from the last value to the next multiple of 64
    g.end[i] = saved + off + used;
    g.len[i++] = (int)((64 - used % 64) % 64);
  };
  end(sv.S, sl * c.m * c.d);
  end(sv.z, sl * c.m);
  end(sv.qbar, sl * c.d);
  end(sv.s, sl * (c.L + 1));
  end(sv.F, sl * (c.L + 1));
  end(sv.D, sl * c.n);
  end(sv.scalars, 4);
  end(sv.coef, sl * kCoefStride);
  if (c.L > kTileL)
    for (const int64_t off : {sv.tileQ, sv.tileK, sv.addQ, sv.addK}) end(off, sl * ((c.n + 63) / 64) * c.d);
  g.coef = saved + sv.coef;   // (the gate, which comes later, writes as many levels as there are)
  g.tile[0] = saved + sv.OA + z.OA - tileA;
  g.tile_len[0] = (int)((64 - z.OA % 64) % 64 + tileA);
  g.tile[1] = saved + sv.OB + z.OB - tileB;
  g.tile_len[1] = (int)((64 - z.OB % 64) % 64 + tileB);
  return g;
}

template <typename T>
struct OmegaPack {
  const T *omega;      // [matrices][d][m]
  const float *sigma;
  float bw_floor;
  float *scalars;
  bf16_t *OA, *OB;     // features as vectors (k = columns), columns as vectors (k = features)
  int matrices, KS, CT, PT, blocks;   // (the last one clears)
  Gaps gaps;
};
template <typename T>
__device__ void omega_pack_body(const OmegaPack<T> &o, const Dims &s, int block) {
  if (block == o.blocks - 1) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int g = 0; g < 12; ++g)
      if (g % 4 == wave && lane < o.gaps.len[g]) o.gaps.end[g][lane] = 0.f;
#pragma unroll
    for (int g = 0; g < 2; ++g)
      for (int e = threadIdx.x; e < o.gaps.tile_len[g]; e += 256) o.gaps.tile[g][e] = 0.f;
    return;
  }
  if (block == 0 && threadIdx.x == 0) {
    const float sg = *o.sigma, se = fmaxf(sg, o.bw_floor);
    o.scalars[0] = 1.0f / (se * sqrtf((float)s.m));
    o.scalars[1] = se;
    o.scalars[2] = sg > o.bw_floor ? 1.0f : 0.0f;
    o.scalars[3] = 1.0f;
  }
  const int per_ft = 64 * (o.KS + 2 * o.CT), per_mat = s.mt * per_ft;
  const int e = block * 256 + threadIdx.x;
  if (e >= o.matrices * per_mat) return;
  const int mat = e / per_mat, ft = e % per_mat / per_ft, piece = e % per_ft, lane = piece & 63, which = piece >> 6;
  const int l32 = lane & 31, h = lane >> 5;
  const T *om = o.omega + (int64_t)mat * s.d * s.m;
  float v[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    int f, c;
    if (which < o.KS) {
      f = 32 * ft + l32;
      c = 16 * which + 8 * h + q;
    } else {
      const int a = (which - o.KS) / o.CT, ct = (which - o.KS) % o.CT;
      f = 32 * ft + 16 * a + 8 * (q >> 2) + 4 * h + (q & 3);
      c = 32 * ct + l32;
    }
    v[q] = (f < s.m && c < s.d) ? ld(om + (int64_t)c * s.m + f) : 0.f;
  }
  bf16x8 t[3];
  split8(v, t);
  const int64_t tile = which < o.KS ? ((int64_t)(mat * s.mt + ft) * o.KS + which) * o.PT
                                    : ((int64_t)(mat * s.mt + ft) * 2 * o.CT + which - o.KS) * o.PT;
  // OB by its distance from OA: a choice between two members of a kernel argument would be made by their addresses, in scratch
  // memory, and a kernel with scratch starts later (this one, for one slice of 1024 tokens, d 64: 7.8 us with it, 3.8 without).
  bf16_t *dst = o.OA + (which < o.KS ? 0 : o.OB - o.OA) + tile * kTile;
  for (int i = 0; i < o.PT; ++i) store_operand(dst + i * kTile, lane, i == 0 ? t[0] : i == 1 ? t[1] : t[2]);
}
template <typename T>
__global__ __launch_bounds__(256) void pool_kernel(const T *q, const T *k, View v, Dims s, int vec, int rows_per_chunk,
                                                  int chunks, float *partq, float *partk, OmegaPack<T> om) {
  if ((int)blockIdx.x < om.blocks) {
    if (blockIdx.z == 0) omega_pack_body(om, s, blockIdx.x);
    return;
  }
  const int slice = (blockIdx.x - om.blocks) / chunks, chunk = (blockIdx.x - om.blocks) % chunks;
  if (chunk == 0 && blockIdx.z == 0 && threadIdx.x < kCoefStride) om.gaps.coef[slice * kCoefStride + threadIdx.x] = 0.f;
  const int cpr = s.d / 8, rpi = 256 / cpr;   // 8 columns per thread, rpi rows at a time
  const int t0 = chunk * rows_per_chunk, t1 = min(s.n, t0 + rows_per_chunk);
  const int cc = threadIdx.x % cpr, rr = threadIdx.x / cpr;
  const T *xs = (blockIdx.z ? k : q) + v.slice_base(slice) + cc * 8;
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
  if (rr < rpi) {
    int t = t0 + rr;
    for (; t + 3 * rpi < t1; t += 4 * rpi) {   // four rows in flight
      float x[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u) load8(xs + (int64_t)(t + u * rpi) * v.sn, vec, x[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += x[u][e];
    }
    for (; t < t1; t += rpi) {
      float x[8];
      load8(xs + (int64_t)t * v.sn, vec, x);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += x[e];
    }
  }
  __shared__ float red[2048 + 128];   // [rpi][d + 1]: at most 128 x 17
  if (rr < rpi)
#pragma unroll
    for (int e = 0; e < 8; ++e) red[rr * (s.d + 1) + cc * 8 + e] = acc[e];
  __syncthreads();
  // halves of the rows are folded until a few are left (fixed order), then summed per column
  int rows = rpi;
  while (rows > 8) {
    const int half = rows / 2, keep = rows - half;
    for (int e = threadIdx.x; e < half * s.d; e += 256)
      red[(e / s.d) * (s.d + 1) + e % s.d] += red[(e / s.d + keep) * (s.d + 1) + e % s.d];
    __syncthreads();
    rows = keep;
  }
  if ((int)threadIdx.x < s.d) {
    float sum = 0.f;
    for (int r = 0; r < rows; ++r) sum += red[r * (s.d + 1) + threadIdx.x];
    (blockIdx.z ? partk : partq)[((int64_t)slice * chunks + chunk) * s.d + threadIdx.x] = sum;
  }
}

// ------------------------------------------------------------------------------------
// Operands of n x d, 4096 elements per workgroup.
// ------------------------------------------------------------------------------------
template <int DH>
struct Geo {
  static constexpr int KS = DH / 16, CT = DH < 32 ? 1 : DH / 32, CW = DH < 64 ? DH : 64, TR = 4096 / CW,
                       PIECES = DH / CW, LS = CW + 4, SEGS = 256 / CW;
  // Operand tiles per feature tile of S with its columns as vectors.  Head dimension 16 leaves half of the 32 columns
  // free: [S0 | S1] and [S2 | 0] take four products instead of six (see apply_terms).
  static constexpr int NSB = DH == 16 ? 4 : 6 * CT;
};
// acc + Phi S for one half of a feature tile and one column tile; sb: the operand tiles of S from lds_operand.
template <int DH>
__device__ __forceinline__ void apply_terms(f32x16 &acc, const bf16x8 *p, const bf16_t *sb, int a, int ct, int lane) {
  if (DH == 16) {   // columns 0-15: p0 S2 + (p2 + p1 + p0) S0; columns 16-31: (p2 + p1 + p0) S1; added at the end
    const bf16x8 s01 = lds_operand(sb + 2 * a * kTile, lane), s2 = lds_operand(sb + (2 * a + 1) * kTile, lane);
    acc = mfma(p[0], s2, acc);
    acc = mfma(p[2], s01, acc);
    acc = mfma(p[1], s01, acc);
    acc = mfma(p[0], s01, acc);
    return;
  }
  constexpr int CT = DH < 32 ? 1 : DH / 32;
  bf16x8 y[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) y[i] = lds_operand(sb + ((a * CT + ct) * 3 + i) * kTile, lane);
  add_terms<3>(acc, acc, p, y);
}
// sum over the levels above four (up to L) of coef_l * (block sum): levels 5 and 6 from the 16-row sums of a tile
template <int CW>
__device__ __forceinline__ float upper_levels(const float (*segsum)[CW], const float *cf, int seg, int c, int L) {
  if (L < 5) return 0.f;
  const int b = seg & ~3;
  const float s5 = segsum[seg & ~1][c] + segsum[seg | 1][c];
  const float s6 = (segsum[b][c] + segsum[b + 1][c]) + (segsum[b + 2][c] + segsum[b + 3][c]);
  return fmaf(cf[5], s5, L < 6 ? 0.f : cf[6] * s6);
}
// Scratch of a packing kernel: one tile of rows, the 16-row sums or two values per row, and a few scalars.
template <int DH>
struct PrepLds {
  using G = Geo<DH>;
  static constexpr int RB = 4096 / DH, FILTER = G::TR * G::LS, ROWS = RB * (DH + 4);   // rows of a tile of whole rows
  float tile[FILTER > ROWS ? FILTER : ROWS];
  float part[256];
  float small[8];
};
template <int DH> using PrepGate = GateLds<16, DH>;   // in the place of the tile
// TR x CW elements of a strided tensor from row t0, column c0 into LDS; zeros past n and d.
template <typename T, int DH>
__device__ __forceinline__ void load_tile(const T *xs, const View &v, const Dims &s, int vec, int t0, int c0, float *tile) {
  using G = Geo<DH>;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int e = threadIdx.x + 256 * u, r = e / (G::CW / 8), cc = e % (G::CW / 8) * 8;
    float x[8];
    if (t0 + r < s.n && c0 + cc < s.d) load8(xs + (int64_t)(t0 + r) * v.sn + c0 + cc, vec, x);
    else
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = 0.f;
    f32x4 a, b;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      a[i] = x[i];
      b[i] = x[4 + i];
    }
    *reinterpret_cast<f32x4 *>(&tile[r * G::LS + cc]) = a;
    *reinterpret_cast<f32x4 *>(&tile[r * G::LS + cc + 4]) = b;
  }
}
// Gated Haar filter of one signal (steps 3, 5, 6), split and packed with k = columns.  One thread per (column, 16
// rows) in the filter, the 32- and 64-row sums through LDS.  X: X_F (may be nullptr); XS: X_F / D_t (may be nullptr).
template <typename T, int DH>
__device__ __forceinline__ void filter_pack(PrepLds<DH> &lds, const T *x, const View &v, const Dims &s, int vec, int L,
                                            const float *coef, const float *add, const float *D, bf16_t *X, bf16_t *XS) {
  using G = Geo<DH>;
  constexpr int CW = G::CW, TR = G::TR, LS = G::LS;
  float(*segsum)[CW] = reinterpret_cast<float(*)[CW]>(lds.part);
  const int tid = threadIdx.x, slice = blockIdx.y;
  const int rg = blockIdx.x / G::PIECES, piece = blockIdx.x % G::PIECES;
  const int t0 = rg * TR, c0 = piece * CW;
  if (coef && tid < 8) lds.small[tid] = coef[slice * kCoefStride + tid];   // (nullptr: they are there)
  load_tile<T, DH>(x + v.slice_base(slice), v, s, vec, t0, c0, lds.tile);
  __syncthreads();
  const int c = tid % CW, seg = tid / CW;
  float vals[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) vals[i] = lds.tile[(seg * 16 + i) * LS + c];
  segsum[seg][c] = segment_sum<16>(vals);
  __syncthreads();
  float upper = upper_levels<CW>(segsum, lds.small, seg, c, L);
  const int gt = t0 / 64 + seg / 4, ntl = (s.n + 63) / 64;
  if (add && gt < ntl && c0 + c < s.d) upper += add[((int64_t)slice * ntl + gt) * s.d + c0 + c];
  filter_segment<16>(vals, lds.small, upper, L);
  // (rows past n must stay zero: they are padding, not output)
#pragma unroll
  for (int i = 0; i < 16; ++i) lds.tile[(seg * 16 + i) * LS + c] = t0 + seg * 16 + i < s.n ? vals[i] : 0.f;
  __syncthreads();
  constexpr int KSL = CW / 16;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int p = tid + 256 * u, lane = p & 63, ksl = (p >> 6) % KSL, tb = t0 / 32 + (p >> 6) / KSL;
    if (tb >= s.nt) continue;
    float f[8];
    load8(&lds.tile[(((p >> 6) / KSL) * 32 + (lane & 31)) * LS + 16 * ksl + 8 * (lane >> 5)], true, f);
    const int64_t off = (((int64_t)slice * s.nt + tb) * G::KS + piece * KSL + ksl) * 3 * kTile;
    bf16x8 t[3];
    if (X) {
      split8(f, t);
#pragma unroll
      for (int i = 0; i < 3; ++i) store_operand(X + off + i * kTile, lane, t[i]);
    }
    if (XS) {
      const int row = 32 * tb + (lane & 31);
      const float inv = row < s.n ? 1.0f / D[(int64_t)slice * s.n + row] : 1.f;
#pragma unroll
      for (int q = 0; q < 8; ++q) f[q] *= inv;
      split8(f, t);
#pragma unroll
      for (int i = 0; i < 3; ++i) store_operand(XS + off + i * kTile, lane, t[i]);
    }
  }
}

// Forward operands: Q_F and K_F packed with k = columns, V packed with k = tokens.
// Grid (row groups * column pieces, slices, 3: Q, K, V).
// GATE: by workgroups that form the gate first.
template <typename T, int DH, int PT, bool GATE>
__global__ __launch_bounds__(256) void prep_fwd_kernel(const T *q, const T *k, const T *vv, View v, Dims s, int vec, int L,
                                                      const float *coef, const float *addQ, const float *addK,
                                                      bf16_t *XQ, bf16_t *XK, bf16_t *VC, GateFwdArgs gate) {
  using G = Geo<DH>;
  constexpr int CW = G::CW, TR = G::TR, LS = G::LS;
  __shared__ __attribute__((aligned(16))) PrepLds<DH> lds;
  const int side = blockIdx.z;
  if (side < 2) {
    if constexpr (GATE) {
      static_assert(sizeof(PrepGate<DH>) <= sizeof(lds.tile), "the gate's scratch");
      PrepGate<DH> &gl = *reinterpret_cast<PrepGate<DH> *>(lds.tile);
      gate_prologue<16, DH>(gate, blockIdx.y, blockIdx.x == 0 && side == 0, gl);
      if (threadIdx.x < 8) lds.small[threadIdx.x] = gl.coef[threadIdx.x];
      __syncthreads();
    }
    filter_pack<T, DH>(lds, side ? k : q, v, s, vec, L, GATE ? nullptr : coef, side ? addK : addQ, nullptr, side ? XK : XQ, nullptr);
    return;
  }
  const int tid = threadIdx.x, slice = blockIdx.y;
  const int rg = blockIdx.x / G::PIECES, piece = blockIdx.x % G::PIECES;
  const int t0 = rg * TR, c0 = piece * CW;
  load_tile<T, DH>(vv + v.slice_base(slice), v, s, vec, t0, c0, lds.tile);
  __syncthreads();
  constexpr int CTL = CW < 32 ? 1 : CW / 32, NP = TR / 32 * 2 * CTL * 64;
#pragma unroll
  for (int u = 0; u < NP / 256; ++u) {
    const int p = tid + 256 * u, lane = p & 63, ctl = (p >> 6) % CTL, a = (p >> 6) / CTL % 2, tbl = (p >> 6) / (2 * CTL);
    const int tb = t0 / 32 + tbl, c = 32 * ctl + (lane & 31), h = lane >> 5;
    if (tb >= s.nt) continue;
    float x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = tbl * 32 + 16 * a + 8 * (i >> 2) + 4 * h + (i & 3);
      // (head dimension 16: column 16 of the 32 is the column of ones that gives z)
      x[i] = c < CW ? lds.tile[r * LS + c] : (c == 16 ? 1.f : 0.f);
    }
    bf16x8 t[3];
    split8(x, t);
    bf16_t *o = VC + ((((int64_t)slice * s.nt + tb) * 2 + a) * G::CT + piece * CTL + ctl) * PT * kTile;
#pragma unroll
    for (int i = 0; i < PT; ++i) store_operand(o + i * kTile, lane, t[i]);
  }
}

// ------------------------------------------------------------------------------------
// Backward operands.  blockIdx.z = 0, per row: <dO_t, O_t>, then dN_t and dD_t; dN packed with k = tokens for dS.
//   PT == 1 (bf16 storage): dN stays dO, one exact term; 1 / D_t goes into the rows of Q_F of the dS
//   product (XS; ReLU is positively homogeneous) and into the scale of the rows of dQ_F (rowscale), so
//   ddw is then -<dO_t, O_t>.   PT == 3: dN = dO / D in float32, ddw = dD_t = -<dO_t, O_t> / D_t.
//   With the LayerNorm output stage: dN = rstd (dO - mean dO - O mean(dO O)), ddw = 0.
// part[slice][workgroup]: sum of the per-row term of d sigma (dD_t, or -<dO_t, O_t> rstd_t^2).
// blockIdx.z = 1: XS or, with three terms, Q_F as the forward packs it; 2: K_F (see keeps_operands).  dN and V with k = columns are not
// packed: the gradient kernel reads each of their rows once, in the order in which they are stored.
// Grid (row groups, slices, 1 to 3); the row groups of both forms are the same in number.
// ------------------------------------------------------------------------------------
template <typename T, int DH, int PT>
__global__ __launch_bounds__(256) void prep_bwd_kernel(const T *dout, const T *out, const T *q, const T *k, View v, Dims s, int vec,
                                                      int ln, int L, const float *coef, const float *addQ, const float *addK,
                                                      const float *D, bf16_t *NC, bf16_t *XQ, bf16_t *XS, bf16_t *XK, float *ddw,
                                                      float *rowscale, float *part) {
  using G = Geo<DH>;
  __shared__ __attribute__((aligned(16))) PrepLds<DH> lds;
  if (blockIdx.z) {
    if (blockIdx.z == 1) filter_pack<T, DH>(lds, q, v, s, vec, L, coef, addQ, D, XQ, XS);
    else filter_pack<T, DH>(lds, k, v, s, vec, L, coef, addK, nullptr, XK, nullptr);
    return;
  }
  constexpr int RB = PrepLds<DH>::RB, PARTS = DH / 16, LS = DH + 4;
  static_assert(RB <= 256, "one weight per row in LDS");
  float *tile = lds.tile, *wrow = lds.part, *red = lds.small;
  const int tid = threadIdx.x, slice = blockIdx.y, t0 = blockIdx.x * RB;
  const int r = tid / PARTS, pc = tid % PARTS * 16, t = t0 + r;
  const bool ok = t < s.n && pc < s.d;
  const int64_t base = v.slice_base(slice) + (int64_t)(t < s.n ? t : 0) * v.sn + (pc < s.d ? pc : 0);
  float g[16], o[16];
  load8(dout + base, vec, g);
  load8(dout + base + 8, vec, g + 8);
  load8(out + base, vec, o);
  load8(out + base + 8, vec, o + 8);
  if (!ok)
#pragma unroll
    for (int i = 0; i < 16; ++i) g[i] = o[i] = 0.f;
  float dot = 0.f, sum = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    dot = fmaf(g[i], o[i], dot);
    sum += g[i];
  }
#pragma unroll
  for (int w = 1; w < PARTS; w <<= 1) {
    dot += __shfl_xor(dot, w, 64);
    sum += __shfl_xor(sum, w, 64);
  }
  const float Dt = t < s.n ? D[(int64_t)slice * s.n + t] : 1.f;
  float w = 0.f, sig, inv = 1.f;
  if (ln) {
    const float m1 = sum / (float)s.d, m2 = dot / (float)s.d;
#pragma unroll
    for (int i = 0; i < 16; ++i) g[i] = ok ? Dt * (g[i] - m1 - o[i] * m2) : 0.f;
    sig = -dot * Dt * Dt;
  } else if (PT == 1) {
    w = -dot;
    inv = 1.0f / Dt;
    sig = w * inv;
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) g[i] = g[i] / Dt;
    w = sig = -dot / Dt;
  }
  if (t >= s.n) w = sig = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f32x4 x;
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = g[4 * i + j];
    *reinterpret_cast<f32x4 *>(&tile[r * LS + pc + 4 * i]) = x;
  }
  if (pc == 0) {
    wrow[r] = w;
    if (t < 32 * s.nt) {
      ddw[(int64_t)slice * 32 * s.nt + t] = w;
      if (PT == 1) rowscale[(int64_t)slice * 32 * s.nt + t] = inv;
    }
  } else {
    sig = 0.f;
  }
  sig = wave_sum(sig);
  if ((tid & 63) == 0) red[tid >> 6] = sig;
  __syncthreads();
  if (tid == 0) part[(int64_t)slice * gridDim.x + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
  constexpr int NP = RB / 32 * 2 * G::CT * 64;
#pragma unroll
  for (int u = 0; u < NP / 256; ++u) {   // k = tokens
    const int p = tid + 256 * u, lane = p & 63, ct = (p >> 6) % G::CT, a = (p >> 6) / G::CT % 2, tbl = (p >> 6) / (2 * G::CT);
    const int tb = t0 / 32 + tbl, c = 32 * ct + (lane & 31), h = lane >> 5;
    if (tb >= s.nt) continue;
    float x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int rr = tbl * 32 + 16 * a + 8 * (i >> 2) + 4 * h + (i & 3);
      // (head dimension 16: the weights w_t of dz = Phi^T w sit in column 16, with one term per operand in
      // columns 16, 17, 18)
      x[i] = c < DH ? tile[rr * LS + (c < DH ? c : 0)] : (c < (PT == 1 ? 19 : 17) ? wrow[rr] : 0.f);
    }
    bf16x8 tt[3];
    split8(x, tt);
    if (DH == 16 && PT == 1) {
      if (c == 17) tt[0] = tt[1];
      if (c == 18) tt[0] = tt[2];
    }
    bf16_t *dd = NC + ((((int64_t)slice * s.nt + tb) * 2 + a) * G::CT + ct) * PT * kTile;
#pragma unroll
    for (int i = 0; i < PT; ++i) store_operand(dd + i * kTile, lane, tt[i]);
  }
}

// ------------------------------------------------------------------------------------
// part[slice][p][f][c] = sum over the p-th share of the tokens of ReLU(X Omega)[t, f] Y[t, c], and the
// same against the weights w_t (1 where w is nullptr) into zpart[slice][p][f]; head dimension 16 has that
// column among the 32 of Y.  Eight waves: FW of them own one feature tile each, and TW such groups take the token
// tiles of a stage in turn (each group a share of its own).  X and Y go through LDS, one stage of SG token
// tiles ahead in registers; Omega stays in registers.  Grid (splits, feature tiles / FW, slices).
// ------------------------------------------------------------------------------------
// Token tiles (32 rows) per stage: the double-buffered stage stays below 100 KiB of LDS, and below 50 KiB where that lets
// the registers of a second workgroup in (head dimension 32 with three terms: 359 -> 334 us with half the stage).
constexpr int stage_tokens(int DH, int PT) { return DH == 128 ? 1 : (DH == 64 || (DH == 32 && PT == 3) ? 2 : 4); }
template <int DH, int PT, bool BITS>
__global__ __launch_bounds__(512, 2) void contract_kernel(const bf16_t *X, const bf16_t *Y, const float *w, const bf16_t *OA,
                                                         Dims s, int FW, int TW, int tiles_per_split, float *part, float *zpart,
                                                         unsigned short *bits) {
  using G = Geo<DH>;
  constexpr int SG = stage_tokens(DH, PT), NX = G::KS * 3, NY = 2 * G::CT * PT, NS = SG * (NX + NY),
                NW = 8, U = (NS + NW - 1) / NW;
  // The leading product in an accumulator of its own, where its registers cost no wave: S (4096 tokens, d 16) 0.70e-7 -> 0.49e-7 from
  // the exact sum, d 64, 3000 tokens 0.92e-7 -> 0.71e-7; 118 -> 120 us, 48.9 -> 49.0.
  constexpr bool LO = DH <= 64 && !(DH == 32 && PT == 3);
  __shared__ __attribute__((aligned(16))) bf16_t lds[2][NS * kTile];
  __shared__ __attribute__((aligned(16))) float lw[2][SG * 32];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slice = blockIdx.z, fw = wave % FW, tw = wave / FW;
  const int ft = blockIdx.y * FW + fw;
  const int tb0 = blockIdx.x * tiles_per_split, tb1 = min(s.nt, tb0 + tiles_per_split);
  const bf16_t *xs = X + (int64_t)slice * s.nt * NX * kTile, *ys = Y + (int64_t)slice * s.nt * NY * kTile;
  bf16x8 om[G::KS][PT];
#pragma unroll
  for (int ks = 0; ks < G::KS; ++ks)
#pragma unroll
    for (int i = 0; i < PT; ++i) om[ks][i] = lds_operand(OA + (((int64_t)ft * G::KS + ks) * PT + i) * kTile, lane);
  u32x4 st[U];
  float stw = 0.f;
  auto fetch = [&](int tb) {   // (consecutive token tiles are contiguous; what lies past the slice is clamped and not used)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(wave + NW * u, NS - 1);   // (no branch: a last tile may be moved twice)
      const int64_t tile = i < SG * NX ? min(tb * NX + i, s.nt * NX - 1) : min(tb * NY + i - SG * NX, s.nt * NY - 1);
      st[u] = *reinterpret_cast<const u32x4 *>((i < SG * NX ? xs : ys) + tile * kTile + lane * 8);
    }
    if (DH > 16 && w) stw = w[(int64_t)slice * s.nt * 32 + min(tb * 32 + (tid & (SG * 32 - 1)), s.nt * 32 - 1)];
  };
  auto put = [&](int b) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(wave + NW * u, NS - 1);
      *reinterpret_cast<u32x4 *>(&lds[b][i * kTile + lane * 8]) = st[u];
    }
    if (DH > 16) lw[b][tid & (SG * 32 - 1)] = w ? stw : 1.f;
  };
  f32x16 acc[G::CT], lo[LO ? G::CT : 1];
#pragma unroll
  for (int ct = 0; ct < G::CT; ++ct) {
    acc[ct] = zero16();
    if (LO) lo[LO ? ct : 0] = zero16();
  }
  float zacc = 0.f;
  const NegIdentity ni(lane);
  if (tb0 < tb1) {
    fetch(tb0);
    put(0);
    wait_loads();
    __syncthreads();
    int b = 0;
    for (int tb = tb0; tb < tb1; tb += SG, b ^= 1) {
      const bool more = tb + SG < tb1;
      if (more) fetch(tb + SG);
      for (int g = tw < TW ? tw : SG; g < SG && tb + g < tb1; g += TW) {
        const bf16_t *lx = &lds[b][g * NX * kTile], *ly = &lds[b][(SG * NX + g * NY) * kTile];
        f32x16 R = zero16();
#pragma unroll
        for (int ks = 0; ks < G::KS; ++ks) {
          bf16x8 x[3];
#pragma unroll
          for (int i = 0; i < 3; ++i) x[i] = lds_operand(lx + (ks * 3 + i) * kTile, lane);
          R = mfma_terms<PT, false>(R, x, om[ks]);   // rows: tokens, columns (lanes): features
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) R[i] = relu(R[i]);
        if (DH > 16) {
          f32x4 w4[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) w4[j] = *reinterpret_cast<const f32x4 *>(&lw[b][g * 32 + 8 * j + 4 * h]);
          zacc += dot16(R, w4);
        }
        bf16x8 lead[2];
        with_split<mfma_residuals(DH, PT, true)>(R, ni, [&](int a, const bf16x8 *p) {
          if (BITS) lead[a] = p[0];
#pragma unroll
          for (int ct = 0; ct < G::CT; ++ct) {
            bf16x8 y[PT];
#pragma unroll
            for (int i = 0; i < PT; ++i) y[i] = lds_operand(ly + ((a * G::CT + ct) * PT + i) * kTile, lane);
            add_terms<PT>(acc[ct], LO ? lo[LO ? ct : 0] : acc[ct], p, y);   // rows: features, columns: columns of Y
          }
        });
        if (BITS)
          bits[(((int64_t)slice * s.nt + tb + g) * s.mt + ft) * 64 + ((lane & ~36) | (lane & 4) << 3 | (lane & 32) >> 3)] =
              (unsigned short)decisions(lead);
      }
      if (more) put(b ^ 1);
      __syncthreads();
    }
  }
  if (tw >= TW) return;
  const int64_t pidx = (int64_t)slice * gridDim.x * TW + blockIdx.x * TW + tw;
  constexpr int PW = 32 * G::CT;
  float *po = part + (pidx * s.mt + ft) * 32 * PW;
#pragma unroll
  for (int ct = 0; ct < G::CT; ++ct)
#pragma unroll
    for (int i = 0; i < 16; ++i) po[(8 * (i >> 2) + 4 * h + (i & 3)) * PW + 32 * ct + l32] = LO ? acc[ct][i] + lo[LO ? ct : 0][i] : acc[ct][i];
  if (DH > 16) {
    zacc = xor32_sum(zacc);
    if (h == 0) zpart[(pidx * s.mt + ft) * 32 + l32] = zacc;
  }
}

// ------------------------------------------------------------------------------------
// S (or dS) and z (or dz) of one feature tile: fixed-order sum of the shares, times c; in the forward the float32
// results [m][d] and [m], and the operand tiles of the kernels that follow: columns as vectors with k = features (SB);
// in the backward also features as vectors (SA) with the extension tile that carries the rank-one term dD z^T
// (three-term products in six k-slots), for dS and, from the forward's S and z (blockIdx.z = 1), SAin.
// Grid (feature tiles, slices, forward 1, backward 2).
// ------------------------------------------------------------------------------------
// Sum of the values at p, p + step, ...: eight at a time (in flight together) as a tree, eight of these in a chain, and a
// chain of those.  In one chain, the hundreds of shares of a long sequence would lose more than the products do.
// SHORT: up to 32 shares in few workgroups, sixteen in flight together.
template <bool SHORT, typename V>
__device__ __forceinline__ V sum_shares(const float *p, int64_t step, int shares) {
  V acc = (V)(0.f), part = (V)(0.f);
  int sh = 0;
  if constexpr (SHORT) {
#pragma unroll 1
    for (; sh < shares; sh += 16) {
      V x[16];
#pragma unroll
      for (int k = 0; k < 16; k += 8)
        if (sh + k < shares)
#pragma unroll
          for (int i = k; i < k + 8; ++i) x[i] = *reinterpret_cast<const V *>(p + min(sh + i, shares - 1) * step);
#pragma unroll
      for (int k = 0; k < 16; k += 8) {
        if (sh + k + 8 <= shares) {
          part += ((x[k] + x[k + 1]) + (x[k + 2] + x[k + 3])) + ((x[k + 4] + x[k + 5]) + (x[k + 6] + x[k + 7]));
        } else {
#pragma unroll
          for (int i = k; i < k + 7; ++i)
            if (sh + i < shares) part += x[i];
        }
      }
    }
    return part;
  }
  for (; sh + 8 <= shares; sh += 8) {
    V x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = *reinterpret_cast<const V *>(p + (sh + i) * step);
    part += ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
    if (sh % 64 == 56) {
      acc += part;
      part = (V)(0.f);
    }
  }
  for (; sh < shares; ++sh) part += *reinterpret_cast<const V *>(p + sh * step);
  return acc + part;
}
template <int DH, bool SHORT>
__global__ __launch_bounds__(256) void reduce_kernel(const float *part, const float *zpart, int shares, int zcols,
                                                    const float *scalars, Dims s, float *S, float *z, float *zpad,
                                                    bf16_t *SA, bf16_t *SB, bf16_t *SAin) {
  using G = Geo<DH>;
  constexpr int PW = 32 * G::CT, LS = PW + 1;
  __shared__ float tile[32 * LS];
  __shared__ float zt[32];
  const int tid = threadIdx.x, ft = blockIdx.x, slice = blockIdx.y;
  const bool given = SAin && blockIdx.z;   // S and z are there already
  const float c = scalars[0];
  if (given) {
    for (int e = tid; e < 32 * DH; e += 256) {
      const int f = e / DH, cc = e % DH;
      tile[f * LS + cc] = (32 * ft + f < s.m && cc < s.d) ? S[((int64_t)slice * s.m + 32 * ft + f) * s.d + cc] : 0.f;
    }
    if (tid < 32) zt[tid] = 32 * ft + tid < s.m ? z[(int64_t)slice * s.m + 32 * ft + tid] : 0.f;
    __syncthreads();
  } else {
    const int64_t step = (int64_t)s.mt * 32 * PW;
    const float *p0 = part + ((int64_t)slice * shares * s.mt + ft) * 32 * PW;
#pragma unroll
    for (int u = 0; u < 32 * PW / 1024; ++u) {
      const int e = (tid + 256 * u) * 4;
      const f32x4 acc = sum_shares<SHORT, f32x4>(p0 + e, step, shares);
#pragma unroll
      for (int i = 0; i < 4; ++i) tile[(e / PW) * LS + e % PW + i] = acc[i] * c;
    }
    if (DH > 16 && tid < 32)
      zt[tid] = sum_shares<SHORT, float>(zpart + ((int64_t)slice * shares * s.mt + ft) * 32 + tid, (int64_t)s.mt * 32, shares) * c;
    __syncthreads();
    if (DH == 16 && tid < 32) {
      float acc = 0.f;
      for (int j = zcols - 1; j >= 0; --j) acc += tile[tid * LS + 16 + j];
      zt[tid] = acc;
    }
    __syncthreads();
    if (!SAin) {   // forward
      for (int e = tid; e < 32 * s.d; e += 256) {
        const int f = e / s.d, cc = e % s.d;
        if (32 * ft + f < s.m) S[((int64_t)slice * s.m + 32 * ft + f) * s.d + cc] = tile[f * LS + cc];
      }
      if (tid < 32) {
        if (32 * ft + tid < s.m) z[(int64_t)slice * s.m + 32 * ft + tid] = zt[tid];
        zpad[((int64_t)slice * s.mt + ft) * 32 + tid] = zt[tid];
      }
    }
  }
  bf16_t *sa = (given ? SAin : SA) + ((int64_t)slice * s.mt + ft) * (3 * G::KS + 1) * kTile;
  bf16_t *sb = SB + ((int64_t)slice * s.mt + ft) * G::NSB * kTile;
  const int first = SA ? 0 : G::KS + 1, last = given ? G::KS + 1 : G::KS + 1 + 2 * G::CT;   // (the forward needs SB only)
  for (int p = tid + 64 * first; p < 64 * last; p += 256) {
    const int lane = p & 63, which = p >> 6, l32 = lane & 31, h = lane >> 5;
    bf16x8 t[3];
    if (which < G::KS) {
      float x[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) x[q] = tile[l32 * LS + 16 * which + 8 * h + q];
      split8(x, t);
#pragma unroll
      for (int i = 0; i < 3; ++i) store_operand(sa + (3 * which + i) * kTile, lane, t[i]);
    } else if (which == G::KS) {
      __bf16 zz[3];
      split1(h == 0 ? zt[l32] : 0.f, zz);
      const __bf16 o = (__bf16)0.f;
      const bf16x8 e = {zz[0], zz[1], zz[0], zz[2], zz[0], zz[1], o, o};
      store_operand(sa + 3 * G::KS * kTile, lane, e);
    } else {
      const int a = (which - G::KS - 1) / G::CT, ct = (which - G::KS - 1) % G::CT, cc = 32 * ct + l32;
      float x[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        x[q] = tile[(16 * a + 8 * (q >> 2) + 4 * h + (q & 3)) * LS + (DH == 16 ? cc & 15 : cc)];
      }
      split8(x, t);
      if (DH == 16) {
        const bf16x8 none = {};
        store_operand(sb + 2 * a * kTile, lane, cc < 16 ? t[0] : t[1]);
        store_operand(sb + (2 * a + 1) * kTile, lane, cc < 16 ? t[2] : none);
      } else {
#pragma unroll
        for (int i = 0; i < 3; ++i) store_operand(sb + ((a * G::CT + ct) * 3 + i) * kTile, lane, t[i]);
      }
    }
  }
}

// ------------------------------------------------------------------------------------
// Kernels that own token rows and walk over the features: RT token tiles per wave, NW waves, the operands
// of FC feature tiles per stage through LDS (shared by the waves), the next stage ahead in registers.
// Sections of a stage: up to four packed arrays, each contiguous per feature tile.
// ------------------------------------------------------------------------------------
template <int N0, int N1, int N2, int N3, int FC, int NW>
struct Stager {
  static constexpr int NS = FC * (N0 + N1 + N2 + N3), U = (NS + NW - 1) / NW;
  static constexpr int O1 = FC * N0, O2 = O1 + FC * N1, O3 = O2 + FC * N2;   // first tile of each section in LDS
  const bf16_t *p0, *p1, *p2, *p3;
  u32x4 st[U];
  __device__ __forceinline__ void fetch(int ft, int wave, int lane) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(wave + NW * u, NS - 1);   // (no branch: a last tile may be moved twice)
      const bf16_t *src = i < O1   ? p0 + ((int64_t)ft * N0 + i) * kTile
                          : i < O2 ? p1 + ((int64_t)ft * N1 + (i - O1)) * kTile
                          : i < O3 ? p2 + ((int64_t)ft * N2 + (i - O2)) * kTile
                                   : p3 + ((int64_t)ft * N3 + (i - O3)) * kTile;
      st[u] = *reinterpret_cast<const u32x4 *>(src + lane * 8);
    }
  }
  __device__ __forceinline__ void put(bf16_t *lds, int wave, int lane) const {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(wave + NW * u, NS - 1);
      *reinterpret_cast<u32x4 *>(&lds[i * kTile + lane * 8]) = st[u];
    }
  }
};

// A sum over the features is taken sum_tiles feature tiles at a time where the registers hold a second accumulator: the
// matrix cores round an accumulator after every product (and a little towards zero: the same in all columns of a row, which
// <dO, O> does not average out), and with one for the whole sum its error grows with the square root of m.  An accumulator for the
// leading products and one for the others are as many registers, but halve the error only.  2048 tokens, d 32, 4096 features, against float64:
// O 3.4e-7 -> 1.1e-7, dK 3.1e-7 -> 1.0e-7, dV (one accumulator) 5.9e-7 -> 0.9e-7; 4000 tokens, 1024 features: 1.7e-7 -> 0.8e-7,
// 1.3e-7 -> 0.9e-7, 3.3e-7 -> 0.7e-7.  Their training step (128 slices of the latter) 2430 -> 2463 us.  With one-term operands the results are
// rounded to bf16, and the registers are worth more (head dimension 16, 8 slices of 131072 tokens: 382 us without, 397 with).
constexpr int sum_tiles(int DH) { return DH <= 32 ? 4 : 1; }
constexpr bool sum_in_parts(int PT) { return PT == 3; }
// Waves per SIMD that the register budget is set for.
constexpr int row_occupancy(int DH, int NW) { return NW >= 4 && DH < 128 ? 2 : 1; }

// MODE 0: O = (Phi S) / (Phi z + eps) and D.   1: N = Phi S in float32 (LayerNorm follows).
// MODE 2: dV = Phi_K dS.     X: operand tiles of Q_F or K_F.  Grid (row groups, slices).
template <typename T, int DH, int PT, int MODE, int RT, int NW>
__global__ __launch_bounds__(NW * 64, row_occupancy(DH, NW)) void apply_kernel(const bf16_t *X, const bf16_t *OA, const bf16_t *SB,
                                                                       const float *zpad, const float *scalars, float eps,
                                                                       Dims s, T *out, View v, float *N, float *D,
                                                                       unsigned short *bits) {
  using G = Geo<DH>;
  constexpr bool BITS = MODE == 2;
  constexpr int FC = DH <= 32 ? 2 : 1, NA = G::KS * PT, NB = G::NSB;
  constexpr bool ZV = MODE == 0;   // the normaliser, on the vector units
  typedef Stager<NA, NB, 0, 0, FC, NW> Stg;
  __shared__ __attribute__((aligned(16))) bf16_t lds[2][Stg::NS * kTile];
  __shared__ __attribute__((aligned(16))) float lz[2][ZV ? FC * 32 : 1];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slice = blockIdx.y, tb0 = (blockIdx.x * NW + wave) * RT;
  bf16x8 x[RT][G::KS][3];
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    const bf16_t *xp = X + ((int64_t)slice * s.nt + min(tb0 + r, s.nt - 1)) * G::KS * 3 * kTile;
#pragma unroll
    for (int ks = 0; ks < G::KS; ++ks)
#pragma unroll
      for (int i = 0; i < 3; ++i) x[r][ks][i] = lds_operand(xp + (ks * 3 + i) * kTile, lane);
  }
  Stg sg;
  sg.p0 = OA;
  sg.p1 = SB + (int64_t)slice * s.mt * NB * kTile;
  sg.p2 = sg.p3 = nullptr;
  constexpr bool PARTS = sum_in_parts(PT);
  f32x16 acc[RT][G::CT], total[PARTS ? RT : 1][G::CT];
  float dsum[RT], dpart[RT];   // Phi z: of all groups of eight feature tiles before, of this one
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    dsum[r] = dpart[r] = 0.f;
#pragma unroll
    for (int ct = 0; ct < G::CT; ++ct) {
      acc[r][ct] = zero16();
      if (PARTS) total[PARTS ? r : 0][ct] = zero16();
    }
  }
  const NegIdentity ni(lane);
  const float *zs = zpad + (int64_t)slice * s.mt * 32;
  const int zi = tid & (FC * 32 - 1);
  float zr = 0.f;
  sg.fetch(0, wave, lane);
  if (ZV) zr = zs[min(zi, s.mt * 32 - 1)];
  sg.put(lds[0], wave, lane);
  if (ZV) lz[0][zi] = zr;
  wait_loads();
  __syncthreads();
  int b = 0;
  for (int f0 = 0; f0 < s.mt; f0 += FC, b ^= 1) {
    const bool more = f0 + FC < s.mt;
    if (more) {
      sg.fetch(f0 + FC, wave, lane);
      if (ZV) zr = zs[min((f0 + FC) * 32 + zi, s.mt * 32 - 1)];
    }
#pragma unroll
    for (int fi = 0; fi < FC; ++fi) {
      if (f0 + fi >= s.mt) break;
      const bf16_t *la = &lds[b][fi * NA * kTile], *lb = &lds[b][(Stg::O1 + fi * NB) * kTile];
      f32x4 z4[4];
      if (ZV)
#pragma unroll
        for (int j = 0; j < 4; ++j) z4[j] = *reinterpret_cast<const f32x4 *>(&lz[b][fi * 32 + 8 * j + 4 * h]);
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        f32x16 R = zero16();
#pragma unroll
        for (int ks = 0; ks < G::KS; ++ks) {
          bf16x8 o[PT];
#pragma unroll
          for (int i = 0; i < PT; ++i) o[i] = lds_operand(la + (ks * PT + i) * kTile, lane);
          R = mfma_terms<PT, true>(R, x[r][ks], o);   // rows: features, lanes: tokens
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) R[i] = relu(R[i]);
        if (ZV) dpart[r] += dot16(R, z4);
        bf16x8 lead[2];
        with_split<mfma_residuals(DH, PT)>(R, ni, [&](int a, const bf16x8 *p) {
          if (BITS) lead[a] = p[0];
#pragma unroll
          for (int ct = 0; ct < G::CT; ++ct) apply_terms<DH>(acc[r][ct], p, lb, a, ct, lane);   // rows: tokens, lanes: columns
        });
        if (BITS && tb0 + r < s.nt)
          bits[(((int64_t)slice * s.nt + tb0 + r) * s.mt + f0 + fi) * 64 + lane] =
              (unsigned short)TransposeDecisions(lane)(decisions(lead));
      }
    }
    if (ZV && (!more || (f0 + FC) % 8 == 0)) {
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        dsum[r] += dpart[r];
        dpart[r] = 0.f;
      }
    }
    if (PARTS && (!more || (f0 + FC) % sum_tiles(DH) == 0)) {
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int ct = 0; ct < G::CT; ++ct) {
          total[PARTS ? r : 0][ct] += acc[r][ct];
          acc[r][ct] = zero16();
        }
    }
    if (more) {
      sg.put(lds[b ^ 1], wave, lane);
      if (ZV) lz[b ^ 1][zi] = zr;
    }
    __syncthreads();
  }
  const float c = scalars[0];
  T *const ob = MODE == 1 ? nullptr : out + v.slice_base(slice);
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    const int tb = tb0 + r;
    if (tb >= s.nt) continue;
    float Dl = 0.f;
    if (ZV) Dl = fmaf(c, xor32_sum(dsum[r]), eps);   // token l32
    if (ZV && h == 0 && 32 * tb + l32 < s.n) D[(int64_t)slice * s.n + 32 * tb + l32] = Dl;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int row = 8 * (i >> 2) + 4 * h + (i & 3), t = 32 * tb + row;
      float Dt = 1.f;
      if (ZV) Dt = __shfl(Dl, row, 64);
      if (PARTS)
#pragma unroll
        for (int ct = 0; ct < G::CT; ++ct) acc[r][ct][i] = total[PARTS ? r : 0][ct][i];
      if (DH == 16) acc[r][0][i] += __shfl_xor(acc[r][0][i], 16, 64);
#pragma unroll
      for (int ct = 0; ct < G::CT; ++ct) {
        const int col = 32 * ct + l32;
        if (t < s.n && col < s.d) {
          const float val = c * acc[r][ct][i];
          if (MODE == 1) N[((int64_t)slice * s.n + t) * s.d + col] = val;
          else st(ob + (int64_t)t * v.sn + col, MODE == 0 ? val / Dt : val);
        }
      }
    }
  }
}

// The gradient kernel's dX_F likewise, and dV where it rides along (at head dimension 64 it has no registers left for either).
constexpr bool grad_in_parts(int DH, int PT, bool DV) { return sum_in_parts(PT) && (DH <= 32 || (DH == 64 && !DV)); }
// dX_F of one side: G = Y S^T + w z^T (Y = dN, S, w = dD on the query side; Y = V, dS, w = 1
// on the key side), dX_F = c rowscale ((G masked where R = X Omega > 0) Omega^T) in float32, row t of a slice at
// grad_row(t) (in the place of X's operand tiles, which at most the wave that writes them still needs, and it has read its own).
// DV: dV = c ReLU(R) dS rides along, R is formed here; without DV the decisions come as bits.
// Bits instead of the projection, query side, us: 128 slices of 4000 tokens, d 32, m 1024, float32 525 -> 371 (the registers of X
// hold a second token tile), the contraction that leaves them 328 -> 344; 8 of 131072, d 16, m 1024, bf16 385 -> 330, 280 -> 305; 8 of 16384,
// m 256, float32, d 64 85 -> 64, 51 -> 52; d 128 both sides 193 -> 134, dV's kernel 156 -> 159.  dV on its own at d 32, with
// the key side's gradient on bits, would take 329 and 371 where the two in one take 729.  ddw, rowscale nullptr: 1.
// The rows of Y come from the tensors as they are: y, divided by D (one term: not), or with the LayerNorm output
// stage (o given) rstd (y - mean y - o mean(y o)).
template <int DH> constexpr int64_t grad_tile() { return 48 * DH; }   // floats of a tile of 32 rows: its operand tiles' size
template <int DH>
__device__ __forceinline__ int64_t grad_row(int t) { return (int64_t)(t >> 5) * grad_tile<DH>() + (t & 31) * DH; }
template <typename T>
struct GradRows {
  const T *y, *o;
  const float *D;
  int vec;
};
template <typename T, int DH, int PT, bool DV, int RT, int NW>
__global__ __launch_bounds__(NW * 64, row_occupancy(DH, NW)) void grad_kernel(const bf16_t *X, const unsigned short *bits, GradRows<T> Y, const float *ddw,
                                                                      const float *rowscale, const bf16_t *OA,
                                                                      const bf16_t *SA, const bf16_t *OB, const bf16_t *SB,
                                                                      const float *scalars, Dims s, float *dXF, T *dv, View v) {
  using G = Geo<DH>;
  constexpr int FC = DH == 16 || (DH == 32 && PT == 1 && !DV) ? 2 : 1, NA = DV ? G::KS * PT : 0, NSA = 3 * G::KS + 1, NOB = 2 * G::CT * PT, NSB = DV ? G::NSB : 0;
  typedef Stager<NA, NSA, NOB, NSB, FC, NW> Stg;
  __shared__ __attribute__((aligned(16))) bf16_t lds[2][Stg::NS * kTile];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slice = blockIdx.y, tb0 = (blockIdx.x * NW + wave) * RT;
  bf16x8 x[DV ? RT : 1][G::KS][3], y[RT][G::KS][PT], ext[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    const bool mine = tb0 + r < s.nt;   // (a wave past the last tile only helps to stage)
    const int64_t tb = (int64_t)slice * s.nt + (mine ? tb0 + r : 0);
    if constexpr (DV) {
      const bf16_t *xp = X + tb * G::KS * 3 * kTile;
#pragma unroll
      for (int ks = 0; ks < G::KS; ++ks)
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          x[r][ks][i] = bf16x8{};
          if (mine) x[r][ks][i] = lds_operand(xp + (ks * 3 + i) * kTile, lane);
        }
    }
    const int t = 32 * (tb0 + r) + l32;
    const bool ok = t < s.n;
    const int64_t row = v.slice_base(slice) + (int64_t)(ok ? t : 0) * v.sn;
    float g[G::KS][8];
#pragma unroll
    for (int ks = 0; ks < G::KS; ++ks) {
      const int col = 16 * ks + 8 * h;
      load8(Y.y + row + (col < s.d ? col : 0), Y.vec, g[ks]);
#pragma unroll
      for (int q = 0; q < 8; ++q) g[ks][q] = ok && col < s.d ? g[ks][q] : 0.f;
    }
    if (!DV && PT == 3 && Y.D) {
      const float Dt = ok ? Y.D[(int64_t)slice * s.n + t] : 1.f;
      if (Y.o) {
        float sum = 0.f, dot = 0.f, o[G::KS][8];
#pragma unroll
        for (int ks = 0; ks < G::KS; ++ks) {
          const int col = 16 * ks + 8 * h;
          load8(Y.o + row + (col < s.d ? col : 0), Y.vec, o[ks]);
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            o[ks][q] = ok && col < s.d ? o[ks][q] : 0.f;
            sum += g[ks][q];
            dot = fmaf(g[ks][q], o[ks][q], dot);
          }
        }
        const float m1 = xor32_sum(sum) / (float)s.d, m2 = xor32_sum(dot) / (float)s.d;
#pragma unroll
        for (int ks = 0; ks < G::KS; ++ks)
#pragma unroll
          for (int q = 0; q < 8; ++q) g[ks][q] = ok && 16 * ks + 8 * h < s.d ? Dt * (g[ks][q] - m1 - o[ks][q] * m2) : 0.f;
      } else {
#pragma unroll
        for (int ks = 0; ks < G::KS; ++ks)
#pragma unroll
          for (int q = 0; q < 8; ++q) g[ks][q] = g[ks][q] / Dt;
      }
    }
#pragma unroll
    for (int ks = 0; ks < G::KS; ++ks) {
      bf16x8 t3[3];
      split8(g[ks], t3);
#pragma unroll
      for (int i = 0; i < PT; ++i) y[r][ks][i] = t3[i];
    }
    __bf16 w[3];
    split1(h ? 0.f : (ddw ? ddw[tb * 32 + l32] : 1.f), w);
    const __bf16 o = (__bf16)0.f;
    ext[r] = bf16x8{w[0], w[0], w[1], w[0], w[2], w[1], o, o};   // against z0, z1, z0, z2, z0, z1
  }
  Stg sg;
  sg.p0 = OA;
  sg.p1 = SA + (int64_t)slice * s.mt * NSA * kTile;
  sg.p2 = OB;
  sg.p3 = DV ? SB + (int64_t)slice * s.mt * NSB * kTile : nullptr;
  constexpr bool PARTS = grad_in_parts(DH, PT, DV), VPARTS = PARTS && DV;
  f32x16 acc[RT][G::CT], total[PARTS ? RT : 1][G::CT], accv[DV ? RT : 1][G::CT], totalv[VPARTS ? RT : 1][G::CT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int ct = 0; ct < G::CT; ++ct) {
      acc[r][ct] = zero16();
      if (PARTS) total[PARTS ? r : 0][ct] = zero16();
      if (DV) accv[DV ? r : 0][ct] = zero16();
      if (VPARTS) totalv[VPARTS ? r : 0][ct] = zero16();
    }
  const NegIdentity ni(lane);
  // the decisions of a stage's feature tiles, one stage ahead (two token tiles share a word)
  const TransposeDecisions transpose(lane);
  constexpr int WR = (RT + 1) / 2;
  unsigned short next[DV ? 1 : FC][DV ? 1 : RT];
  uint32_t word[DV ? 1 : FC][WR];
  auto fetch_bits = [&](int f0) {
#pragma unroll
    for (int fi = 0; fi < FC; ++fi)
#pragma unroll
      for (int r = 0; r < RT; ++r)
        next[fi][r] = bits[(((int64_t)slice * s.nt + min(tb0 + r, s.nt - 1)) * s.mt + min(f0 + fi, s.mt - 1)) * 64 + lane];
  };
  auto take_bits = [&]() {
#pragma unroll
    for (int fi = 0; fi < FC; ++fi)
#pragma unroll
      for (int u = 0; u < WR; ++u)
        word[fi][u] = transpose(2 * u + 1 < RT ? (uint32_t)next[fi][2 * u] | (uint32_t)next[fi][2 * u + 1 < RT ? 2 * u + 1 : 0] << 16
                                               : (uint32_t)next[fi][2 * u]);
  };
  sg.fetch(0, wave, lane);
  if constexpr (!DV) fetch_bits(0);
  sg.put(lds[0], wave, lane);
  wait_loads();
  __syncthreads();
  int b = 0;
  for (int f0 = 0; f0 < s.mt; f0 += FC, b ^= 1) {
    const bool more = f0 + FC < s.mt;
    if constexpr (!DV) take_bits();
    if (more) {
      sg.fetch(f0 + FC, wave, lane);
      if constexpr (!DV) fetch_bits(f0 + FC);
    }
#pragma unroll
    for (int fi = 0; fi < FC; ++fi) {
      if (f0 + fi >= s.mt) break;
      const bf16_t *la = &lds[b][fi * NA * kTile], *ls = &lds[b][(Stg::O1 + fi * NSA) * kTile],
                   *lo = &lds[b][(Stg::O2 + fi * NOB) * kTile], *lv = &lds[b][(Stg::O3 + fi * NSB) * kTile];
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        f32x16 R = zero16(), Gr = zero16();
        if constexpr (DV)
#pragma unroll
          for (int ks = 0; ks < G::KS; ++ks) {
            bf16x8 o[PT];
#pragma unroll
            for (int i = 0; i < PT; ++i) o[i] = lds_operand(la + (ks * PT + i) * kTile, lane);
            R = mfma_terms<PT, true>(R, x[r][ks], o);   // rows: features, lanes: tokens
          }
        // (the small products of the whole sum first: while they are added the accumulator is small, and so is its rounding)
        auto go = [&](int ks, int i, int j) { Gr = mfma(lds_operand(ls + (ks * 3 + i) * kTile, lane), y[r][ks][j], Gr); };
#pragma unroll
        for (int ks = 0; ks < G::KS; ++ks) {
          if (PT == 3) {
            go(ks, 0, PT - 1);
            go(ks, 1, PT / 2);
          }
          go(ks, 2, 0);
          if (PT == 3) go(ks, 0, PT / 2);
          go(ks, 1, 0);
        }
#pragma unroll
        for (int ks = 0; ks < G::KS; ++ks) go(ks, 0, 0);
        Gr = mfma(lds_operand(ls + 3 * G::KS * kTile, lane), ext[r], Gr);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          if constexpr (DV) {
            const float mask = positive(R[i]);
            Gr[i] = masked(Gr[i], mask);
            R[i] = masked(R[i], mask);
          } else {
            Gr[i] = masked(Gr[i], word[fi][r / 2], i, r % 2);
          }
        }
        with_split<mfma_residuals(DH, PT, DV)>(Gr, ni, [&](int a, const bf16x8 *p) {
#pragma unroll
          for (int ct = 0; ct < G::CT; ++ct) {
            bf16x8 o[PT];
#pragma unroll
            for (int i = 0; i < PT; ++i) o[i] = lds_operand(lo + ((a * G::CT + ct) * PT + i) * kTile, lane);
            add_terms<PT>(acc[r][ct], acc[r][ct], p, o);   // rows: tokens, lanes: columns
          }
        });
        if (DV)
          with_split<mfma_residuals(DH, PT, DV)>(R, ni, [&](int a, const bf16x8 *p) {
#pragma unroll
            for (int ct = 0; ct < G::CT; ++ct) apply_terms<DH>(accv[r][ct], p, lv, a, ct, lane);
          });
      }
    }
    if (PARTS && (!more || (f0 + FC) % sum_tiles(DH) == 0)) {
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int ct = 0; ct < G::CT; ++ct) {
          total[PARTS ? r : 0][ct] += acc[r][ct];
          acc[r][ct] = zero16();
          if (VPARTS) {
            totalv[VPARTS ? r : 0][ct] += accv[DV ? r : 0][ct];
            accv[DV ? r : 0][ct] = zero16();
          }
        }
    }
    if (more) sg.put(lds[b ^ 1], wave, lane);
    __syncthreads();
  }
  const float c = scalars[0];
  T *const vb = DV ? dv + v.slice_base(slice) : nullptr;
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    const int tb = tb0 + r;
    if (tb >= s.nt) continue;
    const float rs = rowscale ? c * rowscale[((int64_t)slice * s.nt + tb) * 32 + l32] : c;   // token l32
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int row = 8 * (i >> 2) + 4 * h + (i & 3), t = 32 * tb + row;
      const float sc = rowscale ? __shfl(rs, row, 64) : c;
      if (PARTS)
#pragma unroll
        for (int ct = 0; ct < G::CT; ++ct) acc[r][ct][i] = total[PARTS ? r : 0][ct][i];
      if (VPARTS)
#pragma unroll
        for (int ct = 0; ct < G::CT; ++ct) accv[DV ? r : 0][ct][i] = totalv[VPARTS ? r : 0][ct][i];
      if (DV && DH == 16) accv[r][0][i] += __shfl_xor(accv[r][0][i], 16, 64);
#pragma unroll
      for (int ct = 0; ct < G::CT; ++ct) {
        const int col = 32 * ct + l32;
        if (col < DH) dXF[((int64_t)slice * s.nt + tb) * grad_tile<DH>() + row * DH + col] = sc * acc[r][ct][i];
        if (DV && t < s.n && col < s.d) st(vb + (int64_t)t * v.sn + col, c * accv[r][ct][i]);
      }
    }
  }
}

// ------------------------------------------------------------------------------------
// Band inner products of X and dX_F on 64-row tiles (band l - 1: details of level l; band L: the
// approximation) -> part[slice][workgroup][L + 1].  One thread per (column, 16 rows); with block sums A, B of the halves of a
// 2^l-row block the detail coefficients are (A - B) / sqrt(2^l).  tgq, tgk (L > 6): the tile
// sums of dX_F.  Grid (row groups * column pieces, slices, 2: Q, K).
// ------------------------------------------------------------------------------------
template <typename T, int DH>
__global__ __launch_bounds__(256) void dots_kernel(const T *q, const T *k, View v, const float *gq, const float *gk, Dims s,
                                                  int L, int rows_out, float *partq, float *partk, float *tgq, float *tgk) {
  using G = Geo<DH>;
  constexpr int CW = G::CW, TR = G::TR;
  __shared__ float sg[G::SEGS][CW], sx[G::SEGS][CW];
  __shared__ float red[4][8];
  const int tid = threadIdx.x, slice = blockIdx.y, side = blockIdx.z;
  const int rg = blockIdx.x / G::PIECES, piece = blockIdx.x % G::PIECES;
  const int c = tid % CW, seg = tid / CW, col = piece * CW + c, t0 = rg * TR + seg * 16;
  const bool cok = col < s.d;
  const T *xp = (side ? k : q) + v.slice_base(slice) + (cok ? col : 0);
  // (16 rows from a multiple of 16: in one tile of 32, at most the last one)
  const float *gp = (side ? gk : gq) + (int64_t)slice * s.nt * grad_tile<DH>() + grad_row<DH>(min(t0, 32 * s.nt - 16)) + col;
  float a[16], b[16], e[8];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int t = t0 + i;
    a[i] = ld(xp + (int64_t)min(t, s.n - 1) * v.sn);
    b[i] = gp[i * DH];
  }
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if (!cok || t0 + i >= s.n) a[i] = b[i] = 0.f;
#pragma unroll
  for (int l = 0; l < 8; ++l) e[l] = 0.f;
  auto top = [&](int l, int cnt) {   // e[7]: the approximation band, once level L is reached
    if (l == L)
#pragma unroll
      for (int i = 0; i < cnt; ++i) e[7] = fmaf(a[i], b[i], e[7]);
  };
  top(0, 16);
#pragma unroll
  for (int l = 1; l <= 4; ++l) {
#pragma unroll
    for (int i = 0; i < (16 >> l); ++i) {
      e[l] = fmaf(a[2 * i] - a[2 * i + 1], b[2 * i] - b[2 * i + 1], e[l]);
      a[i] = a[2 * i] + a[2 * i + 1];
      b[i] = b[2 * i] + b[2 * i + 1];
    }
    top(l, 16 >> l);
  }
  sx[seg][c] = a[0];
  sg[seg][c] = b[0];
  __syncthreads();
  if ((seg & 1) == 0) {
    const float x1 = sx[seg + 1][c], g1 = sg[seg + 1][c];
    e[5] = (a[0] - x1) * (b[0] - g1);
    a[0] += x1;
    b[0] += g1;
    top(5, 1);
    if ((seg & 2) == 0) {
      const float x2 = sx[seg + 2][c] + sx[seg + 3][c], g2 = sg[seg + 2][c] + sg[seg + 3][c];
      e[6] = (a[0] - x2) * (b[0] - g2);
      a[0] += x2;
      b[0] += g2;
      top(6, 1);
      float *tg = side ? tgk : tgq;
      const int ntl = (s.n + 63) / 64, gt = (rg * TR) / 64 + seg / 4;
      if (tg && cok && gt < ntl) tg[((int64_t)slice * ntl + gt) * s.d + col] = b[0];
    }
  }
#pragma unroll
  for (int l = 1; l < 8; ++l) {
    const float t = wave_sum(e[l]);
    if ((tid & 63) == 0) red[tid >> 6][l] = t;
  }
  __syncthreads();
  if (tid <= L) {
    float val = 0.f;
    const int l = tid < L ? tid + 1 : 7;   // (bands of levels above 6 are left at zero here)
    if (tid < L ? tid < 6 : L <= 6)
      val = ((red[0][l] + red[1][l]) + (red[2][l] + red[3][l])) / (float)(1 << (tid < L ? tid + 1 : L));
    (side ? partk : partq)[((int64_t)slice * rows_out + blockIdx.x) * (L + 1) + tid] = val;
  }
}

// dQ = G_F dQ_F + dqbar / n and dK = G_F dK_F: the filter's backward (symmetric matrix) with the pooled query's
// share.  addq, addk: the per-tile addends of the levels above 6.  Grid (row groups * column pieces, slices + rows of
// the gate's parameter gradients (see gate_bwd_params_rows), 2: Q, K).
template <typename T, int DH>
__global__ __launch_bounds__(256) void filter_bwd_kernel(const float *gq, const float *gk, T *dq, T *dk, View v, Dims s, int L,
                                                        const float *coef, const float *addq, const float *addk,
                                                        const float *dqbar, float inv_n, GateBwdParams gp) {
  if (gate_bwd_params_rows(gp)) return;
  using G = Geo<DH>;
  constexpr int CW = G::CW, TR = G::TR;
  __shared__ float segsum[G::SEGS][CW];
  __shared__ float cf[8];
  const int tid = threadIdx.x, slice = blockIdx.y, side = blockIdx.z;
  if (tid < 8) cf[tid] = coef[slice * kCoefStride + tid];
  const int rg = blockIdx.x / G::PIECES, piece = blockIdx.x % G::PIECES;
  const int c = tid % CW, seg = tid / CW, col = piece * CW + c, t0 = rg * TR + seg * 16;
  const bool cok = col < s.d;
  const float *xp = (side ? gk : gq) + (int64_t)slice * s.nt * grad_tile<DH>() + grad_row<DH>(min(t0, 32 * s.nt - 16)) + col;
  float x[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] = xp[i * DH];
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if (t0 + i >= s.n) x[i] = 0.f;
  segsum[seg][c] = segment_sum<16>(x);
  __syncthreads();
  float upper = upper_levels<CW>(segsum, cf, seg, c, L);
  const float *add = side ? addk : addq;
  const int ntl = (s.n + 63) / 64, gt = (rg * TR) / 64 + seg / 4;
  if (add && cok && gt < ntl) upper += add[((int64_t)slice * ntl + gt) * s.d + col];
  filter_segment<16>(x, cf, upper, L);
  const float extra = !side && cok ? inv_n * dqbar[(int64_t)slice * s.d + col] : 0.f;
  T *yp = (side ? dk : dq) + v.slice_base(slice) + (cok ? col : 0);
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if (cok && t0 + i < s.n) st(yp + (int64_t)(t0 + i) * v.sn, x[i] + extra);
}

// ------------------------------------------------------------------------------------
// Levels above 6 (see build_tile_pyramid): addends of Q_F, K_F from the tile sums of Q and K; in the backward
// the addends of dQ, dK from the tile sums of dQ_F, dK_F, and the band inner products of the levels
// above 6 into d / 16 extra rows of the partials.  Grid (slices, 2, d / 16) of 1024 threads.
// ------------------------------------------------------------------------------------
// IN_LDS: the pyramids are (pyramid_in_lds bytes of dynamic LDS).
template <bool IN_LDS>
__global__ __launch_bounds__(1024) void deep_addend_kernel(const float *Tq, const float *Tk, const float *coef, int ntiles, int d, int L,
                                                          float *pyr, float *Aq, float *Ak) {
  extern __shared__ float lds_pyr[];
  const int slice = blockIdx.x, side = blockIdx.y, cl = threadIdx.x & (kCoarseCols - 1);
  const int c = kCoarseCols * blockIdx.z + cl, g = threadIdx.x / kCoarseCols;
  const int64_t base = (int64_t)slice * ntiles * d;
  const float *T = (side ? Tk : Tq) + base, *cf = coef + slice * kCoefStride;
  float *A = (side ? Ak : Aq) + base, *P = pyr + ((int64_t)slice * 2 + side) * pyramid_floats(ntiles, d);
  if constexpr (IN_LDS) coarse_addends(T, cf, ntiles, d, L - 6, first_level((lds_float *)lds_pyr, ntiles, kCoarseCols, cl), A, c, g);
  else coarse_addends(T, cf, ntiles, d, L - 6, first_level(P, ntiles, d, c), A, c, g);
}
template <bool IN_LDS>
__global__ __launch_bounds__(1024) void deep_bwd_kernel(const float *TgQ, const float *TgK, const float *TxQ, const float *TxK,
                                                       const float *coef, int ntiles, int d, int L, float *pyr, float *AQ,
                                                       float *AK, float *partQ, float *partK, int row) {
  extern __shared__ float lds_pyr[];
  const int slice = blockIdx.x, side = blockIdx.y, J = L - 6, cl = threadIdx.x & (kCoarseCols - 1);
  const int c = kCoarseCols * blockIdx.z + cl, g = threadIdx.x / kCoarseCols;
  const int64_t base = (int64_t)slice * ntiles * d;
  float *Pg = pyr + (((int64_t)slice * 2 + side) * 2) * pyramid_floats(ntiles, d);
  float *Px = Pg + pyramid_floats(ntiles, d);
  const float *tg = (side ? TgK : TgQ) + base, *tx = (side ? TxK : TxQ) + base, *cf = coef + slice * kCoefStride;
  float *A = (side ? AK : AQ) + base;
  __shared__ float detail[kMaxBands][16], sum[kMaxBands][16];
  if constexpr (IN_LDS) {
    lds_float *p = (lds_float *)lds_pyr;
    coarse_bwd<true>(tg, tx, cf, ntiles, d, J, first_level(p, ntiles, kCoarseCols, cl), first_level(p + (ntiles + 32) * kCoarseCols, ntiles, kCoarseCols, cl), A,
               c, g, detail, sum);
  } else {
    coarse_bwd<true>(tg, tx, cf, ntiles, d, J, first_level(Pg, ntiles, d, c), first_level(Px, ntiles, d, c), A, c, g, detail, sum);
  }
  float *part = (side ? partK : partQ) + ((int64_t)slice * (row + gridDim.z) + row + blockIdx.z) * (L + 1);
  if ((int)threadIdx.x < 6) part[threadIdx.x] = 0.f;
  if ((int)threadIdx.x >= 6 && (int)threadIdx.x <= L) {   // band 5 + j: the details of level 6 + j; band L: the approximation
    const int j = min((int)threadIdx.x - 5, J);
    float tot = 0.f;
    for (int i = 0; i < 16; ++i) tot += (int)threadIdx.x == L ? sum[J][i] : detail[j][i];
    part[threadIdx.x] = tot / (float)(1 << (6 + j));
  }
}

// Output stage of Algorithm 1 (LayerNorm over the d columns of a row, rstd kept in D); one wave per row.
template <typename T>
__global__ __launch_bounds__(256) void ln_out_kernel(const float *N, T *out, View v, int n, int d, float eps, float *D) {
  const int slice = blockIdx.y;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (t >= n) return;
  const float *p = N + ((int64_t)slice * n + t) * d;
  float x[2], acc = 0.f;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    x[u] = lane + 64 * u < d ? p[lane + 64 * u] : 0.f;
    acc += x[u];
  }
  const float mu = wave_sum(acc) / (float)d;
  acc = 0.f;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const float e = lane + 64 * u < d ? x[u] - mu : 0.f;
    acc += e * e;
  }
  const float rstd = 1.0f / sqrtf(wave_sum(acc) / (float)d + eps);
  T *o = out + v.slice_base(slice) + (int64_t)t * v.sn;
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (lane + 64 * u < d) st(o + lane + 64 * u, (x[u] - mu) * rstd);
  if (lane == 0) D[(int64_t)slice * n + t] = rstd;
}

// ------------------------------------------------------------------------------------
// Host side
// ------------------------------------------------------------------------------------
constexpr int kFillBlocks = 1024;   // workgroups of the contraction: four per compute unit, so that the last ones to end leave little idle

int dh_of(int d) { return d <= 16 ? 16 : d <= 32 ? 32 : d <= 64 ? 64 : 128; }
// One term for what comes in as bf16 (head dimensions up to 32, where that pays for instances of its own; the LayerNorm
// output stage has a float32 dN); otherwise three terms for every operand.
int terms_of(const wersa_desc &c) {
  return c.dtype == WERSA_BF16 && c.d <= 32 && !(c.flags & WERSA_FLAG_LAYERNORM) ? 1 : 3;
}
struct Plan {
  Dims s;
  int DH, KS, CT, PT, NSB, matrices;
  int chunks, rows_per_chunk;         // pooling
  int FW, TW, splits, tiles_per_split, shares;
  int groups;                         // 4096-element workgroups per slice
  int ntl;                            // 64-row tiles per slice
};
Plan plan_least(const wersa_desc &c, int least) {   // least: token tiles of a workgroup of the contraction at least
  Plan p{};
  const int slices = c.B * c.H;
  p.DH = dh_of(c.d);
  p.KS = p.DH / 16;
  p.CT = p.DH < 32 ? 1 : p.DH / 32;
  p.PT = terms_of(c);
  p.NSB = p.DH == 16 ? 4 : 6 * p.CT;
  p.matrices = (c.flags & WERSA_FLAG_SEPARATE_OMEGA) ? 2 : 1;
  p.s = Dims{c.n, c.d, c.m, (c.n + 63) / 64 * 2, (c.m + 31) / 32};
  p.ntl = (c.n + 63) / 64;
  if (c.L > kTileL) {
    p.rows_per_chunk = 64;   // the partial sums are the tile sums of the levels above 6
  } else {
    // about 2048 workgroups, at most 256 partials per slice (the gate kernel sums them), at least 64 rows
    int want = (2048 + slices - 1) / slices;
    want = want > 256 ? 256 : (want < 1 ? 1 : want);
    const int rows = (c.n + want - 1) / want;
    p.rows_per_chunk = rows < 64 ? 64 : rows;
  }
  p.chunks = (c.n + p.rows_per_chunk - 1) / p.rows_per_chunk;
  p.FW = 8;
  while (p.s.mt % p.FW) p.FW /= 2;
  p.TW = 8 / p.FW;
  const int sg = stage_tokens(p.DH, p.PT);
  p.TW = p.TW < sg ? p.TW : sg;
  const int base = slices * (p.s.mt / p.FW);
  int splits = (kFillBlocks + base - 1) / base;
  const int most = (p.s.nt + least - 1) / least;
  splits = splits > most ? most : splits;
  p.tiles_per_split = (p.s.nt + splits - 1) / splits;
  p.splits = (p.s.nt + p.tiles_per_split - 1) / p.tiles_per_split;
  p.shares = p.splits * p.TW;
  const int cw = p.DH < 64 ? p.DH : 64, tr = 4096 / cw;
  p.groups = (c.n + tr - 1) / tr * (p.DH / cw);
  return p;
}

struct Ws {
  float *qpart, *part, *zpart, *zpad, *Nbuf, *pyr;
  bf16_t *VC, *SB, *XQ, *XK;   // (XQ, XK: see keeps_operands)
  // backward
  bf16_t *NC, *XS, *SA, *dSA, *dSB;
  float *ddw, *rowscale, *dpart, *gq, *gk, *partQ, *partK, *dF, *dlogit, *dqbar, *tgq, *tgk, *aq, *ak;
  unsigned short *bitsQ, *bitsK;   // the ReLU's decisions (bitsK at head dimension 128)
  int64_t total;
};
int64_t tile_floats(int64_t tiles) { return tiles * (kTile / 2); }
Ws ws_of(const wersa_desc &c, const Plan &p, int bwd, bool keep, float *base) {
  Ws w{};
  Bump b(base);
  const int64_t sl = (int64_t)c.B * c.H;
  auto op = [&](int64_t tiles) { return (bf16_t *)b.take(tile_floats(tiles)); };
  const int64_t rows = sl * p.s.nt;
  const bool deep = c.L > kTileL;
  w.part = b.take(sl * p.shares * p.s.mt * 32 * 32 * p.CT);
  w.zpart = b.take(sl * p.shares * p.s.mt * 32);
  if (!bwd) {
    w.zpad = b.take(sl * p.s.mt * 32);
    w.qpart = b.take(sl * p.chunks * c.d);
    w.VC = op(rows * 2 * p.CT * p.PT);
    if (!keep) {
      w.XQ = op(rows * p.KS * 3);
      w.XK = op(rows * p.KS * 3);
    }
    w.SB = op((sl * p.s.mt + 1) * p.NSB);       // (one feature tile more: a stage reads whole groups)
    if (c.flags & WERSA_FLAG_LAYERNORM) w.Nbuf = b.take(sl * c.n * c.d);
    if (deep) w.pyr = b.take(2 * sl * pyramid_floats(p.ntl, c.d));
  } else {
    w.NC = op(rows * 2 * p.CT * p.PT);
    // dQ_F and dK_F, in the place of operands that nothing else needs
    w.gq = (float *)op(rows * p.KS * 3);
    w.gk = (float *)op(rows * p.KS * 3);
    if (p.PT == 1) w.XS = (bf16_t *)w.gq;
    else if (!keep) w.XQ = (bf16_t *)w.gq;
    if (!keep) w.XK = (bf16_t *)w.gk;
    w.SA = op((sl * p.s.mt + 1) * (3 * p.KS + 1));
    w.dSA = op((sl * p.s.mt + 1) * (3 * p.KS + 1));
    w.dSB = op((sl * p.s.mt + 1) * p.NSB);
    w.bitsQ = (unsigned short *)b.take(rows * p.s.mt * 32);
    if (p.DH == 128) w.bitsK = (unsigned short *)b.take(rows * p.s.mt * 32);
    w.ddw = b.take(rows * 32);
    if (p.PT == 1) w.rowscale = b.take(rows * 32);
    w.dpart = b.take(sl * p.groups);
    const int64_t prow = p.groups + (deep ? c.d / kCoarseCols : 0);
    w.partQ = b.take(sl * prow * (c.L + 1));
    w.partK = b.take(sl * prow * (c.L + 1));
    w.dF = b.take(sl * (c.L + 1));
    w.dlogit = b.take(sl * (c.L + 1));
    w.dqbar = b.take(sl * c.d);
    if (deep) {
      w.tgq = b.take(sl * p.ntl * c.d);
      w.tgk = b.take(sl * p.ntl * c.d);
      w.aq = b.take(sl * p.ntl * c.d);
      w.ak = b.take(sl * p.ntl * c.d);
      w.pyr = b.take(4 * sl * pyramid_floats(p.ntl, c.d));
    }
  }
  w.total = b.off;
  return w;
}

// Eight token tiles for a workgroup of the contraction at least, four or two where compute units are left without one: the chain of tiles is
// the kernel's time then, and up to 24 or 16 shares the kernel that adds them does not lose it again (SHORT in sum_shares).  No more workgroups than
// compute units: at head dimensions 64 and 128 one is all that a compute unit holds, and a second round costs what the shorter chain gave.  us of
// forward and backward with the coarser split and the finer, workgroups of each in brackets: 160 slices of 185 tokens, d 64, m 64, float32 (160, 320) 122.2,
// 134.1; 54 of 961, d 64, m 128 (216, 432) 223.9, 244.3; 120 of 382, d 96, m 128, bf16 (240, 360) 313.8, 330.9; but 13 of 490, d 64, m 128, float32
// (26, 52) 108.9, 99.1; 2 of 217, d 96, m 64, bf16 (2, 4) 128.7, 111.7; 26 of 715, d 32, m 32, float32 (78, 156) 79.7, 73.7.  Two tiles with 16 shares and with
// more: 5 of 986, d 96, m 96, bf16 (16 shares) 142.9, 139.0; 8 of 460, d 48, m 128, float32 (16) 93.1, 91.6; 3 of 893, d 48, m 64 (28) 76.8, 79.1; 10 of 2950,
// d 96, m 128 (47) 204.6, 244.7.
// Below head dimension 128 not to fewer than eight shares from more than one, which are added one after the other (16 of 182 tokens, d 48, m 32, bf16, two
// shares, four and six 69.9, 73.1, 73.1), and not with head dimension 16 or one-term operands, whose tiles are short: 8 to 4 there 9 slices of 3940, d 16, m 64
// 78.9, 91.9; 2 of 2882, d 32, m 64, bf16 70.4, 81.0; at best 5 us less (1 of 589, d 32, m 128).
// us of the contraction and the sum, at eight, four and two tiles: one slice of 1024 tokens, d 64, m 64, float32 8.3 5.1, 6.0 5.5, 4.5 8.2 (32 shares);
// 4 of 1000, d 128, m 256 34.9 8.8, 20.9 8.3, 14.1 9.0; 16 of 1000, d 64, m 256 19.3 6.6, 13.2 6.9, 11.5 7.6.
// What fits wersa_forward_static's scratch, with Q_F and K_F or without, still does.
Plan plan_of(const wersa_desc &c) {
  const Plan whole = plan_least(c, 8);
  if (whole.PT == 1 || whole.DH == 16) return whole;
  auto fits = [&](const Plan &q, bool keep) { return (size_t)ws_of(c, q, 0, keep, nullptr).total * sizeof(float) <= kStaticScratchBytes; };
  Plan p = whole;
  for (int least = 4; least >= (p.DH >= 64 ? 2 : 4); least /= 2) {
    const Plan q = plan_least(c, least);
    if ((int64_t)c.B * c.H * (q.s.mt / q.FW) * q.splits > 256 || q.shares > (least == 4 ? 24 : 16)) break;
    if (!fits(q, false) && (fits(p, false) || (fits(p, true) && !fits(q, true)))) break;
    p = q;
  }
  return p.DH < 128 && p.shares < 8 && whole.shares > 1 ? whole : p;
}

// Where Q_F and K_F, packed (6 bytes per element each), live between the forward and the backward.  In `saved` where the rest
// of the forward's workspace fits wersa_forward_static's scratch: the backward has less to do where latency counts (64 slices
// of 1000 tokens, d 64, m 64, float32: 110 us, 122 us where it packs them again), and what the static call takes does not
// shrink by them.  Beyond, `saved` would hold three times a tensor for every layer of a model (811 MB for 8 slices of 131072
// tokens, d 64, against 5), and the backward packs them again, from Q and K, in the launch that packs dN: 8 x 16384 tokens, d 64,
// m 256 367 us -> 374, 128 x 4000, d 32, m 1024 1716 -> 1763.
bool keeps_operands(const wersa_desc &c, const Plan &p) {
  return (size_t)ws_of(c, p, 0, true, nullptr).total * sizeof(float) <= kStaticScratchBytes;
}

// Rows of the strided tensors can be read in 16-byte pieces.
bool rows_aligned(const wersa_desc &c, std::initializer_list<const void *> ptrs) {
  const int64_t es = c.dtype == WERSA_BF16 ? 2 : 4;
  if (c.stride_n * es % 16 || c.stride_h * es % 16 || c.stride_b * es % 16) return false;
  for (const void *q : ptrs)
    if ((uintptr_t)q % 16) return false;
  return true;
}

// Workgroup sizes of the row kernels.  Head dimensions up to 32: 4 waves, several workgroups per compute unit, so that one
// runs while another waits for its stage (d 16, m 1024, 8 x 131072 tokens: the forward's kernel 420 -> 392 us against 8 waves).
// 64: 8 waves, the stage fills the LDS.  128: 4 waves with the whole register file.  2 waves where the rows are too few
// to give every compute unit a full workgroup (each wave walks all features whatever the size, so more and
// smaller workgroups cost only the staging).
constexpr int full_waves(int DH) { return DH <= 32 ? 4 : 8; }
// Token tiles per wave: two (DH <= 32, where the registers hold them) halve what a wave reads from LDS per product, but a wave of two
// is a coarser piece of work.  A round is 512 workgroups of four waves, two per SIMD; two tiles where they do not make more rounds of tiles,
// and from four rounds on.
// us of the forward's kernel and of the query side's gradient, one tile and two, d 32, m 512, float32, token tiles in all:
// 512: 18.8 26.6, 21.5 30.2; 1536: 27.8 32.2, 31.2 34.6; 8192: 114.5 106.2, 127.1 113.8; 16128 (m 1024): 365 346, 405 371.
// d 16, bf16: 512: 14.5 21.9, 14.1 20.1; 3072: 24.4 30.2, 23.3 27.5; 4096: 30.6 32.5, 28.7 29.5; 8192: 61.0 61.0, 57.1 54.8; 32768 (m 1024):
// 386 365, 362 330.
template <int DH, int MOST>
int row_tiles(const Plan &p, int slices) {
  if (MOST == 1) return 1;
  const int64_t one = (int64_t)slices * ((p.s.nt + 3) / 4), two = (int64_t)slices * ((p.s.nt + 7) / 8);
  return one >= 2048 || 2 * ((two + 511) / 512) <= (one + 511) / 512 ? 2 : 1;
}
template <int DH>
int row_waves(const Plan &p, int RT, int slices) {
  if (DH == 128) return 4;
  const int full = full_waves(DH);
  return (int64_t)slices * ((p.s.nt + full * RT - 1) / (full * RT)) >= 256 ? full : 2;
}
// Calls go(token tiles per wave, waves, grid) of the instance that a row kernel runs as.
template <int DH, int MOST, typename F>
void row_launch(const Plan &p, int slices, F go) {
  using std::integral_constant;
  const int rt = row_tiles<DH, MOST>(p, slices), nw = row_waves<DH>(p, rt, slices);
  const dim3 grid((p.s.nt + nw * rt - 1) / (nw * rt), slices);
  using Full = integral_constant<int, DH == 128 ? 4 : full_waves(DH)>;
  if constexpr (MOST == 2)
    if (rt == 2) return go(integral_constant<int, 2>(), Full(), grid);   // (more than 256 workgroups)
  if constexpr (DH < 128)
    if (nw == 2) return go(integral_constant<int, 1>(), integral_constant<int, 2>(), grid);
  go(integral_constant<int, 1>(), Full(), grid);
}

// Calls go(kernel): with more workgroups the registers of sixteen loads cost more than the chain (128 slices of 32 workgroups, 2 shares: 21.8 -> 25.2 us).
template <int DH, typename F>
void reduce_launch(const Plan &p, int slices, F go) {
  if (p.shares > 8 && p.shares <= 32 && slices * p.s.mt <= 256) go(&reduce_kernel<DH, true>);
  else go(&reduce_kernel<DH, false>);
}

template <typename T, int DH, int PT, int MODE>
void launch_apply(const wersa_desc &c, const Plan &p, const bf16_t *X, const bf16_t *OA, const bf16_t *SB, const float *zpad,
                  const float *scalars, T *out, View v, float *N, float *D, unsigned short *bits, hipStream_t st) {
  row_launch<DH, DH == 16 || (DH == 32 && PT == 3) ? 2 : 1>(p, c.B * c.H, [&](auto RT, auto NW, dim3 grid) {
    WERSA_STAGE(MODE == 2 ? "split_apply_dv" : "split_apply", st, apply_kernel<T, DH, PT, MODE, RT.value, NW.value><<<grid, 64 * NW.value, 0, st>>>(
        X, OA, SB, zpad, scalars, c.eps, p.s, out, v, N, D, bits));
  });
}
template <typename T, int DH, int PT, bool DV>
void launch_grad(const wersa_desc &c, const Plan &p, const bf16_t *X, const unsigned short *bits, const GradRows<T> &Y,
                 const float *ddw, const float *rowscale, const bf16_t *OA, const bf16_t *SA, const bf16_t *OB, const bf16_t *SB,
                 const float *scalars, float *dXF, T *dv, View v, hipStream_t st) {
  constexpr int MOST = DH == 16 ? (DV && PT == 3 ? 1 : 2) : DH == 32 && PT == 3 && !DV ? 2 : 1;   // (as the registers of two waves per SIMD hold)
  row_launch<DH, MOST>(p, c.B * c.H, [&](auto RT, auto NW, dim3 grid) {
    WERSA_STAGE(DV ? "split_grad_k" : "split_grad", st, grad_kernel<T, DH, PT, DV, RT.value, NW.value><<<grid, 64 * NW.value, 0, st>>>(
        X, bits, Y, ddw, rowscale, OA, SA, OB, SB, scalars, p.s, dXF, dv, v));
  });
}

template <typename T, int DH, int PT>
wersa_status forward_t(const wersa_desc &c, const T *q, const T *k, const T *v, const T *omega, const float *sigma,
                       const float *gate_w, const float *gate_b, const float *scale_w, T *out, float *saved, float *ws,
                       hipStream_t st) {
  const Plan p = plan_of(c);
  const bool keep = keeps_operands(c, p);
  const Ws w = ws_of(c, p, 0, keep, ws);
  const SavedLayout sv = saved_layout(c);
  const int slices = c.B * c.H;
  const View tv{c.stride_b, c.stride_h, c.stride_n, c.H};
  const bool deep = c.L > kTileL, ln = (c.flags & WERSA_FLAG_LAYERNORM) != 0;
  float *scalars = saved + sv.scalars, *coef = saved + sv.coef;
  bf16_t *XQ = keep ? (bf16_t *)(saved + sv.XQ) : w.XQ, *XK = keep ? (bf16_t *)(saved + sv.XK) : w.XK,
         *OA = (bf16_t *)(saved + sv.OA), *OB = (bf16_t *)(saved + sv.OB);
  const bf16_t *OAk = OA + (p.matrices == 2 ? (int64_t)p.s.mt * p.KS * PT * kTile : 0);
  float *addQ = deep ? saved + sv.addQ : nullptr, *addK = deep ? saved + sv.addK : nullptr;
  float *qpart = deep ? saved + sv.tileQ : w.qpart, *kpart = deep ? saved + sv.tileK : nullptr;
  const int vec = rows_aligned(c, {q, k, v});
  const int pieces = p.matrices * p.s.mt * 64 * (p.KS + 2 * p.CT);
  const OmegaPack<T> om{omega, sigma, c.bw_floor, scalars, OA, OB, p.matrices, p.KS, p.CT, PT, (pieces + 255) / 256 + 1,
                        gaps_of(c, sv, saved, tile_floats(p.KS * PT), tile_floats(2 * p.CT * PT), split_sizes(c))};
  WERSA_STAGE("split_pool", st, pool_kernel<T><<<dim3(om.blocks + p.chunks * slices, 1, deep ? 2 : 1), 256, 0, st>>>(
      q, k, tv, p.s, vec, p.rows_per_chunk, p.chunks, qpart, kpart, om));
  const bool pooled_gate = (c.flags & WERSA_FLAG_POOLED_GATE) != 0;
  GateFwdArgs gate{qpart, p.chunks, c.n, c.d, c.L, c.H, gate_w, gate_b, scale_w, saved + sv.qbar, saved + sv.s, saved + sv.F, coef,
                   PooledLayout{(int64_t)c.H * p.chunks * c.d, (int64_t)p.chunks * c.d, c.d}, nullptr, 0, AmaxLayout{0, 0, 0, 1}, scalars};
  // One round of packing workgroups: they form the gate themselves (one slice of 1024 tokens, d 64, m 64: 34.0 -> 31.4 us per call, 8 of 1500,
  // d 32, m 512: 54.3 -> 52.9); with more rounds each would wait for it again (2460 workgroups, d 64 268.3, 271.7).  Above head dimension 64 a workgroup waits
  // for a round of loads per four chunks and 64 columns, and the launch of its own is the shorter one from nine chunks on (4 slices of 276
  // tokens, d 128, m 224, five chunks 62.3, 60.2; 4 of 786, m 160, thirteen 70.4, 70.9; 6 of 2190, m 160, 35 chunks 92.5, 95.9).
  const bool fused = !deep && !pooled_gate && p.chunks <= (DH == 128 ? 8 : kGatePrologueChunks) && (int64_t)p.groups * slices * 3 <= 2048;
  if (!fused)
    WERSA_STAGE("gate_fwd_kernel", st, gate_fwd_kernel<<<slices, kGateFwdThreads, 0, st>>>(
        qpart, p.chunks, c.n, c.d, c.L, c.H, gate_w, gate_b, scale_w, gate.qbar, gate.s_out, gate.F_out, coef, pooled_gate ? 1 : 0, gate.ql, nullptr, 0,
        scalars, gate.al, 1));
  if (deep) {
    auto go = [&](auto kern, size_t lds) {
      WERSA_STAGE("split_deep", st, kern<<<dim3(slices, 2, c.d / kCoarseCols), 1024, lds, st>>>(qpart, kpart, coef, p.ntl, c.d, c.L, w.pyr, addQ, addK));
    };
    if (const size_t lds = pyramid_in_lds(&deep_addend_kernel<true>, p.ntl, 1)) go(&deep_addend_kernel<true>, lds);
    else go(&deep_addend_kernel<false>, 0);
  }
  auto pack = [&](auto kern) {
    WERSA_STAGE("split_prep_fwd", st, kern<<<dim3(p.groups, slices, 3), 256, 0, st>>>(q, k, v, tv, p.s, vec, c.L, coef, addQ, addK, XQ, XK, w.VC, gate));
  };
  if (fused) pack(&prep_fwd_kernel<T, DH, PT, true>);
  else pack(&prep_fwd_kernel<T, DH, PT, false>);
  WERSA_STAGE("split_contract", st, contract_kernel<DH, PT, false><<<dim3(p.splits, p.s.mt / p.FW, slices), 512, 0, st>>>(
      XK, w.VC, nullptr, OAk, p.s, p.FW, p.TW, p.tiles_per_split, w.part, w.zpart, nullptr));
  reduce_launch<DH>(p, slices, [&](auto kern) {
    WERSA_STAGE("split_reduce", st, kern<<<dim3(p.s.mt, slices), 256, 0, st>>>(
        w.part, w.zpart, p.shares, 1, scalars, p.s, saved + sv.S, saved + sv.z, w.zpad, nullptr, w.SB, nullptr));
  });
  if (ln) {
    launch_apply<T, DH, PT, 1>(c, p, XQ, OA, w.SB, w.zpad, scalars, out, tv, w.Nbuf, nullptr, nullptr, st);
    WERSA_STAGE("split_ln", st, ln_out_kernel<T><<<dim3((c.n + 3) / 4, slices), 256, 0, st>>>(w.Nbuf, out, tv, c.n, c.d, c.eps, saved + sv.D));
  } else {
    launch_apply<T, DH, PT, 0>(c, p, XQ, OA, w.SB, w.zpad, scalars, out, tv, nullptr, saved + sv.D, nullptr, st);
  }
  return hipGetLastError() == hipSuccess ? WERSA_OK : WERSA_ERR_LAUNCH;
}

template <typename T, int DH, int PT>
wersa_status backward_t(const wersa_desc &c, const T *q, const T *k, const T *v, const float *gate_w, const float *scale_w,
                        const T *out, const T *dout, const float *saved, T *dq, T *dk, T *dv, float *dgate_w, float *dgate_b,
                        float *dscale_w, float *dsigma, float *ws, hipStream_t st) {
  const Plan p = plan_of(c);
  const bool keep = keeps_operands(c, p);
  const Ws w = ws_of(c, p, 1, keep, ws);
  const SavedLayout sv = saved_layout(c);
  const int slices = c.B * c.H;
  const View tv{c.stride_b, c.stride_h, c.stride_n, c.H};
  const bool deep = c.L > kTileL, ln = (c.flags & WERSA_FLAG_LAYERNORM) != 0;
  const float *scalars = saved + sv.scalars, *coef = saved + sv.coef, *D = saved + sv.D;
  // (with one-term operands the contraction takes Phi of Q_F / D: the same decisions)
  const bf16_t *XQ = PT == 1 ? w.XS : keep ? (const bf16_t *)(saved + sv.XQ) : w.XQ,
               *XK = keep ? (const bf16_t *)(saved + sv.XK) : w.XK, *OA = (const bf16_t *)(saved + sv.OA),
               *OB = (const bf16_t *)(saved + sv.OB);
  const int64_t two = p.matrices == 2 ? p.s.mt : 0;
  const bf16_t *OAk = OA + two * p.KS * PT * kTile, *OBk = OB + two * 2 * p.CT * PT * kTile;
  const int vec = rows_aligned(c, {q, k, v, out, dout});
  WERSA_STAGE("split_prep_bwd", st, prep_bwd_kernel<T, DH, PT><<<dim3(p.groups, slices, keep ? (PT == 1 ? 2 : 1) : 3), 256, 0, st>>>(
      dout, out, q, k, tv, p.s, vec, ln, c.L, coef, deep ? saved + sv.addQ : nullptr, deep ? saved + sv.addK : nullptr, D, w.NC,
      w.XQ, w.XS, w.XK, w.ddw, w.rowscale, w.dpart));
  WERSA_STAGE("split_contract", st, contract_kernel<DH, PT, true><<<dim3(p.splits, p.s.mt / p.FW, slices), 512, 0, st>>>(
      XQ, w.NC, w.ddw, OA, p.s, p.FW, p.TW, p.tiles_per_split, w.part, w.zpart, w.bitsQ));
  reduce_launch<DH>(p, slices, [&](auto kern) {
    WERSA_STAGE("split_reduce", st, kern<<<dim3(p.s.mt, slices, 2), 256, 0, st>>>(
        w.part, w.zpart, p.shares, PT == 1 ? 3 : 1, scalars, p.s, const_cast<float *>(saved + sv.S), const_cast<float *>(saved + sv.z),
        nullptr, w.dSA, w.dSB, w.SA));
  });
  const GradRows<T> rowsK{v, nullptr, nullptr, vec}, rowsQ{dout, ln ? out : nullptr, PT == 1 ? nullptr : D, vec};
  if constexpr (DH == 128) {   // (dV on its own: no registers left for its accumulators; first, dK_F may go in the place of K_F)
    launch_apply<T, DH, PT, 2>(c, p, XK, OAk, w.dSB, nullptr, scalars, dv, tv, nullptr, nullptr, w.bitsK, st);
    launch_grad<T, DH, PT, false>(c, p, nullptr, w.bitsK, rowsK, nullptr, nullptr, nullptr, w.dSA, OBk, nullptr, scalars, w.gk, nullptr, tv, st);
  } else {
    launch_grad<T, DH, PT, true>(c, p, XK, nullptr, rowsK, nullptr, nullptr, OAk, w.dSA, OBk, w.dSB, scalars, w.gk, dv, tv, st);
  }
  launch_grad<T, DH, PT, false>(c, p, nullptr, w.bitsQ, rowsQ, w.ddw, PT == 1 ? w.rowscale : nullptr, nullptr, w.SA, OB, nullptr, scalars, w.gq,
                                nullptr, tv, st);
  const int prow = p.groups + (deep ? c.d / kCoarseCols : 0);
  WERSA_STAGE("split_dots", st, dots_kernel<T, DH><<<dim3(p.groups, slices, 2), 256, 0, st>>>(
      q, k, tv, w.gq, w.gk, p.s, c.L, prow, w.partQ, w.partK, w.tgq, w.tgk));
  if (deep) {
    auto go = [&](auto kern, size_t lds) {
      WERSA_STAGE("split_deep", st, kern<<<dim3(slices, 2, c.d / kCoarseCols), 1024, lds, st>>>(
          w.tgq, w.tgk, saved + sv.tileQ, saved + sv.tileK, coef, p.ntl, c.d, c.L, w.pyr, w.aq, w.ak, w.partQ, w.partK, p.groups));
    };
    if (const size_t lds = pyramid_in_lds(&deep_bwd_kernel<true>, p.ntl, 2)) go(&deep_bwd_kernel<true>, lds);
    else go(&deep_bwd_kernel<false>, 0);
  }
  WERSA_STAGE("gate_bwd_slice_kernel", st, gate_bwd_slice_kernel<<<slices, kGateBwdThreads, 0, st>>>(
      w.partQ, w.partK, prow, c.L, c.d, c.H, saved + sv.s, gate_w, scale_w, w.dF, w.dlogit, w.dqbar,
      (c.flags & WERSA_FLAG_POOLED_GATE) ? 1 : 0));
  const GateBwdParams gp{w.dF, w.dlogit, saved + sv.s, saved + sv.qbar, w.dpart, slices * p.groups, c.B, c.H, c.L, c.d, c.eps, scalars,
                         dgate_w, dgate_b, dscale_w, dsigma, gate_bwd_params_blocks(c.H, c.L, c.d)};
  WERSA_STAGE("split_filter_bwd", st, filter_bwd_kernel<T, DH><<<with_gate_bwd_params(dim3(p.groups, slices, 2), gp), 256, 0, st>>>(
      w.gq, w.gk, dq, dk, tv, p.s, c.L, coef, w.aq, w.ak, w.dqbar, 1.0f / (float)c.n, gp));
  return hipGetLastError() == hipSuccess ? WERSA_OK : WERSA_ERR_LAUNCH;
}

// Calls f(element type tag, head dimension, terms) of the instance that serves the descriptor.
template <typename F>
wersa_status dispatch(const wersa_desc &c, F f) {
  using std::integral_constant;
  const int DH = dh_of(c.d), PT = terms_of(c);
  auto by_dh = [&](auto tag) -> wersa_status {
    using T = decltype(tag);
    if constexpr (sizeof(T) == 2) {
      if (PT == 1) return DH == 16 ? f(tag, integral_constant<int, 16>(), integral_constant<int, 1>())
                                   : f(tag, integral_constant<int, 32>(), integral_constant<int, 1>());
    }
    switch (DH) {
      case 16: return f(tag, integral_constant<int, 16>(), integral_constant<int, 3>());
      case 32: return f(tag, integral_constant<int, 32>(), integral_constant<int, 3>());
      case 64: return f(tag, integral_constant<int, 64>(), integral_constant<int, 3>());
      default: return f(tag, integral_constant<int, 128>(), integral_constant<int, 3>());
    }
  };
  return c.dtype == WERSA_F32 ? by_dh(float()) : by_dh(bf16_t());
}

}  // namespace

SplitSizes split_sizes(const wersa_desc &c) {
  const Plan p = plan_of(c);
  const int64_t X = keeps_operands(c, p) ? tile_floats((int64_t)c.B * c.H * p.s.nt * p.KS * 3) : 0;
  // (one feature tile more than there are: a stage of the row kernels reads whole groups of them)
  return SplitSizes{X, tile_floats((int64_t)(p.matrices * p.s.mt + 1) * p.KS * p.PT),
                    tile_floats((int64_t)(p.matrices * p.s.mt + 1) * 2 * p.CT * p.PT)};
}
size_t split_workspace_bytes(const wersa_desc &c, int for_backward) {
  const Plan p = plan_of(c);
  return (size_t)ws_of(c, p, for_backward, keeps_operands(c, p), nullptr).total * sizeof(float);
}
wersa_status split_forward(const wersa_desc &c, const void *q, const void *k, const void *v, const void *omega_rf,
                           const float *sigma, const float *gate_w, const float *gate_b, const float *scale_w, void *out,
                           float *saved, float *ws, hipStream_t st) {
  return dispatch(c, [&](auto tag, auto DH, auto PT) {
    using T = decltype(tag);
    return forward_t<T, DH.value, PT.value>(c, (const T *)q, (const T *)k, (const T *)v, (const T *)omega_rf, sigma, gate_w,
                                            gate_b, scale_w, (T *)out, saved, ws, st);
  });
}
wersa_status split_backward(const wersa_desc &c, const void *q, const void *k, const void *v, const float *gate_w,
                            const float *scale_w, const void *out, const void *dout, const float *saved, void *dq, void *dk,
                            void *dv, float *dgate_w, float *dgate_b, float *dscale_w, float *dsigma, float *ws,
                            hipStream_t st) {
  return dispatch(c, [&](auto tag, auto DH, auto PT) {
    using T = decltype(tag);
    return backward_t<T, DH.value, PT.value>(c, (const T *)q, (const T *)k, (const T *)v, gate_w, scale_w, (const T *)out,
                                             (const T *)dout, saved, (T *)dq, (T *)dk, (T *)dv, dgate_w, dgate_b, dscale_w,
                                             dsigma, ws, st);
  });
}

}  // namespace wersa
