// MFMA path for bf16 tensors on gfx950 (Section 3.1 steps 3-8 and their derivatives).
//
// Staging (all intermediates that reach HBM are n x d sized; the n x m feature matrices live
// only in registers):
//   haar_stage      X (bf16) -> X_F = W^-1(F (.) W X) as fp16, LDS-staged 64-row tiles
//                   (steps 3, 5, 6 fused; the block-mean form of the gated Haar filter)
//   phiT_contract   sum_t ReLU(X_F Omega)[t,:]^T Y[t,:]  and  sum_t w_t ReLU(X_F Omega)[t,:]
//                   split over n into partials (step 7 + the reductions of step 8;
//                   reused in the backward for dS = Phi_Q^T dN, dz = Phi_Q^T dD)
//   reduce_contract fixed-order sum of the partials, scaled; also bf16 copies as MFMA operands
//   rows            per 64-row block: ReLU(X_F Omega) again, then either the step-8 apply +
//                   normaliser (forward; the same apply form gives dV = Phi_K dS), or
//                   dPhi -> mask -> dX_F -> gated Haar filter of the gradient + per-band
//                   inner products (backward, Q side and K side; the mask comes as bits from the kernel
//                   that formed the projection before: phiT_contract and the dV rows)
// The projection uses fp16 MFMA operands (X_F in fp16 keeps the sign of X_F Omega right to
// 2^-12, which the ReLU derivative needs); everything downstream of the ReLU uses bf16 MFMA.
#include "wersa_internal.h"

#include <type_traits>

namespace wersa {
namespace {

#include "wersa_small_kernels.inc"
#include "wersa_filter.inc"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

// MFMA 32x32x16 lane layout (wave64; l32 = lane % 32, h = lane / 32):
//   A operand: row l32, k = 8h + q (q = 0..7)      B operand: column l32, k = 8h + q
//   C/D: acc[i] is row 8*(i/4) + 4h + (i%4), column l32.
__device__ __forceinline__ int acc_row(int i, int h) { return 8 * (i >> 2) + 4 * h + (i & 3); }

__device__ __forceinline__ f32x16 mfma_f16(f16x8 a, f16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mfma_bf16(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.f;
  return z;
}
// x[lane] + x[lane ^ 32] in every lane: one swap of the upper half of a register with the lower
// half of its copy (a VALU instruction of gfx950) and an add, instead of an exchange through LDS.
__device__ __forceinline__ float xor32_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Sum over the 32 columns of a tile, which a row holds as s[i] = column 16 (i / 8) + 8 h + i % 8 in lanes of half-wave h (rows on
// lanes): pairs, quads, then the four quads of a sixteen two by two, then the two sixteens; 7 roundings in a row where a chain over the lane's
// registers has 32 and 64.  even: quads added as (Q0 + Q3) + (Q1 + Q2), odd: as (Q0 + Q1) + (Q2 + Q3).  The columns of even and of odd quads
// take their own: that is what a butterfly over lanes gives with columns on the lanes, and the results are its bits.
struct TileSum {
  float even, odd;
  __device__ __forceinline__ float of(int i) const { return i & 4 ? odd : even; }   // for the column of register i
};
__device__ __forceinline__ TileSum tile_sum(const float (&s)[16]) {
  float e[2], o[2];
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const float u = (s[8 * g] + s[8 * g + 1]) + (s[8 * g + 2] + s[8 * g + 3]);
    const float v = (s[8 * g + 4] + s[8 * g + 5]) + (s[8 * g + 6] + s[8 * g + 7]);
    const auto q02 = __builtin_amdgcn_permlane32_swap(__float_as_uint(u), __float_as_uint(u), false, false);
    const auto q13 = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    const float q0 = __uint_as_float(q02[0]), q1 = __uint_as_float(q13[0]), q2 = __uint_as_float(q02[1]), q3 = __uint_as_float(q13[1]);
    e[g] = (q0 + q3) + (q1 + q2);
    o[g] = (q0 + q1) + (q2 + q3);
  }
  return TileSum{e[0] + e[1], o[0] + o[1]};
}
__device__ __forceinline__ float wave_sum64(float v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
// Pack accumulator registers 8a .. 8a+7 into one bf16 MFMA operand. With this choice k-slot
// (h, q) of the consuming MFMA stands for accumulator row 16a + 8*(q/4) + 4h + (q%4); the other
// operand must be fetched in the same order (two runs of four consecutive indices).
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ bf16x8 pack_half(const f32x16 &v, int a) {
  bf16x8 p;
#pragma unroll
  for (int j = 0; j < 4; ++j) {   // one packed conversion per pair
    f32x2 f;
    f[0] = v[8 * a + 2 * j];
    f[1] = v[8 * a + 2 * j + 1];
    const bf16x2_t c = __builtin_convertvector(f, bf16x2_t);
    p[2 * j] = c[0];
    p[2 * j + 1] = c[1];
  }
  return p;
}
// The matching operand: indices base + 4h + {0..3} and base + 8 + 4h + {0..3} of a row in LDS.
__device__ __forceinline__ bf16x8 lds_perm8(const bf16_t *row, int base, int h) {
  const bf16x4 lo = *reinterpret_cast<const bf16x4 *>(row + base + 4 * h);
  const bf16x4 hi = *reinterpret_cast<const bf16x4 *>(row + base + 8 + 4 * h);
  bf16x8 r;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    r[q] = lo[q];
    r[4 + q] = hi[q];
  }
  return r;
}

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}

// ------------------------------------------------------------------------------------
// Per-call constants: block 0 writes the scalars; every block transposes its share of Omega
// into Omega^T in fp16 ([m][d]), the projection's MFMA operand.  (The filter coefficients of
// the block-mean form come from the gate kernel.)
// ------------------------------------------------------------------------------------
struct SetupArgs {
  const float *sigma;
  float bw_floor;
  const bf16_t *omega;
  int d, m, matrices;
  float *scalars;
  _Float16 *omT;
  int blocks;   // workgroups of 256 threads that cover matrices * d * m elements (0: nothing to do)
};
inline int setup_blocks(int d, int m, int matrices) { return (matrices * d * m + 255) / 256; }
__device__ __forceinline__ void setup_body(const SetupArgs &a, int block) {
  if (block == 0 && threadIdx.x == 0) {
    const float s = *a.sigma;
    const float se = fmaxf(s, a.bw_floor);
    a.scalars[0] = 1.0f / (se * sqrtf((float)a.m));
    a.scalars[1] = se;
    a.scalars[2] = s > a.bw_floor ? 1.0f : 0.0f;
    a.scalars[3] = 1.0f;
  }
  const int e = block * 256 + threadIdx.x;
  if (e < a.matrices * a.d * a.m) {   // one or two d x m matrices, each transposed on its own
    const int mat = e / (a.d * a.m), w = e % (a.d * a.m);
    const int r = w / a.d, j = w % a.d;
    a.omT[e] = (_Float16)bf16_to_f32(a.omega[(int64_t)mat * a.d * a.m + (int64_t)j * a.m + r]);
  }
}
__global__ __launch_bounds__(256) void setup_kernel(SetupArgs a) { setup_body(a, blockIdx.x); }

// ------------------------------------------------------------------------------------
// Column sums of Q for the pooled query: 16-byte loads, one partial per (slice, chunk).
// Grid (chunks + su.blocks, slices): the workgroups past `chunks` of slice 0 carry the per-call
// constants (one launch fewer at the head of the forward pass); those of the other slices exit.
// ------------------------------------------------------------------------------------
template <int DH>
__global__ __launch_bounds__(256) void qbar_partial_kernel(const bf16_t *q, View v, int n,
                                                          int rows_per_chunk, float *part, int chunks,
                                                          SetupArgs su, float *amax_part) {
  constexpr int CPR = DH / 8;        // 16-byte chunks per row
  constexpr int RPI = 256 / CPR;     // rows per iteration
  if ((int)blockIdx.x >= chunks) {
    if (blockIdx.y == 0) setup_body(su, blockIdx.x - chunks);
    return;
  }
  const int slice = blockIdx.y, chunk = blockIdx.x;
  const int t0 = chunk * rows_per_chunk, t1 = min(n, t0 + rows_per_chunk);
  const int cc = threadIdx.x % CPR, rr = threadIdx.x / CPR;
  const bf16_t *qs = q + v.slice_base(slice) + cc * 8;
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
  // largest magnitude seen: integer maximum of the values with their sign bits cleared (packed 16-bit)
  u16x8 mx = {0, 0, 0, 0, 0, 0, 0, 0};
  const u16x8 magn = {0x7fff, 0x7fff, 0x7fff, 0x7fff, 0x7fff, 0x7fff, 0x7fff, 0x7fff};
  auto track = [&](const u16x8 &x) { mx = __builtin_elementwise_max(mx, x & magn); };
  int t = t0 + rr;
  for (; t + 7 * RPI < t1; t += 8 * RPI) {   // eight independent loads in flight
    u16x8 x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = *reinterpret_cast<const u16x8 *>(qs + (int64_t)(t + u * RPI) * v.sn);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      track(x[u]);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += bf16_to_f32(x[u][e]);
    }
  }
  for (; t < t1; t += RPI) {
    const u16x8 x = *reinterpret_cast<const u16x8 *>(qs + (int64_t)t * v.sn);
    track(x);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += bf16_to_f32(x[e]);
  }
  __shared__ float red[RPI][DH + 1];
  __shared__ float amax_w[4];
#pragma unroll
  for (int e = 0; e < 8; ++e) red[rr][cc * 8 + e] = acc[e];
  if (amax_part) {   // (NaN and infinity compare as the largest magnitudes and are passed on as such)
    unsigned short m16 = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) m16 = mx[e] > m16 ? mx[e] : m16;
    float m = bf16_to_f32(m16);
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if ((threadIdx.x & 63) == 0) amax_w[threadIdx.x >> 6] = m;
  }
  __syncthreads();
  if (threadIdx.x < DH) {
    float s = 0.f;
    for (int r = 0; r < RPI; ++r) s += red[r][threadIdx.x];
    part[((int64_t)slice * chunks + chunk) * DH + threadIdx.x] = s;
  }
  if (amax_part && threadIdx.x == 0)
    amax_part[(int64_t)slice * chunks + chunk] = fmaxf(fmaxf(amax_w[0], amax_w[1]), fmaxf(amax_w[2], amax_w[3]));
}

// Q and K (bf16, strided; blockIdx.z) -> Q_F, K_F (fp16, contiguous [slices][n][DH]); one 64-row tile per workgroup.
// Steps: coalesced 16-byte loads into LDS; one thread per (column, row segment) computes the
// nested block sums (in registers up to the segment, through LDS above it) and the filtered
// values; fp16 results go back to LDS and leave with coalesced 16-byte stores.
// tile_add (L > 6, else nullptr): [slices][ceil(n / 64)][DH], the per-tile addend of the levels above 6.
template <int DH>
__global__ __launch_bounds__(256) void haar_stage_kernel(const bf16_t *q, const bf16_t *k, View v, int n, const float *coef,
                                                        const float *addQ, const float *addK, _Float16 *qf, _Float16 *kf) {
  const bf16_t *x = blockIdx.z ? k : q;
  const float *tile_add = blockIdx.z ? addK : addQ;
  _Float16 *xf = blockIdx.z ? kf : qf;
  constexpr int SEGS = 256 / DH;   // row segments per column: 4 (DH=64) or 2 (DH=128)
  constexpr int RS = 64 / SEGS;    // rows per segment: 16 or 32
  constexpr int CPR = DH / 8;
  __shared__ __attribute__((aligned(16))) bf16_t tile[64 * DH];
  __shared__ float segsum[SEGS][DH];
  __shared__ float cf[8];
  const int slice = blockIdx.y, t0 = blockIdx.x * 64;
  const int tid = threadIdx.x;
  if (tid < 8) cf[tid] = coef[slice * kCoefStride + tid];
  const bf16_t *xs = x + v.slice_base(slice);
  for (int e = tid; e < 64 * CPR; e += 256) {
    const int r = e / CPR, cc = e % CPR;
    u16x8 val;
    if (t0 + r < n) val = *reinterpret_cast<const u16x8 *>(xs + (int64_t)(t0 + r) * v.sn + cc * 8);
    else
#pragma unroll
      for (int q = 0; q < 8; ++q) val[q] = 0;
    *reinterpret_cast<u16x8 *>(&tile[r * DH + cc * 8]) = val;
  }
  __syncthreads();
  const int c = tid % DH, seg = tid / DH;
  float vals[RS];
#pragma unroll
  for (int i = 0; i < RS; ++i) vals[i] = bf16_to_f32(tile[(seg * RS + i) * DH + c]);
  segsum[seg][c] = segment_sum<RS>(vals);
  __syncthreads();
  float upper;
  if (SEGS == 4) {
    const float s5 = segsum[seg & ~1][c] + segsum[seg | 1][c];
    const float s6 = (segsum[0][c] + segsum[1][c]) + (segsum[2][c] + segsum[3][c]);
    upper = fmaf(cf[5], s5, cf[6] * s6);
  } else {
    upper = cf[6] * (segsum[0][c] + segsum[1][c]);
  }
  if (tile_add) upper += tile_add[((int64_t)slice * gridDim.x + blockIdx.x) * DH + c];
  filter_segment<RS>(vals, cf, upper);
  _Float16 *tile16 = reinterpret_cast<_Float16 *>(tile);
#pragma unroll
  for (int i = 0; i < RS; ++i) tile16[(seg * RS + i) * DH + c] = (_Float16)vals[i];
  __syncthreads();
  _Float16 *out = xf + ((int64_t)slice * n + t0) * DH;
  for (int e = tid; e < 64 * CPR; e += 256) {
    const int r = e / CPR, cc = e % CPR;
    if (t0 + r < n)
      *reinterpret_cast<u16x8 *>(out + (int64_t)r * DH + cc * 8) =
          *reinterpret_cast<const u16x8 *>(&tile[r * DH + cc * 8]);
  }
}

// float32 -> bf16 storage with the hardware conversion (round to nearest even)
__device__ __forceinline__ bf16_t cvt_bf16(float f) {
  return __builtin_bit_cast(bf16_t, (__bf16)f);
}

// The gated Haar filter as a stage of its own on bf16 tensors (steps 3, 5, 6 of Section 3.1; the
// stage entry point): X -> X_F in the same layout and dtype, up to six levels, one tile of 64 rows x
// 64 columns per workgroup.  Rows move in 16-byte pieces both ways; the filter is evaluated in
// block-mean form, one thread per (column, 16-row segment), the 32- and 64-row sums through LDS;
// no float copy of the tile exists anywhere.  filt: [slices][L + 1] (band order of Algorithm 2).
__global__ __launch_bounds__(256) void haar_filter_bf16_kernel(const bf16_t *x, bf16_t *y, View v, int n, int d,
                                                              const float *filt, int L) {
  constexpr int TC = 64, RS = 16, CPR = TC / 8;
  __shared__ __attribute__((aligned(16))) bf16_t tile[64 * TC];
  __shared__ float segsum[4][TC];
  __shared__ float cf[8];
  const int slice = blockIdx.z, t0 = blockIdx.x * 64, c0 = blockIdx.y * TC;
  const int tid = threadIdx.x;
  if (tid < 8) {   // block-mean coefficients: coef_0 = F_0, coef_l = (F_l - F_{l-1}) / 2^l, 0 above L
    const float *F = filt + (int64_t)slice * (L + 1);
    cf[tid] = tid == 0 ? F[0] : (tid <= L ? (F[tid] - F[tid - 1]) / (float)(1 << tid) : 0.f);
  }
  const int64_t base = v.slice_base(slice);
  u16x8 piece[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int e = tid + 256 * u, r = e / CPR, cc = e % CPR;
    const bool ok = t0 + r < n && c0 + cc * 8 < d;
    // (rows past n and columns past d read as zeros: Algorithm 2's padding)
    piece[u] = *reinterpret_cast<const u16x8 *>(x + base + (int64_t)(ok ? t0 + r : 0) * v.sn + (ok ? c0 + cc * 8 : 0));
    if (!ok)
#pragma unroll
      for (int q = 0; q < 8; ++q) piece[u][q] = 0;
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int e = tid + 256 * u;
    *reinterpret_cast<u16x8 *>(&tile[(e / CPR) * TC + (e % CPR) * 8]) = piece[u];
  }
  __syncthreads();
  const int c = tid % TC, seg = tid / TC;
  float vals[RS];
#pragma unroll
  for (int i = 0; i < RS; ++i) vals[i] = bf16_to_f32(tile[(seg * RS + i) * TC + c]);
  segsum[seg][c] = segment_sum<RS>(vals);
  __syncthreads();
  const float s5 = segsum[seg & ~1][c] + segsum[seg | 1][c];
  const float s6 = (segsum[0][c] + segsum[1][c]) + (segsum[2][c] + segsum[3][c]);
  filter_segment<RS>(vals, cf, fmaf(cf[5], s5, cf[6] * s6));
#pragma unroll
  for (int i = 0; i < RS; ++i) tile[(seg * RS + i) * TC + c] = cvt_bf16(vals[i]);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int e = tid + 256 * u, r = e / CPR, cc = e % CPR;
    if (t0 + r < n && c0 + cc * 8 < d)
      *reinterpret_cast<u16x8 *>(y + base + (int64_t)(t0 + r) * v.sn + c0 + cc * 8) =
          *reinterpret_cast<const u16x8 *>(&tile[r * TC + cc * 8]);
  }
}

// ------------------------------------------------------------------------------------
// Small helpers for the chained MFMAs.
// ------------------------------------------------------------------------------------
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// ReLU on a packed bf16 operand: as 16-bit integers, negative floats are negative integers.
__device__ __forceinline__ bf16x8 relu_bf16x8(bf16x8 p) {
  s16x8 s = __builtin_bit_cast(s16x8, p);
  const s16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
  s = __builtin_elementwise_max(s, zero);
  return __builtin_bit_cast(bf16x8, s);
}
// A weighted sum over the k-slots of a packed operand (D = Phi z) beside the products: the 4 x 4 x 4 matrix instruction,
// sixteen blocks of four lanes, with the weights of the lane's half-wave in every column.  Accumulator i of a lane is the sum of lane
// 4 (lane / 4) + i; own() picks its own.  Two of them per eight values take 8 cycles each of the matrix pipe; pair dot products do not run
// beside matrix instructions either and take 7.5 each, four per eight values.  Forward rows kernel, 8 slices of 131072 rows, m 256: 94.9 -> 90.0 us,
// 64 of 4096, m 128: 20.8 -> 19.8; in phiT_contract, which waits at its barriers, and at head dimension 128 nothing or less.  D against
// float64 sums of the same operands: 2.2e-7 rms at 4096 features, 2.55e-7 with pair dot products.
struct WeightedSum {
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  __device__ __forceinline__ void add(bf16x8 p, bf16x8 w) {
    const s16x8 a = __builtin_bit_cast(s16x8, p), b = __builtin_bit_cast(s16x8, w);
    acc = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_shufflevector(a, a, 0, 1, 2, 3), __builtin_shufflevector(b, b, 0, 1, 2, 3), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_shufflevector(a, a, 4, 5, 6, 7), __builtin_shufflevector(b, b, 4, 5, 6, 7), acc, 0, 0, 0);
  }
  __device__ __forceinline__ float own(int lane) const {
    const float lo = lane & 1 ? acc[1] : acc[0], hi = lane & 1 ? acc[3] : acc[2];
    return lane & 2 ? hi : lo;
  }
};
// acc + sum_q p[q] * w[q] with bf16 pair dot products (float32 accumulate)
__device__ __forceinline__ float dot8_bf16(bf16x8 p, bf16x8 w, float acc) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    bf16x2 a, b;
    a[0] = p[2 * j]; a[1] = p[2 * j + 1];
    b[0] = w[2 * j]; b[1] = w[2 * j + 1];
    acc = __builtin_amdgcn_fdot2_f32_bf16(a, b, acc, false);
  }
  return acc;
}
__device__ __forceinline__ bf16x8 splat_bf16x8(float v) {
  bf16x8 r;
#pragma unroll
  for (int q = 0; q < 8; ++q) r[q] = (__bf16)v;
  return r;
}

// Transposing LDS read of gfx950 (ds_read_b64_tr_b16): within each group of 16 lanes, lane i
// passes the address of four consecutive 16-bit values, taken as row i / 4, columns
// 4 (i % 4) .. + 3 of a 4 x 16 block, and receives column i of that block.  (Lane mapping
// checked on the GPU with an index-valued LDS array.)
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x4 lds_read_tr4(const bf16_t *p) {
  typedef s16x4 __attribute__((address_space(3))) * lds_s16x4_ptr;
  return __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)p));
}

// The same packing as pack_half into an fp16 operand.
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f16x8 pack_half_f16(const f32x16 &v, int a) {
  f16x8 p;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    f32x2 f;
    f[0] = v[8 * a + 2 * j];
    f[1] = v[8 * a + 2 * j + 1];
    const f16x2_t c = __builtin_convertvector(f, f16x2_t);
    p[2 * j] = c[0];
    p[2 * j + 1] = c[1];
  }
  return p;
}

// In-kernel stage A (head dimension 64): the gated Haar filter of one aligned 64-row block is
// the product with a 64 x 64 matrix G (from the block-mean coefficients of the slice), so the kernels
// that consume X_F take the raw rows of Q or K and form X_F^T = X^T G^T on the matrix cores.
// G[t'][t] depends only on the highest bit in which t' and t differ: g_k = sum of coef_l over
// l >= k, k = 0 for t' == t, else (position of that bit) + 1.  For the matrix cores G is split
// into a bf16 high part and a bf16 low part (the gradients are sensitive to a relative error of
// 2^-9 in the filter), and its B operands (column t', k-slot t = 8 j + q) come out of a small
// table T[part][t' % 8][(t' / 8) ^ j][q] = part of g at t' ^ t, one 16-byte read each.
__device__ __forceinline__ void build_filter_table(bf16_t *T, const float *coef8, int tid, int nthreads) {
  float g[7], acc = 0.f;
#pragma unroll
  for (int l = 6; l >= 0; --l) {
    acc += coef8[l];
    g[l] = acc;
  }
  for (int e = tid; e < 512; e += nthreads) {
    const int b = e >> 6, xh = (e >> 3) & 7, q = e & 7;
    const int x = 8 * xh + (b ^ q);
    const int lvl = x ? 32 - __clz(x) : 0;
    float v = g[0];
#pragma unroll
    for (int k = 1; k < 7; ++k) v = (lvl == k) ? g[k] : v;
    const __bf16 hi = (__bf16)v;
    const __bf16 lo = (__bf16)(v - (float)hi);
    T[e] = __builtin_bit_cast(bf16_t, hi);
    T[512 + e] = __builtin_bit_cast(bf16_t, lo);
  }
}
__device__ __forceinline__ bf16x8 filter_operand(const bf16_t *T, int part, int trow, int j) {
  return *reinterpret_cast<const bf16x8 *>(&T[part * 512 + (((trow & 7) << 3) | ((trow >> 3) ^ j)) * 8]);
}
// This is the A operand of that product from a row-major bf16 tile [t][stride]: operand row
// lane % 32 is tile column col0 + lane % 32 (PERM: with bits 2 and 3 of lane % 32 swapped),
// k-slot (h, q) is tile row 16 ks + 8 h + q.  With PERM, pack_half of the result delivers the
// columns in natural order (k-slot (h, q) of half a is column 16 a + 8 h + q).
template <bool PERM>
__device__ __forceinline__ bf16x8 tile_cols_operand(const bf16_t *tile, int stride, int col0, int ks, int lane) {
  const int i16 = lane & 15, g16 = lane >> 4;
  int k = i16 & 3;
  if (PERM) k = ((k & 1) << 1) | (k >> 1);
  const bf16_t *p = tile + (16 * ks + 8 * (g16 >> 1) + (i16 >> 2)) * stride + col0 + 16 * (g16 & 1) + 4 * k;
  const bf16x4 lo = lds_read_tr4(p), hi = lds_read_tr4(p + 4 * stride);
  bf16x8 r;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    r[q] = lo[q];
    r[4 + q] = hi[q];
  }
  return r;
}

// A value that the compiler re-derives from in every block: offsets that depend on the lane alone would otherwise be
// kept in registers across the feature loop and spill (the gradient kernels).
__device__ __forceinline__ uint32_t opaque(uint32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}

// ------------------------------------------------------------------------------------
// The ReLU's decisions 1[R > 0] of the backward as bits: the kernel that forms the projection of a side for dS (queries) or dV
// (keys) leaves them for the gradient kernel of that side, which then needs neither X_F nor the projection.
// One 32-bit word per (64-row block, half ti of its rows, 64 features 64 w ..) and position p:
//   bits[slice][block][ti][w / 2][p][w % 2]; n m / 8 bytes per slice.
// With r, f the row and the feature inside 32 (r_k, f_k: their bits) and u the feature tile inside 64, p and the bit are
//   from a kernel that has rows on lanes:     p = r0 + 2 r1 + 4 f3 + 8 r3 + 16 r4 + 32 r2, bit 16 f0 + 8 u + 4 f4 + 2 f2 + f1;
//   from one that has features on lanes:      p = f0 + 2 f1 + 4 f3 + 8 f2 + 16 f4 + 32 r2, bit 16 r0 + 8 u + 4 r4 + 2 r3 + r1
// (transpose_bits takes the second form to the first).  In memory bytes 1 and 2 of a word are exchanged, so that the bits of a
// feature tile are one half of it.
// ------------------------------------------------------------------------------------
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
// Features (operand rows) with bits 2 and 3 exchanged: accumulator register i of half-wave h then is feature
// 16 (i / 8) + 8 h + i % 8 of its tile, and the packed registers 8 a .. 8 a + 7 contract with one 16-byte piece.
__device__ __forceinline__ int swap23(int r) { return (r & ~12) | (r & 4) << 1 | (r & 8) >> 1; }
// One bit per element of a packed accumulator tile after the ReLU: register pair (2 j, 2 j + 1) gives bits j and 16 + j.  A
// positive bf16 is at least 2^7 as an integer (R is a sum of fp16 products, multiples of 2^-48, and never a denormal).
__device__ __forceinline__ uint32_t positive_bits(const bf16x8 *pa) {
  uint32_t w = 0;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      bf16x2 e;
      e[0] = pa[a][2 * jj];
      e[1] = pa[a][2 * jj + 1];
      const unsigned short one = (unsigned short)(1u << (4 * a + jj));
      u16x2 bit = {one, one};
      if (one == 1) asm("" : "+s"(bit));   // (of min(x, 1) the compiler makes two comparisons and two selections)
      w |= __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, e), bit));
    }
  return w;
}
__device__ __forceinline__ uint32_t swap_bytes12(uint32_t w) { return __builtin_amdgcn_perm(w, w, 0x03010200); }
// Rows on word bits and features on lanes -> features on word bits and rows on lanes, for a lane that sits at position p (bits 0 to 5:
// l0, l1, l5, l4, l2, l3 of its number): lane bits 0, 1, 4, 2 change places with the word's bits 16, 1, 2, 4 (place values), one
// exchange between two lanes each.
__device__ __forceinline__ uint32_t transpose_bits(uint32_t w, int lane) {
  auto merge = [](uint32_t own, int other, bool upper, uint32_t mask, int shift) {
    const uint32_t m = upper ? ~mask : mask, t = (uint32_t)other;
    return (own & m) | (__builtin_amdgcn_alignbit(t, t, upper ? shift : 32 - shift) & ~m);
  };
  const uint32_t t = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xB1, 0xF, 0xF, false);   // lane ^ 1
  w = __builtin_amdgcn_perm(w, t, lane & 1 ? 0x07060302u : 0x01000504u);
  w = merge(w, __builtin_amdgcn_update_dpp(0, (int)w, 0x4E, 0xF, 0xF, false), lane & 2, 0x55555555u, 1);   // lane ^ 2
  w = merge(w, __builtin_amdgcn_ds_swizzle((int)w, 0x401F), lane & 16, 0x33333333u, 2);                    // lane ^ 16
  return merge(w, __builtin_amdgcn_ds_swizzle((int)w, 0x101F), lane & 4, 0x0F0F0F0Fu, 4);                  // lane ^ 4
}
// Row of 32 that operand lane l32 takes where the accumulator registers of the result shall hold 16 consecutive rows 16 h + i.
__device__ __forceinline__ int lane_row(int ln) { return (ln & 3) | (ln >> 3 & 3) << 2 | (ln & 4) << 2; }
// The position (see above) at which such a lane's words are.
__device__ __forceinline__ int lane_position(int ln) {
  return (ln & 3) | (ln >> 5) << 2 | (ln & 16) >> 1 | (ln & 4) << 2 | (ln & 8) << 2;
}
// Half a of an accumulator tile packed to bf16, elements whose bit is not set as zero; w in register form, u: which feature tile of the word.
__device__ __forceinline__ bf16x8 pack_masked(const f32x16 &v, int a, uint32_t w, int u) {
  const bf16x8 p = pack_half(v, a);
  bf16x8 r;
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) {
    bf16x2 e;
    e[0] = p[2 * jj];
    e[1] = p[2 * jj + 1];
    const s16x2 m = (__builtin_bit_cast(s16x2, w) << (short)(15 - 8 * u - 4 * a - jj)) >> (short)15;
    e = __builtin_bit_cast(bf16x2, (uint32_t)(__builtin_bit_cast(uint32_t, e) & __builtin_bit_cast(uint32_t, m)));
    r[2 * jj] = e[0];
    r[2 * jj + 1] = e[1];
  }
  return r;
}

// ------------------------------------------------------------------------------------
// phiT_contract: for the rows of one chunk and the features [f0, f0 + NW*FW) of one slice
//   Spart[r][c] = sum_t ReLU(X_F Omega)[t][r] * (Y[t][c] / rowdiv_t)
//   zpart[r]    = sum_t w_t * ReLU(X_F Omega)[t][r]
// NW waves split the features; each wave keeps its Omega operands in registers and chains
// the projection's accumulators (rows t on registers) straight into the second MFMA as the
// A operand.  X_F and Y tiles of 64 rows go through double-buffered LDS (Y transposed so that
// t runs along the operand's k index); the next tile is fetched while the current one is used.
// ------------------------------------------------------------------------------------
// PREP (backward, Q side): Y = dO, rowdiv = D, and the weights are computed here instead of
// read: w_t = dD_t = -<dO_t, O_t> / D_t from the rows of O (`orows`, laid out like Y).  The
// feature block 0 also writes dD [slices][n] for the gradient rows kernel and one partial sum
// of dD per (slice, chunk) for d sigma.
// Head dimension 64 (FUSE): `xf` is not read; the rows of X (Q or K, bf16, view vx) are staged
// raw and each step starts with X_F = G X for its tile, one 32 x 32 quarter per wave, written
// to LDS in fp16 for the projection.
// NW = 8 (head dimension 128): four waves are two workgroups per compute unit that each bring every row into LDS, divide
// it by D and take its product with O, for 128 features; eight do that once for 256, and keep the matrix cores fed by
// halves (see next_tile).  32 slices of 65536 rows, m 512, training step of the attention block: 16708 -> 16441 us; per launch
// (forward, backward form) there 628, 908 -> 521, 667; 12 slices of 16384 rows, m 512: 69.2, 95.6 -> 59.0, 72.8 us; 256 of 1024, m 256: 55.6, 73.5 -> 45.3, 56.7;
// 8 of 4096, m 512: 17.2, 20.6 -> 17.1, 18.6.  The sums are the same bits.
// BITS (the backward): the ReLU's decisions go to `bits` for the gradient kernel (see positive_bits), 12.5 vector instructions per 32 x 32 tile
// (8 slices of 131072 rows, d 64, m 256: 118 -> 121 us; 32 of 65536, d 128, m 512: 682 -> 715).
// RAGGED: n % 64 != 0, rows past n count as zeros with weight 0.  DEEP: L > 6, the filter's levels
// above 6 enter as the per-tile addend tile_add [slices][ceil(n / 64)][DH] (the accumulators of X_F start there).
template <int DH, int FW, bool PREP, bool RAGGED, bool DEEP, bool BITS, int NW = 4>
__global__ __launch_bounds__(64 * NW, 2) void phiT_contract_kernel(
    const _Float16 *xf, const bf16_t *xraw, View vx, const float *coef, const float *tile_add,
    const bf16_t *y, View vy, const float *rowdiv, const float *w,
    const bf16_t *orows, float *dDout, float *dDpart,
    const _Float16 *omT, int n, int m, int rows_per_chunk, float *Spart, float *zpart, uint32_t *bits, GateFwdArgs gate) {
  constexpr bool FUSE = (DH == 64);
  constexpr bool GATE = FUSE && !BITS && !DEEP;   // (the forward) `gate` may be given: the first launch that filters
  static_assert(NW == 4 || (NW == 8 && !FUSE), "the filter of head dimension 64 is dealt to four waves");
  constexpr int NT = 64 * NW;
  constexpr int KS = DH / 16;   // k-steps of the projection
  constexpr int RT = FW / 32;   // feature tiles per wave
  constexpr int CT = DH / 32;   // column tiles of Y
  constexpr int CPR = DH / 8;   // 16-byte pieces per row
  constexpr int LPT = 64 * CPR / NT;   // pieces per thread per tile
  constexpr int YS = DH + 32;   // row stride (elements) of the Y tile [t][column]: 64 bytes past a multiple
                                // of 256, so the four rows of a transposing read fall into different bank quarters
  constexpr int XS = DH + 8;    // row stride (elements) of the X_F tile
  __shared__ __attribute__((aligned(16))) bf16_t yt[2][64 * YS];
  __shared__ __attribute__((aligned(16))) _Float16 xt[2][64 * XS];   // FUSE: raw bf16 rows of X
  __shared__ __attribute__((aligned(16))) _Float16 xq[FUSE ? 64 * XS : 8];   // FUSE: X_F of the current tile
  __shared__ __attribute__((aligned(16))) bf16_t gt[FUSE ? 1024 : 8];        // FUSE: filter operand table
  __shared__ __attribute__((aligned(16))) bf16_t wl[2][64];
  const int slice = blockIdx.z, chunk = blockIdx.x, chunks = gridDim.x;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int f0 = blockIdx.y * (NW * FW) + wave * FW;
  const int t_begin = chunk * rows_per_chunk, t_end = min(n, t_begin + rows_per_chunk);
  const int steps = (t_end - t_begin + 63) / 64;   // the last tile of the sequence may be partial

  // Omega^T operands of this wave's features: B operand, column = feature (in the order of swap23), k = 8h + q.
  const int fl = swap23(l32);
  f16x8 om[RT][KS];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      om[rt][ks] = *reinterpret_cast<const f16x8 *>(omT + (int64_t)(f0 + 32 * rt + fl) * DH + 16 * ks + 8 * h);

  f32x16 S[RT][CT];
  float zacc[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    zacc[rt] = 0.f;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) S[rt][ct] = zero16();
  }
  const _Float16 *xs = FUSE ? nullptr : xf + (int64_t)slice * n * DH;
  const bf16_t *xrs = FUSE ? xraw + vx.slice_base(slice) : nullptr;
  const bf16_t *ys = y + vy.slice_base(slice);
  const float *rd = rowdiv ? rowdiv + (int64_t)slice * n : nullptr;
  const float *ws = w ? w + (int64_t)slice * n : nullptr;

  // X_F and Y pieces are taken row-major (coalesced) and stored as they are; the Y operand
  // (t along k) comes out of its tile through transposing LDS reads.
  u16x8 yr[LPT], xr[LPT];
  float inv[LPT], wv = 1.0f;
  // PREP: the rows of O come in like those of Y (the thread that holds piece cc of row r of dO
  // holds the same piece of O); the CPR partial dot products of a row sit in neighbouring lanes.
  u16x8 orw[PREP ? LPT : 1];
  float dsum = 0.f;
  const bf16_t *os = PREP ? orows + vy.slice_base(slice) : nullptr;
  // RAGGED: rows past n (partial last tile) count as zeros with weight 0: the address is clamped
  // to the last row and the value replaced.
  // Whole tiles (the plain instances): one running pointer per tensor, advanced by a tile per
  // call (the tiles are requested in order); piece i sits i * (NT / CPR) rows further on.
  constexpr int RPP = NT / CPR;   // rows between a thread's pieces
  const int r0 = tid / CPR, c0 = (tid % CPR) * 8;
  const int64_t xsn = FUSE ? vx.sn : DH;
  const u16x8 *px = reinterpret_cast<const u16x8 *>((FUSE ? xrs : reinterpret_cast<const bf16_t *>(xs)) +
                                                    (int64_t)(t_begin + r0) * xsn + c0);
  const u16x8 *py = reinterpret_cast<const u16x8 *>(ys + (int64_t)(t_begin + r0) * vy.sn + c0);
  const u16x8 *po = PREP ? reinterpret_cast<const u16x8 *>(os + (int64_t)(t_begin + r0) * vy.sn + c0) : nullptr;
  const float *prd = rd ? rd + t_begin + r0 : nullptr;
  const float *pws = ws ? ws + t_begin + tid : nullptr;
  auto fetch = [&](int t0) {
    if (!RAGGED) {
#pragma unroll
      for (int i = 0; i < LPT; ++i) {
        xr[i] = *reinterpret_cast<const u16x8 *>(reinterpret_cast<const bf16_t *>(px) + i * RPP * xsn);
        yr[i] = *reinterpret_cast<const u16x8 *>(reinterpret_cast<const bf16_t *>(py) + i * RPP * vy.sn);
        if (PREP) orw[i] = *reinterpret_cast<const u16x8 *>(reinterpret_cast<const bf16_t *>(po) + i * RPP * vy.sn);
        inv[i] = prd ? prd[i * RPP] : 1.0f;   // divided at the stash, when the load has landed
      }
      if (!PREP && tid < 64) wv = pws ? *pws : 1.0f;
      px = reinterpret_cast<const u16x8 *>(reinterpret_cast<const bf16_t *>(px) + 64 * xsn);
      py = reinterpret_cast<const u16x8 *>(reinterpret_cast<const bf16_t *>(py) + 64 * vy.sn);
      if (PREP) po = reinterpret_cast<const u16x8 *>(reinterpret_cast<const bf16_t *>(po) + 64 * vy.sn);
      if (prd) prd += 64;
      if (pws) pws += 64;
      return;
    }
    const int last = RAGGED ? n - t0 - 1 : 63;
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      const int e = tid + NT * i, r = e / CPR, cc = e % CPR;
      const bool bad = RAGGED && r > last;
      const int rc = t0 + (RAGGED ? min(r, last) : r);
      xr[i] = FUSE ? *reinterpret_cast<const u16x8 *>(xrs + (int64_t)rc * vx.sn + cc * 8)
                   : *reinterpret_cast<const u16x8 *>(xs + (int64_t)rc * DH + cc * 8);
      yr[i] = *reinterpret_cast<const u16x8 *>(ys + (int64_t)rc * vy.sn + cc * 8);
      if (PREP) orw[i] = *reinterpret_cast<const u16x8 *>(os + (int64_t)rc * vy.sn + cc * 8);
      inv[i] = rd ? rd[rc] : 1.0f;   // divided at the stash, when the load has landed
      if (bad) {
#pragma unroll
        for (int q = 0; q < 8; ++q) { xr[i][q] = 0; yr[i][q] = 0; }
        inv[i] = 1.0f;
      }
    }
    if (!PREP && tid < 64) wv = (RAGGED && tid > last) ? 0.f : (ws ? ws[t0 + tid] : 1.0f);
  };
  int t_stash = t_begin;   // first row of the tile the registers hold
  auto stash = [&](int buf) {
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      const int e = tid + NT * i, r = e / CPR, cc = e % CPR;
      *reinterpret_cast<u16x8 *>(&xt[buf][r * XS + cc * 8]) = xr[i];
      if (rd) {
        const float rinv = 1.0f / inv[i];
        u16x8 sc;
#pragma unroll
        for (int q = 0; q < 8; ++q) sc[q] = cvt_bf16(bf16_to_f32(yr[i][q]) * rinv);
        *reinterpret_cast<u16x8 *>(&yt[buf][r * YS + cc * 8]) = sc;
      } else {
        *reinterpret_cast<u16x8 *>(&yt[buf][r * YS + cc * 8]) = yr[i];
      }
    }
    if (PREP) {
      static_assert(!PREP || CPR == 8 || CPR == 16, "row pieces sit in 8 or 16 neighbouring lanes");
#pragma unroll
      for (int i = 0; i < LPT; ++i) {
        const int e = tid + NT * i, r = e / CPR, cc = e % CPR;
        // (rows past n hold zeros in yr and 1 in inv: their dD is 0)
        float dot = dot8_bf16(__builtin_bit_cast(bf16x8, orw[i]), __builtin_bit_cast(bf16x8, yr[i]), 0.f);
        dot += dpp_move<0xB1>(dot);    // lane ^ 1
        dot += dpp_move<0x4E>(dot);    // lane ^ 2
        dot += dpp_move<0x141>(dot);   // mirror inside each group of 8 lanes: the other quad's sum
        if (CPR == 16) dot += dpp_move<0x140>(dot);   // mirror inside the row of 16 lanes: the other half's sum
        const float dDt = -dot / inv[i];
        if (cc == 0) {
          wl[buf][r] = cvt_bf16(dDt);
          dsum += dDt;
          if (blockIdx.y == 0 && (!RAGGED || t_stash + r < n)) dDout[(int64_t)slice * n + t_stash + r] = dDt;
        }
      }
    } else if (tid < 64) {
      wl[buf][tid] = cvt_bf16(wv);
    }
  };

  // The filter's table is visible after the barrier below.  (Loads return in order: the coefficients, where they are there, before the rows.)
  const bool form_gate = GATE && gate.qpart;
  if (FUSE && !form_gate) build_filter_table(gt, coef + slice * kCoefStride, tid, 256);
  if (steps > 0) fetch(t_begin);
  if (form_gate) {
    typedef GateLds<4, 64> Lds;
    static_assert(sizeof(Lds) <= sizeof(xq) || !GATE, "the gate's scratch lies where X_F goes later");
    Lds &lds = *reinterpret_cast<Lds *>(&xq[0]);
    gate_prologue<4, 64>(gate, slice, chunk == 0 && blockIdx.y == 0, lds);
    build_filter_table(gt, lds.coef, tid, 256);
  }
  if (steps > 0) stash(0);
  __syncthreads();
  // FUSE: rows 32 (wave / 2) + l32 of G are this wave's B operands in every step: high part for the four k-steps, low part for
  // the two of the quarter's own half.  Forward: kept in registers, own half first (ks_own, ks_own + 1: high and low part),
  // then the other half (high part only), so that the step loop has no branch and its LDS reads go out together.
  // BITS: read again in every step (kept they would be spilled), and the sum is that of rows_kernel, k-steps upwards and the low part
  // after the high one: X_F then has the bits it has in the forward, and dQ the forward's decisions.  (Own half first, a pre-activation
  // within a rounding of zero went the other way here and there: dQ was further from float64, 4.74494e-3 against 4.74480e-3 at 8 slices of
  // 131072 rows, m 256, 3.04324e-3 against 3.04244e-3 at 12 of 6000, m 1024, L 7.  The time is the same, with L > 6 less: 297 -> 292 us
  // per training step at 8 slices of 30000 rows, L 10.)
  bf16x8 ghi[4], glo[2];
  const int ks_own = 2 * (wave >> 1), ks_oth = ks_own ^ 2;
  auto read_filter = [&](int ln) {
    const int trow = 32 * (wave >> 1) + (ln & 31), hh = ln >> 5;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      ghi[u] = filter_operand(gt, 0, trow, 2 * (ks_own + u) + hh);
      ghi[2 + u] = filter_operand(gt, 0, trow, 2 * (ks_oth + u) + hh);
      glo[u] = filter_operand(gt, 1, trow, 2 * (ks_own + u) + hh);
    }
  };
  if (FUSE && !BITS) read_filter(lane);
  // Eight waves: the registers hold the tile after the current one when a step begins.  The waves of one half put it into
  // LDS (and request the one after it) before their matrix instructions, those of the other half, their partners on the
  // same SIMDs, after them.
  auto next_tile = [&](int s) {
    if (s + 1 >= steps) return;
    stash((s & 1) ^ 1);
    if (s + 2 < steps) {
      t_stash = t_begin + 64 * (s + 2);
      fetch(t_stash);
    }
  };
  if (NW == 8 && steps > 1) {
    t_stash = t_begin + 64;
    fetch(t_stash);
  }
  // BITS: the words of this wave's features, block by block
  // (a buffer of the slice's words, n m / 8 bytes: the running offset stays scalar)
  const int fb = __builtin_amdgcn_readfirstlane(f0);
  __amdgpu_buffer_rsrc_t bb;
  if (BITS)
    bb = __builtin_amdgcn_make_buffer_rsrc(bits + (int64_t)slice * ((n + 63) / 64) * 2 * m, 0, (int)((uint32_t)((n + 63) / 64) * 8 * (uint32_t)m), 0x00020000);
  uint32_t bo = (uint32_t)(t_begin / 64) * 8 * m + fb / 128 * 512 + (fb / 64 & 1) * 4 + (RT == 1 ? (fb / 32 & 1) * 2 : 0);
  for (int s = 0; s < steps; ++s) {
    const int buf = s & 1;
    const bool more = s + 1 < steps;
    if (NW == 8) {
      if (wave < 4) next_tile(s);
    } else if (more) {
      t_stash = t_begin + 64 * (s + 1);
      fetch(t_stash);
    }
    if (FUSE) {
      // X_F^T quarter: columns 32 (wave % 2) .. + 31 of the tile, rows 32 (wave / 2) .. + 31.
      const bf16_t *raw = reinterpret_cast<const bf16_t *>(&xt[buf][0]);
      f32x16 q = zero16();
      if (DEEP) {   // register i is column 32 (wave % 2) + acc_row(i, h) for every row of the quarter
        const float *ta = tile_add + ((int64_t)slice * ((n + 63) / 64) + (t_begin / 64 + s)) * DH + 32 * (wave & 1);
#pragma unroll
        for (int i = 0; i < 16; ++i) q[i] = ta[acc_row(i, h)];
      }
      if (BITS) {
        const int ln = (int)opaque(lane), trow = 32 * (wave >> 1) + (ln & 31), hh = ln >> 5, lower = wave >> 1;   // 1: rows 32 ..
        // (k-step, part) of the six products, without a branch: (0, hi), (0, lo | 1, hi), (k23, hi), (k23, lo), (2 | 3, hi), (3, hi | lo)
        const int k1 = lower, k23 = 1 + lower, k4 = 2 + lower;
        auto rows = [&](int ks) { return tile_cols_operand<false>(raw, XS, 32 * (wave & 1), ks, ln); };
        auto gop = [&](int part, int ks) { return filter_operand(gt, part, trow, 2 * ks + hh); };
        const bf16x8 x0 = rows(0), x1 = rows(k1), x23 = rows(k23), x4 = rows(k4), x5 = rows(3);
        const bf16x8 g0 = gop(0, 0), g1 = gop(1 - lower, k1), g2 = gop(0, k23), g3 = gop(1, k23), g4 = gop(0, k4), g5 = gop(lower, 3);
        q = mfma_bf16(x0, g0, q);
        q = mfma_bf16(x1, g1, q);
        q = mfma_bf16(x23, g2, q);
        q = mfma_bf16(x23, g3, q);
        q = mfma_bf16(x4, g4, q);
        q = mfma_bf16(x5, g5, q);
      } else {
        f32x16 q2 = zero16();
        bf16x8 xa[4];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          xa[u] = tile_cols_operand<false>(raw, XS, 32 * (wave & 1), ks_own + u, lane);
          xa[2 + u] = tile_cols_operand<false>(raw, XS, 32 * (wave & 1), ks_oth + u, lane);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {   // the low part matters inside the quarter's own 32-row half only
          q = mfma_bf16(xa[u], ghi[u], q);
          q2 = mfma_bf16(xa[u], glo[u], q2);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) q = mfma_bf16(xa[2 + u], ghi[2 + u], q);
#pragma unroll
        for (int i = 0; i < 16; ++i) q[i] += q2[i];
      }
      // accumulator register i is column 32 (wave % 2) + acc_row(i, h), lane l32 is row 32 (wave / 2) + l32
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
        f16x4 pk;
#pragma unroll
        for (int e = 0; e < 4; ++e) pk[e] = (_Float16)q[4 * g + e];
        *reinterpret_cast<f16x4 *>(&xq[(32 * (wave >> 1) + l32) * XS + 32 * (wave & 1) + 8 * g + 4 * h]) = pk;
      }
      __syncthreads();
    }
    const _Float16 *xcur = FUSE ? &xq[0] : &xt[buf][0];
    uint32_t word = 0;   // BITS
    __builtin_amdgcn_s_setprio(3);   // the matrix phase goes ahead of the other workgroup's tile traffic (-1 %)
#pragma unroll
    for (int ti = 0; ti < 2; ++ti) {
      f16x8 xa[KS];   // projection A operand: rows 32 ti + l32, k = 8h + q (+16 per k-step)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        xa[ks] = *reinterpret_cast<const f16x8 *>(&xcur[(32 * ti + l32) * XS + 16 * ks + 8 * h]);
      bf16x8 yb[2][CT], wp[2];
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        wp[a] = lds_perm8(&wl[buf][0], 32 * ti + 16 * a, h);
        // k-slot (h, q) of the chained MFMA stands for row 16 a + 8 (q / 4) + 4 h + (q % 4): two
        // transposing reads of four consecutive rows each, at column 32 ct + l32.
        const int i16 = lane & 15, c16 = 16 * ((lane >> 4) & 1) + 4 * (i16 & 3);
        const int trow = 32 * ti + 16 * a + 4 * h + (i16 >> 2);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          const bf16x4 lo = lds_read_tr4(&yt[buf][trow * YS + 32 * ct + c16]);
          const bf16x4 hi = lds_read_tr4(&yt[buf][(trow + 8) * YS + 32 * ct + c16]);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            yb[a][ct][q] = lo[q];
            yb[a][ct][4 + q] = hi[q];
          }
        }
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        f32x16 R = zero16();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) R = mfma_f16(xa[ks], om[rt][ks], R);
        bf16x8 pa[2];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          pa[a] = relu_bf16x8(pack_half(R, a));
          zacc[rt] = dot8_bf16(pa[a], wp[a], zacc[rt]);
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) S[rt][ct] = mfma_bf16(pa[a], yb[a][ct], S[rt][ct]);
        }
        if (BITS) {   // two feature tiles, or two row tiles of one, share a word
          const uint32_t b = positive_bits(pa);
          word = (RT == 2 ? rt : ti) == 0 ? b : word | b << 8;
        }
      }
      if (BITS && RT == 2) __builtin_amdgcn_raw_buffer_store_b32(swap_bytes12(word), bb, 8 * opaque(lane), bo + ti * 4 * m, 0);
    }
    if (BITS) {
      if (RT == 1) {
        word = swap_bytes12(word);
        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)word, bb, 8 * opaque(lane), bo, 0);
        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(word >> 16), bb, 8 * opaque(lane), bo + 4 * m, 0);
      }
      bo += 8 * m;
    }
    __builtin_amdgcn_s_setprio(0);
    if (NW == 8) {
      if (wave >= 4) next_tile(s);
    } else if (more) {
      stash(buf ^ 1);
    }
    __syncthreads();
  }
  float *sp = Spart + ((int64_t)slice * chunks + chunk) * (int64_t)m * DH;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        sp[(int64_t)(f0 + 32 * rt + swap23(acc_row(i, h))) * DH + 32 * ct + l32] = S[rt][ct][i];
    const float zt = xor32_sum(zacc[rt]);
    if (h == 0) zpart[((int64_t)slice * chunks + chunk) * m + f0 + 32 * rt + fl] = zt;
  }
  if (PREP && blockIdx.y == 0) {   // sum of dD over this chunk's rows, fixed order
    __shared__ float red[NW];
    const float wsum = wave_sum64(dsum);
    if (lane == 0) red[wave] = wsum;
    __syncthreads();
    if (tid == 0) {
      float sum = (red[0] + red[1]) + (red[2] + red[3]);
      if constexpr (NW == 8) sum += (red[4] + red[5]) + (red[6] + red[7]);
      dDpart[(int64_t)slice * chunks + chunk] = sum;
    }
  }
}

// M[slice][e] = scale[slice] * sum_chunk part[slice][chunk][e]  (e over m*DH; scale_ptr points at the
// slice rows' c * 2^-k entries, kCoefStride apart) and the vector part
// b likewise; plus the bf16 MFMA operand copies:
//   Mx  [m][DH+16]: row r = (M[r][0..DH), b[r], 0 x 15)   (A operand of dPhi = Y M^T + a b^T)
//   MT  [DH][m]   : M transposed                           (B operand of Phi M)
//   bb  [m]       : b in bf16
// One workgroup = 64 VEC consecutive outputs x 4 waves; wave g sums the chunks g, g+4, ... with up
// to 16 loads in flight, the four partial sums meet in LDS in a fixed order.  Workgroups
// [0, m*DH/(64 VEC)) handle M, the ones after those b.
// Where there are few outputs (reduce_short_kernel takes the others).  Two widths: VEC = 4 columns per lane (16-byte loads, S^T leaves as one
// piece per column through LDS instead of 2-byte stores m apart) where that still gives every compute unit a workgroup; 1 where it does not
// (one slice of 131072 rows: 64 workgroups would read 32 MB).  Both add in the same order: the results are the same bits.
template <int DH, int VEC>
__global__ __launch_bounds__(256) void reduce_contract_kernel(const float *Spart, const float *zpart,
                                                             int chunks, int m, const float *scale_ptr,
                                                             float *S, float *z, bf16_t *Mx, bf16_t *MT,
                                                             bf16_t *bb) {
  constexpr int DX = DH + 16, COLS = 64 * VEC;   // elements of a workgroup
  typedef float fv __attribute__((ext_vector_type(VEC)));
  const int slice = blockIdx.y, tid = threadIdx.x, lane = tid & 63, grp = tid >> 6;
  const int64_t W = (int64_t)m * DH;
  const int wblocks = (int)(W / COLS);
  const bool is_z = (int)blockIdx.x >= wblocks;
  const int64_t count = is_z ? m : W;
  const int64_t e0 = (int64_t)(is_z ? blockIdx.x - wblocks : blockIdx.x) * COLS, el = e0 + lane * VEC;
  __shared__ __align__(16) float part[4][COLS];
  fv acc = (fv)(0.f);
  if (el < count) {   // (m may end inside the last workgroup of z)
    const float *p = (is_z ? zpart : Spart) + (int64_t)slice * chunks * count + el;
    int c = grp;
    for (; c + 60 < chunks; c += 64) {
      fv v16[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v16[u] = *reinterpret_cast<const fv *>(p + (int64_t)(c + 4 * u) * count);
#pragma unroll
      for (int u = 0; u < 16; ++u) acc += v16[u];
    }
    for (; c + 12 < chunks; c += 16) {
      fv v4[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v4[u] = *reinterpret_cast<const fv *>(p + (int64_t)(c + 4 * u) * count);
#pragma unroll
      for (int u = 0; u < 4; ++u) acc += v4[u];
    }
    for (; c < chunks; c += 4) acc += *reinterpret_cast<const fv *>(p + (int64_t)c * count);
  }
  *reinterpret_cast<fv *>(&part[grp][lane * VEC]) = acc;
  __syncthreads();
  const int64_t e = e0 + tid;
  const bool mine = tid < COLS && e < count;
  bf16_t b = 0;
  if (mine) {
    const float sum = ((part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid])) * scale_ptr[slice * kCoefStride];
    b = f32_to_bf16(sum);
    if (!is_z) {
      S[(int64_t)slice * W + e] = sum;
      const int r = (int)(e / DH), cidx = (int)(e % DH);
      Mx[((int64_t)slice * m + r) * DX + cidx] = b;
      if (VEC == 1) MT[(int64_t)slice * W + (int64_t)cidx * m + r] = b;
    } else {
      z[(int64_t)slice * m + e] = sum;
      bb[(int64_t)slice * m + e] = b;
      bf16_t *ext = Mx + ((int64_t)slice * m + e) * DX + DH;
      ext[0] = b;
#pragma unroll
      for (int q = 1; q < 16; ++q) ext[q] = 0;
    }
  }
  if constexpr (VEC == 4) {
    if (is_z) return;
    constexpr int RW = COLS / DH;   // features of this workgroup: 4 or 2, so pieces of 8 or 4 bytes
    typedef bf16_t bv __attribute__((ext_vector_type(RW)));
    __shared__ bf16_t tile[COLS];
    tile[tid] = b;
    __syncthreads();
    if (tid < DH) {
      bv o;
#pragma unroll
      for (int q = 0; q < RW; ++q) o[q] = tile[q * DH + tid];
      *reinterpret_cast<bv *>(MT + (int64_t)slice * W + (int64_t)tid * m + e0 / DH) = o;
    }
  }
}

// The same sums, by threads that add all chunks of their four columns themselves: the four interleaved sums of above in four accumulators, the
// same bits.  1024 elements per workgroup (RW features), 16-byte stores of S.
// What bounds it: the latency of one round of loads, and the loads and stores in flight; four waves that share the chunks have two each where
// a problem has many slices, a barrier, and four times the workgroups.  us, four waves and one thread: 64 workgroups of this kernel 8.0, 9.7 (4 slices,
// d 64, m 256: 128 partials) and 5.4, 6.4; 128 8.1, 7.9 (8 slices) and 5.8, 5.6; 64 slices, d 64, m 128 7.9, 5.6; 16, d 128, m 512 13.3, 9.6;
// 64, m 512, d 64 16.3, 11.2, d 128 28.5, 16.8.
template <int DH>
__global__ __launch_bounds__(256) void reduce_short_kernel(const float *Spart, const float *zpart, int chunks, int m, const float *scale_ptr,
                                                          float *S, float *z, bf16_t *Mx, bf16_t *MT, bf16_t *bb) {
  constexpr int DX = DH + 16, COLS = 1024, RW = COLS / DH;
  const int slice = blockIdx.y, tid = threadIdx.x;
  const int64_t W = (int64_t)m * DH;
  const int wblocks = (int)(W / COLS);
  const bool is_z = (int)blockIdx.x >= wblocks;
  const int64_t count = is_z ? m : W, e = (int64_t)(is_z ? blockIdx.x - wblocks : blockIdx.x) * COLS + tid * 4;
  f32x4 acc[4] = {};
  const bool mine = e < count;   // (m may end inside the workgroup of z)
  if (mine) {
    const float *p = (is_z ? zpart : Spart) + (int64_t)slice * chunks * count + e;
    int c = 0;
    for (; c + 8 <= chunks; c += 8) {
      f32x4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const f32x4 *>(p + (int64_t)(c + u) * count);
#pragma unroll
      for (int u = 0; u < 8; ++u) acc[u & 3] += v[u];
    }
    f32x4 v[7];
#pragma unroll
    for (int u = 0; u < 7; ++u) v[u] = c + u < chunks ? *reinterpret_cast<const f32x4 *>(p + (int64_t)(c + u) * count) : (f32x4)(0.f);
#pragma unroll
    for (int u = 0; u < 7; ++u) acc[u & 3] += v[u];
  }
  const f32x4 sum = ((acc[0] + acc[1]) + (acc[2] + acc[3])) * scale_ptr[slice * kCoefStride];
  typedef bf16_t b16x4 __attribute__((ext_vector_type(4)));
  b16x4 b;
#pragma unroll
  for (int q = 0; q < 4; ++q) b[q] = f32_to_bf16(sum[q]);
  if (is_z) {
    if (!mine) return;
    *reinterpret_cast<f32x4 *>(z + (int64_t)slice * m + e) = sum;
    *reinterpret_cast<b16x4 *>(bb + (int64_t)slice * m + e) = b;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      u16x8 lo = {}, hi = {};
      lo[0] = b[q];
      u16x8 *ext = reinterpret_cast<u16x8 *>(Mx + ((int64_t)slice * m + e + q) * DX + DH);
      ext[0] = lo;
      ext[1] = hi;
    }
    return;
  }
  *reinterpret_cast<f32x4 *>(S + (int64_t)slice * W + e) = sum;
  const int r = (int)(e / DH), cidx = (int)(e % DH);
  *reinterpret_cast<b16x4 *>(Mx + ((int64_t)slice * m + r) * DX + cidx) = b;
  // M transposed: column c of the RW features as pieces of eight; LDS rows of RW + 4 values
  __shared__ __align__(16) bf16_t tile[DH * (RW + 4)];
#pragma unroll
  for (int q = 0; q < 4; ++q) tile[(cidx + q) * (RW + 4) + tid * 4 / DH] = b[q];
  __syncthreads();
  constexpr int PIECES = RW / 8;
  if (tid < DH * PIECES) {
    const int c = tid / PIECES, k = tid % PIECES * 8;
    u16x8 o;
#pragma unroll
    for (int q = 0; q < 8; ++q) o[q] = tile[c * (RW + 4) + k + q];
    *reinterpret_cast<u16x8 *>(MT + (int64_t)slice * W + (int64_t)c * m + (int64_t)blockIdx.x * RW + k) = o;
  }
}

// ------------------------------------------------------------------------------------
// rows kernels.  A wave owns 64 consecutive rows at a time (one Haar block of the largest
// size; 32 at head dimension 128); the workgroup's waves share the feature-side operands in LDS and walk over the
// row groups of their slice (the operands are staged once when all features fit).  The
// projection is computed transposed (features on the accumulator's register index, rows on
// lanes) so that the ReLU output chains into MFMAs that contract over the features.
//   MODE 0 (forward, Q side):   N = relu(R) S,  D = c * relu(R) z + eps,  O = c N / D
//   MODE 1 (backward, Q side):  G = dN S^T + dD z^T; dR = 1[R>0] G; dX_F = c dR Omega^T
//   MODE 2 (backward, K side):  G = V dS^T + 1 dz^T; dR, dX_F as above
//   MODE 3 (backward, K side):  dV = c relu(R) dS  (apply form, like MODE 0 without the normaliser)
// The rank-one term a b^T of G rides along as one extra k-step of the dPhi MFMA (operand
// rows extended by (b_r, 0, ...) and (a_t, 0, ...)).
// Backward epilogue: dX = gated Haar filter of dX_F (block-mean form on the accumulator
// layout, rows on registers), per-band inner products with X for dF, bf16 stores.
// ------------------------------------------------------------------------------------

// The rows of one 64-row block as a buffer of `valid` rows of `sn` elements (values v of 2 or 4 bytes): loads past
// the last row return zeros and stores past it do nothing, by the bounds check of the buffer instructions, so a
// partial last block runs the code of a whole one.  All arguments are the same for the whole wave; 64 rows must
// stay below 2^32 bytes (see kMaxBufferStride).
typedef __amdgpu_buffer_rsrc_t RowBuf;
constexpr int64_t kMaxBufferStride = 1 << 24;   // row stride (elements) up to which a partial last block is a buffer
constexpr int64_t kMaxGroupStride = 1 << 26;    // and up to which a lane of the gradient kernels reaches 32 rows with a 32-bit offset in bytes
template <typename T>
__device__ __forceinline__ RowBuf row_buffer(const T *rows, int64_t sn, int valid) {
  const uint64_t a = reinterpret_cast<uint64_t>(rows);   // (the compiler does not see that a wave's index is uniform)
  const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
  const int v = __builtin_amdgcn_readfirstlane(valid < 0 ? 0 : (valid < 64 ? valid : 64));
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(hi << 32 | lo), 0,
                                           (int)(uint32_t)((uint64_t)v * (uint64_t)sn * sizeof(T)), 0x00020000);
}
template <typename V> __device__ __forceinline__ V buf_load16(RowBuf r, uint32_t off) {
  return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
__device__ __forceinline__ float buf_load4(RowBuf r, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
typedef unsigned int u32x2v __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4v __attribute__((ext_vector_type(4)));
template <typename V> __device__ __forceinline__ void buf_store16(RowBuf r, uint32_t off, V v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4v, v), r, off, 0, 0);
}
__device__ __forceinline__ void buf_store4(RowBuf r, uint32_t off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, off, 0, 0);
}

// The apply modes of head dimension 64.  8 slices of 131072 rows, m 256 (forward, dV): 86 and 84 us; with the accumulators' rows on
// registers (128 two-byte LDS writes per block, 8-byte stores, D through LDS) 90 and 90.  LN (MODE 0): LayerNorm over the columns of a row instead of the normaliser.  RAGGED: n is
// not a multiple of 64; rows are read and written through buffers that end at row n (see row_buffer).  The plain instance has
// none of that code.  DEEP: L > 6: X_F starts from the per-tile addend of the levels above 6 (tile_add
// [slices][ceil(n / 64)][DH]).
constexpr int kWavesApply = 8;   // two per SIMD: one's epilogue runs under the other's matrix instructions (four with few rows, see fast_plan)
template <int MODE, int MC, bool LN, bool RAGGED, bool DEEP, int NW = kWavesApply>
__global__ __launch_bounds__(NW * 64, 2) void rows_kernel(
    const bf16_t *x, View vx,  // X (Q or K)
    const _Float16 *omT,       // Omega^T fp16 [m][DH]
    const bf16_t *MT,          // S^T (MODE 0) / dS^T (MODE 3), bf16 [slices][DH][m]
    const bf16_t *bb,          // z bf16 [slices][m] (MODE 0)
    const float *coef,         // block-mean filter coefficients [slices][kCoefStride]
    float eps, int n, int m, int row_groups,
    bf16_t *out, View vo,      // O (MODE 0) / dV (MODE 3)
    float *Dout,               // D (MODE 0)
    const float *tile_add,     // DEEP (see above)
    uint32_t *bits)            // MODE 3: the ReLU's decisions (see positive_bits)
{
  static_assert(MODE == 0 || MODE == 3, "the gradient modes have masked_rows_kernel");
  constexpr int DH = 64;
  constexpr int KS = DH / 16, CT = DH / 32;
  constexpr int AS = DH + 8;            // stride of the [feature][DH] fp16 array (16-byte reads)
  constexpr int NT = NW * 64;
  // Stage A runs here.  Each wave keeps the raw rows of its 64-row block in
  // LDS (one 64 x 32 panel per column tile), forms X_F^T = X^T G^T with 16 MFMAs at the top of
  // the block and packs the result into the projection's fp16 operands; the output tiles go through a panel once its X
  // values are used up.
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  constexpr int mc = MC;
  constexpr int BS = MC + 8;            // stride of [DH][feature] arrays (16-byte reads)
  _Float16 *s_omT = reinterpret_cast<_Float16 *>(smem_raw);                 // [mc][AS]
  unsigned char *p = smem_raw + (size_t)mc * AS * 2;
  bf16_t *s_bb = nullptr, *s_MT = reinterpret_cast<bf16_t *>(p);                       // [DH][BS]
  p += (size_t)DH * BS * 2;
  if (MODE == 0) { s_bb = reinterpret_cast<bf16_t *>(p); p += (size_t)mc * 2; }        // [mc]
  constexpr int TS = 36;                // row stride (elements) of the per-wave 64 x 32 epilogue tile
  bf16_t *s_tile = reinterpret_cast<bf16_t *>(p);            // [waves][CT][64][TS]
  p += (size_t)NW * CT * 64 * TS * 2;
  bf16_t *s_T = reinterpret_cast<bf16_t *>(p);               // filter operand table [2][512]

  const int slice = blockIdx.y;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const float cscale = coef[slice * kCoefStride + kCoefCscale];   // c * 2^-k of this slice (X_F carries 2^k)
  const int nchunks = m / mc;

  // Feature-side operands of features [m0, m0 + MC) into LDS: every piece count is a compile-time
  // constant, loads go out in batches of eight before the first LDS write.
  auto stage = [&](int m0) {
    constexpr int CPRX = DH / 8;          // 16-byte pieces per Omega^T row
    constexpr int CPC = MC / 4;           // 8-byte pieces per column row (padded stride is 8-byte aligned)
    constexpr int B = 8;
    for (int e0 = 0; e0 < MC * CPRX; e0 += NT * B) {
      u16x8 tmp[B];
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int e = e0 + NT * u + tid;
        if (e < MC * CPRX)
          tmp[u] = *reinterpret_cast<const u16x8 *>(omT + (int64_t)(m0 + e / CPRX) * DH + (e % CPRX) * 8);
      }
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int e = e0 + NT * u + tid;
        if (e < MC * CPRX) *reinterpret_cast<u16x8 *>(&s_omT[(e / CPRX) * AS + (e % CPRX) * 8]) = tmp[u];
      }
    }
    for (int e0 = 0; e0 < DH * CPC; e0 += NT * B) {
      bf16x4 t1[B];
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int e = e0 + NT * u + tid;
        if (e < DH * CPC) {
          const int cidx = e / CPC, cc = e % CPC;
          t1[u] = *reinterpret_cast<const bf16x4 *>(MT + ((int64_t)slice * DH + cidx) * m + m0 + cc * 4);
        }
      }
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int e = e0 + NT * u + tid;
        if (e < DH * CPC) {
          const int cidx = e / CPC, cc = e % CPC;
          *reinterpret_cast<bf16x4 *>(&s_MT[cidx * BS + cc * 4]) = t1[u];
        }
      }
    }
    if (MODE == 0)
      for (int e = tid; e < MC; e += NT) s_bb[e] = bb[(int64_t)slice * m + m0 + e];
  };

  build_filter_table(s_T, coef + slice * kCoefStride, tid, NT);
  if (nchunks == 1) stage(0);
  __syncthreads();

  // ---- per-wave row-side operands; the next row group's are fetched right after the feature
  // loop of the current one (their registers are free by then), so that the latency of these
  // loads hides behind the epilogue.
  f16x8 xb[2][KS];      // X_F rows: B operand of the transposed projection
  u16x8 xp[8];          // raw X rows of the next block, 16-byte row-major pieces (row lane / 8 + 8 j, columns 8 (lane % 8) ..)
  auto load_rows = [&](int t0) {
    const int valid = RAGGED ? n - t0 : 64;   // rows of this block that exist
    if (!RAGGED) {
      // one running pointer (eight separately scaled row offsets would each be kept in registers)
      const bf16_t *xsrc = x + vx.slice_base(slice) + (int64_t)(t0 + (lane >> 3)) * vx.sn + (lane & 7) * 8;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        xp[j] = *reinterpret_cast<const u16x8 *>(xsrc);
        xsrc += 8 * vx.sn;
      }
    } else {
      const RowBuf xr = row_buffer(x + vx.slice_base(slice) + (int64_t)t0 * vx.sn, vx.sn, valid);
      const uint32_t sn2 = (uint32_t)vx.sn * 2;
      const uint32_t ln = opaque(lane);
      uint32_t off = (ln >> 3) * sn2 + (ln & 7) * 16;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        xp[j] = buf_load16<u16x8>(xr, off);
        off += 8 * sn2;
      }
    }
  };
  // The raw rows go from the registers into the wave's panels as soon as the panels are
  // free (end of the epilogue), so that they do not occupy registers during the feature loop.
  bf16_t *panels = s_tile + wave * (CT * 64 * TS);
  auto put_rows = [&]() {
    __builtin_amdgcn_wave_barrier();
    // a 16-byte piece lies inside one panel (columns 8 (lane % 8) .. + 7); two 8-byte writes
    // because odd panel rows are only 8-byte aligned
    bf16_t *dstp = panels + ((lane & 7) >> 2) * (64 * TS) + (lane >> 3) * TS + ((lane & 3) << 3);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
      u16x4 lo4, hi4;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        lo4[q] = xp[j][q];
        hi4[q] = xp[j][4 + q];
      }
      *reinterpret_cast<u16x4 *>(dstp + 8 * j * TS) = lo4;
      *reinterpret_cast<u16x4 *>(dstp + 8 * j * TS + 4) = hi4;
    }
    __builtin_amdgcn_wave_barrier();
  };
  {
    const int t_first = (blockIdx.x * NW + wave) * 64;
    if ((int)blockIdx.x < row_groups && t_first < n) {
      load_rows(t_first);
      put_rows();
    }
  }
  // (Two waves per SIMD: the wave priorities set around the feature loop below are what lets one
  // wave's epilogue run under the other's matrix work; an explicit start delay for the second wave
  // group, used before the priorities were there, no longer gains anything.)

  const int frow = swap23(l32);   // operand rows of features and of columns (see swap23)
  for (int rg = blockIdx.x; rg < row_groups; rg += gridDim.x) {
    const int t0 = (rg * NW + wave) * 64;
    const bool active = t0 < n;
    const int valid = RAGGED ? n - t0 : 64;

    if (active) {
      // X_F^T = X^T G^T per (column tile, row tile) from the raw rows in the panels (written at
      // the end of the previous block's epilogue), then the projection's fp16 operands.
      __builtin_amdgcn_wave_barrier();
      // (one column tile at a time: the 256-register budget has no room for four accumulators next to the operands
      // being built)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        f32x16 q[2];
        q[0] = zero16();
        if (DEEP) {
          // register i stands for column 32 ct + (acc_row(i, h) with bits 2 and 3 swapped), every lane's row alike
          const float *ta = tile_add + ((int64_t)slice * ((n + 63) / 64) + t0 / 64) * DH + 32 * ct;
#pragma unroll
          for (int i = 0; i < 16; ++i) q[0][i] = ta[16 * (i >> 3) + 8 * h + 4 * ((i >> 2) & 1) + (i & 3)];
        }
        q[1] = q[0];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          bf16x8 gop[2][2];
#pragma unroll
          for (int tt = 0; tt < 2; ++tt) {
            gop[tt][0] = filter_operand(s_T, 0, 32 * tt + l32, 2 * ks + h);
            gop[tt][1] = filter_operand(s_T, 1, 32 * tt + l32, 2 * ks + h);
          }
          const bf16x8 xa = tile_cols_operand<true>(panels + ct * (64 * TS), TS, 0, ks, lane);
          // The low part matters inside the row tile's own 32-row half only: across the halves
          // every entry of G is the single coarsest-level coefficient.
#pragma unroll
          for (int tt = 0; tt < 2; ++tt) {
            q[tt] = mfma_bf16(xa, gop[tt][0], q[tt]);
            if ((ks >> 1) == tt) q[tt] = mfma_bf16(xa, gop[tt][1], q[tt]);
          }
        }
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
          xb[tt][2 * ct] = pack_half_f16(q[tt], 0);
          xb[tt][2 * ct + 1] = pack_half_f16(q[tt], 1);
        }
      }
    }
    // N or dV, rows on lanes: register i of half-wave h is column 32 ct + 16 (i / 8) + 8 h + i % 8 of row 32 ti + l32, so that the row's
    // scale is one value per lane and a lane's registers are two 16-byte pieces of its row.
    f32x16 acc0[2][CT];
    WeightedSum dacc[2];   // D partial of this lane's row (MODE 0)
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) acc0[ti][ct] = zero16();

    for (int m0 = 0; m0 < m; m0 += mc) {
      if (nchunks > 1) {
        __syncthreads();
        stage(m0);
        __syncthreads();
      }
      if (!active) continue;

      // Two waves per SIMD: the wave in its feature loop goes first, so that the other wave's epilogue
      // (no matrix work) fills the gaps instead of competing for issue slots (forward kernel -3 %).
      __builtin_amdgcn_s_setprio(3);
      uint32_t word[2], *bw = nullptr;   // MODE 3
      if (MODE == 3) {
        const int ln = (int)opaque(lane);   // the lane's position: row l32, half h of the features
        bw = bits + ((int64_t)slice * ((n + 63) / 64) + t0 / 64) * 2 * m + m0 + 2 * ((ln & 27) | (ln & 4) << 3 | (ln >> 5) << 2);
      }
#pragma unroll 2
      for (int rt = 0; rt < mc / 32; ++rt) {
        f16x8 oa[KS];     // Omega^T rows of this feature tile: A operand of the projection
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          oa[ks] = *reinterpret_cast<const f16x8 *>(&s_omT[(32 * rt + frow) * AS + 16 * ks + 8 * h]);
#pragma unroll
        for (int ti = 0; ti < 2; ++ti) {
          f32x16 R = zero16();
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) R = mfma_f16(oa[ks], xb[ti][ks], R);
          bf16x8 pa[2];
#pragma unroll
          for (int a = 0; a < 2; ++a) {
            pa[a] = relu_bf16x8(pack_half(R, a));
            if (MODE == 0) dacc[ti].add(pa[a], *reinterpret_cast<const bf16x8 *>(&s_bb[32 * rt + 16 * a + 8 * h]));
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
              acc0[ti][ct] = mfma_bf16(*reinterpret_cast<const bf16x8 *>(&s_MT[(32 * ct + frow) * BS + 32 * rt + 16 * a + 8 * h]), pa[a], acc0[ti][ct]);
          }
          if (MODE == 3) {
            const uint32_t b = positive_bits(pa);
            if ((rt & 1) == 0) word[ti] = b;
            else bw[ti * m + (rt >> 2) * 128 + (rt >> 1 & 1)] = swap_bytes12(word[ti] | b << 8);
          }
        }
      }
    }
    __builtin_amdgcn_s_setprio(0);
    if (!active) continue;

    // ---- epilogues -----------------------------------------------------------------
    {
      // Unconditional (the last round re-requests its own rows): a branch around these loads
      // would leave two paths with different numbers of outstanding memory operations, and the
      // waits the compiler then places further down would cover the loads just issued.
      const int t_next = ((rg + gridDim.x) * NW + wave) * 64;
      load_rows((rg + (int)gridDim.x < row_groups && t_next < n) ? t_next : t0);
    }
    bf16_t *os = out + vo.slice_base(slice) + (int64_t)t0 * vo.sn;
    float *Dp = MODE == 0 ? Dout + (int64_t)slice * n + t0 : nullptr;
    RowBuf osb, Dpb;
    if (RAGGED) {
      osb = row_buffer(os, vo.sn, valid);
      if (MODE == 0) Dpb = row_buffer(Dp, 1, valid);
    }
    const int ln = (int)opaque(lane), row32 = ln & 31, hh = ln >> 5;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int ti = 0; ti < 2; ++ti) {
      float scale = cscale, scale_odd = 0.f, Dt = 0.f;   // scale_odd: LN, columns of odd quads (see tile_sum)
      if (MODE == 0 && LN) {
        // Output stage of Algorithm 1: O_t = (N_t - mean N_t) / sqrt(var N_t + eps), N = c * acc: mean first, then the centred
        // second moment (the other half of the row is in the other half-wave).  1 / sqrt(var + eps) goes to D.
        float v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = acc0[ti][0][i] + acc0[ti][1][i];
        const TileSum mu = tile_sum(v);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          v[i] = 0.f;
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            const float e = (acc0[ti][ct][i] - mu.of(i) * (1.0f / (float)DH)) * cscale;
            acc0[ti][ct][i] = e;
            v[i] = fmaf(e, e, v[i]);
          }
        }
        const TileSum q = tile_sum(v);
        scale = Dt = 1.0f / sqrtf(q.even * (1.0f / (float)DH) + eps);
        scale_odd = 1.0f / sqrtf(q.odd * (1.0f / (float)DH) + eps);
      } else if (MODE == 0) {   // normaliser D_t = c * sum_r relu(R) z + eps, row scale c / D_t
        Dt = fmaf(cscale, xor32_sum(dacc[ti].own(ln)), eps);
        scale = cscale * __builtin_amdgcn_rcpf(Dt);
      }
      if (MODE == 0) {   // (both half-waves write the same values: no branch around the store)
        if (RAGGED) buf_store4(Dpb, 4 * (32 * ti + row32), Dt);
        else Dp[32 * ti + row32] = Dt;
      }
      // bf16 through the wave's panel, [64 rows][64]: 16-byte piece c of row r at slot c ^ (r % 8)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          bf16x8 pk;
#pragma unroll
          for (int e = 0; e < 8; ++e) pk[e] = (__bf16)(acc0[ti][ct][8 * a + e] * (LN && (e & 4) ? scale_odd : scale));
          *reinterpret_cast<bf16x8 *>(panels + (32 * ti + row32) * 64 + (((4 * ct + 2 * a + hh) ^ (row32 & 7)) << 3)) = pk;
        }
    }
    __builtin_amdgcn_wave_barrier();
    u16x8 piece[8];   // row 8 j + lane / 8, columns 8 (lane % 8) ..
#pragma unroll
    for (int j = 0; j < 8; ++j) piece[j] = *reinterpret_cast<const u16x8 *>(panels + (8 * j + (ln >> 3)) * 64 + (((ln & 7) ^ (ln >> 3)) << 3));
    if (RAGGED) {
      const uint32_t off = (uint32_t)(ln >> 3) * ((uint32_t)vo.sn * 2) + (ln & 7) * 16;
#pragma unroll
      for (int j = 0; j < 8; ++j) buf_store16(osb, off + (uint32_t)j * ((uint32_t)vo.sn * 16), piece[j]);
    } else {   // (64-bit: the forward takes rows any distance apart)
      bf16_t *orow = os + (int64_t)(ln >> 3) * vo.sn + (ln & 7) * 8;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        *reinterpret_cast<u16x8 *>(orow) = piece[j];
        orow += 8 * vo.sn;
      }
    }
    put_rows();
  }
}

// 16 bytes per lane from base + voff (bytes) to LDS at lds (bytes, wave-uniform) + 16 * lane, without passing through
// registers.  Written as a statement because the compiler waits for every such load before the next LDS read, whatever it
// reads; the kernel waits (vmcnt) before its barrier instead.  It has no register outputs.
__device__ __forceinline__ void lds_dma16(uint32_t lds, uint32_t voff, const void *base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base)
               : "memory", "m0");
}
// ------------------------------------------------------------------------------------
// Gradient rows kernel of head dimension 64 (MODE 1: query side, MODE 2: key side, as above) where the ReLU's decisions are
// there as bits (see positive_bits): two contractions per feature tile, dPhi and dX_F, and no filter of the rows at the top.
// Eight waves of 64 rows, two per SIMD with 256 registers each, so that one wave's epilogue runs under the other's matrix
// instructions; the feature-side operands of MC features are staged once per workgroup (once per pass and row group
// where there are more).
// What bounds it: no single unit.  8 slices of 131072 rows, m 256, key side (query side): 384 MiB of X, V (dO) and dX and 32 (40) of bits (dD
// and D too) are necessary in this form, 453 (461) move by the counters (in its last round a wave requests its own rows again), 83 (85) us at the 5.7 TB/s of
// a large copy; it takes 107 (116).  Without seven eighths of the feature loop the key side takes 87, without the epilogue's arithmetic 102; matrix cores 38 %
// busy, vector units 55 %.
// The kernel before it formed the projection, too, with one wave of 512 registers per SIMD: 175 us on the query side, 235 on the key
// side with dV beside dX_F; now 116 and 107, and 84 for dV (its kernel has the projection in hand and leaves the bits).
// A lane's row: operand row l32 of dN or V is row 32 ti + r with r's bits (l0, l1, l3, l4, l2), so that the accumulator registers of
// dX_F hold 16 consecutive rows 32 ti + 16 h + i of column 32 ct + l32: of the Haar filter's levels only 32 and 64 rows leave the lane.
// X comes straight from memory into the wave's panels, one of 4 KiB per 32 columns ([64 rows][32], requested a row group ahead), and
// dX goes out through the same panel ([32 columns][64 rows]: 16-byte piece q of column c at slot q ^ (c % 8)).
// ------------------------------------------------------------------------------------
template <int MODE, int MC, bool RAGGED, bool DEEP, int NW = kWavesApply>
__global__ __launch_bounds__(NW * 64, 2) void masked_rows_kernel(
    const bf16_t *x, View vx, const bf16_t *y, View vy, const float *Dsaved, const float *arow, const uint32_t *bits,
    const bf16_t *omega, const bf16_t *Mx, const float *coef, int n, int m, int row_groups, bf16_t *out, View vo,
    float *partF, int L, float *tile_gsum) {
  constexpr int DH = 64, KS = 4, KSX = 5, CT = 2, NT = NW * 64;
  constexpr int AM = DH + 16 + 8, BS = MC + 8, WORDS = MC / 64;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  bf16_t *s_Mx = reinterpret_cast<bf16_t *>(smem_raw);                      // [MC][AM]: (S | z) or (dS | dz)
  bf16_t *s_om = s_Mx + MC * AM;                                            // [DH][BS]: Omega
  float *s_wave = reinterpret_cast<float *>(s_om + DH * BS);                // [waves][64]
  bf16_t *s_panel = reinterpret_cast<bf16_t *>(s_wave + NW * 64);           // [waves][CT][2048]
  typedef __attribute__((address_space(3))) unsigned char lds_byte;
  const int slice = blockIdx.y, tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float cscale = coef[slice * kCoefStride + kCoefCscale];
  const int nchunks = m / MC, blocks = (n + 63) / 64;
  // (What depends on the lane alone is formed anew where it is used, from a value that the compiler does not see through: kept
  // across the feature loop, it would be spilled.)
  auto stage = [&](int m0) {
    // 16-byte pieces per row, pieces, and pieces per thread (all requested before the first is stored)
    constexpr int CPRM = (DH + 16) / 8, CPC = MC / 8, PM = MC * CPRM, PO = DH * CPC, UM = (PM + NT - 1) / NT, UO = (PO + NT - 1) / NT;
    u16x8 tm[UM], to[UO];
    const int tid = (int)opaque(threadIdx.x);
#pragma unroll
    for (int u = 0; u < UM; ++u) {
      const int e = NT * u + tid;
      if (e < PM) tm[u] = *reinterpret_cast<const u16x8 *>(Mx + ((int64_t)slice * m + m0 + e / CPRM) * (DH + 16) + (e % CPRM) * 8);
    }
#pragma unroll
    for (int u = 0; u < UO; ++u) {
      const int e = NT * u + tid;
      if (e < PO) to[u] = *reinterpret_cast<const u16x8 *>(omega + (int64_t)(e / CPC) * m + m0 + (e % CPC) * 8);
    }
#pragma unroll
    for (int u = 0; u < UM; ++u) {
      const int e = NT * u + tid;
      if (e < PM) *reinterpret_cast<u16x8 *>(&s_Mx[(e / CPRM) * AM + (e % CPRM) * 8]) = tm[u];
    }
#pragma unroll
    for (int u = 0; u < UO; ++u) {
      const int e = NT * u + tid;
      if (e < PO) *reinterpret_cast<u16x8 *>(&s_om[(e / CPC) * BS + (e % CPC) * 8]) = to[u];
    }
  };
  float u[kTileBands], cf[kTileBands];   // u_l = sum over blocks of bs_l(g) * bs_l(x), this lane's share
#pragma unroll
  for (int l = 0; l < kTileBands; ++l) {
    u[l] = 0.f;
    cf[l] = coef[slice * kCoefStride + l];
  }
  // Row-side operands; those of the next row group are requested after the feature loop of the current one.
  bf16x8 yb[2][KSX];    // dO or V rows (+ the a_t extension): B operand of dPhi
  float dval[2] = {1.f, 1.f}, aval[2] = {1.f, 1.f};   // D and dD of the lane's rows (MODE 1)
  uint32_t words[2][WORDS];
  const uint32_t *wrow = bits + (int64_t)slice * blocks * 2 * (m / 64) * 64;
  auto load_words = [&](int t0, int m0) {
    const uint32_t *p = wrow + (int64_t)(t0 >> 6) * 2 * m + m0;
    const uint32_t off = 8 * (uint32_t)lane_position((int)opaque(lane));
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
      for (int w = 0; w < WORDS; w += 2) {
        const u32x2v pair = *reinterpret_cast<const u32x2v *>(reinterpret_cast<const char *>(p + ti * m + w * 64) + off);
        words[ti][w] = pair[0];
        words[ti][w + 1] = pair[1];
      }
  };
  auto finish_words = [&]() {
    const int ln = (int)opaque(lane);
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
      for (int w = 0; w < WORDS; ++w) {
        words[ti][w] = swap_bytes12(words[ti][w]);
        if (MODE == 1) words[ti][w] = transpose_bits(words[ti][w], ln);   // (from the contraction: features on lanes)
      }
  };
  u16x8 yraw[8];   // rows of dO or V on their way: 16-byte row-major pieces (row 8 j + lane / 8, columns 8 (lane % 8) ..)
  auto load_rows = [&](int t0) {
    const int valid = RAGGED ? n - t0 : 64;
    const bf16_t *ys = y + vy.slice_base(slice) + (int64_t)t0 * vy.sn;
    const int ln = (int)opaque(lane), lrow = lane_row(ln);
    const uint32_t yoff = (uint32_t)(ln >> 3) * ((uint32_t)vy.sn * 2) + (ln & 7) * 16;
    if (RAGGED) {
      const RowBuf yr = row_buffer(ys, vy.sn, valid);
#pragma unroll
      for (int j = 0; j < 8; ++j) yraw[j] = buf_load16<u16x8>(yr, yoff + (uint32_t)j * ((uint32_t)vy.sn * 16));
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) yraw[j] = *reinterpret_cast<const u16x8 *>(reinterpret_cast<const char *>(ys + 8 * j * vy.sn) + yoff);
    }
    RowBuf dr, ar;
    if (RAGGED && MODE == 1) {
      dr = row_buffer(Dsaved + (int64_t)slice * n + t0, 1, valid);
      ar = row_buffer(arow + (int64_t)slice * n + t0, 1, valid);
    }
#pragma unroll
    for (int ti = 0; ti < 2; ++ti) {
      const int row = 32 * ti + lrow;
      if (MODE == 1) {   // only requested here: used at the top of the next round
        const uint32_t off = 4 * (uint32_t)row;
        dval[ti] = RAGGED ? buf_load4(dr, off) : *reinterpret_cast<const float *>(reinterpret_cast<const char *>(Dsaved + (int64_t)slice * n + t0) + off);
        aval[ti] = RAGGED ? buf_load4(ar, off) : *reinterpret_cast<const float *>(reinterpret_cast<const char *>(arow + (int64_t)slice * n + t0) + off);
      } else if (RAGGED) {
        aval[ti] = row >= valid ? 0.f : 1.f;
      }
    }
    if (nchunks == 1) load_words(t0, 0);
  };
  bf16_t *panels = s_panel + wave * (CT * 2048);
  // The rows of Y through the (free) panels, [64 rows][64], into the order of the operand; then X into its panels, 16 rows of 32
  // columns per request (rows past n: the last one, see below).  (A load of the operand as it is used would touch 32 rows of memory with
  // 32 bytes each; with such loads and stores the kernel took 120 us, with these 107.)
  auto turn_rows = [&](int t0) {
    const int ln = (int)opaque(lane), lrow = lane_row(ln), hh = ln >> 5;
    auto key = [](int row) { return (row & 3) | (row >> 2 & 4); };
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int row = 8 * j + (ln >> 3);
      *reinterpret_cast<u16x8 *>(panels + row * 64 + (((ln & 7) ^ key(row)) << 3)) = yraw[j];
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        yb[ti][ks] = *reinterpret_cast<const bf16x8 *>(panels + (32 * ti + lrow) * 64 + (((2 * ks + hh) ^ key(lrow)) << 3));
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (what is read from the panels has arrived)
    const uint32_t at = (uint32_t)(uintptr_t)(lds_byte *)panels;
    const bf16_t *xs = x + vx.slice_base(slice) + (int64_t)t0 * vx.sn;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int ct = i >> 2, j = i & 3, r = ln >> 2;
      if (RAGGED)
        lds_dma16(at + 1024 * i, (uint32_t)min(16 * j + r, n - t0 - 1) * ((uint32_t)vx.sn * 2) + (ln & 3) * 16, xs + 32 * ct);
      else
        lds_dma16(at + 1024 * i, (uint32_t)r * ((uint32_t)vx.sn * 2) + (ln & 3) * 16, xs + 16 * j * vx.sn + 32 * ct);
    }
  };
  {
    const int t_first = (blockIdx.x * NW + wave) * 64;
    const bool any = (int)blockIdx.x < row_groups && t_first < n;
    if (any) load_rows(t_first);
    if (nchunks == 1) stage(0);
    if (any) turn_rows(t_first);
  }
  __syncthreads();
  const int frow = swap23(l32);   // feature-side operand rows (see swap23)

  for (int rg = blockIdx.x; rg < row_groups; rg += gridDim.x) {
    const int t0 = (rg * NW + wave) * 64;
    const bool active = t0 < n;
    const int valid = RAGGED ? n - t0 : 64;
    if (active) {
      const int lrow = lane_row((int)opaque(lane));
      // MODE 1 works with the raw dO rows: G' = D_t * G (the extension carries dD_t * D_t), and row t of dX_F is scaled by
      // c / D_t at the end; MODE 2 scales by c (extension 1, or 0 for a row past n, which must not pick up the vector part).
#pragma unroll
      for (int ti = 0; ti < 2; ++ti) {
        bf16x8 ext = splat_bf16x8(0.f);
        if (h == 0) ext[0] = (__bf16)(MODE == 1 ? aval[ti] * dval[ti] : (RAGGED ? aval[ti] : 1.0f));
        yb[ti][KS] = ext;
        if (MODE == 1 && h == 0)   // (rows past n: D reads as 0 there, and their scale must be finite for the sums over the block)
          s_wave[wave * 64 + 32 * ti + lrow] =
              (RAGGED && 32 * ti + lrow >= valid) ? 0.f : cscale * __builtin_amdgcn_rcpf(dval[ti]);
      }
    }
    f32x16 acc[2][CT];   // dX_F: rows on registers, columns on lanes
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) acc[ti][ct] = zero16();
    for (int m0 = 0; m0 < m; m0 += MC) {
      if (nchunks > 1) {
        if (active) load_words(t0, m0);
        __syncthreads();
        stage(m0);
        __syncthreads();
      }
      if (!active) continue;
      finish_words();
      __builtin_amdgcn_s_setprio(3);   // ahead of the other wave's epilogue
      // Software pipeline over the row tiles of the feature tiles: the dPhi chain of the next one among the vector instructions
      // that mask and pack the current one (a matrix instruction takes 32 cycles and leaves room for four vector instructions).
      bf16x8 ma[KSX], ob[2][CT];   // (M | b) rows: A operand of dPhi; Omega: B operand of dX_F
      auto read_ma = [&](int ft) {
#pragma unroll
        for (int ks = 0; ks < KSX; ++ks) ma[ks] = *reinterpret_cast<const bf16x8 *>(&s_Mx[(32 * ft + frow) * AM + 16 * ks + 8 * h]);
      };
      auto read_ob = [&](int ft) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct)
            ob[a][ct] = *reinterpret_cast<const bf16x8 *>(&s_om[(32 * ct + l32) * BS + 32 * ft + 16 * a + 8 * h]);
      };
      auto chain = [&](int ti) {
        f32x16 G = zero16();
#pragma unroll
        for (int ks = 0; ks < KSX; ++ks) G = mfma_bf16(ma[ks], yb[ti][ks], G);
        return G;
      };
      auto consume = [&](int ti, const f32x16 &G, uint32_t word, int uu) {
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          const bf16x8 pg = pack_masked(G, a, word, uu);
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) acc[ti][ct] = mfma_bf16(pg, ob[a][ct], acc[ti][ct]);
        }
      };
      // five matrix instructions of the chain, four of the product; the first half is packed when 16 vector instructions are through
      auto pattern = [&](auto early, auto late) {   // LDS reads after the chain, and after the first half's product
#pragma unroll
        for (int i = 0; i < 7; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
          if (i == 4) __builtin_amdgcn_sched_group_barrier(0x100, decltype(early)::value, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, decltype(late)::value, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
        __builtin_amdgcn_sched_barrier(0);
      };
      constexpr int TILES = MC / 32;
      read_ma(0);
      read_ob(0);
      f32x16 G0 = chain(0), G1;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ft = 0; ft < TILES; ++ft) {
        G1 = chain(1);
        consume(0, G0, words[0][ft / 2], ft & 1);
        if (ft + 1 < TILES) read_ma(ft + 1);
        pattern(std::integral_constant<int, KSX>{}, std::integral_constant<int, 0>{});
        if (ft + 1 < TILES) G0 = chain(0);
        consume(1, G1, words[1][ft / 2], ft & 1);
        if (ft + 1 < TILES) {
          read_ob(ft + 1);
          pattern(std::integral_constant<int, 0>{}, std::integral_constant<int, 2 * CT>{});
        }
      }
      __builtin_amdgcn_s_setprio(0);
    }
    if (!active) continue;

    // ---- epilogue.  The next rows' request is unconditional (the last round re-requests its own): see rows_kernel.
    __builtin_amdgcn_s_waitcnt(0x0F70);   // X is in its panels
    asm volatile("" ::: "memory");
    const int t_after = ((rg + (int)gridDim.x) * NW + wave) * 64;
    const int t_next = (rg + (int)gridDim.x < row_groups && t_after < n) ? t_after : t0;
    if (RAGGED && valid < 64) {   // rows past n are zeros
      const u16x8 zero = {};
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (16 * (j & 3) + (lane >> 2) >= valid) *reinterpret_cast<u16x8 *>(panels + (j >> 2) * 2048 + 512 * (j & 3) + lane * 8) = zero;
    }
    load_rows(t_next);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int ti = 0; ti < 2; ++ti) {   // row scale of dX_F
      float sc[16];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4 s4 = {cscale, cscale, cscale, cscale};
        if (MODE == 1) s4 = *reinterpret_cast<const f32x4 *>(&s_wave[wave * 64 + 32 * ti + 16 * h + 4 * g]);
#pragma unroll
        for (int q = 0; q < 4; ++q) sc[4 * g + q] = s4[q];
      }
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[ti][ct][i] *= sc[i];
    }
    // Gated Haar filter of dX_F and band inner products, per column tile: X comes out of the wave's panel, dX goes in (transposed,
    // [column][row]) and leaves in 16-byte row-major pieces through transposing reads.
    bf16_t *os = out + vo.slice_base(slice) + (int64_t)t0 * vo.sn;
    RowBuf osb;
    if (RAGGED) osb = row_buffer(os, vo.sn, valid);
    u16x8 piece[CT][4];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const int ln = (int)opaque(lane), i16 = ln & 15, g16 = ln >> 4, l32 = ln & 31, h = ln >> 5;
      bf16_t *tl = panels + ct * 2048;
      float g5[2], x5[2];
#pragma unroll
      for (int ti = 0; ti < 2; ++ti) {
        float g1[8], x1[8];
        bf16x4 xq[4];   // X at this lane's accumulator positions: rows 32 ti + 16 h + 4 g .. + 3 of column l32
#pragma unroll
        for (int g = 0; g < 4; ++g)
          xq[g] = lds_read_tr4(&tl[(32 * ti + 16 * h + 4 * g + (i16 >> 2)) * 32 + 16 * (g16 & 1) + 4 * (i16 & 3)]);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const float ga = acc[ti][ct][2 * k], gb = acc[ti][ct][2 * k + 1];
          const float xa = (float)xq[k >> 1][2 * (k & 1)], xb = (float)xq[k >> 1][2 * (k & 1) + 1];
          u[0] = fmaf(ga, xa, fmaf(gb, xb, u[0]));
          g1[k] = ga + gb;
          x1[k] = xa + xb;
          u[1] = fmaf(g1[k], x1[k], u[1]);
        }
        float g2[4], x2[4], g3[2], x3[2];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          g2[k] = g1[2 * k] + g1[2 * k + 1];
          x2[k] = x1[2 * k] + x1[2 * k + 1];
          u[2] = fmaf(g2[k], x2[k], u[2]);
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          g3[k] = g2[2 * k] + g2[2 * k + 1];
          x3[k] = x2[2 * k] + x2[2 * k + 1];
          u[3] = fmaf(g3[k], x3[k], u[3]);
        }
        const float g4 = g3[0] + g3[1], x4 = x3[0] + x3[1];
        u[4] = fmaf(g4, x4, u[4]);
        g5[ti] = xor32_sum(g4);   // 32 rows: both half-waves hold the same sums
        x5[ti] = xor32_sum(x4);
        u[5] = fmaf(0.5f * g5[ti], x5[ti], u[5]);
      }
      const float g6 = g5[0] + g5[1], x6 = x5[0] + x5[1];
      u[6] = fmaf(0.5f * g6, x6, u[6]);
      // (both half-waves hold the same sum and write the same value)
      if (DEEP) tile_gsum[((int64_t)slice * blocks + t0 / 64) * DH + 32 * ct + l32] = g6;
      __builtin_amdgcn_wave_barrier();
      // filtered gradient, top-down (block sums rebuilt), bf16 into the panel
#pragma unroll
      for (int ti = 0; ti < 2; ++ti) {
        const float T5 = fmaf(cf[5], g5[ti], cf[6] * g6);
        float g1[8], g2[4], g3[2], o16[16];
#pragma unroll
        for (int k = 0; k < 8; ++k) g1[k] = acc[ti][ct][2 * k] + acc[ti][ct][2 * k + 1];
#pragma unroll
        for (int k = 0; k < 4; ++k) g2[k] = g1[2 * k] + g1[2 * k + 1];
#pragma unroll
        for (int k = 0; k < 2; ++k) g3[k] = g2[2 * k] + g2[2 * k + 1];
        const float T4 = fmaf(cf[4], g3[0] + g3[1], T5);
#pragma unroll
        for (int k3 = 0; k3 < 2; ++k3) {
          const float T3 = fmaf(cf[3], g3[k3], T4);
#pragma unroll
          for (int k2 = 2 * k3; k2 < 2 * k3 + 2; ++k2) {
            const float T2 = fmaf(cf[2], g2[k2], T3);
#pragma unroll
            for (int k1 = 2 * k2; k1 < 2 * k2 + 2; ++k1) {
              const float T1 = fmaf(cf[1], g1[k1], T2);
#pragma unroll
              for (int e = 0; e < 2; ++e) o16[2 * k1 + e] = fmaf(cf[0], acc[ti][ct][2 * k1 + e], T1);
            }
          }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          bf16x8 pk;
#pragma unroll
          for (int e = 0; e < 8; ++e) pk[e] = (__bf16)o16[8 * q + e];
          *reinterpret_cast<bf16x8 *>(&tl[l32 * 64 + (((4 * ti + 2 * h + q) ^ (l32 & 7)) << 3)]) = pk;
        }
      }
      __builtin_amdgcn_wave_barrier();
      // back as rows 16 v + i16, columns 8 g16 .. + 7 of the tile
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int c = i16 >> 2, q = 2 * v + ((i16 & 3) >> 1), e = 4 * (i16 & 1);
        const bf16x4 lo = lds_read_tr4(&tl[(8 * g16 + c) * 64 + ((q ^ c) << 3) + e]);
        const bf16x4 hi = lds_read_tr4(&tl[(8 * g16 + 4 + c) * 64 + ((q ^ (4 + c)) << 3) + e]);
        piece[ct][v] = __builtin_bit_cast(u16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      }
    }
    // whole rows through the panels once more, so that a store covers 8 rows of 128 bytes
    __builtin_amdgcn_wave_barrier();
    {
      const int ln = (int)opaque(lane), i16 = ln & 15, g16 = ln >> 4;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          *reinterpret_cast<u16x8 *>(panels + (16 * v + i16) * 64 + (((4 * ct + g16) ^ (i16 & 7)) << 3)) = piece[ct][v];
      __builtin_amdgcn_wave_barrier();
      const uint32_t off = (uint32_t)(ln >> 3) * ((uint32_t)vo.sn * 2) + (ln & 7) * 16;
      u16x8 row[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) row[j] = *reinterpret_cast<const u16x8 *>(panels + (8 * j + (ln >> 3)) * 64 + (((ln & 7) ^ (ln >> 3)) << 3));
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (RAGGED) buf_store16(osb, off + (uint32_t)j * ((uint32_t)vo.sn * 16), row[j]);
        else *reinterpret_cast<u16x8 *>(reinterpret_cast<char *>(os + 8 * j * vo.sn) + off) = row[j];
      }
    }
    turn_rows(t_next);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the last request: nothing reads it, but it must not outlive the workgroup

  // With u_l = <dX_F, P_l X> the band gradients are dF_L = u_L and dF_{l-1} = u_{l-1} - u_l (l = 1..L).
  __syncthreads();
#pragma unroll
  for (int l = 0; l < kTileBands; ++l) {
    const float s = wave_sum64(u[l]) / (float)(1 << l);
    if (lane == 0) s_wave[wave * 8 + l] = s;
  }
  __syncthreads();
  if (tid <= L) {
    // DEEP: levels above 6 are not seen here; band 6 keeps u_6 alone (its -u_7, and the bands above, come from the tile-sum
    // kernel in extra rows of the partials), bands above get 0.
    float ul = 0.f, ul1 = 0.f;
    if (tid < kTileBands)
      for (int wv = 0; wv < NW; ++wv) {
        ul += s_wave[wv * 8 + tid];
        if (tid < L && tid + 1 < kTileBands) ul1 += s_wave[wv * 8 + tid + 1];
      }
    const int rows = DEEP ? gridDim.x + DH / 16 : gridDim.x;
    partF[((int64_t)slice * rows + blockIdx.x) * (L + 1) + tid] = tid < L ? ul - ul1 : ul;
  }
}
constexpr size_t masked_smem_bytes(int mc, int waves) {
  return (size_t)mc * 88 * 2 + (size_t)64 * (mc + 8) * 2 + (size_t)waves * (64 * 4 + 8192);
}

// ------------------------------------------------------------------------------------
// The rows kernels of head dimension 128 (modes as above).  A wave owns 32 rows and all 128 columns, eight waves per workgroup
// (256 rows), two per SIMD with 256 registers each, so one wave's conversions, masks and LDS latency run under the other's matrix
// instructions.  They share the feature-side operands, which pass through LDS in stages of kWideTiles feature tiles, double-buffered,
// by direct global-to-LDS loads: one barrier per stage, the next stage in flight during it.  A feature tile is
//   Omega^T rows (apply modes) or (M | b) rows (gradient modes)  [32 features][128], 256-byte rows: 16-byte piece c of row r at
//   slot c ^ (r % 16); gradient modes also the 32 extensions of 32 bytes;
//   S^T or Omega  [128 columns][32 features] bf16, 64-byte rows: piece c of row r at slot c ^ ((r / 4) % 4).
// An instruction's row l32 is feature swap23(l32): the features that accumulator registers 8 a .. 8 a + 7 of
// half-wave h stand for are then 16 a + 8 h .. + 7, one 16-byte piece of the second array.
// Rows of X_F, dN or V come in as whole 256-byte lines, a row group ahead, and go through the wave's panel into the order of the operand.
// ------------------------------------------------------------------------------------
constexpr int kWideWaves = 8, kWideTiles = 2, kWideRows = 32 * kWideWaves;
constexpr bool wide_grad(int MODE) { return MODE == 1 || MODE == 2; }
constexpr int wide_tile_bytes(int MODE) { return (wide_grad(MODE) ? 17 : 16) * 1024; }
constexpr int kWidePanel = 8192;   // bytes of a wave's panel
inline size_t wide_smem_bytes(int MODE, int m) {
  return 2 * kWideTiles * wide_tile_bytes(MODE) + kWideWaves * (kWidePanel + (wide_grad(MODE) ? 32 * 4 + 2 * 128 * 4 : 0)) + (MODE == 0 ? m * 2 : 0);
}
// A panel of 32 rows of 256 bytes: 16-byte piece c of row r at slot c ^ wide_key(r).  Rows in the order of a lane's number (natural, or as
// lane_row gives them) meet all eight keys in eight lanes.
__device__ __forceinline__ int wide_key(int r) { return (r & 3) | (r >> 2 & 4) | (r & 4) << 1; }
// The rows' raw pieces (row 4 j + lane / 16, piece lane % 16) -> operands (row `row`, k = 16 ks + 8 h ..).
__device__ __forceinline__ void wide_turn(unsigned char *panel, const u16x8 (&raw)[8], int ln, int row, u16x8 (&op)[8]) {
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int r = 4 * j + (ln >> 4);
    *reinterpret_cast<u16x8 *>(panel + r * 256 + (((ln & 15) ^ wide_key(r)) << 4)) = raw[j];
  }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int ks = 0; ks < 8; ++ks)
    op[ks] = *reinterpret_cast<const u16x8 *>(panel + row * 256 + (((2 * ks + (ln >> 5)) ^ wide_key(row)) << 4));
  __builtin_amdgcn_wave_barrier();
}
// 32 rows of 128 columns from `rows`, row stride sn elements, as raw pieces (RAGGED: zeros from row `valid` on).
template <bool RAGGED, typename T>
__device__ __forceinline__ void wide_load(const T *rows, int64_t sn, int valid, int ln, u16x8 (&raw)[8]) {
  const uint32_t off = (uint32_t)(ln >> 4) * ((uint32_t)sn * 2) + (ln & 15) * 16;
  if (RAGGED) {
    const RowBuf b = row_buffer(rows, sn, valid);
#pragma unroll
    for (int j = 0; j < 8; ++j) raw[j] = buf_load16<u16x8>(b, off + (uint32_t)j * ((uint32_t)sn * 8));
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) raw[j] = *reinterpret_cast<const u16x8 *>(reinterpret_cast<const char *>(rows + 4 * j * sn) + off);
  }
}

// Apply modes.  32 slices of 65536 rows, m 512 (forward, dV): 528 and 544 us (with rows of the accumulators on registers, written
// to LDS two bytes at a time: 559 and 592; with rows of X_F read in the order of the operand, 32 bytes of a line at a time, and without
// the bits: 617 and 584; four waves of 64 rows and 512 registers: 896 and 782).  Matrix cores busy about half of
// the time: an operand of 1 KiB read from LDS serves one matrix instruction, and the waits of two waves per SIMD are not all covered.
template <int MODE, bool LN, bool RAGGED>
__global__ __launch_bounds__(kWideWaves * 64, 2) void wide_rows_kernel(
    const _Float16 *xf, const _Float16 *omT, const bf16_t *MT, const bf16_t *bb, const float *coef, float eps,
    int n, int m, int row_groups, bf16_t *out, View vo, float *Dout, uint32_t *bits) {
  static_assert(!wide_grad(MODE), "the gradient modes have wide_grad_kernel");
  constexpr int DH = 128, KS = 8, CT = 4, TB = wide_tile_bytes(MODE), OO = 8192;   // a feature tile and its second array
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  typedef __attribute__((address_space(3))) unsigned char lds_byte;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte *)smem_raw;
  unsigned char *p = smem_raw + 2 * kWideTiles * TB;
  const int slice = blockIdx.y, tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  unsigned char *panel = p + wave * kWidePanel;
  bf16_t *s_bb = reinterpret_cast<bf16_t *>(p + kWideWaves * kWidePanel);   // MODE 0: z
  const float cscale = coef[slice * kCoefStride + kCoefCscale];

  // ---- staging: wave w moves pieces 4 w .. 4 w + 3 (rows) or 16 w .. 16 w + 15 (columns) of every array
  const int ra = 4 * wave + (lane >> 4), ca = (lane & 15) ^ (ra & 15), ro = 16 * wave + (lane >> 2), co = (lane & 3) ^ ((ro >> 2) & 3);
  const uint32_t va = ra * 256 + ca * 16, vcol = (uint32_t)ro * (uint32_t)(2 * m) + co * 16;
  const bf16_t *cols = MT + (int64_t)slice * DH * m;
  auto request = [&](int buf, int f0) {
#pragma unroll
    for (int ft = 0; ft < kWideTiles; ++ft, f0 += 32) {
      const uint32_t at = lds0 + (uint32_t)((buf * kWideTiles + ft) * TB + wave * 1024);
      lds_dma16(at, va, omT + (int64_t)f0 * DH);
      lds_dma16(at + OO, vcol, cols + f0);
    }
  };
  // (the wait as a builtin: the compiler then knows that the rows' loads have landed, too, and waits for none in the loop)
  auto landed = [&]() {
    __builtin_amdgcn_s_waitcnt(0x0070);
    asm volatile("s_barrier" ::: "memory");
  };
  u16x8 raw[8], xb[KS];
  auto load_rows = [&](int t0) { wide_load<RAGGED>(xf + ((int64_t)slice * n + t0) * DH, DH, n - t0, (int)opaque(lane), raw); };
  auto turn_rows = [&]() {
    const int ln = (int)opaque(lane);
    wide_turn(panel, raw, ln, ln & 31, xb);
  };
  // (with a partial last block both waves of a 64-row block take part: rows past n are zeros)
  auto in_range = [&](int t0) { return (RAGGED ? t0 & ~63 : t0) < n; };

  const int stages = m / (32 * kWideTiles);
  int buf = 0;
  request(0, 0);
  if (MODE == 0)
    for (int e = tid; e < m; e += kWideWaves * 64) s_bb[e] = bb[(int64_t)slice * m + e];
  {
    const int t_first = blockIdx.x * kWideRows + wave * 32;
    if ((int)blockIdx.x < row_groups && in_range(t_first)) {
      load_rows(t_first);
      turn_rows();
    }
  }
  const int prow = swap23(l32), o_row = prow * 256 + ((h ^ (prow & 15)) << 4), o_col0 = prow * 64 + ((h ^ ((prow >> 2) & 3)) << 4);

  for (int rg = blockIdx.x; rg < row_groups; rg += gridDim.x) {
    const int t0 = rg * kWideRows + wave * 32;
    const bool active = in_range(t0);
    const int valid = RAGGED ? n - t0 : 32;
    f32x16 acc[CT];   // rows on lanes, as in rows_kernel
    float dacc = 0.f;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[ct] = zero16();
    uint32_t *bw = nullptr;   // MODE 3: the lane's words (row l32, half h of the features), see positive_bits
    if (MODE == 3)
      bw = bits + (((int64_t)slice * ((n + 63) / 64) + (t0 >> 6)) * 2 + (t0 >> 5 & 1)) * m + 2 * ((l32 & 27) | (l32 & 4) << 3 | h << 2);
    for (int s = 0; s < stages; ++s, buf ^= 1) {
      landed();   // stage s is there; every wave is done with the one before it, which is overwritten now
      request(buf ^ 1, s + 1 < stages ? (s + 1) * 32 * kWideTiles : 0);   // (the last: for the next row group)
      if (!active) continue;
      uint32_t word = 0;
#pragma unroll
      for (int ft = 0; ft < kWideTiles; ++ft) {
        const unsigned char *st = smem_raw + (buf * kWideTiles + ft) * TB;
        f32x16 R = zero16();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          R = mfma_f16(*reinterpret_cast<const f16x8 *>(st + (o_row ^ (32 * ks))), __builtin_bit_cast(f16x8, xb[ks]), R);
        bf16x8 pa[2];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          pa[a] = relu_bf16x8(pack_half(R, a));
          if (MODE == 0)
            dacc = dot8_bf16(pa[a], *reinterpret_cast<const bf16x8 *>(s_bb + (s * kWideTiles + ft) * 32 + 16 * a + 8 * h), dacc);
#pragma unroll
          for (int ct = 0; ct < CT; ++ct)
            acc[ct] = mfma_bf16(*reinterpret_cast<const bf16x8 *>(st + OO + ct * 2048 + (o_col0 ^ (32 * a))), pa[a], acc[ct]);
        }
        if (MODE == 3) word |= positive_bits(pa) << 8 * ft;
      }
      if (MODE == 3) bw[(s >> 1) * 128 + (s & 1)] = swap_bytes12(word);
      // operand reads kAhead matrix instructions before their use (left alone, the compiler reads one and waits for it)
      constexpr int kAhead = 6, MF = kWideTiles * 16;
      __builtin_amdgcn_sched_group_barrier(0x100, kAhead, 0);
#pragma unroll
      for (int i = 0; i < MF - kAhead; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, kAhead, 0);
    }

    // ---- epilogue
    if (!active) continue;   // (no later row group of the wave is in range either)
    const int t_next = t0 + (int)gridDim.x * kWideRows;
    const bool more = rg + (int)gridDim.x < row_groups && in_range(t_next);
    if (more) load_rows(t_next);
    bf16_t *os = out + vo.slice_base(slice) + (int64_t)t0 * vo.sn;
    RowBuf osb;
    if (RAGGED) osb = row_buffer(os, vo.sn, valid);
    const int ln = (int)opaque(lane), row32 = ln & 31, hh = ln >> 5;
    float scale = cscale, scale_odd = 0.f, Dt = 0.f;   // scale_odd: LN, columns of odd quads (see tile_sum)
    if (MODE == 0 && LN) {   // O_t = (N_t - mean N_t) / sqrt(var N_t + eps), N = c * acc; 1 / sqrt(var + eps) goes to D
      float v[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = (acc[0][i] + acc[1][i]) + (acc[2][i] + acc[3][i]);
      const TileSum mu = tile_sum(v);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        v[i] = 0.f;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          const float e = (acc[ct][i] - mu.of(i) * (1.0f / (float)DH)) * cscale;
          acc[ct][i] = e;
          v[i] = fmaf(e, e, v[i]);
        }
      }
      const TileSum q = tile_sum(v);
      scale = Dt = 1.0f / sqrtf(q.even * (1.0f / (float)DH) + eps);
      scale_odd = 1.0f / sqrtf(q.odd * (1.0f / (float)DH) + eps);
    } else if (MODE == 0) {   // D_t = c * sum_r relu(R) z + eps, row scale c / D_t
      Dt = fmaf(cscale, xor32_sum(dacc), eps);
      scale = cscale * __builtin_amdgcn_rcpf(Dt);
    }
    if (MODE == 0 && row32 < valid) Dout[(int64_t)slice * n + t0 + row32] = Dt;   // (both half-waves hold and write the same)
    // bf16 through the wave's panel, [32 rows][128]: 16-byte piece c of row r at slot c ^ (r % 16); a store covers 4 rows of 256 bytes
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        bf16x8 pk;
#pragma unroll
        for (int e = 0; e < 8; ++e) pk[e] = (__bf16)(acc[ct][8 * a + e] * (LN && (e & 4) ? scale_odd : scale));
        *reinterpret_cast<bf16x8 *>(panel + row32 * 256 + (((4 * ct + 2 * a + hh) ^ (row32 & 15)) << 4)) = pk;
      }
    __builtin_amdgcn_wave_barrier();
    u16x8 piece[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int r = 4 * j + (ln >> 4);
      piece[j] = *reinterpret_cast<const u16x8 *>(panel + r * 256 + (((ln & 15) ^ (r & 15)) << 4));
    }
    if (RAGGED) {
      const uint32_t off = (uint32_t)(ln >> 4) * ((uint32_t)vo.sn * 2) + (ln & 15) * 16;
#pragma unroll
      for (int j = 0; j < 8; ++j) buf_store16(osb, off + (uint32_t)j * ((uint32_t)vo.sn * 8), piece[j]);
    } else {   // (64-bit: the forward takes rows any distance apart)
      bf16_t *orow = os + (int64_t)(ln >> 4) * vo.sn + (ln & 15) * 8;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        *reinterpret_cast<u16x8 *>(orow) = piece[j];
        orow += 4 * vo.sn;
      }
    }
    if (more) turn_rows();
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the last request: nothing reads it, but it must not outlive the workgroup
}

// Gradient modes, with the ReLU's decisions given (see masked_rows_kernel, whose epilogue this one shares): the 64-row level of the
// Haar filter, the only one that crosses waves, goes through LDS and costs a barrier.
// 32 slices of 65536 rows, m 512 (Q side, K side): 808 and 797 us.  With the projection in the kernel, X_F among the operands (28 to 148
// bytes per lane of scratch) and rows read and written 16 and 8 bytes at a time: 1132 and 1096.  16 slices of 4096 rows: 40, 36 -> 30, 29.
template <int MODE, bool RAGGED, bool DEEP>
__global__ __launch_bounds__(kWideWaves * 64, 2) void wide_grad_kernel(
    const bf16_t *x, View vx, const bf16_t *y, View vy, const float *Dsaved, const float *arow, const uint32_t *bits,
    const bf16_t *omega, const bf16_t *Mx, const float *coef, int n, int m, int row_groups, bf16_t *out, View vo,
    float *partF, int L, float *tile_gsum) {
  constexpr int DH = 128, KS = 8, CT = 4, TB = wide_tile_bytes(MODE), OO = 8192, OE = 16384;   // a feature tile and its arrays
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  typedef __attribute__((address_space(3))) unsigned char lds_byte;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte *)smem_raw;
  unsigned char *p = smem_raw + 2 * kWideTiles * TB;
  const int slice = blockIdx.y, tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  unsigned char *panel = p + wave * kWidePanel;
  float *s_wave = reinterpret_cast<float *>(p + kWideWaves * kWidePanel), *s_pair = s_wave + kWideWaves * 32;   // [waves][32]; [waves][2][128]: 32-row sums of dX_F and X
  float *sw = s_wave + wave * 32, *mine = s_pair + wave * 256, *other = s_pair + (wave ^ 1) * 256;
  const float cscale = coef[slice * kCoefStride + kCoefCscale];

  // ---- staging, as above
  const int ra = 4 * wave + (lane >> 4), ca = (lane & 15) ^ (ra & 15), ro = 16 * wave + (lane >> 2), co = (lane & 3) ^ ((ro >> 2) & 3);
  const uint32_t vm = ra * 288 + ca * 16, vcol = (uint32_t)ro * (uint32_t)(2 * m) + co * 16, ve = (lane & 31) * 288 + 256 + (lane >> 5) * 16;
  const bf16_t *mx = Mx + (int64_t)slice * m * (DH + 16);
  auto request = [&](int buf, int f0) {
#pragma unroll
    for (int ft = 0; ft < kWideTiles; ++ft, f0 += 32) {
      const uint32_t at = lds0 + (uint32_t)((buf * kWideTiles + ft) * TB + wave * 1024);
      lds_dma16(at, vm, mx + (int64_t)f0 * (DH + 16));
      lds_dma16(at + OO, vcol, omega + f0);
      if (wave == ft) lds_dma16(at + OE - wave * 1024, ve, mx + (int64_t)f0 * (DH + 16));
    }
  };
  auto landed = [&]() {
    __builtin_amdgcn_s_waitcnt(0x0070);
    asm volatile("s_barrier" ::: "memory");
  };
  float u[kTileBands], cf[kTileBands];   // u_l = sum over blocks of bs_l(g) * bs_l(x), this lane's share
#pragma unroll
  for (int l = 0; l < kTileBands; ++l) {
    u[l] = 0.f;
    cf[l] = coef[slice * kCoefStride + l];
  }

  // ---- row-side operands of the wave's 32 rows, and X in the panel as [4 column tiles][32 rows][32]
  u16x8 raw[8], yb[KS];
  float dval = 1.f, aval = 1.f;   // D and dD of the lane's row (MODE 1)
  auto load_rows = [&](int t0) {
    const int ln = (int)opaque(lane), lrow = lane_row(ln), valid = RAGGED ? n - t0 : 32;
    wide_load<RAGGED>(y + vy.slice_base(slice) + (int64_t)t0 * vy.sn, vy.sn, valid, ln, raw);
    if (MODE == 1) {
      const float *Dp = Dsaved + (int64_t)slice * n + t0, *ap = arow + (int64_t)slice * n + t0;
      const uint32_t off = 4 * (uint32_t)lrow;
      dval = RAGGED ? buf_load4(row_buffer(Dp, 1, valid), off) : *reinterpret_cast<const float *>(reinterpret_cast<const char *>(Dp) + off);
      aval = RAGGED ? buf_load4(row_buffer(ap, 1, valid), off) : *reinterpret_cast<const float *>(reinterpret_cast<const char *>(ap) + off);
    } else if (RAGGED) {
      aval = lrow < valid ? 1.f : 0.f;
    }
  };
  auto turn_rows = [&](int t0) {
    const int ln = (int)opaque(lane);
    wide_turn(panel, raw, ln, lane_row(ln), yb);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (what is read from the panel has arrived)
    const uint32_t at = (uint32_t)(uintptr_t)(lds_byte *)panel;
    // (a wave past row n whose block's other half is there: any rows in range will do, they are replaced by zeros)
    const int last = RAGGED ? max(n - t0 - 1, 0) : 31;
    const bf16_t *xs = x + vx.slice_base(slice) + (int64_t)(RAGGED ? min(t0, n - 1) : t0) * vx.sn;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int ct = i >> 1, r = 16 * (i & 1) + (ln >> 2);
      lds_dma16(at + 1024 * i, (uint32_t)(RAGGED ? min(r, last) : r) * ((uint32_t)vx.sn * 2) + (ln & 3) * 16, xs + 32 * ct);
    }
  };
  // (with a partial last block both waves of a 64-row block take part: rows past n are zeros)
  auto in_range = [&](int t0) { return (RAGGED ? t0 & ~63 : t0) < n; };

  const int stages = m / (32 * kWideTiles);
  int buf = 0;
  request(0, 0);
  {
    const int t_first = blockIdx.x * kWideRows + wave * 32;
    if ((int)blockIdx.x < row_groups && in_range(t_first)) {
      load_rows(t_first);
      turn_rows(t_first);
    }
  }
  const int prow = swap23(l32), o_row = prow * 256 + ((h ^ (prow & 15)) << 4), o_ext = (h * 32 + prow) * 16;
  const int o_col0 = l32 * 64 + ((h ^ ((l32 >> 2) & 3)) << 4);

  for (int rg = blockIdx.x; rg < row_groups; rg += gridDim.x) {
    const int t0 = rg * kWideRows + wave * 32;
    const bool active = in_range(t0);
    const int valid = RAGGED ? n - t0 : 32;
    bf16x8 ext = splat_bf16x8(0.f);
    const uint32_t *wp = bits;
    uint32_t next_word = 0;
    if (active) {   // the rank-one extension (a_t, 0, ...); MODE 1 works with the raw dO rows: G' = D_t G
      const int ln = (int)opaque(lane), lrow = lane_row(ln);
      if (h == 0) ext[0] = (__bf16)(MODE == 1 ? aval * dval : aval);
      // row scale c / D_t (rows past n: D reads as 0 there, and their scale must be finite for the sums over the block)
      if (MODE == 1 && h == 0) sw[lrow] = (RAGGED && lrow >= valid) ? 0.f : cscale * __builtin_amdgcn_rcpf(dval);
      wp = bits + (((int64_t)slice * ((n + 63) / 64) + (t0 >> 6)) * 2 + (t0 >> 5 & 1)) * m +
           2 * lane_position(ln);
      next_word = wp[0];
    }
    f32x16 acc[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[ct] = zero16();
    for (int s = 0; s < stages; ++s, buf ^= 1) {
      landed();   // stage s is there; every wave is done with the one before it, which is overwritten now
      request(buf ^ 1, s + 1 < stages ? (s + 1) * 32 * kWideTiles : 0);   // (the last: for the next row group)
      if (!active) continue;
      uint32_t word = swap_bytes12(next_word);
      if (MODE == 1) word = transpose_bits(word, (int)opaque(lane));   // (from the contraction: features on lanes)
      const int sn = s + 1 < stages ? s + 1 : s;
      next_word = wp[(sn >> 1) * 128 + (sn & 1)];
      f32x16 G[kWideTiles];
#pragma unroll
      for (int ft = 0; ft < kWideTiles; ++ft) {
        const unsigned char *st = smem_raw + (buf * kWideTiles + ft) * TB;
        G[ft] = zero16();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          G[ft] = mfma_bf16(*reinterpret_cast<const bf16x8 *>(st + (o_row ^ (32 * ks))), __builtin_bit_cast(bf16x8, yb[ks]), G[ft]);
        G[ft] = mfma_bf16(*reinterpret_cast<const bf16x8 *>(st + OE + o_ext), ext, G[ft]);
      }
#pragma unroll
      for (int ft = 0; ft < kWideTiles; ++ft) {
        const unsigned char *st = smem_raw + (buf * kWideTiles + ft) * TB;
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          const bf16x8 pg = pack_masked(G[ft], a, word, ft);
#pragma unroll
          for (int ct = 0; ct < CT; ++ct)
            acc[ct] = mfma_bf16(pg, *reinterpret_cast<const bf16x8 *>(st + OO + ct * 2048 + (o_col0 ^ (32 * a))), acc[ct]);
        }
      }
      // operand reads kAhead matrix instructions before their use (left alone, the compiler reads one and waits for it)
      constexpr int kAhead = 6, MF = kWideTiles * 17;
      __builtin_amdgcn_sched_group_barrier(0x100, kAhead, 0);
#pragma unroll
      for (int i = 0; i < MF - kAhead; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, kAhead, 0);
    }

    // ---- epilogue.  Lane (l32, h) holds column 32 ct + l32 and rows 16 h + i.
    const int t_next = t0 + (int)gridDim.x * kWideRows;
    const bool more = active && rg + (int)gridDim.x < row_groups && in_range(t_next);
    if (active) {
      // (X is in the panel: the stages' waits were for every load)
      if (RAGGED && valid < 32) {   // rows past n are zeros
        const u16x8 zero = {};
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (16 * (i & 1) + (lane >> 2) >= valid) *reinterpret_cast<u16x8 *>(panel + 1024 * i + lane * 16) = zero;
      }
      if (more) load_rows(t_next);
      __builtin_amdgcn_wave_barrier();
      float sc[16];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4 s4 = {cscale, cscale, cscale, cscale};
        if (MODE == 1) s4 = *reinterpret_cast<const f32x4 *>(&sw[16 * h + 4 * g]);
#pragma unroll
        for (int q = 0; q < 4; ++q) sc[4 * g + q] = s4[q];
      }
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[ct][i] *= sc[i];
        const int ln = (int)opaque(lane), i16 = ln & 15, g16 = ln >> 4;
        const bf16_t *tl = reinterpret_cast<const bf16_t *>(panel) + ct * 1024;
        float g1[8], x1[8];
        bf16x4 xq[4];   // X at this lane's accumulator positions: rows 16 h + 4 g .. + 3 of column l32
#pragma unroll
        for (int g = 0; g < 4; ++g)
          xq[g] = lds_read_tr4(&tl[(16 * (ln >> 5) + 4 * g + (i16 >> 2)) * 32 + 16 * (g16 & 1) + 4 * (i16 & 3)]);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const float ga = acc[ct][2 * k], gb = acc[ct][2 * k + 1];
          const float xa = (float)xq[k >> 1][2 * (k & 1)], xb = (float)xq[k >> 1][2 * (k & 1) + 1];
          u[0] = fmaf(ga, xa, fmaf(gb, xb, u[0]));
          g1[k] = ga + gb;
          x1[k] = xa + xb;
          u[1] = fmaf(g1[k], x1[k], u[1]);
        }
        float g2[4], x2[4], g3[2], x3[2];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          g2[k] = g1[2 * k] + g1[2 * k + 1];
          x2[k] = x1[2 * k] + x1[2 * k + 1];
          u[2] = fmaf(g2[k], x2[k], u[2]);
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          g3[k] = g2[2 * k] + g2[2 * k + 1];
          x3[k] = x2[2 * k] + x2[2 * k + 1];
          u[3] = fmaf(g3[k], x3[k], u[3]);
        }
        const float g4 = g3[0] + g3[1], x4 = x3[0] + x3[1];
        u[4] = fmaf(g4, x4, u[4]);
        const float g5 = xor32_sum(g4), x5 = xor32_sum(x4);   // 32 rows: both half-waves hold the same sums
        u[5] = fmaf(0.5f * g5, x5, u[5]);
        mine[32 * ct + l32] = g5;   // (both half-waves write the same)
        mine[128 + 32 * ct + l32] = x5;
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // (the loads of the next stage stay in flight)
    if (active) {
      bf16_t *os = out + vo.slice_base(slice) + (int64_t)t0 * vo.sn;
      RowBuf osb;
      if (RAGGED) osb = row_buffer(os, vo.sn, valid);
      u16x8 piece[CT][2];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const int ln = (int)opaque(lane), i16 = ln & 15, g16 = ln >> 4, c32 = ln & 31, hh = ln >> 5;
        bf16_t *tl = reinterpret_cast<bf16_t *>(panel) + ct * 1024;
        const float g5 = mine[32 * ct + c32], o5 = other[32 * ct + c32];
        const float g6 = g5 + o5;
        if ((wave & 1) == 0) {
          u[6] = fmaf(0.5f * g6, mine[128 + 32 * ct + c32] + other[128 + 32 * ct + c32], u[6]);
          if (DEEP) tile_gsum[((int64_t)slice * ((n + 63) / 64) + t0 / 64) * DH + 32 * ct + c32] = g6;
        }
        const float T5 = fmaf(cf[5], g5, cf[6] * g6);
        float g1[8], g2[4], g3[2], o16[16];
#pragma unroll
        for (int k = 0; k < 8; ++k) g1[k] = acc[ct][2 * k] + acc[ct][2 * k + 1];
#pragma unroll
        for (int k = 0; k < 4; ++k) g2[k] = g1[2 * k] + g1[2 * k + 1];
#pragma unroll
        for (int k = 0; k < 2; ++k) g3[k] = g2[2 * k] + g2[2 * k + 1];
        const float T4 = fmaf(cf[4], g3[0] + g3[1], T5);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const float T1 = fmaf(cf[1], g1[k], fmaf(cf[2], g2[k >> 1], fmaf(cf[3], g3[k >> 2], T4)));
#pragma unroll
          for (int e = 0; e < 2; ++e) o16[2 * k + e] = fmaf(cf[0], acc[ct][2 * k + e], T1);
        }
        __builtin_amdgcn_wave_barrier();
        // the tile transposed, [32 columns][32 rows]: 16-byte piece q of column c at slot q ^ (c / 2 % 4)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          bf16x8 pk;
#pragma unroll
          for (int e = 0; e < 8; ++e) pk[e] = (__bf16)o16[8 * q + e];
          *reinterpret_cast<bf16x8 *>(&tl[c32 * 32 + (((2 * hh + q) ^ (c32 >> 1 & 3)) << 3)]) = pk;
        }
        __builtin_amdgcn_wave_barrier();
        // back as rows 16 v + i16, columns 8 g16 .. + 7
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          const int c = i16 >> 2, q = 2 * v + ((i16 & 3) >> 1), e = 4 * (i16 & 1);
          const bf16x4 lo = lds_read_tr4(&tl[(8 * g16 + c) * 32 + ((q ^ (c >> 1)) << 3) + e]);
          const bf16x4 hi = lds_read_tr4(&tl[(8 * g16 + 4 + c) * 32 + ((q ^ (2 + (c >> 1))) << 3) + e]);
          piece[ct][v] = __builtin_bit_cast(u16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
      }
      // whole rows through the panel once more, so that a store covers 4 rows of 256 bytes
      __builtin_amdgcn_wave_barrier();
      {
        const int ln = (int)opaque(lane), i16 = ln & 15, g16 = ln >> 4;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
          for (int v = 0; v < 2; ++v)
            *reinterpret_cast<u16x8 *>(panel + (16 * v + i16) * 256 + (((4 * ct + g16) ^ i16) << 4)) = piece[ct][v];
        __builtin_amdgcn_wave_barrier();
        const uint32_t off = (uint32_t)(ln >> 4) * ((uint32_t)vo.sn * 2) + i16 * 16;
        u16x8 row[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int r = 4 * j + (ln >> 4);
          row[j] = *reinterpret_cast<const u16x8 *>(panel + r * 256 + ((i16 ^ (r & 15)) << 4));
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          if (RAGGED) buf_store16(osb, off + (uint32_t)j * ((uint32_t)vo.sn * 8), row[j]);
          else *reinterpret_cast<u16x8 *>(reinterpret_cast<char *>(os + 4 * j * vo.sn) + off) = row[j];
        }
      }
      if (more) turn_rows(t_next);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the last request: nothing reads it, but it must not outlive the workgroup
  // With u_l = <dX_F, P_l X> the band gradients are dF_L = u_L and dF_{l-1} = u_{l-1} - u_l (l = 1..L).
  __syncthreads();
#pragma unroll
  for (int l = 0; l < kTileBands; ++l) {
    const float s = wave_sum64(u[l]) / (float)(1 << l);
    if (lane == 0) sw[l] = s;
  }
  __syncthreads();
  if (tid <= L) {   // DEEP: see masked_rows_kernel
    float ul = 0.f, ul1 = 0.f;
    if (tid < kTileBands)
      for (int wv = 0; wv < kWideWaves; ++wv) {
        ul += s_wave[wv * 32 + tid];
        if (tid < L && tid + 1 < kTileBands) ul1 += s_wave[wv * 32 + tid + 1];
      }
    const int rows = DEEP ? gridDim.x + DH / 16 : gridDim.x;
    partF[((int64_t)slice * rows + blockIdx.x) * (L + 1) + tid] = tid < L ? ul - ul1 : ul;
  }
}

// dX[t][:] += dqbar / n (the pooled-query path; dqbar may be nullptr) + tile_add[t / 64][:] (the
// part of the gated filter above level 6; may be nullptr), bf16 read-modify-write with 16-byte
// accesses, four independent pieces per thread.
// TILE: tile_add is given (the plain instance has none of its code), and blockIdx.z = 1 is dK with its own addends and
// without the pooled term (a launch of its own before: 8 slices of 30000 rows, 17 + 14 us for the two, 26 us now).
// Grid (chunks, slices + rows of the gate's parameter gradients (see gate_bwd_params_rows), 1 or 2).
template <int DH, bool TILE>
__global__ __launch_bounds__(256) void add_pooled_kernel(bf16_t *dq, View v, const float *dqbar, int n,
                                                        float inv_n, const float *tile_add, bf16_t *dk,
                                                        const float *tile_add_k, GateBwdParams gp) {
  constexpr int CPR = DH / 8;
  const int slice = blockIdx.y;
  if (gate_bwd_params_rows(gp)) return;
  if (TILE && blockIdx.z) {
    dq = dk;
    tile_add = tile_add_k;
    dqbar = nullptr;
  }
  const int64_t total = (int64_t)n * CPR;
  const int64_t e0 = (int64_t)blockIdx.x * 1024 + threadIdx.x;
  const int cc = threadIdx.x % CPR;   // 256 and 1024 are multiples of CPR: same columns for all four
  const int ntiles = (n + 63) / 64;
  float add[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) add[q] = (!TILE || dqbar) ? dqbar[(int64_t)slice * DH + cc * 8 + q] * inv_n : 0.f;
  bf16_t *base = dq + v.slice_base(slice) + cc * 8;
  u16x8 val[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t e = e0 + 256 * u;
    if (e < total) val[u] = *reinterpret_cast<u16x8 *>(base + (e / CPR) * v.sn);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t e = e0 + 256 * u;
    if (e < total) {
      const int64_t row = e / CPR;
      float tadd[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      if (TILE) {   // two 16-byte loads of the tile's addend (32-byte aligned: DH and 8 cc are multiples of 8)
        const f32x4 *ta = reinterpret_cast<const f32x4 *>(tile_add + ((int64_t)slice * ntiles + (row >> 6)) * DH + cc * 8);
        const f32x4 t0 = ta[0], t1 = ta[1];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          tadd[q] = t0[q];
          tadd[4 + q] = t1[q];
        }
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) val[u][q] = f32_to_bf16(bf16_to_f32(val[u][q]) + add[q] + tadd[q]);
      *reinterpret_cast<u16x8 *>(base + row * v.sn) = val[u];
    }
  }
}

// Forward: blockIdx.y = 0 for Q, 1 for K; blockIdx.z = group of 16 columns.  T*: tile sums
// [S][ntiles][d]; A*: addends, same shape; pyr: 2 * S pyramids of pyramid_floats(ntiles, d).
// IN_LDS: the pyramid is (pyramid_in_lds bytes of dynamic LDS).
template <bool IN_LDS>
__global__ __launch_bounds__(1024) void coarse_addend_kernel(const float *Tq, const float *Tk, const float *coef,
                                                            int ntiles, int d, int L, float *pyr, float *Aq, float *Ak) {
  extern __shared__ float lds_pyr[];
  const int slice = blockIdx.x, side = blockIdx.y, cl = threadIdx.x & (kCoarseCols - 1);
  const int c = kCoarseCols * blockIdx.z + cl, g = threadIdx.x / kCoarseCols;
  const int64_t base = (int64_t)slice * ntiles * d;
  const float *T = (side ? Tk : Tq) + base, *cf = coef + slice * kCoefStride;
  float *A = (side ? Ak : Aq) + base, *P = pyr + ((int64_t)slice * 2 + side) * pyramid_floats(ntiles, d);
  if constexpr (IN_LDS) coarse_addends(T, cf, ntiles, d, L - 6, first_level((lds_float *)lds_pyr, ntiles, kCoarseCols, cl), A, c, g);
  else coarse_addends(T, cf, ntiles, d, L - 6, first_level(P, ntiles, d, c), A, c, g);
}

// Backward, after both gradient kernels: Tg* = tile sums of dX_F (written by their epilogues),
// Tx* = tile sums of X.  Writes the addends of dX (the filter is symmetric) and, into the extra
// rows row .. row + d / 16 - 1 (one per workgroup) of the band partials part*[S][row + d / 16][L + 1], the
// contribution of the levels above 6: with u_l = 2^-l * sum over 2^l-row blocks and columns of
// blocksum(dX_F) * blocksum(X), band 6 gets -u_7, band l (7 .. L-1) gets u_l - u_{l+1}, band L
// gets u_L (the gradient kernels leave u_6 alone in band 6 and zeros above).
template <bool IN_LDS>
__global__ __launch_bounds__(1024) void coarse_bwd_kernel(const float *TgQ, const float *TgK, const float *TxQ,
                                                         const float *TxK, const float *coef, int ntiles, int d, int L,
                                                         float *pyr, float *AQ, float *AK, float *partQ,
                                                         float *partK, int row) {
  extern __shared__ float lds_pyr[];
  const int slice = blockIdx.x, side = blockIdx.y, J = L - 6, cl = threadIdx.x & (kCoarseCols - 1);
  const int c = kCoarseCols * blockIdx.z + cl, g = threadIdx.x / kCoarseCols;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t base = (int64_t)slice * ntiles * d;
  float *Pg = pyr + (((int64_t)slice * 2 + side) * 2) * pyramid_floats(ntiles, d);
  float *Px = Pg + pyramid_floats(ntiles, d);
  __shared__ float red[kMaxBands][16];
  __shared__ float u[kMaxBands + 1];
  const float *tg = (side ? TgK : TgQ) + base, *tx = (side ? TxK : TxQ) + base, *cf = coef + slice * kCoefStride;
  float *A = (side ? AK : AQ) + base;
  if constexpr (IN_LDS) {
    lds_float *p = (lds_float *)lds_pyr;
    coarse_bwd<false>(tg, tx, cf, ntiles, d, J, first_level(p, ntiles, kCoarseCols, cl), first_level(p + (ntiles + 32) * kCoarseCols, ntiles, kCoarseCols, cl), A,
               c, g, nullptr, red);
  } else {
    coarse_bwd<false>(tg, tx, cf, ntiles, d, J, first_level(Pg, ntiles, d, c), first_level(Px, ntiles, d, c), A, c, g, nullptr, red);
  }
  if (wave == 0 && lane >= 1 && lane <= J) {
    float tot = 0.f;
    for (int i = 0; i < 16; ++i) tot += red[lane][i];
    u[6 + lane] = tot / (float)(1 << (6 + lane));
  }
  __syncthreads();
  if ((int)threadIdx.x <= L) {
    const int i = threadIdx.x;
    float val = 0.f;
    if (i == 6) val = -u[7];
    else if (i > 6) val = i < L ? u[i] - u[i + 1] : u[i];
    float *part = side ? partK : partQ;
    part[((int64_t)slice * (row + gridDim.z) + row + blockIdx.z) * (L + 1) + i] = val;
  }
}

// Backward of the LayerNorm output stage (Algorithm 1), row by row:
//   dN_t = rstd_t (dO_t - mean dO_t - O_t mean(dO_t * O_t))   -> bf16 [slices][n][DH]
// The gradient kernels then run as without a normaliser: D = 1 and dD = 0 (written here).
// part[slice][chunk] = sum over the chunk's rows of -<dO_t, O_t> rstd_t^2, the per-row term of
// d sigma (N scales with 1 / sigma^2 and <dN_t, N_t> = <dO_t, O_t> eps rstd_t^2).
// DH / 8 lanes share a row, 16 bytes each.  Bound by memory; its workgroups have a split of their own, enough of
// them (kLnWgs) to fill every compute unit: with the contraction's split (16 slices of 4096 rows: 128 workgroups of
// 32 dependent rounds of loads) it took 34 us, now 11 us for 50 MB.
template <int DH>
__global__ __launch_bounds__(256) void ln_prep_kernel(const bf16_t *dout, const bf16_t *out, View v,
                                                     const float *rstd, int n, int rows_per_chunk,
                                                     bf16_t *dN, float *ones, float *zeros, float *part) {
  constexpr int CPR = DH / 8, RPB = 256 / CPR;
  const int slice = blockIdx.y, chunk = blockIdx.x, tid = threadIdx.x;
  const int t_begin = chunk * rows_per_chunk, t_end = min(n, t_begin + rows_per_chunk);
  const int r = tid / CPR, cc = tid % CPR;
  const int64_t base = v.slice_base(slice);
  float acc = 0.f;
#pragma unroll 2
  for (int t = t_begin + r; t < t_end; t += RPB) {
    const int64_t off = base + (int64_t)t * v.sn + cc * 8;
    const u16x8 g8 = *reinterpret_cast<const u16x8 *>(dout + off);
    const u16x8 o8 = *reinterpret_cast<const u16x8 *>(out + off);
    float g[8], o[8], sg = 0.f, sgo = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      g[q] = bf16_to_f32(g8[q]);
      o[q] = bf16_to_f32(o8[q]);
      sg += g[q];
      sgo = fmaf(g[q], o[q], sgo);
    }
#pragma unroll
    for (int d = 1; d < CPR; d <<= 1) {
      sg += __shfl_xor(sg, d, 64);
      sgo += __shfl_xor(sgo, d, 64);
    }
    const int64_t row = (int64_t)slice * n + t;
    const float rs = rstd[row];
    const float m1 = sg * (1.0f / (float)DH), m2 = sgo * (1.0f / (float)DH);
    u16x8 d8;
#pragma unroll
    for (int q = 0; q < 8; ++q) d8[q] = cvt_bf16(rs * (g[q] - m1 - o[q] * m2));
    *reinterpret_cast<u16x8 *>(dN + row * DH + cc * 8) = d8;
    if (cc == 0) {
      ones[row] = 1.0f;
      zeros[row] = 0.0f;
      acc -= sgo * rs * rs;
    }
  }
  acc = wave_sum64(acc);
  __shared__ float red[4];
  if ((tid & 63) == 0) red[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) part[(int64_t)slice * gridDim.x + chunk] = (red[0] + red[1]) + (red[2] + red[3]);
}

// ---------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------
constexpr int kLnWgs = 2048;   // workgroups of ln_prep: eight of 256 threads per compute unit

struct FastPlan {
  int DH, FW, NWC, MB, mc;   // NWC: waves of a phiT_contract workgroup; mc: features staged in LDS per pass by the rows kernels of head dimension 64
  int chunksQ, rowsQ;   // pooled-query partial sums
  int chunksC, rowsC;   // split of n in phiT_contract
  int rowWaves, rowGroups, rowsWgs;   // rows kernels: groups of 64 rowWaves rows (head dimension 64) or 256 (128), workgroups per slice
  int chunksL, rowsL;   // split of n in ln_prep
};

FastPlan fast_plan(const wersa_desc &c) {
  FastPlan p{};
  p.DH = c.d;
  if (c.m % 256 == 0 && c.d == 64) { p.FW = 64; p.MB = 256; } else { p.FW = 32; p.MB = 128; }
  p.mc = (c.d == 64 && c.m % 256 == 0) ? 256 : 128;
  const int slices = c.B * c.H, blocks = (c.n + 63) / 64;
  int cq = (c.n + 1023) / 1024;
  p.chunksQ = cq < 1 ? 1 : (cq > 512 ? 512 : cq);
  p.rowsQ = (c.n + p.chunksQ - 1) / p.chunksQ;
  p.chunksQ = (c.n + p.rowsQ - 1) / p.rowsQ;
  if (c.L > kTileL) {   // the pooled-query partial sums double as the 64-row tile sums
    p.rowsQ = 64;
    p.chunksQ = blocks;
  }
  int want = 512 / (slices * (c.m / p.MB));   // two resident workgroups per compute unit, one round
  if (want < 1) want = 1;
  if (want > blocks) want = blocks;
  const int bpc = (blocks + want - 1) / want;
  // Eight waves per workgroup (256 features) from two 64-row blocks per workgroup on: what they save is the second time that a row
  // is brought in and prepared, and from the second block on loads run under products.  With one block four waves on twice the
  // workgroups have less to wait for.  Both kernels' time (forward and backward form), eight waves against four, at 96 to 256
  // workgroups of eight: one block 1.18 times at 96 to 128 workgroups, 0.92 to 1.11 at 140 to 256 (10.9 + 12.9 us against 10.5 + 12.9 in
  // the mean); two blocks 0.92 to 0.99, from 129 workgroups (43 slices of 384 rows, m 256: 24.2 us against 24.8) to 256; three 0.86 to 0.97,
  // four 0.86 to 0.98, six and more 0.73 to 0.89.  (More blocks than one always make 128 workgroups or more.)
  p.NWC = 4;
  if (c.d == 128 && c.m % 256 == 0 && bpc >= 2) { p.NWC = 8; p.MB = 256; }
  p.rowsC = bpc * 64;
  p.chunksC = (blocks + bpc - 1) / bpc;
  const int wantL = kLnWgs / slices < 1 ? 1 : kLnWgs / slices, bpl = (blocks + wantL - 1) / wantL;
  p.rowsL = bpl * 64;
  p.chunksL = (blocks + bpl - 1) / bpl;
  // Few rows (head dimension 64): workgroups of four waves, one per SIMD, where eight waves leave compute units without one and four give each one at
  // most; the time is that of one wave's block then, and two on a SIMD share it.  us of the query side's and the key side's gradient, forward and dV,
  // eight waves and four: 16 workgroups of four (4 slices of 1000 rows, m 256) 16.0 15.2 11.0 11.1, 13.9 12.7 10.1 9.9; 128 (8 of 4096) 17.4 16.6 11.8 12.1,
  // 15.8 14.7 11.1 11.3, with m 512 23.9 22.6 18.1 17.9, 20.3 18.7 16.4 15.7.  Of forward and backward: 200 workgroups (8 of 6400, m 128, 256, 512) 97.1
  // 114.8 147.1, 92.3 110.0 136.8; 240 (20 of 3000) 102.4 121.6 156.0, 98.7 118.7 148.6; 250 (125 of 500, m 256, 512) 128.1 171.4, 127.7 168.3; 256 (8 of 8192)
  // 123.0 152.5, 119.4 143.5, (64 of 1000, m 256) 127.4, 126.8, (128 of 320, m 256, 512) 115.3 158.0, 116.8 155.2.  (Instances with the LayerNorm output stage
  // or levels above 6 have eight.)
  // Not where eight waves hold all rows of a slice and four would too: as many workgroups, and half the threads to stage the operands.  us of forward and
  // backward, eight waves and four: 1 slice of 200 rows, m 256 66.3, 69.5; 8 of 256, m 1024 131.5, 141.8; 32 of 128, m 256 74.6, 77.8, of 256, m 128 67.6, 69.0;
  // 192 of 200, m 256 117.0, 119.1, m 512 156.3, 161.3; but 8 of 320, m 256 82.0, 75.9; 96 of 320 111.6, 109.3.
  p.rowWaves = kWavesApply;
  if (c.d == 64 && c.L <= kTileL && !(c.flags & WERSA_FLAG_LAYERNORM) && blocks > 4 && (int64_t)slices * ((blocks + 3) / 4) <= 256) p.rowWaves = 4;
  p.rowGroups = c.d == 64 ? (blocks + p.rowWaves - 1) / p.rowWaves : (c.n + kWideRows - 1) / kWideRows;
  // One resident workgroup per compute unit (the operand arrays fill most of the LDS): at most
  // 256 workgroups in total, so that no second, mostly empty round follows the first.
  const int wgs = 256 / slices < 1 ? 1 : 256 / slices;
  p.rowsWgs = wgs < p.rowGroups ? wgs : p.rowGroups;
  return p;
}

struct FastWs {
  float *qamax;   // largest |Q| per (slice, chunk) of the pooling pass
  float *scalars, *coef, *qpart, *Spart, *zpart, *dD, *dDpart, *dS, *dz, *partQ, *partK, *dF,
      *dlogit, *dqbar;
  _Float16 *omT;
  bf16_t *Sx, *ST, *zb, *dSx, *dST, *dzb;
  bf16_t *dN;    // LayerNorm output stage: gradient with respect to the un-normalised rows
  float *ones;   // and the stand-in for D in the gradient kernels
  // L > 6: tile sums of Q and K and the addends of the levels above 6 (saved buffer); tile sums
  // of dQ_F and dK_F, the addends of dQ and dK, and the pyramids (workspace)
  float *tileQ, *tileK, *addQ, *addK, *gsumQ, *gsumK, *gaddQ, *gaddK, *pyr;
  uint32_t *bitsQ, *bitsK;   // the ReLU's decisions of the two sides (see positive_bits)
  int64_t total;
};

// Workspace pieces; the per-call constants and the forward's bf16 operand copies live in the
// saved buffer (the backward reads them back instead of rebuilding them).
// 32-bit words of the ReLU's decisions of one side: n m / 8 bytes per slice (n to the next 64).
inline int64_t bits_words(const wersa_desc &c) { return (int64_t)c.B * c.H * ((c.n + 63) / 64) * 2 * c.m; }
// Tensors from 512 MiB on, twice the last-level cache: the two sides' decisions share one buffer, and the query side goes first.
// Below it goes last, so that the pass that adds the pooled query's share finds part of dQ in the cache, and the second buffer
// is 2 GiB at most (d 64, m 4096).  us per training step with two buffers and with one: tensors of 512 MiB, d 64, m 256 2483, 2488,
// m 512 4333, 4345, d 128, m 256 3024, 3019; of 256 MiB, m 256 1285, 1296; of 128 MiB, m 1024 1848, 1853, m 2048 3318, 3345.
inline bool one_bits_buffer(const wersa_desc &c) { return (int64_t)c.B * c.H * c.n * c.d * 2 >= ((int64_t)512 << 20); }

FastWs fast_ws(const wersa_desc &c, const FastPlan &p, int bwd, float *base, float *saved) {
  FastWs w{};
  Bump b(base);
  const int64_t sl = (int64_t)c.B * c.H, md = (int64_t)c.m * c.d;
  if (saved) {   // (asked for the size alone, this may be called to find out which path a descriptor takes)
    const SavedLayout sv = saved_layout(c);
    w.scalars = saved + sv.scalars;
    w.coef = saved + sv.coef;
    w.omT = reinterpret_cast<_Float16 *>(saved + sv.omT);
    w.Sx = reinterpret_cast<bf16_t *>(saved + sv.Sx);
    w.ST = reinterpret_cast<bf16_t *>(saved + sv.ST);
    w.zb = reinterpret_cast<bf16_t *>(saved + sv.zb);
    if (sv.tileQ >= 0) {
      w.tileQ = saved + sv.tileQ;
      w.tileK = saved + sv.tileK;
      w.addQ = saved + sv.addQ;
      w.addK = saved + sv.addK;
    }
  }
  const bool deep = c.L > kTileL;
  const int ntiles = (c.n + 63) / 64;
  w.qpart = b.take(sl * p.chunksQ * c.d);
  w.qamax = b.take(sl * p.chunksQ);
  w.Spart = b.take(sl * p.chunksC * md);
  w.zpart = b.take(sl * p.chunksC * c.m);
  const int64_t mx = (int64_t)c.m * (c.d + 16);
  if (bwd) {
    w.dD = b.take(sl * c.n);
    w.dDpart = b.take(sl * (c.flags & WERSA_FLAG_LAYERNORM ? p.chunksL : p.chunksC));
    w.dS = b.take(sl * md);
    w.dz = b.take(sl * c.m);
    w.dSx = reinterpret_cast<bf16_t *>(b.take(sl * mx / 2));
    w.dST = reinterpret_cast<bf16_t *>(b.take(sl * md / 2));
    w.dzb = reinterpret_cast<bf16_t *>(b.take(sl * c.m / 2));
    w.partQ = b.take(sl * (p.rowsWgs + c.d / kCoarseCols) * (c.L + 1));   // (+ the rows of the levels above 6)
    w.partK = b.take(sl * (p.rowsWgs + c.d / kCoarseCols) * (c.L + 1));
    if (deep) {
      const int64_t tiles = sl * ntiles * c.d;
      w.gsumQ = b.take(tiles);
      w.gsumK = b.take(tiles);
      w.gaddQ = b.take(tiles);
      w.gaddK = b.take(tiles);
    }
    w.bitsQ = reinterpret_cast<uint32_t *>(b.take(bits_words(c)));
    w.bitsK = one_bits_buffer(c) ? w.bitsQ : reinterpret_cast<uint32_t *>(b.take(bits_words(c)));
    w.dF = b.take(sl * (c.L + 1));
    w.dlogit = b.take(sl * (c.L + 1));
    w.dqbar = b.take(sl * c.d);
    if (c.flags & WERSA_FLAG_LAYERNORM) {
      w.dN = reinterpret_cast<bf16_t *>(b.take(sl * c.n * c.d / 2));
      w.ones = b.take(sl * c.n);
    }
  }
  if (deep) w.pyr = b.take(sl * 4 * pyramid_floats(ntiles, c.d));
  w.total = b.off;
  return w;
}

template <int MODE>
size_t rows_smem_bytes(int mc, int NW) {   // of rows_kernel
  constexpr int DH = 64;
  size_t s = (size_t)mc * (DH + 8) * 2 + (size_t)DH * (mc + 8) * 2;
  if (MODE == 0) s += (size_t)mc * 2;
  s += (size_t)NW * (DH / 32) * 64 * 36 * 2 + 2 * 512 * 2;   // X panels per wave and the filter table
  return s;
}

// Head dimension 128.
template <int MODE>
hipError_t launch_wide_rows(const wersa_desc &c, const FastPlan &p, const _Float16 *xf, const bf16_t *x, const bf16_t *y,
                            const float *Dsaved, const float *arow, const FastWs &w, const bf16_t *omega, const bf16_t *Mx,
                            const bf16_t *MT, const bf16_t *bb, bf16_t *out, float *Dout, float *partF, hipStream_t st,
                            const View *yview) {
  const int64_t side = ((c.flags & WERSA_FLAG_SEPARATE_OMEGA) && MODE >= 2) ? (int64_t)c.d * c.m : 0;
  const View tv{c.stride_b, c.stride_h, c.stride_n, c.H};
  const size_t smem = wide_smem_bytes(MODE, c.m);
  const dim3 grid(p.rowsWgs, c.B * c.H);
  auto allow = [&](auto kern) {
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  };
  const bool ragged = c.n % 64 != 0;
  if constexpr (wide_grad(MODE)) {
    auto go = [&](auto kern) -> hipError_t {
      const hipError_t e = allow(kern);
      if (e != hipSuccess) return e;
      WERSA_STAGE(MODE == 1 ? "wersa_grad_q" : "wersa_grad_k", st,
                  kern<<<grid, kWideWaves * 64, smem, st>>>(x, tv, y, yview ? *yview : tv, Dsaved, arow, MODE == 1 ? w.bitsQ : w.bitsK,
                                                            omega + side, Mx, w.coef, c.n, c.m, p.rowGroups, out, tv, partF, c.L,
                                                            MODE == 1 ? w.gsumQ : w.gsumK));
      return hipSuccess;
    };
    if (c.L > kTileL) return ragged ? go(&wide_grad_kernel<MODE, true, true>) : go(&wide_grad_kernel<MODE, false, true>);
    return ragged ? go(&wide_grad_kernel<MODE, true, false>) : go(&wide_grad_kernel<MODE, false, false>);
  } else {
    auto go = [&](auto kern) -> hipError_t {
      const hipError_t e = allow(kern);
      if (e != hipSuccess) return e;
      WERSA_STAGE(MODE == 0 ? "wersa_rows_fwd" : "wersa_rows_bwd_v", st,
                  kern<<<grid, kWideWaves * 64, smem, st>>>(xf, w.omT + side, MT, bb, w.coef, c.eps, c.n, c.m, p.rowGroups, out, tv, Dout,
                                                            w.bitsK));
      return hipSuccess;
    };
    if (MODE == 0 && (c.flags & WERSA_FLAG_LAYERNORM))
      return ragged ? go(&wide_rows_kernel<MODE, MODE == 0, true>) : go(&wide_rows_kernel<MODE, MODE == 0, false>);
    return ragged ? go(&wide_rows_kernel<MODE, false, true>) : go(&wide_rows_kernel<MODE, false, false>);
  }
}

// Head dimension 64, MODE 0 and 3.
template <int MODE>
hipError_t launch_rows64(const wersa_desc &c, const FastPlan &p, const bf16_t *x, const FastWs &w, const bf16_t *MT, const bf16_t *bb,
                         bf16_t *out, float *Dout, hipStream_t st) {
  // key-side modes take the second random matrix when the descriptor has two
  const _Float16 *omT = w.omT + (((c.flags & WERSA_FLAG_SEPARATE_OMEGA) && MODE >= 2) ? (int64_t)c.d * c.m : 0);
  const View tv{c.stride_b, c.stride_h, c.stride_n, c.H};
  const size_t smem = rows_smem_bytes<MODE>(p.mc, p.rowWaves);
  auto go = [&](auto kern) -> hipError_t {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    WERSA_STAGE(MODE == 0 ? "wersa_rows_fwd" : "wersa_rows_bwd_v", st,
                kern<<<dim3(p.rowsWgs, c.B * c.H), p.rowWaves * 64, smem, st>>>(
                    x, tv, omT, MT, bb, w.coef, c.eps, c.n, c.m, p.rowGroups, out, tv, Dout, MODE == 3 ? w.addK : w.addQ, w.bitsK));
    return hipSuccess;
  };
  const bool ln = MODE == 0 && (c.flags & WERSA_FLAG_LAYERNORM), ragged = c.n % 64 != 0, deep = c.L > kTileL;
  // partial last block, levels above one block: instances of their own
  auto pick = [&](auto mcv, auto lnv) -> hipError_t {
    constexpr int MC = decltype(mcv)::value;
    constexpr bool LNV = decltype(lnv)::value;
    if (deep) return ragged ? go(&rows_kernel<MODE, MC, LNV, true, true>) : go(&rows_kernel<MODE, MC, LNV, false, true>);
    if constexpr (!LNV)
      if (p.rowWaves == 4) return ragged ? go(&rows_kernel<MODE, MC, false, true, false, 4>) : go(&rows_kernel<MODE, MC, false, false, false, 4>);
    return ragged ? go(&rows_kernel<MODE, MC, LNV, true, false>) : go(&rows_kernel<MODE, MC, LNV, false, false>);
  };
  using M128 = std::integral_constant<int, 128>;
  using M256 = std::integral_constant<int, 256>;
  using LNV = std::bool_constant<MODE == 0>;
  if (ln) return p.mc == 256 ? pick(M256{}, LNV{}) : pick(M128{}, LNV{});
  return p.mc == 256 ? pick(M256{}, std::false_type{}) : pick(M128{}, std::false_type{});
}

// Gradient of one side at head dimension 64 with the ReLU's decisions given.
template <int MODE>
hipError_t launch_masked64(const wersa_desc &c, const FastPlan &p, const bf16_t *x, const bf16_t *y, const float *Dsaved,
                           const float *arow, const FastWs &w, const bf16_t *omega, const bf16_t *Mx, bf16_t *out, float *partF,
                           hipStream_t st, const View *yview) {
  if ((c.flags & WERSA_FLAG_SEPARATE_OMEGA) && MODE == 2) omega += (int64_t)c.d * c.m;
  const View tv{c.stride_b, c.stride_h, c.stride_n, c.H};
  auto go = [&](auto kern) -> hipError_t {
    const size_t smem = masked_smem_bytes(p.mc, p.rowWaves);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    WERSA_STAGE(MODE == 1 ? "wersa_grad_q" : "wersa_grad_k", st,
                kern<<<dim3(p.rowsWgs, c.B * c.H), p.rowWaves * 64, smem, st>>>(
                    x, tv, y, yview ? *yview : tv, Dsaved, arow, MODE == 1 ? w.bitsQ : w.bitsK, omega, Mx, w.coef, c.n, c.m,
                    p.rowGroups, out, tv, partF, c.L, MODE == 1 ? w.gsumQ : w.gsumK));
    return hipSuccess;
  };
  const bool ragged = c.n % 64 != 0, deep = c.L > kTileL;
  auto pick = [&](auto MC) -> hipError_t {
    constexpr int M = MC.value;
    if (deep) return ragged ? go(&masked_rows_kernel<MODE, M, true, true>) : go(&masked_rows_kernel<MODE, M, false, true>);
    if (p.rowWaves == 4) return ragged ? go(&masked_rows_kernel<MODE, M, true, false, 4>) : go(&masked_rows_kernel<MODE, M, false, false, 4>);
    return ragged ? go(&masked_rows_kernel<MODE, M, true, false>) : go(&masked_rows_kernel<MODE, M, false, false>);
  };
  return p.mc == 256 ? pick(std::integral_constant<int, 256>{}) : pick(std::integral_constant<int, 128>{});
}

template <int DH, int MODE>
hipError_t launch_rows(const wersa_desc &c, const FastPlan &p, const _Float16 *xf, const bf16_t *x,
                       const bf16_t *y, const float *Dsaved, const float *arow, const FastWs &w,
                       const bf16_t *omega, const bf16_t *Mx, const bf16_t *MT, const bf16_t *bb,
                       bf16_t *out, float *Dout, float *partF, hipStream_t st, const View *yview = nullptr) {
  if constexpr (DH == 128)
    return launch_wide_rows<MODE>(c, p, xf, x, y, Dsaved, arow, w, omega, Mx, MT, bb, out, Dout, partF, st, yview);
  else if constexpr (MODE == 1 || MODE == 2)
    return launch_masked64<MODE>(c, p, x, y, Dsaved, arow, w, omega, Mx, out, partF, st, yview);
  else
    return launch_rows64<MODE>(c, p, x, w, MT, bb, out, Dout, st);
}

// orows != nullptr selects the backward form that derives dD from the rows of O itself;
// otherwise the row weights of the vector part are `wts` (all ones when nullptr).
template <int DH>
void launch_contract(const wersa_desc &c, const FastPlan &p, const _Float16 *xf, const bf16_t *xraw,
                     const bf16_t *y, const View &yv, const float *rowdiv, const float *wts, const bf16_t *orows,
                     bool key_side, const FastWs &w, float *S, float *z, bf16_t *Mx, bf16_t *MT,
                     bf16_t *bb, const GateFwdArgs &gate, hipStream_t st) {
  const int slices = c.B * c.H;
  dim3 grid(p.chunksC, c.m / p.MB, slices);
  const _Float16 *omT = w.omT + (((c.flags & WERSA_FLAG_SEPARATE_OMEGA) && key_side) ? (int64_t)c.d * c.m : 0);
  // The backward's launch is the one on the query side: it leaves the ReLU's decisions for the gradient kernel.
  const bool bwd = !key_side;
  auto go = [&](auto kern) {
    WERSA_STAGE("wersa_phiT_contract", st,
                kern<<<grid, 64 * p.NWC, 0, st>>>(xf, xraw, View{c.stride_b, c.stride_h, c.stride_n, c.H}, w.coef,
                                           key_side ? w.addK : w.addQ, y, yv,
                                           rowdiv, wts, orows, w.dD, w.dDpart, omT, c.n, c.m, p.rowsC, w.Spart,
                                           w.zpart, bwd ? w.bitsQ : nullptr, gate));
  };
  const bool ragged = c.n % 64 != 0, deep = DH == 64 && c.L > kTileL;
  constexpr bool D64 = DH == 64;
  // forward; backward with the rows of O (dD derived here); backward after the LayerNorm output stage
  auto form = [&](auto FW, auto NW, auto RAG, auto DEEP) {
    constexpr int F = FW.value, N = NW.value;
    if (!bwd) go(&phiT_contract_kernel<DH, F, false, RAG.value, DEEP.value, false, N>);
    else if (orows) go(&phiT_contract_kernel<DH, F, true, RAG.value, DEEP.value, true, N>);
    else go(&phiT_contract_kernel<DH, F, false, RAG.value, DEEP.value, true, N>);
  };
  using Yes = std::true_type;
  using No = std::false_type;
  auto shape = [&](auto FW, auto NW) {
    if (deep) ragged ? form(FW, NW, Yes{}, std::bool_constant<D64>{}) : form(FW, NW, No{}, std::bool_constant<D64>{});
    else ragged ? form(FW, NW, Yes{}, No{}) : form(FW, NW, No{}, No{});
  };
  using I4 = std::integral_constant<int, 4>;
  if constexpr (DH == 128) {
    if (p.NWC == 8) shape(std::integral_constant<int, 32>{}, std::integral_constant<int, 8>{});
    else shape(std::integral_constant<int, 32>{}, I4{});
  } else {   // (64 features per wave exist for head dimension 64 only, see fast_plan)
    if (p.FW == 64) shape(std::integral_constant<int, 64>{}, I4{});
    else shape(std::integral_constant<int, 32>{}, I4{});
  }
  const int64_t W = (int64_t)c.m * DH;
  auto reduce = [&](auto VEC) {
    constexpr int cols = 64 * VEC.value;
    WERSA_STAGE("wersa_reduce_contract", st,
                (reduce_contract_kernel<DH, VEC.value><<<dim3((unsigned)(W / cols + (c.m + cols - 1) / cols), slices), 256, 0, st>>>(
                    w.Spart, w.zpart, p.chunksC, c.m, w.coef + kCoefCscale, S, z, Mx, MT, bb)));
  };
  if (slices * (W / 1024) >= 128)   // (see reduce_short_kernel)
    WERSA_STAGE("wersa_reduce_contract", st,
                (reduce_short_kernel<DH><<<dim3((unsigned)(W / 1024 + (c.m + 1023) / 1024), slices), 256, 0, st>>>(
                    w.Spart, w.zpart, p.chunksC, c.m, w.coef + kCoefCscale, S, z, Mx, MT, bb)));
  else if (slices * (W / 256) >= 256) reduce(std::integral_constant<int, 4>());
  else reduce(std::integral_constant<int, 1>());
}

template <int DH>
wersa_status fast_forward_t(const wersa_desc &c, const bf16_t *q, const bf16_t *k, const bf16_t *v,
                            const bf16_t *omega, const float *sigma, const float *gate_w,
                            const float *gate_b, const float *scale_w, bf16_t *out, float *saved,
                            float *ws, hipStream_t st, const PooledSums *pooled) {
  const FastPlan p = fast_plan(c);
  const FastWs w = fast_ws(c, p, 0, ws, saved);
  const SavedLayout sv = saved_layout(c);
  const int slices = c.B * c.H;
  const View tv{c.stride_b, c.stride_h, c.stride_n, c.H};
  float *S = saved + sv.S, *z = saved + sv.z, *qbar = saved + sv.qbar, *s = saved + sv.s,
        *F = saved + sv.F, *D = saved + sv.D;
  _Float16 *QF = sv.QF >= 0 ? reinterpret_cast<_Float16 *>(saved + sv.QF) : nullptr;
  _Float16 *KF = sv.KF >= 0 ? reinterpret_cast<_Float16 *>(saved + sv.KF) : nullptr;

  const int nmat = (c.flags & WERSA_FLAG_SEPARATE_OMEGA) ? 2 : 1;
  SetupArgs su{sigma, c.bw_floor, omega, c.d, c.m, nmat, w.scalars, w.omT, setup_blocks(c.d, c.m, nmat)};
  const SetupArgs none{};
  const bool deep = c.L > kTileL;
  const bool pooled_gate = (c.flags & WERSA_FLAG_POOLED_GATE) != 0;
  GateFwdArgs gate{};
  gate.n = c.n, gate.d = c.d, gate.L = c.L, gate.H = c.H;
  gate.gate_w = gate_w, gate.gate_b = gate_b, gate.scale_w = scale_w, gate.scalars = w.scalars;
  gate.qbar = qbar, gate.s_out = s, gate.F_out = F, gate.coef_out = w.coef;
  if (pooled && c.n % 128 == 0 && !deep) {
    WERSA_STAGE("wersa_setup", st, setup_kernel<<<su.blocks, 256, 0, st>>>(su));
    // the caller's column sums per 128 token rows: batch b owns row blocks [b n/128, (b+1) n/128)
    const int groups = c.d / kPooledMaxCols;
    const int64_t all = pooled->hidden / kPooledMaxCols;
    gate.qpart = pooled->sums;
    gate.chunks = c.n / 128;
    gate.ql = PooledLayout{gate.chunks * pooled->hidden, c.d, pooled->hidden};
    gate.amax_part = pooled->amax;
    gate.amax_chunks = gate.chunks * groups;
    gate.al = AmaxLayout{gate.chunks * all, groups, all, groups};
  } else {
    // deep: one partial per 64-row tile, kept (with those of K) as the tile sums of the levels above 6
    float *qpart = deep ? w.tileQ : w.qpart;
    WERSA_STAGE("wersa_qbar", st,
                qbar_partial_kernel<DH><<<dim3(p.chunksQ + su.blocks, slices), 256, 0, st>>>(q, tv, c.n, p.rowsQ, qpart,
                                                                                             p.chunksQ, su, w.qamax));
    gate.qpart = qpart;
    gate.chunks = gate.amax_chunks = p.chunksQ;
    gate.ql = PooledLayout{(int64_t)c.H * p.chunksQ * c.d, (int64_t)p.chunksQ * c.d, c.d};
    gate.amax_part = w.qamax;
    gate.al = AmaxLayout{(int64_t)c.H * p.chunksQ, p.chunksQ, 0, p.chunksQ};
  }
  // Head dimension 64: the contraction's workgroups form the gate themselves where they are one round, two per compute unit (us per call, forward: 64 slices
  // of 4096 rows, m 128 60.6 -> 58.5, 4 of 2000, m 256 34.9 -> 32.5, 128 of 1000 67.0 -> 64.8, attention block with 8 heads of 2048 rows 51.8 -> 49.0).
  // In further rounds each waits for it again: there where a slice's features are on one or two workgroups, and with them the launch of its own has many
  // slices (gate apart and inside: 1000 slices of 256 rows, m 128 105.9, 93.6, m 256 154.2, 142.0; 512 of 1000, m 512 261.0, 254.9; 750 of 256, m 512
  // 208.9, 205.0), up to where the two meet (1000 of 256, m 512 298.2, 299.4); not with more (128 of 64, m 2048 127.3, 128.8; 160 of 1000, m 2048
  // 317.8, 323.4; 1000 of 256, m 1024 567.5, 585.2; 1000 of 64, m 4096 2104, 2186).
  // Not the thousands of workgroups of head dimension 128's filter, nor a gate that pools heads or has many partial sums.
  const int64_t contracting = (int64_t)p.chunksC * (c.m / p.MB) * slices;
  const bool inside = contracting <= 512 || (c.m <= 2 * p.MB && contracting <= 1536);
  if (DH != 64 || deep || pooled_gate || gate.chunks > kGatePrologueChunks || !inside) {
    WERSA_STAGE("gate_fwd_kernel", st,
                gate_fwd_kernel<<<slices, kGateFwdThreads, 0, st>>>(gate.qpart, gate.chunks, c.n, c.d, c.L, c.H, gate_w, gate_b, scale_w,
                                                       qbar, s, F, w.coef, pooled_gate ? 1 : 0, gate.ql,
                                                       gate.amax_part, gate.amax_chunks, w.scalars, gate.al));
    gate.qpart = nullptr;
  }
  if (deep) {
    WERSA_STAGE("wersa_qbar", st,
                qbar_partial_kernel<DH><<<dim3(p.chunksQ, slices), 256, 0, st>>>(k, tv, c.n, p.rowsQ, w.tileK,
                                                                                 p.chunksQ, none, nullptr));
    auto go = [&](auto kern, size_t lds) {
      WERSA_STAGE("wersa_coarse_addend", st, kern<<<dim3(slices, 2, DH / kCoarseCols), 1024, lds, st>>>(w.tileQ, w.tileK, w.coef, p.chunksQ, DH, c.L,
                                                                                                       w.pyr, w.addQ, w.addK));
    };
    if (const size_t lds = pyramid_in_lds(&coarse_addend_kernel<true>, p.chunksQ, 1)) go(&coarse_addend_kernel<true>, lds);
    else go(&coarse_addend_kernel<false>, 0);
  }
  if (DH != 64) {   // head dimension 64 runs stage A inside the kernels that consume X_F
    WERSA_STAGE("wersa_haar_stage", st,
                haar_stage_kernel<DH><<<dim3((c.n + 63) / 64, slices, 2), 256, 0, st>>>(q, k, tv, c.n, w.coef, deep ? w.addQ : nullptr,
                                                                                       deep ? w.addK : nullptr, QF, KF));
  }
  launch_contract<DH>(c, p, KF, k, v, tv, nullptr, nullptr, nullptr, true, w, S, z, w.Sx, w.ST, w.zb, gate, st);
  if (launch_rows<DH, 0>(c, p, QF, q, nullptr, nullptr, nullptr, w, omega, nullptr, w.ST, w.zb, out, D,
                         nullptr, st) != hipSuccess)
    return WERSA_ERR_LAUNCH;
  return hipGetLastError() == hipSuccess ? WERSA_OK : WERSA_ERR_LAUNCH;
}

template <int DH>
wersa_status fast_backward_t(const wersa_desc &c, const bf16_t *q, const bf16_t *k, const bf16_t *v,
                             const bf16_t *omega, const float *sigma, const float *gate_w,
                             const float *scale_w, const bf16_t *out, const bf16_t *dout,
                             const float *saved, bf16_t *dq, bf16_t *dk, bf16_t *dv, float *dgate_w,
                             float *dgate_b, float *dscale_w, float *dsigma, float *ws,
                             hipStream_t st) {
  const FastPlan p = fast_plan(c);
  const FastWs w = fast_ws(c, p, 1, ws, const_cast<float *>(saved));   // operand copies are only read
  const SavedLayout sv = saved_layout(c);
  const int slices = c.B * c.H;
  const View tv{c.stride_b, c.stride_h, c.stride_n, c.H};
  const float *qbar = saved + sv.qbar, *s = saved + sv.s, *D = saved + sv.D;
  const _Float16 *QF = sv.QF >= 0 ? reinterpret_cast<const _Float16 *>(saved + sv.QF) : nullptr;
  const _Float16 *KF = sv.KF >= 0 ? reinterpret_cast<const _Float16 *>(saved + sv.KF) : nullptr;

  // dS = Phi_Q^T dN, dz = Phi_Q^T dD; the same pass derives dD_t = -<dO_t, O_t> / D_t from the
  // rows of O and leaves it in the workspace for the Q-side gradient kernel.
  const bool ln = (c.flags & WERSA_FLAG_LAYERNORM) != 0;
  // LayerNorm output stage: dN first, then the same kernels with D = 1 and dD = 0 (so dz = 0).
  const View nv{(int64_t)c.H * c.n * DH, (int64_t)c.n * DH, DH, c.H};
  if (ln) {
    WERSA_STAGE("wersa_ln_prep", st,
                ln_prep_kernel<DH><<<dim3(p.chunksL, slices), 256, 0, st>>>(dout, out, tv, D, c.n, p.rowsL, w.dN,
                                                                           w.ones, w.dD, w.dDpart));
    launch_contract<DH>(c, p, QF, q, w.dN, nv, nullptr, w.dD, nullptr, false, w, w.dS, w.dz, w.dSx, w.dST, w.dzb, GateFwdArgs{}, st);
  } else {
    launch_contract<DH>(c, p, QF, q, dout, tv, D, nullptr, out, false, w, w.dS, w.dz, w.dSx, w.dST, w.dzb, GateFwdArgs{}, st);
  }
  auto key_side = [&]() {
    const hipError_t e = launch_rows<DH, 3>(c, p, KF, k, nullptr, nullptr, nullptr, w, omega, nullptr, w.dST, nullptr, dv, nullptr, nullptr, st);
    if (e != hipSuccess) return e;
    return launch_rows<DH, 2>(c, p, KF, k, v, nullptr, nullptr, w, omega, w.dSx, nullptr, nullptr, dk, nullptr, w.partK, st);
  };
  auto query_side = [&]() {
    return ln ? launch_rows<DH, 1>(c, p, QF, q, w.dN, w.ones, w.dD, w, omega, w.Sx, nullptr, nullptr, dq, nullptr, w.partQ, st, &nv)
              : launch_rows<DH, 1>(c, p, QF, q, dout, D, w.dD, w, omega, w.Sx, nullptr, nullptr, dq, nullptr, w.partQ, st);
  };
  // K side first: the Q-side kernel then is the last writer of a large tensor before the pass
  // that adds the pooled-query term to dQ, which finds part of dQ still in the last-level cache.
  const bool q_first = one_bits_buffer(c);
  if ((q_first && query_side() != hipSuccess) || key_side() != hipSuccess || (!q_first && query_side() != hipSuccess)) return WERSA_ERR_LAUNCH;
  const bool deep = c.L > kTileL;
  if (deep) {   // levels above 6: addends of dQ and dK and the bands' extra row, from the tile sums
    auto go = [&](auto kern, size_t lds) {
      WERSA_STAGE("wersa_coarse_bwd", st, kern<<<dim3(slices, 2, DH / kCoarseCols), 1024, lds, st>>>(
          w.gsumQ, w.gsumK, w.tileQ, w.tileK, w.coef, (c.n + 63) / 64, DH, c.L, w.pyr, w.gaddQ, w.gaddK, w.partQ, w.partK, p.rowsWgs));
    };
    if (const size_t lds = pyramid_in_lds(&coarse_bwd_kernel<true>, (c.n + 63) / 64, 2)) go(&coarse_bwd_kernel<true>, lds);
    else go(&coarse_bwd_kernel<false>, 0);
  }
  WERSA_STAGE("gate_bwd_slice_kernel", st,
              gate_bwd_slice_kernel<<<slices, kGateBwdThreads, 0, st>>>(w.partQ, w.partK, deep ? p.rowsWgs + DH / kCoarseCols : p.rowsWgs, c.L,
                                                           c.d, c.H, s, gate_w, scale_w, w.dF, w.dlogit, w.dqbar,
                                                           (c.flags & WERSA_FLAG_POOLED_GATE) ? 1 : 0, w.coef));
  const GateBwdParams gp{w.dF, w.dlogit, s, qbar, w.dDpart, slices * (ln ? p.chunksL : p.chunksC), c.B, c.H, c.L, c.d, c.eps, w.scalars,
                         dgate_w, dgate_b, dscale_w, dsigma, gate_bwd_params_blocks(c.H, c.L, c.d)};
  const int64_t chunks = (int64_t)c.n * (DH / 8);
  const dim3 agrid = with_gate_bwd_params(dim3((unsigned)((chunks + 1023) / 1024), slices, deep ? 2 : 1), gp);
  if (deep) {
    WERSA_STAGE("wersa_add_pooled", st,
                (add_pooled_kernel<DH, true><<<agrid, 256, 0, st>>>(dq, tv, w.dqbar, c.n, 1.0f / (float)c.n, w.gaddQ, dk, w.gaddK, gp)));
  } else {
    WERSA_STAGE("wersa_add_pooled", st,
                (add_pooled_kernel<DH, false><<<agrid, 256, 0, st>>>(dq, tv, w.dqbar, c.n, 1.0f / (float)c.n, nullptr, nullptr, nullptr, gp)));
  }
  return hipGetLastError() == hipSuccess ? WERSA_OK : WERSA_ERR_LAUNCH;
}

// Rows too far apart for a buffer with a partial last block (kMaxBufferStride), or, in the backward, for the gradient kernels' 32-bit offsets
// (kMaxGroupStride): the tensors are copied to dense ones in the workspace and the results back.  Rows of more than 32 MB: there are
// never many.
bool rows_far_apart(const wersa_desc &c, int for_backward) {
  return c.n % 64 ? c.stride_n > kMaxBufferStride : for_backward && c.stride_n > kMaxGroupStride;
}
wersa_desc dense_desc(const wersa_desc &c) {
  wersa_desc o = c;
  o.stride_n = c.d;
  o.stride_h = (int64_t)c.n * c.d;
  o.stride_b = c.H * o.stride_h;
  return o;
}
size_t dense_floats(const wersa_desc &c) { return ((size_t)c.B * c.H * c.n * c.d / 2 + 63) / 64 * 64; }   // of one bf16 tensor
struct CopyJob {
  const bf16_t *src[5];
  bf16_t *dst[5];
};
__global__ __launch_bounds__(256) void copy_rows_kernel(CopyJob job, View vs, View vd, int n, int d) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int pieces = d / 8, slice = blockIdx.y;
  if (e >= (int64_t)n * pieces) return;
  const int t = (int)(e / pieces), c = (int)(e % pieces) * 8;
  *reinterpret_cast<u16x8 *>(job.dst[blockIdx.z] + vd.slice_base(slice) + (int64_t)t * vd.sn + c) =
      *reinterpret_cast<const u16x8 *>(job.src[blockIdx.z] + vs.slice_base(slice) + (int64_t)t * vs.sn + c);
}
void copy_rows(const wersa_desc &from, const wersa_desc &to, const CopyJob &job, int count, hipStream_t st) {
  const View vs{from.stride_b, from.stride_h, from.stride_n, from.H}, vd{to.stride_b, to.stride_h, to.stride_n, to.H};
  const int64_t pieces = (int64_t)from.n * (from.d / 8);
  WERSA_STAGE("wersa_copy_rows", st, copy_rows_kernel<<<dim3((unsigned)((pieces + 255) / 256), from.B * from.H, count), 256, 0, st>>>(
      job, vs, vd, from.n, from.d));
}

}  // namespace

bool fast_haar_filter_supported(const wersa_desc &c, const void *x, const void *xf) {
  return c.dtype == WERSA_BF16 && c.L <= kTileL && c.d % 8 == 0 && c.stride_n % 8 == 0 && c.stride_h % 8 == 0 &&
         c.stride_b % 8 == 0 && ((uintptr_t)x % 16) == 0 && ((uintptr_t)xf % 16) == 0;
}

wersa_status fast_haar_filter(const wersa_desc &c, const void *x, const float *filt, void *xf, hipStream_t st) {
  const View tv{c.stride_b, c.stride_h, c.stride_n, c.H};
  const dim3 grid((unsigned)((c.n + 63) / 64), (unsigned)((c.d + 63) / 64), (unsigned)(c.B * c.H));
  WERSA_STAGE("wersa_haar_filter_bf16", st,
              haar_filter_bf16_kernel<<<grid, 256, 0, st>>>((const bf16_t *)x, (bf16_t *)xf, tv, c.n, c.d, filt, c.L));
  return hipGetLastError() == hipSuccess ? WERSA_OK : WERSA_ERR_LAUNCH;
}

bool fast_supported(const wersa_desc &c) {
  if (c.dtype != WERSA_BF16 || (c.d != 64 && c.d != 128) || c.m % 128 || c.stride_n % 8 || c.stride_h % 8 || c.stride_b % 8)
    return false;
  // (the copies do not take a call away from wersa_forward_static)
  return !rows_far_apart(c, 0) || fast_workspace_bytes(c, 0) <= kStaticScratchBytes ||
         (split_workspace_bytes(c, 0) > kStaticScratchBytes && generic_workspace_bytes(c, 0) > kStaticScratchBytes);
}

size_t fast_workspace_bytes(const wersa_desc &c, int for_backward) {
  size_t floats = (size_t)fast_ws(c, fast_plan(c), for_backward, nullptr, nullptr).total;
  if (rows_far_apart(c, for_backward)) floats += (for_backward ? 8 : 4) * dense_floats(c);
  return floats * sizeof(float);
}

wersa_status fast_forward(const wersa_desc &c, const void *q, const void *k, const void *v,
                          const void *omega_rf, const float *sigma, const float *gate_w,
                          const float *gate_b, const float *scale_w, void *out, float *saved,
                          float *ws, hipStream_t st, const PooledSums *pooled) {
  if (rows_far_apart(c, 0)) {
    const wersa_desc dc = dense_desc(c);
    const size_t one = dense_floats(c);
    float *p = ws + fast_workspace_bytes(dc, 0) / sizeof(float);
    bf16_t *t[4];
    for (int i = 0; i < 4; ++i) t[i] = (bf16_t *)(p + i * one);
    copy_rows(c, dc, CopyJob{{(const bf16_t *)q, (const bf16_t *)k, (const bf16_t *)v}, {t[0], t[1], t[2]}}, 3, st);
    const wersa_status rc = fast_forward(dc, t[0], t[1], t[2], omega_rf, sigma, gate_w, gate_b, scale_w, t[3], saved, ws, st, nullptr);
    if (rc != WERSA_OK) return rc;
    copy_rows(dc, c, CopyJob{{t[3]}, {(bf16_t *)out}}, 1, st);
    return hipGetLastError() == hipSuccess ? WERSA_OK : WERSA_ERR_LAUNCH;
  }
  if (c.d == 64)
    return fast_forward_t<64>(c, (const bf16_t *)q, (const bf16_t *)k, (const bf16_t *)v,
                              (const bf16_t *)omega_rf, sigma, gate_w, gate_b, scale_w, (bf16_t *)out,
                              saved, ws, st, pooled);
  return fast_forward_t<128>(c, (const bf16_t *)q, (const bf16_t *)k, (const bf16_t *)v,
                             (const bf16_t *)omega_rf, sigma, gate_w, gate_b, scale_w, (bf16_t *)out,
                             saved, ws, st, pooled);
}

wersa_status fast_backward(const wersa_desc &c, const void *q, const void *k, const void *v,
                           const void *omega_rf, const float *sigma, const float *gate_w,
                           const float *scale_w, const void *out, const void *dout,
                           const float *saved, void *dq, void *dk, void *dv, float *dgate_w,
                           float *dgate_b, float *dscale_w, float *dsigma, float *ws,
                           hipStream_t st) {
  if (rows_far_apart(c, 1)) {
    const wersa_desc dc = dense_desc(c);
    const size_t one = dense_floats(c);
    float *p = ws + fast_workspace_bytes(dc, 1) / sizeof(float);
    bf16_t *t[8];
    for (int i = 0; i < 8; ++i) t[i] = (bf16_t *)(p + i * one);
    copy_rows(c, dc, CopyJob{{(const bf16_t *)q, (const bf16_t *)k, (const bf16_t *)v, (const bf16_t *)out, (const bf16_t *)dout},
                             {t[0], t[1], t[2], t[3], t[4]}}, 5, st);
    const wersa_status rc = fast_backward(dc, t[0], t[1], t[2], omega_rf, sigma, gate_w, scale_w, t[3], t[4], saved, t[5], t[6],
                                          t[7], dgate_w, dgate_b, dscale_w, dsigma, ws, st);
    if (rc != WERSA_OK) return rc;
    copy_rows(dc, c, CopyJob{{t[5], t[6], t[7]}, {(bf16_t *)dq, (bf16_t *)dk, (bf16_t *)dv}}, 3, st);
    return hipGetLastError() == hipSuccess ? WERSA_OK : WERSA_ERR_LAUNCH;
  }
  if (c.d == 64)
    return fast_backward_t<64>(c, (const bf16_t *)q, (const bf16_t *)k, (const bf16_t *)v,
                               (const bf16_t *)omega_rf, sigma, gate_w, scale_w, (const bf16_t *)out,
                               (const bf16_t *)dout, saved, (bf16_t *)dq, (bf16_t *)dk, (bf16_t *)dv,
                               dgate_w, dgate_b, dscale_w, dsigma, ws, st);
  return fast_backward_t<128>(c, (const bf16_t *)q, (const bf16_t *)k, (const bf16_t *)v,
                              (const bf16_t *)omega_rf, sigma, gate_w, scale_w, (const bf16_t *)out,
                              (const bf16_t *)dout, saved, (bf16_t *)dq, (bf16_t *)dk, (bf16_t *)dv,
                              dgate_w, dgate_b, dscale_w, dsigma, ws, st);
}

}  // namespace wersa
