// fp32 contractions on the bf16 matrix pipe, and the operand helpers they share.
//
// A finite fp32 value is the exact sum of three bf16 values (8 + 8 + 8 significand bits): its leading part, the leading
// part of what is left, and the rest.  The method is published: Henry, Tang and Heinecke, "Leveraging the bfloat16
// artificial intelligence datatype for higher-precision computations" (2019).  A product with a value that is bf16 to
// begin with is then three matrix instructions whose products are exact, accumulated in fp32 -- at 16 times the rate
// of the fp32 matrix instruction and without its restriction to two contraction indices.
#pragma once

#include "ssd_internal.hpp"

namespace ssd {
namespace split {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// One operand of v_mfma_f32_32x32x16_bf16: 8 bf16 per lane.
union Op {
  bf16x8 v;
  u32x4 q;
  u32x2 h[2];
  uint32_t u[4];
};

// D(32x32) += A(32x16) * B(16x32).  Lane (r = lane%32, kg = lane/32) supplies A[r][8kg..8kg+7] and
// B[8kg..8kg+7][r]; it receives D[(i/4)*8 + 4kg + i%4][r] in element i.
__device__ __forceinline__ f32x16 mfma(const Op &a, const Op &b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, b.v, c, 0, 0, 0);
}

// The three parts of eight values, highest first, by truncation (a value next to the top of the range must not round to
// an infinity).
__device__ __forceinline__ void split3(const float v[8], Op o[3]) {
  uint32_t b[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) b[j] = __float_as_uint(v[j]);
#pragma unroll
  for (int part = 0; part < 3; ++part) {
#pragma unroll
    for (int k = 0; k < 4; ++k) o[part].u[k] = __builtin_amdgcn_perm(b[2 * k + 1], b[2 * k], 0x07060302u);
    if (part < 2) {
#pragma unroll
      for (int j = 0; j < 8; ++j) b[j] = __float_as_uint(__uint_as_float(b[j]) - __uint_as_float(b[j] & 0xffff0000u));
    }
  }
}

// D(16x16) += A(16x32) * B(32x16).  Lane (r = lane%16, kg = lane/16) supplies A[r][8kg..8kg+7] and B[8kg..8kg+7][r];
// it receives D[4kg + i][r] in element i.
__device__ __forceinline__ f32x4 mfma16(const Op &a, const Op &b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, c, 0, 0, 0);
}

__device__ __forceinline__ float bf_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {  // two fp32 -> packed bf16, RNE
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
// The parts for a product in which BOTH factors are split: six products stand for the nine (mid lo, lo mid and lo lo are
// left out).  Each part is rounded to nearest, so that mid is at most 2^-8 and lo 2^-17 of the value's leading bit: what
// is left out has no preferred sign and is at most 2^-24 of the product, the rounding of an fp32 product itself (with a
// truncated leading part up to 2^-22).  A state of one token, which is one product per element, is then 2.4 units of
// 2^-24 off at most (4.3), 0.58 rms (0.69); 1.0 and 0.42 from the fp32 matrix instruction.  Sums of many products are
// no further off than with that instruction, since they are rounded less often: 0.84 of its error in the final state of
// 21 drawn prompts, 1.00 in y.  The two products left out cost 2 us more of 52 (2048 tokens x 24 heads) and change none of
// these sums.  (Values of 2^30 and more don't come here; see out_of_range.)  W = values, a multiple of 2; part p of
// values 2k, 2k+1 goes to out[p][k].
template <int W>
__device__ __forceinline__ void split3_even(const float *v, uint32_t (*out)[W / 2]) {
#pragma unroll
  for (int k = 0; k < W / 2; ++k) {
    const uint32_t h = pack2(v[2 * k], v[2 * k + 1]);
    out[0][k] = h;
    const float ra = v[2 * k] - bf_lo(h), rb = v[2 * k + 1] - bf_hi(h);
    const uint32_t m = pack2(ra, rb);
    out[1][k] = m;
    out[2][k] = pack2(ra - bf_lo(m), rb - bf_hi(m));
  }
}
__device__ __forceinline__ void split3_even(const float v[8], Op o[3]) {
  uint32_t t[3][4];
  split3_even<8>(v, t);
#pragma unroll
  for (int p = 0; p < 3; ++p)
#pragma unroll
    for (int k = 0; k < 4; ++k) o[p].u[k] = t[p][k];
}
// The larger, and the smaller, of two values, or NaN if one is.
__device__ __forceinline__ float max_or_nan(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ float min_or_nan(float a, float b) { return __builtin_elementwise_minimum(a, b); }
// The six products, smallest first.
constexpr int kPairA[6] = {1, 2, 0, 1, 0, 0}, kPairB[6] = {1, 0, 2, 0, 1, 0};
__device__ __forceinline__ f32x16 mfma6(const Op a[3], const Op b[3], f32x16 c) {
#pragma unroll
  for (int t = 0; t < 6; ++t) c = mfma(a[kPairA[t]], b[kPairB[t]], c);
  return c;
}

__device__ __forceinline__ float exp2_fast(float v) { return __builtin_amdgcn_exp2f(v); }

// The log2 decays of a block's steps, so that differences of their prefix sums -- the decay between two steps -- come
// out right also behind steps that decay everything away.  A step is cut off (cut_decay) and taken apart into a multiple
// of 2^-8, whose sums over 32 steps are exact (at most 5120, 21 bits), and the rest, whose sums stay below 2^-4 (error
// 2^-27).
__device__ __forceinline__ float coarse_part(float d) { return __builtin_rintf(d * 256.f) * 0.00390625f; }

// Transposed LDS read (ds_read_b64_tr_b16).  Inside each group of 16 lanes, lane j names four consecutive
// 16-bit elements -- a quad --; lane i receives element i % 4 of the quads of lanes i/4, 4 + i/4, 8 + i/4 and
// 12 + i/4.  With quad j of a group at row j/4, four columns per j%4, lane i gets four rows of one column: the
// contraction index of a row-major [token][column] tile becomes contiguous per lane.
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x2 lds_read_tr(const uint16_t *p) {
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p));
}

// Sums over 32 lanes (both halves of the wave hold the same values), by lane moves of the vector ALU inside rows of
// 16 lanes and one row's total for the other.  (Every lane must be active where a move is evaluated.)
template <int kCtrl>
__device__ __forceinline__ float dpp_or_zero(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xf, 0xf, true));
}
__device__ __forceinline__ float read_lane(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ float prefix32(float v) {  // the lanes up to and including this one
  v += dpp_or_zero<0x111>(v);  // row_shr:1
  v += dpp_or_zero<0x112>(v);
  v += dpp_or_zero<0x114>(v);
  v += dpp_or_zero<0x118>(v);
  const float first = read_lane(v, 15);
  return v + ((threadIdx.x & 16) ? first : 0.f);
}
__device__ __forceinline__ float suffix32(float v) {  // the lanes behind this one
  const float over = read_lane(v, 16), next = dpp_or_zero<0x101>(v);  // row_shl:1
  v = (threadIdx.x & 31) == 15 ? over : next;
  v += dpp_or_zero<0x101>(v);
  v += dpp_or_zero<0x102>(v);
  v += dpp_or_zero<0x104>(v);
  v += dpp_or_zero<0x108>(v);
  const float second = read_lane(v, 16);
  return v + ((threadIdx.x & 16) ? 0.f : second);
}

// Buffer addressing: loads beyond the descriptor's size return zero, stores beyond it are dropped.
using Rsrc = __amdgpu_buffer_rsrc_t;
__device__ __forceinline__ Rsrc make_rsrc(const void *base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, static_cast<int>(bytes), 0x00020000);
}
// (kPolicy: the instruction's cache-policy field, 0 = default, 2 = nt)
template <int kPolicy = 0>
__device__ __forceinline__ u32x4 buf_load16(Rsrc r, uint32_t voff) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, kPolicy);
}
__device__ __forceinline__ u32x2 buf_load8(Rsrc r, uint32_t voff) { return __builtin_amdgcn_raw_buffer_load_b64(r, voff, 0, 0); }
template <int kPolicy = 0>
__device__ __forceinline__ void buf_store16(Rsrc r, uint32_t voff, u32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, voff, 0, kPolicy);
}

// The MFMA writes row m of a 32-row result to lane group kg = (m >> 2) & 1, element 4 (m >> 3) + (m & 3).
// Giving row m the column 16 ((m >> 2) & 1) + 4 (m >> 3) + (m & 3) makes every lane own 16 consecutive columns.
__device__ __forceinline__ int pi_of_row(int m) { return 16 * ((m >> 2) & 1) + 4 * (m >> 3) + (m & 3); }

}  // namespace split
}  // namespace ssd
