// fp32 contractions on the bf16 matrix pipe, and the operand helpers they share.
//
// A finite fp32 value is the exact sum of three bf16 values: its upper 16 bits, the upper 16 bits of what is
// left, and the rest (8 + 8 + 8 significand bits).  A product with a value that is bf16 to begin with is then
// three matrix instructions whose products are exact, accumulated in fp32 -- at 16 times the rate of the fp32
// matrix instruction and without its restriction to two contraction indices.
// (Truncation, not rounding: the upper part of a value next to the top of the range must not round to infinity.)
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

// The three parts of eight values, highest first.
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

__device__ __forceinline__ float bf_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {  // two fp32 -> packed bf16, RNE
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float exp2_fast(float v) { return __builtin_amdgcn_exp2f(v); }

// Transposed LDS read (ds_read_b64_tr_b16).  Inside each group of 16 lanes, lane j names four consecutive
// 16-bit elements -- a quad --; lane i receives element i % 4 of the quads of lanes i/4, 4 + i/4, 8 + i/4 and
// 12 + i/4.  With quad j of a group at row j/4, four columns per j%4, lane i gets four rows of one column: the
// contraction index of a row-major [token][column] tile becomes contiguous per lane.
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x2 lds_read_tr(const uint16_t *p) {
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p));
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
template <int kPolicy = 0>
__device__ __forceinline__ void buf_store16(Rsrc r, uint32_t voff, u32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, voff, 0, kPolicy);
}

// The MFMA writes row m of a 32-row result to lane group kg = (m >> 2) & 1, element 4 (m >> 3) + (m & 3).
// Giving row m the column 16 ((m >> 2) & 1) + 4 (m >> 3) + (m & 3) makes every lane own 16 consecutive columns.
__device__ __forceinline__ int pi_of_row(int m) { return 16 * ((m >> 2) & 1) + 4 * (m >> 3) + (m & 3); }

}  // namespace split
}  // namespace ssd
