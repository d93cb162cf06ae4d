// Prefill for fp32 io (x, B, C, y in fp32) on the bf16 matrix pipe: every fp32 operand is split into three bf16
// parts (ssd_split_bf16.hpp) and a product of two of them is six matrix instructions, accumulated in fp32 -- fp32
// accuracy at 16 / 6 times the rate of the fp32 matrix instruction, and the prompt cut up over the whole chip.
// Shapes: headdim a multiple of 32, dstate a multiple of 8 up to 128.
//
// The chunked algorithm (Alg. 1; Eq. 3) on blocks of 32 tokens, with cs_l the block-relative inclusive prefix sum of
// dt*A and S the state entering the block:
//     G[l][s] = C_l . B_s                                                     (s <= l; once per workgroup)
//     y[l][p] = exp(cs_l) sum_n C[l][n] S[p][n] + sum_s (G[l][s] dt_s exp(cs_l - cs_s)) x[s][p] + D x[l][p]
//     S'      = exp(cs_31) S + sum_s (dt_s exp(cs_31 - cs_s) x[s][p]) B[s][n]
// The mask is applied on the scores in registers.  Its exponents are differences of prefix sums in two parts, cs = ch +
// cl (cut_decay, coarse_part): the weights are (dt_s exp(-cl_s)) (exp(cl_l) exp(ch_l - ch_s)), right to some 2^-23 for
// any step sizes.
//
// A block whose x, B, C or entering state holds an infinity, a NaN or a value of 2^30 and more (or a step size of 2^40)
// would lose what the recurrence keeps -- an infinity has no parts, a masked score of zero times it is a NaN, sums of
// products overflow --; from there on its workgroup applies the recurrence as it stands, in the same registers.
//
// One wave per slice of 32 headdim columns x dstate, its state in MFMA accumulators; four slices of one B/C group
// per workgroup, which stages the split B and C once for them.  Layouts as in ssd_decode_steps_mfma.hip.
// The sequence is cut into S segments: a states-only launch computes every segment's end state from zero, a pass
// chains them (Alg. 1, "InterChunkRecurrence"), and the full launch walks every segment from its entering state.  The
// states between the launches lie in the caller's workspace where it holds that many -- it is sized for one per chunk,
// 8 for 2048 tokens at a chunk length of 256 where 16 are wanted --, and otherwise in y, each in the rows of the segment
// it enters: a wave reads the state of its slice and later writes its outputs there, and no other wave touches those
// columns.  A segment then has at least as many tokens as a state slice has 128-byte pieces.
// With one segment only the full launch runs; `sub` workgroups may then share the sequence, each first carrying the
// state over the blocks of the ones before it (a third of a block's work, no output).
// Where the states-only launch leaves CUs idle, workgroups of their own split B and C there and form the scores, once for all
// heads (make_image); the full launch then copies a block's image to LDS.
// Bound: issue.  A block of four slices without an image takes 5.2 us where one workgroup has the chip, 7.3 with one per CU, 10.3
// with two each (dstate 128); the matrix instructions are 1.6 of it (3840 cycles a wave), about 1150 vector instructions a wave
// (the splits: 700) come between them.  One wave on a SIMD issues a vector instruction every 5 cycles and they hardly overlap with
// the matrix instructions (eight of them and one of those: 59 cycles, 32 by itself; 49 with two waves), so that operands
// read from LDS a step ahead changed nothing.  Of a block's 12700 cycles (2048 tokens x 24 heads, by time stamps)
// staging is 3270, the scores 810; with an image 11600, of which copying it is 3040.  Two waves per slice (half of dstate
// each, outputs summed through LDS) were 6 % faster alone and half as fast for two; matrix and vector instructions
// interleaved by hand or by scheduling groups 15 % slower and more (spills).
// Measured against the fp32 matrix instruction kernel (ssd_prefill_mfma_f32.hip), us: 2048 tokens x 24 heads x 64 x 128
// 108.7 / 49.0 (12 of it the chain and the gaps), 8 such prompts 504 / 191, 3 x 2428 x 20 190 / 90, 2 x 3593 x 11 x 64 x
// 16 70 / 43, 4096 x 4 x 32 x 16 55 / 37; final state against 64 bits 1.4e-7 / 9.5e-8, y
// 2.6e-8 both.  Of it the checks for values out of range take 1 us of the first, the leading parts rounded instead of cut
// off 0.7, the mask's sums in two parts 0.3.
#include <type_traits>

#include "ssd_split_bf16.hpp"

namespace ssd {
namespace {
using namespace split;

constexpr int kTok = 32;             // tokens per block
constexpr int kCols = 32;            // headdim columns per wave
constexpr int kWaves = 4;
constexpr int kThr = 64 * kWaves;
constexpr int kXStride = kCols + 8;  // floats per row of an x tile (four rows apart: 32 of the 64 banks)
constexpr int kGStride = kTok + 4;   // floats per row of the score tile
constexpr int kTurnStride = 32 + 4;  // floats per row of a state tile on its way through LDS
constexpr float kLog2e = 1.4426950408889634f;
constexpr uint32_t kNowhere = 0xFFFFFF00u;  // an offset beyond any descriptor

struct SplitParams {
  const float *x, *dt, *A, *B, *C, *D, *h0;
  float *y, *final_state;
  float *slots;                    // states entering the segments, [batch row][head][segment]; nullptr: they lie in y
  float *decay;                    // decay: log2 of every segment's total decay, [batch row][head][segment]
  int T, H, P, N, G, Bt, hpg;
  int nslice, cpg;               // slices per group; workgroups per group
  uint32_t S_inv, cpg_inv, rows_inv, G_inv, per_head_inv, sub_inv, nblocks_inv;  // for quotient(); rows: Bt * G, per head: P / 32
  int S;                         // segments per sequence; segment s begins at block segment_begin(s)
  int sub, sub_blocks;           // S = 1: workgroups that share the sequence, output blocks of each
  uint8_t *images;               // with several segments: [batch row][group][block] as SplitLds::kImage; nullptr: none
  int slot0;                     // the first segment starts from its slot in y, not from h0 (which final_state aliases)
  DtXform dtx;
  int dt_plain;                    // the step sizes are used as given
};

inline int segment_begin(int s, int S, int nblocks) { return static_cast<int>(static_cast<long long>(s) * nblocks / S); }
// (A division of 64 bits is some hundred instructions, and the pass over the states had two per segment: 8.1 -> 6.8 us at 2048
// tokens x 24 heads in 16 segments.  The product is below 2^31, see split_plan.)
__device__ __forceinline__ int segment_begin(int s, const SplitParams &p, int nblocks) {
  return quotient(static_cast<uint32_t>(s) * static_cast<uint32_t>(nblocks), p.S, p.S_inv);
}
// The state slice of (batch row b, head h, columns p0 ..) that enters segment s: 32 rows (headdim) of NT pieces of 32
// floats.  In the workspace they lie as in any state; in y, piece (c, nt) is the 32 columns of y's row number c NT + nt
// of the segment.
__device__ __forceinline__ float *state_slot(const SplitParams &p, int b, int h, int p0, int s, int nblocks) {
  if (p.slots != nullptr) return p.slots + (((static_cast<size_t>(b) * p.H + h) * p.S + s) * p.P + p0) * p.N;
  const size_t tok = static_cast<size_t>(b) * p.T + static_cast<size_t>(segment_begin(s, p, nblocks)) * kTok;
  return p.y + (tok * p.H + h) * p.P + p0;
}

template <int NT, bool kStatesOnly>
struct SplitLds {
  static constexpr int kN = 32 * NT;
  static constexpr int kRow = kN + 8;                       // bf16 elements per row of a part of B or C
  static constexpr int kPart = kTok * kRow;
  static constexpr int kB = 3 * kPart * 2, kBC = 2 * kB;    // bytes
  static constexpr int kG = kTok * kGStride * 4;
  // The image of a block: the parts of B and C, the scores, and whether a value is out of range (an int behind the scores).
  static constexpr int kFlag = kBC + kG, kImage = (kFlag + 4 + 4095) / 4096 * 4096, kImagePieces = kImage / (16 * kThr);
  static constexpr int kX = kWaves * kTok * kXStride * 4, kXAt = kStatesOnly ? kB : kImage;
  static constexpr int kTurn = kWaves * kCols * kTurnStride * 4;
  static constexpr int kTiles = kXAt + kX > kBC ? kXAt + kX : kBC;  // (the states-only launch also makes the images)
  static constexpr int kBytes = kTiles > kTurn ? kTiles : kTurn;
};

// The largest magnitude of four values and one seen before, or NaN if one is (two v_maximum3), and whether it is outside
// the range of the contractions.
__device__ __forceinline__ float larger(float seen, f32x4 v) {
  return max_or_nan(max_or_nan(max_or_nan(max_or_nan(seen, fabsf(v.x)), fabsf(v.y)), fabsf(v.z)), fabsf(v.w));
}
__device__ __forceinline__ bool out_of_range(float seen) { return !(seen < 0x1p30f); }

// Descriptor of the rows of block j that exist, `width` bytes of each.
__device__ __forceinline__ Rsrc block_rows(const uint8_t *base, uint32_t row, uint32_t width, int j, int T) {
  const int n = min(kTok, T - j * kTok);
  return make_rsrc(base + static_cast<size_t>(j) * kTok * row, n > 0 ? (n - 1) * row + width : 0u);
}
// Four values of 16-byte piece `item` of a B or C tile, split into its three parts; the columns of a group of 16 in the order
// 0-3, 8-11, 4-7, 12-15.
template <int NT>
__device__ __forceinline__ void put_parts(uint16_t *tile, int item, f32x4 v) {
  using L = SplitLds<NT, false>;
  const int c4 = item % (L::kN / 4), dst = (item / (L::kN / 4)) * L::kRow + 16 * (c4 >> 2) + 8 * (c4 & 1) + 4 * ((c4 >> 1) & 1);
  const float v4[4] = {v.x, v.y, v.z, v.w};
  uint32_t t[3][2];
  split3_even<4>(v4, t);
#pragma unroll
  for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x2 *>(tile + q * L::kPart + dst) = u32x2{t[q][0], t[q][1]};
}
// A quarter of the scores (16 tokens s of `sb`, 16 tokens l of `sc`): lane (tj = lane % 16, lane / 16) gets l = tj, four s.
template <int NT>
__device__ __forceinline__ f32x4 scores_quarter(const uint16_t *sb, const uint16_t *sc) {
  using L = SplitLds<NT, false>;
  f32x4 acc = {};
#pragma unroll
  for (int kk = 0; kk < L::kN / 32; ++kk) {
    Op bq[3], cq[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      bq[q].q = *reinterpret_cast<const u32x4 *>(sb + q * L::kPart + 32 * kk);
      cq[q].q = *reinterpret_cast<const u32x4 *>(sc + q * L::kPart + 32 * kk);
    }
#pragma unroll
    for (int t = 0; t < 6; ++t) acc = mfma16(bq[kPairA[t]], cq[kPairB[t]], acc);
  }
  return acc;
}

// The image of block j of batch row and group bg (see SplitLds): what every workgroup of the group would otherwise work out of B
// and C again (2048 tokens x 24 heads: twelve workgroups a block, 12700 cycles each, 11600 with the image).  Made by workgroups of the
// states-only launch, which leaves CUs idle.
template <int NT>
__device__ __forceinline__ void make_image(const SplitParams &p, uint8_t *smem, int *s_odd, int bg, int j, int nblocks) {
  using L = SplitLds<NT, false>;
  constexpr int N = L::kN, kPieces = kTok * (N / 4) / kThr;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint16_t *const sB = reinterpret_cast<uint16_t *>(smem), *const sC = sB + 3 * L::kPart;
  const uint32_t brow = static_cast<uint32_t>(p.G) * p.N * 4;
  const size_t first = (static_cast<size_t>(bg / p.G) * p.T * p.G + bg % p.G) * p.N;
  const Rsrc rB = block_rows(reinterpret_cast<const uint8_t *>(p.B + first), brow, p.N * 4, j, p.T);
  const Rsrc rC = block_rows(reinterpret_cast<const uint8_t *>(p.C + first), brow, p.N * 4, j, p.T);
  u32x4 b[kPieces], c[kPieces];
#pragma unroll
  for (int k = 0; k < kPieces; ++k) {
    const int item = tid + kThr * k, n0 = 4 * (item % (N / 4));
    const uint32_t at = n0 < p.N ? static_cast<uint32_t>(item / (N / 4)) * brow + 4 * n0 : kNowhere;
    b[k] = buf_load16(rB, at);
    c[k] = buf_load16(rC, at);
  }
  if (tid == 0) *s_odd = 0;
  float seen = 0.f;
#pragma unroll
  for (int k = 0; k < kPieces; ++k) {
    const f32x4 vb = __builtin_bit_cast(f32x4, b[k]), vc = __builtin_bit_cast(f32x4, c[k]);
    put_parts<NT>(sB, tid + kThr * k, vb);
    put_parts<NT>(sC, tid + kThr * k, vc);
    seen = larger(larger(seen, vb), vc);
  }
  __syncthreads();
  if (__builtin_amdgcn_ballot_w64(out_of_range(seen)) != 0 && lane == 0) *s_odd = 1;
  uint8_t *const image = p.images + (static_cast<size_t>(bg) * nblocks + j) * L::kImage;
  for (int at = 16 * tid; at < L::kBC; at += 16 * kThr)
    *reinterpret_cast<u32x4 *>(image + at) = *reinterpret_cast<const u32x4 *>(smem + at);
  if (wave < 3) {
    const int sq = wave >> 1, lq = wave > 0 ? 1 : 0, tj = lane & 15, at = tj * L::kRow + 8 * (lane >> 4);
    const f32x4 acc = scores_quarter<NT>(sB + 16 * sq * L::kRow + at, sC + 16 * lq * L::kRow + at);
    *reinterpret_cast<f32x4 *>(image + L::kBC + ((16 * lq + tj) * kGStride + 16 * sq + 4 * (lane >> 4)) * 4) = acc;
  }
  __syncthreads();
  if (tid == 0) *reinterpret_cast<int *>(image + L::kFlag) = *s_odd;
}

// kImages: the full launch where the states-only launch has left the images of its blocks.
template <int NT, bool kStatesOnly, bool kImages = false>
__global__ __launch_bounds__(kThr, 2) void split_f32_kernel(const SplitParams p) {
  static_assert(!(kStatesOnly && kImages), "the states-only launch makes the images");
  using L = SplitLds<NT, kStatesOnly>;
  constexpr int N = L::kN;                       // dstate padded to whole tiles
  constexpr int kPieces = kTok * (N / 4) / kThr;  // 16-byte pieces of a B or C tile per thread
  __shared__ __align__(16) uint8_t smem[L::kBytes];
  __shared__ __align__(16) float s_ch[kWaves][kTok], s_in[kWaves][kTok], s_w[kWaves][kTok];
  __shared__ int s_odd;                                     // a value outside the range of the contractions was met
  uint16_t *const sB = reinterpret_cast<uint16_t *>(smem);  // three parts of B, then of C: [token][n]
  uint16_t *const sC = sB + 3 * L::kPart;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, kg = lane >> 5;
  float *const sX = reinterpret_cast<float *>(smem + L::kXAt) + wave * (kTok * kXStride);  // x [token][column], this wave's
  float *const sG = reinterpret_cast<float *>(smem + L::kBC);                              // scores [l][s]

  // ---- which slice, segment and blocks ----
  const int nblocks = (p.T + kTok - 1) / kTok;
  int wg = blockIdx.x;
  if constexpr (kStatesOnly) {
    const int n_images = p.images != nullptr ? nblocks * p.Bt * p.G : 0;
    if (wg < n_images) {
      const int row = quotient(wg, nblocks, p.nblocks_inv);
      make_image<NT>(p, smem, &s_odd, row, wg - row * nblocks, nblocks);
      return;
    }
    wg -= n_images;
  }
  const int item = quotient(wg, p.cpg, p.cpg_inv), col = wg - item * p.cpg;
  const int piece = quotient(item, p.Bt * p.G, p.rows_inv), bg = item - piece * (p.Bt * p.G);
  const int b = quotient(bg, p.G, p.G_inv), g = bg - b * p.G;
  const int seg = kStatesOnly || kImages ? piece : quotient(piece, p.sub, p.sub_inv), part = kStatesOnly || kImages ? 0 : piece - seg * p.sub;
  const int j0 = segment_begin(seg, p, nblocks), jend = segment_begin(seg + 1, p, nblocks);
  // the state alone over [j0, j1), everything over [j1, j2)
  const int j1 = kStatesOnly ? jend : min(jend, j0 + part * p.sub_blocks);
  const int j2 = kStatesOnly ? jend : min(jend, j1 + p.sub_blocks);
  if (!kStatesOnly && j1 >= j2) return;  // uniform over the workgroup

  const int slice_raw = kWaves * col + wave;
  const bool live = slice_raw < p.nslice;  // (a wave without a slice repeats the last one and stores nothing)
  const int slice = live ? slice_raw : p.nslice - 1;
  const int per_head = p.P / kCols;
  const int in_group = quotient(slice, per_head, p.per_head_inv);
  const int h = g * p.hpg + in_group, p0 = kCols * (slice - in_group * per_head);
  const size_t bh = static_cast<size_t>(b) * p.H + h;
  const float alog = p.A[h] * kLog2e;
  const float Dh = p.D[h];
  const float dbias = p.dtx.bias != nullptr ? p.dtx.bias[h] : 0.f;

  // ---- addressing: rows (tokens) of x / y, of B / C and of dt ----
  const uint32_t xrow = static_cast<uint32_t>(p.H) * p.P * 4, brow = static_cast<uint32_t>(p.G) * p.N * 4,
                 drow = static_cast<uint32_t>(p.H) * 4;
  const size_t tok0 = static_cast<size_t>(b) * p.T;
  const uint8_t *const xb = reinterpret_cast<const uint8_t *>(p.x) + tok0 * xrow + (static_cast<size_t>(h) * p.P + p0) * 4;
  uint8_t *const yb = reinterpret_cast<uint8_t *>(p.y) + tok0 * xrow + (static_cast<size_t>(h) * p.P + p0) * 4;
  const uint8_t *const Bb = reinterpret_cast<const uint8_t *>(p.B) + tok0 * brow + static_cast<size_t>(g) * p.N * 4;
  const uint8_t *const Cb = reinterpret_cast<const uint8_t *>(p.C) + tok0 * brow + static_cast<size_t>(g) * p.N * 4;
  const uint8_t *const db = reinterpret_cast<const uint8_t *>(p.dt) + tok0 * drow + static_cast<size_t>(h) * 4;
  auto rows_of = [&](const uint8_t *base, uint32_t row, uint32_t width, int j) { return block_rows(base, row, width, j, p.T); };

  // ---- data of a block in flight ----
  u32x4 r_b[kImages ? 1 : kPieces], r_c[kStatesOnly || kImages ? 1 : kPieces], r_x[4];
  u32x4 r_img[kImages ? L::kImagePieces : 1];
  float r_dt;
  uint32_t v_bc[kPieces];
#pragma unroll
  for (int k = 0; k < kPieces; ++k) {
    const int item = tid + kThr * k, n0 = 4 * (item % (N / 4));
    v_bc[k] = n0 < p.N ? static_cast<uint32_t>(item / (N / 4)) * brow + 4 * n0 : kNowhere;
  }
  // (with_c, uniform: a block of which only the state is wanted needs no C; its loads are pointed beyond the
  // descriptor, where they cost nothing, rather than put behind a branch)
  auto load_block = [&](int j, bool with_c) __attribute__((always_inline)) {
    if constexpr (kImages) {
      const Rsrc rI = make_rsrc(p.images + (static_cast<size_t>(bg) * nblocks + j) * L::kImage, L::kImage);
#pragma unroll
      for (int k = 0; k < L::kImagePieces; ++k) r_img[k] = buf_load16(rI, 16 * (tid + kThr * k));
    } else {
      const Rsrc rB = rows_of(Bb, brow, p.N * 4, j);
#pragma unroll
      for (int k = 0; k < kPieces; ++k) r_b[k] = buf_load16(rB, v_bc[k]);
    }
    const Rsrc rx = rows_of(xb, xrow, 4 * kCols, j);
#pragma unroll
    for (int k = 0; k < 4; ++k) r_x[k] = buf_load16(rx, static_cast<uint32_t>(8 * k + (lane >> 3)) * xrow + 16 * (lane & 7));
    r_dt = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rows_of(db, drow, 4, j), r * drow, 0, 0));
    if constexpr (!kStatesOnly && !kImages) {
      const Rsrc rC = rows_of(Cb, brow, p.N * 4, j);
#pragma unroll
      for (int k = 0; k < kPieces; ++k) r_c[k] = buf_load16(rC, with_c ? v_bc[k] : kNowhere);
    }
  };

  // ---- the state slice, through LDS into the accumulators: 32 rows of NT pieces of 32 floats, in memory order (row
  //      stride dstate) or in a slot (row stride NT rows of y) ----
  float *const turn = reinterpret_cast<float *>(smem) + wave * (kCols * kTurnStride);
  auto st_off = [&](int nt, int k, bool in_y) {  // byte offset of this lane's 16 bytes of rows 8 k .., tile nt
    const uint32_t row = 8 * k + (lane >> 3);
    const uint32_t at = in_y ? (row * NT + nt) * xrow : row * (p.N * 4u) + 128 * nt;
    return 32 * nt + 4 * (lane & 7) < p.N ? at + 16 * (lane & 7) : kNowhere;
  };
  const uint32_t st_size = kCols * p.N * 4u, slot_size = p.slots != nullptr ? st_size : (kCols * NT - 1) * xrow + 4 * kCols;
  const size_t st_base = (bh * p.P + p0) * p.N;
  f32x16 H[NT];
  if (tid == 0) s_odd = 0;
  bool odd = false;
  if constexpr (kStatesOnly) {
    load_block(j0, false);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) H[nt] = f32x16{};
  } else {
    const bool slot = seg > 0 || p.slot0;
    const float *src = slot ? state_slot(p, b, h, p0, seg, nblocks) : p.h0 != nullptr ? p.h0 + st_base : nullptr;
    const Rsrc rs = make_rsrc(src != nullptr ? src : p.x, src == nullptr ? 0u : slot ? slot_size : st_size);
    u32x4 raw[NT][4];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int k = 0; k < 4; ++k) raw[nt][k] = buf_load16(rs, st_off(nt, k, slot && p.slots == nullptr));
    load_block(j0, j0 == j1);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        *reinterpret_cast<u32x4 *>(turn + (8 * k + (lane >> 3)) * kTurnStride + 4 * (lane & 7)) = raw[nt][k];
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const f32x4 v = *reinterpret_cast<const f32x4 *>(turn + pi_of_row(r) * kTurnStride + 8 * i4 + 4 * kg);
#pragma unroll
        for (int i = 0; i < 4; ++i) H[nt][4 * i4 + i] = v[i];
      }
    }
    float seen[4] = {};
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4)
        seen[i4] = larger(seen[i4], f32x4{H[nt][4 * i4], H[nt][4 * i4 + 1], H[nt][4 * i4 + 2], H[nt][4 * i4 + 3]});
    odd = out_of_range(max_or_nan(max_or_nan(seen[0], seen[1]), max_or_nan(seen[2], seen[3])));
  }

  // LDS addresses of this lane (elements)
  const uint32_t a_c = r * L::kRow + 8 * kg;                                 // C as a 32-row operand, + 16 kk
  const int tj = lane & 15, t_half = (lane >> 4) & 1;                        // transposed reads: quad tj of the group
  const uint32_t a_bt = (4 * kg + (tj >> 2)) * L::kRow + 16 * t_half + 8 * (tj & 1) + 4 * ((tj >> 1) & 1);
  const int sq = wave >> 1, lq = wave > 0 ? 1 : 0;                           // waves 0-2: quarters (0,0), (0,1), (1,1) of the scores
  const uint32_t a_sb = (16 * sq + tj) * L::kRow + 8 * (lane >> 4);          // B, C as 16-row operands, + 32 kk
  const uint32_t a_sc = (16 * lq + tj) * L::kRow + 8 * (lane >> 4);
  float log2_total = 0.f;

  // (false, with the state as it was: the block holds a value outside the range of the contractions)
  auto block = [&](int j, auto full_tag) __attribute__((always_inline)) -> bool {
    constexpr bool kFull = decltype(full_tag)::value;
    __syncthreads();  // the previous block's readers (at first: the turning of the state) are done with LDS
    // ---- registers -> LDS ----
    float seen[3] = {};
    if constexpr (kImages) {
#pragma unroll
      for (int k = 0; k < L::kImagePieces; ++k) *reinterpret_cast<u32x4 *>(smem + 16 * (tid + kThr * k)) = r_img[k];
    } else {
#pragma unroll
      for (int k = 0; k < kPieces; ++k) {
        const f32x4 vb = __builtin_bit_cast(f32x4, r_b[k]);
        put_parts<NT>(sB, tid + kThr * k, vb);
        seen[0] = larger(seen[0], vb);
        if constexpr (kFull) {
          const f32x4 vc = __builtin_bit_cast(f32x4, r_c[k]);
          put_parts<NT>(sC, tid + kThr * k, vc);
          seen[1] = larger(seen[1], vc);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const f32x4 v = __builtin_bit_cast(f32x4, r_x[k]);
      *reinterpret_cast<f32x4 *>(sX + (8 * k + (lane >> 3)) * kXStride + 4 * (lane & 7)) = v;
      seen[2] = larger(seen[2], v);
    }
    // ---- decays: lane r (both halves) = token; tokens beyond the sequence have step size zero.  The decay from a
    //      token to the end of the block is summed from the end: the newest tokens weigh most ----
    float dtv = r_dt;
    if (!p.dt_plain) dtv = dt_apply_branchless(r_dt, dbias, p.dtx);  // (no load is outstanding that a branch would make wait)
    dtv = j * kTok + r < p.T ? dtv : 0.f;
    const float d = cut_decay(dtv * alog), after = suffix32(d), total = read_lane(after + d, 0);
    float ch = 0.f, cl = 0.f;
    if constexpr (kFull) {
      const float dh = coarse_part(d);
      ch = prefix32(dh);
      cl = prefix32(d - dh);
    }
    if (kg == 0) {
      if constexpr (kFull) {
        s_ch[wave][r] = ch;
        s_in[wave][r] = dtv * exp2_fast(-cl);
      }
      s_w[wave][r] = dtv * exp2_fast(after);
    }
    const float el_low = exp2_fast(cl), el = exp2_fast(ch) * el_low, e_all = exp2_fast(total);
    odd |= out_of_range(max_or_nan(max_or_nan(seen[0], seen[1]), seen[2])) || !(fabsf(dtv) < 0x1p40f) || !(fabsf(d) < 1e30f);
    if (__builtin_amdgcn_ballot_w64(odd) != 0 && lane == 0) s_odd = 1;
    load_block(min(j + 1, j2 - 1), j + 1 >= j1);  // (after the last block: a harmless repeat, no branch)
    __syncthreads();
    const int met_odd = kImages ? s_odd | *reinterpret_cast<const int *>(smem + L::kFlag) : s_odd;  // uniform over the workgroup; waited for where the state is about to change

    f32x16 Y = {};
    if constexpr (kFull) {
      // ---- scores: a quarter of the 32 x 32 tile per wave (the fourth wave's, above the diagonal, repeats the third's) ----
      if constexpr (!kImages) {
        if (wave < 3)
          *reinterpret_cast<f32x4 *>(sG + (16 * lq + tj) * kGStride + 16 * sq + 4 * (lane >> 4)) = scores_quarter<NT>(sB + a_sb, sC + a_sc);
      }
      // ---- Y^T[p][l]: the state's part, then scaled by the decay up to token l = r ----
#pragma unroll
      for (int kk = 0; kk < N / 16; ++kk) {
        Op c[3], hp[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) c[q].q = *reinterpret_cast<const u32x4 *>(sC + q * L::kPart + a_c + 16 * kk);
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = H[kk >> 1][8 * (kk & 1) + i];
        split3_even(v, hp);
        Y = mfma6(hp, c, Y);
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) Y[i] *= el;
      if constexpr (!kImages) __syncthreads();  // the scores are in LDS
    }
    if (met_odd != 0) return false;
    if constexpr (kStatesOnly) log2_total += total;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      // x^T: headdim column pi(r), tokens 16 q + {4kg.., 8 + 4kg..}
      float xv[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) xv[i] = sX[(16 * q + 8 * (i >> 2) + 4 * kg + (i & 3)) * kXStride + pi_of_row(r)];
      if constexpr (kFull) {
        // masked scores, transposed: element i is token s of the same order, the column l = r
        Op gm[3], xo[3];
        float v[8];
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          const int sb = 16 * q + 8 * hf + 4 * kg;
          const f32x4 gv = *reinterpret_cast<const f32x4 *>(sG + r * kGStride + sb);
          const f32x4 ch_s = *reinterpret_cast<const f32x4 *>(&s_ch[wave][sb]);
          const f32x4 in_s = *reinterpret_cast<const f32x4 *>(&s_in[wave][sb]);
#pragma unroll
          for (int i = 0; i < 4; ++i)  // (above the diagonal the tile holds whatever was there: selected, not multiplied)
            v[4 * hf + i] = sb + i <= r ? gv[i] * (in_s[i] * (el_low * exp2_fast(ch - ch_s[i]))) : 0.f;
        }
        split3_even(v, gm);
        split3_even(xv, xo);
        Y = mfma6(xo, gm, Y);
      }
      // ---- the state to the end of the block ----
      Op xm[3];
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const f32x4 w = *reinterpret_cast<const f32x4 *>(&s_w[wave][16 * q + 8 * hf + 4 * kg]);
#pragma unroll
        for (int i = 0; i < 4; ++i) xv[4 * hf + i] *= w[i];
      }
      split3_even(xv, xm);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        if (q == 0) {
#pragma unroll
          for (int i = 0; i < 16; ++i) H[nt][i] *= e_all;
        }
        Op bt[3];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
          bt[t].h[0] = lds_read_tr(sB + t * L::kPart + a_bt + 32 * nt + 16 * q * L::kRow);
          bt[t].h[1] = lds_read_tr(sB + t * L::kPart + a_bt + 32 * nt + (16 * q + 8) * L::kRow);
        }
        H[nt] = mfma6(bt, xm, H[nt]);
      }
    }
    if constexpr (kFull) {
      // ---- y: lane (r, kg) holds columns 16 kg .. 16 kg + 15 of token r ----
      const int n = min(kTok, p.T - j * kTok);
      const Rsrc ry = make_rsrc(yb + static_cast<size_t>(j) * kTok * xrow, live ? (n - 1) * xrow + 4 * kCols : 0u);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const f32x4 xr = *reinterpret_cast<const f32x4 *>(sX + r * kXStride + 16 * kg + 4 * c);
        f32x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = fmaf(Dh, xr[i], Y[4 * c + i]);
        buf_store16(ry, static_cast<uint32_t>(r) * xrow + 64 * kg + 16 * c, __builtin_bit_cast(u32x4, o));
      }
    }
    return true;
  };
  int j = j0;
  bool in_range = true;
  if constexpr (!kImages) {
    for (; j < j1 && in_range; j += in_range) in_range = block(j, std::false_type{});
  }
  if constexpr (!kStatesOnly) {
    for (; j < j2 && in_range; j += in_range) in_range = block(j, std::true_type{});
  }
  // ---- what is left of a walk that met such a block: the recurrence, token by token.  A lane holds half of a state row,
  //      the columns 32 nt + 8 i4 + 4 kg + 0 .. 3 of row pi(r) ----
  for (; j < j2; ++j) {
    const int n = min(kTok, p.T - j * kTok);
    const Rsrc rB = rows_of(Bb, brow, p.N * 4, j), rC = rows_of(Cb, brow, p.N * 4, j), rx = rows_of(xb, xrow, 4 * kCols, j);
    const Rsrc ry = make_rsrc(yb + static_cast<size_t>(j) * kTok * xrow, live && j >= j1 && !kStatesOnly ? (n - 1) * xrow + 4 * kCols : 0u);
    const float raw = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rows_of(db, drow, 4, j), r * drow, 0, 0));
    const float dtv = r < n ? dt_apply_branchless(raw, dbias, p.dtx) : 0.f;
    if constexpr (kStatesOnly) log2_total += read_lane(prefix32(cut_decay(dtv * alog)), kTok - 1);
#pragma clang loop unroll(disable)
    for (int t = 0; t < n; ++t) {
      const float dt_t = read_lane(dtv, t), dA = exp2_fast(dt_t * alog);
      const uint32_t at = t * xrow + 4 * pi_of_row(r);
      const float xv = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, at, 0, 0)), ux = dt_t * xv;
      float part = 0.f;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const int n0 = 32 * nt + 8 * i4 + 4 * kg;
          const uint32_t off = n0 < p.N ? t * brow + 4 * n0 : kNowhere;
          const f32x4 bv = __builtin_bit_cast(f32x4, buf_load16(rB, off)), cv = __builtin_bit_cast(f32x4, buf_load16(rC, off));
#pragma unroll
          for (int i = 0; i < 4; ++i) {  // (a column of padding stays zero whatever x is)
            const float v = n0 < p.N ? fmaf(dA, H[nt][4 * i4 + i], ux * bv[i]) : 0.f;
            H[nt][4 * i4 + i] = v;
            part = fmaf(cv[i], v, part);
          }
        }
      }
      part += __shfl_xor(part, 32, 64);
      if (kg == 0) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(fmaf(Dh, xv, part)), ry, at, 0, 0);
    }
  }

  // ---- the state back to memory: the segment's local end state, or the final state (Alg. 1, "Store") ----
  if (!kStatesOnly && j2 < nblocks) return;
  __syncthreads();
  float *const dst = kStatesOnly ? state_slot(p, b, h, p0, seg + 1, nblocks) : p.final_state + st_base;
  const Rsrc rs = make_rsrc(dst, !live ? 0u : kStatesOnly ? slot_size : st_size);
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4)
      *reinterpret_cast<f32x4 *>(turn + pi_of_row(r) * kTurnStride + 8 * i4 + 4 * kg) =
          f32x4{H[nt][4 * i4], H[nt][4 * i4 + 1], H[nt][4 * i4 + 2], H[nt][4 * i4 + 3]};
#pragma unroll
    for (int k = 0; k < 4; ++k)
      buf_store16(rs, st_off(nt, k, kStatesOnly && p.slots == nullptr),
                  *reinterpret_cast<const u32x4 *>(turn + (8 * k + (lane >> 3)) * kTurnStride + 4 * (lane & 7)));
  }
  if (kStatesOnly && live && p0 == 0 && lane == 0) p.decay[bh * p.S + seg] = log2_total;
}

// slot[0] = h0 (only where the full launch reads it there); slot[s] = exp2(decay[s-1]) * slot[s-1] + local[s-1].
// grid (ceil(P*N/1024), Bt*H), four consecutive state elements per thread; the loads, which do not depend on the
// chain, are issued eight segments at a time.
constexpr int kPassThr = 256;
__global__ __launch_bounds__(kPassThr) void split_pass_kernel(const SplitParams p) {
  constexpr int kAhead = 8;
  const int e = (blockIdx.x * kPassThr + threadIdx.x) * 4;
  if (e >= p.P * p.N) return;
  const int nblocks = (p.T + kTok - 1) / kTok, NT = (p.N + 31) / 32;
  const int b = blockIdx.y / p.H, h = blockIdx.y % p.H;
  const int row = e / p.N, n = e % p.N;
  const size_t piece = p.slots != nullptr ? static_cast<size_t>(row % kCols) * p.N + n
                                          : static_cast<size_t>((row % kCols) * NT + n / 32) * p.H * p.P + n % 32;
  auto at = [&](int s) { return reinterpret_cast<f32x4 *>(state_slot(p, b, h, row / kCols * kCols, s, nblocks) + piece); };
  f32x4 run = {};
  if (p.h0 != nullptr) run = *reinterpret_cast<const f32x4 *>(p.h0 + static_cast<size_t>(blockIdx.y) * p.P * p.N + e);
  const float *const dp = p.decay + static_cast<size_t>(blockIdx.y) * p.S;
  if (p.slot0) *at(0) = run;
  for (int s0 = 1; s0 < p.S; s0 += kAhead) {
    f32x4 v[kAhead];
    float d[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      const int s = min(s0 + k, p.S - 1);  // (clamped: the surplus loads of the last group are not used)
      v[k] = *at(s);
      d[k] = dp[s - 1];
    }
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      if (s0 + k < p.S) {
        const float f = exp2_fast(d[k]);
        run = f32x4{fmaf(f, run.x, v[k].x), fmaf(f, run.y, v[k].y), fmaf(f, run.z, v[k].z), fmaf(f, run.w, v[k].w)};
        *at(s0 + k) = run;
      }
    }
  }
}

}  // namespace

// How a sequence is cut up.
struct SplitPlan {
  int segments, sub, sub_blocks;
  double us;  // modelled time
};

// Segments whose states fit: the workspace holds them, or every segment's rows of y do (see state_slot).
static bool slots_in_workspace(const Dims &d, int S) {
  return static_cast<size_t>(d.Bt) * d.H * S * (static_cast<size_t>(d.P) * d.N + 1) * sizeof(float) <= generic_workspace_bytes(d);
}
static size_t image_bytes(const Dims &d) {
  const int nblocks = (d.T + kTok - 1) / kTok;
  constexpr int kImage[4] = {SplitLds<1, false>::kImage, SplitLds<2, false>::kImage, SplitLds<3, false>::kImage, SplitLds<4, false>::kImage};
  return static_cast<size_t>(d.Bt) * d.G * nblocks * kImage[(d.N + 31) / 32 - 1];
}
static bool slots_in_y(const Dims &d, int S) {
  const int nblocks = (d.T + kTok - 1) / kTok, rows = kCols * ((d.N + 31) / 32);
  return nblocks / S * kTok >= rows && d.T - segment_begin(S - 1, S, nblocks) * kTok >= rows;
}
static bool segments_fit(const Dims &d, int S) { return slots_in_workspace(d, S) || slots_in_y(d, S); }

// Microseconds on MI355X, fits to timings of 10 shapes: a full block; a block of which only the state is updated, in
// the states-only launch and in the full one; by state tiles.  A CU holds two workgroups, which slow each other by a
// third; a launch of more runs in rounds.
constexpr double kFullUs[4] = {2.2, 3.2, 4.1, 4.9}, kStateUs[4] = {1.0, 1.2, 1.4, 1.55}, kCarryUs[4] = {0.75, 1.3, 1.7, 2.1};
static double rounds_us(long wgs, double us, double second = 0.33) {
  double t = 0.0;
  for (; wgs > 0; wgs -= 512) t += us * (wgs <= 256 ? 1.0 : 1.0 + second * ((wgs < 512 ? wgs : 512) - 256) / 256.0);
  return t;
}

static SplitPlan split_plan(const Dims &d) {
  const int nblocks = (d.T + kTok - 1) / kTok, NT = (d.N + 31) / 32;
  const long wgs = static_cast<long>(d.Bt) * d.G * ((d.hpg * (d.P / kCols) + kWaves - 1) / kWaves);
  const int ks = knobs().seg_blocks, kp = knobs().seg_parts;
  SplitPlan pl = {1, 1, nblocks, 8.0 + 0.5 * NT + rounds_us(wgs, nblocks * kFullUs[NT - 1])};
  if (ks > 0) {
    pl.segments = (nblocks + ks - 1) / ks;
    while (pl.segments > 1 && (!segments_fit(d, pl.segments) || static_cast<long long>(pl.segments) * nblocks > 0x7FFFFFFFll)) --pl.segments;
    pl.sub = kp > 0 && pl.segments == 1 ? kp : 1;
    pl.sub_blocks = (nblocks + pl.sub - 1) / pl.sub;
    return pl;
  }
  for (int sub = 2; sub <= nblocks && sub <= 16 && wgs * sub <= 512; ++sub) {
    const int len = (nblocks + sub - 1) / sub;
    const double us = 8.0 + 0.5 * NT + rounds_us(wgs * sub, len * kFullUs[NT - 1] + (nblocks - len) * kCarryUs[NT - 1]);
    if (us < pl.us) pl = {1, sub, len, us};
  }
  const double state_mb = static_cast<double>(d.Bt) * d.H * d.P * d.N * 4e-6;
  for (int S = 2; S <= nblocks && S <= 64; ++S) {
    if (!segments_fit(d, S)) continue;
    const int len = (nblocks + S - 1) / S;
    const double us = 16.0 + 2.4 * NT + S * state_mb / 4.5 + rounds_us(wgs * (S - 1), len * kStateUs[NT - 1]) +
                      rounds_us(wgs * S, len * kFullUs[NT - 1]);
    if (us < pl.us) pl = {S, 1, nblocks, us};
  }
  return pl;
}

bool split_f32_supported(const Dims &d) {
  // (the rows of a whole block are addressed, whether they exist or not: 32-bit byte offsets must not wrap)
  const unsigned long long lim = 0xFFFF0000ull, t = static_cast<unsigned long long>(d.T < kTok ? kTok : d.T);
  return !d.bf16 && d.P % kCols == 0 && d.N % 8 == 0 && d.N <= 128 && t * d.H * d.P * 4 <= lim && t * d.G * d.N * 4 <= lim &&
         static_cast<unsigned long long>(d.Bt) * d.H <= 65535 &&
         static_cast<unsigned long long>(d.Bt) * d.H * (d.P / kCols) * 64 <= 0x7fffffffull;
}

// Microseconds of a call with that plan.  split_plan only compares plans with each other; this is fitted to 1600 drawn shapes
// (16 to 5000 tokens, 1 to 48 heads, batches of up to 8; 5 % rms, 4.7 % on 600 others): one launch is some 5 us cheaper
// than that model has it, and the pass over the states takes a quarter of a microsecond a segment however small they are.
static double split_us(const Dims &d, const SplitPlan &pl) {
  constexpr double kFull[4] = {3.43, 4.55, 5.46, 6.49}, kState[4] = {0.4, 0.5, 0.6, 0.7}, kCarry[4] = {1.15, 1.61, 1.9, 2.45};
  const int nblocks = (d.T + kTok - 1) / kTok, NT = (d.N + 31) / 32;
  const long wgs = static_cast<long>(d.Bt) * d.G * ((d.hpg * (d.P / kCols) + kWaves - 1) / kWaves);
  if (pl.segments == 1)
    return 2.9 + 0.53 * NT + rounds_us(wgs * pl.sub, pl.sub_blocks * kFull[NT - 1] + (nblocks - pl.sub_blocks) * kCarry[NT - 1], 0.71);
  const int len = (nblocks + pl.segments - 1) / pl.segments;
  const double state_mb = static_cast<double>(d.Bt) * d.H * d.P * d.N * 4e-6;
  return 10.9 + pl.segments * (0.265 + 0.79 * state_mb) + rounds_us(wgs * (pl.segments - 1), len * kState[NT - 1], 0.71) +
         rounds_us(wgs * pl.segments, len * kFull[NT - 1], 0.71);
}

// Taken where the models have it at most 3 % behind the faster of the other two families.  Over the 600 shapes that is 0.11 %
// behind the faster of the two timed, three are more than 6 % behind, 6.7 at most (without the 3 %: 0.15 %, three, 14).  By
// split_plan's own figure against the fp32 matrix instruction's it was 0.85 %, sixteen more than a tenth behind: prompts
// of up to a hundred tokens and many heads, where one launch suffices (4 x 33 tokens x 40 heads x 64 x 32 in four groups 11.4
// us, 7.9 on split operands), and middling ones (991 x 23 x 64 x 128 51.7, 47.8).
bool split_f32_chosen(const Dims &d) {
  if (!split_f32_supported(d)) return false;
  if (knobs().seg_blocks > 0) return true;
  return 0.97 * split_us(d, split_plan(d)) < f32_other_us(d);
}

// What several segments leave where for each other: the blocks' images, if they are made, first in the workspace, which then
// holds the states if it has room for them (else y does, see state_slot), and the decays.
// Images where the states-only launch has CUs left for them -- at most a workgroup per CU with them -- (2048 tokens x 24 heads
// 51.2 -> 49.0 us, 2 x 712 x 27 x 64 x 64 32.6 -> 31.3).  In a fuller launch they delay the states by what the full launch
// gains: 40 drawn prompts took 0.96 to 1.07 of the time, 6 x 2184 x 30 138 -> 143 us.
struct SplitMemory {
  bool images, states;  // in the workspace
  size_t off_states, off_decay;
};
static SplitMemory split_memory(const Dims &d, const SplitPlan &pl) {
  SplitMemory m = {false, false, 0, 0};
  if (pl.segments == 1) return m;
  const size_t row = static_cast<size_t>(d.Bt) * d.H * pl.segments, have = generic_workspace_bytes(d);
  const size_t images = image_bytes(d), decays = (row * sizeof(float) + 255) / 256 * 256, states = row * d.P * d.N * sizeof(float);
  const long rows = static_cast<long>(d.Bt) * d.G, nblocks = (d.T + kTok - 1) / kTok;
  const long wgs = rows * ((d.hpg * (d.P / kCols) + kWaves - 1) / kWaves);
  const bool idle = wgs * (pl.segments - 1) + rows * nblocks <= 256;
  m.images = knobs().split_images != 2 && idle && images + decays <= have && (images + decays + states <= have || slots_in_y(d, pl.segments));
  m.off_states = m.images ? images : 0;
  m.states = m.images ? images + decays + states <= have : slots_in_workspace(d, pl.segments);
  // (without the states: S decays per head, of which the workspace holds at least one per token and head)
  m.off_decay = m.off_states + (m.states ? states : 0);
  return m;
}

void split_f32_plan(const Dims &d, int *seg_blocks, int *segments, int *parts, int *images, int *states_in_y) {
  const SplitPlan pl = split_plan(d);
  const SplitMemory m = split_memory(d, pl);
  const int nblocks = (d.T + kTok - 1) / kTok;
  *seg_blocks = (nblocks + pl.segments - 1) / pl.segments;
  *segments = pl.segments;
  *parts = pl.sub;
  *images = m.images;
  *states_in_y = pl.segments > 1 && !m.states;
}

template <int NT>
static void launch_nt(const SplitParams &p, unsigned wgs, hipStream_t stream, KernelTrace *trace) {
  if (p.S > 1) {
    const unsigned images = p.images != nullptr ? static_cast<unsigned>((p.T + kTok - 1) / kTok) * p.Bt * p.G : 0;
    hipLaunchKernelGGL((split_f32_kernel<NT, true>), dim3(images + wgs * (p.S - 1)), dim3(kThr), 0, stream, p);
    trace_mark(trace, stream, "segment_states");
    hipLaunchKernelGGL(split_pass_kernel, dim3((p.P * p.N + 4 * kPassThr - 1) / (4 * kPassThr), p.Bt * p.H), dim3(kPassThr), 0,
                       stream, p);
    trace_mark(trace, stream, "segment_pass");
  }
  if (p.images != nullptr)
    hipLaunchKernelGGL((split_f32_kernel<NT, false, true>), dim3(wgs * p.S), dim3(kThr), 0, stream, p);
  else
    hipLaunchKernelGGL((split_f32_kernel<NT, false>), dim3(wgs * p.S * p.sub), dim3(kThr), 0, stream, p);
  trace_mark(trace, stream, "prefill_f32");
}

hipError_t launch_prefill_split_f32(const Dims &d, const void *x, const float *dt, const float *A, const void *B,
                                    const void *C, const float *D, const float *h0, void *y, float *final_state,
                                    void *workspace, hipStream_t stream, KernelTrace *trace) {
  const SplitPlan pl = split_plan(d);
  SplitParams p;
  p.x = static_cast<const float *>(x);
  p.dt = dt;
  p.A = A;
  p.B = static_cast<const float *>(B);
  p.C = static_cast<const float *>(C);
  p.D = D;
  p.h0 = h0;
  p.y = static_cast<float *>(y);
  p.final_state = final_state;
  const SplitMemory m = split_memory(d, pl);
  uint8_t *const ws = static_cast<uint8_t *>(workspace);
  p.images = m.images ? ws : nullptr;
  p.slots = m.states ? reinterpret_cast<float *>(ws + m.off_states) : nullptr;
  p.decay = reinterpret_cast<float *>(ws + m.off_decay);
  p.T = d.T;
  p.H = d.H;
  p.P = d.P;
  p.N = d.N;
  p.G = d.G;
  p.Bt = d.Bt;
  p.hpg = d.hpg;
  p.nslice = d.hpg * (d.P / kCols);
  p.cpg = (p.nslice + kWaves - 1) / kWaves;
  p.S = pl.segments;
  p.sub = pl.sub;
  p.sub_blocks = pl.sub_blocks;
  p.S_inv = inverse_of(p.S);
  p.cpg_inv = inverse_of(p.cpg);
  p.rows_inv = inverse_of(d.Bt * d.G);
  p.G_inv = inverse_of(d.G);
  p.per_head_inv = inverse_of(d.P / kCols);
  p.sub_inv = inverse_of(p.sub);
  p.nblocks_inv = inverse_of((d.T + kTok - 1) / kTok);
  p.dtx = d.dtx;
  p.dt_plain = d.dtx.identity();
  const size_t state_bytes = static_cast<size_t>(d.Bt) * d.H * d.P * d.N * sizeof(float);
  const char *const h = reinterpret_cast<const char *>(h0), *const f = reinterpret_cast<const char *>(final_state);
  const bool aliases = h0 != nullptr && h < f + state_bytes && f < h + state_bytes;
  p.slot0 = aliases && p.S > 1;
  if (aliases && p.S == 1) {  // the workgroup that stores the final state must be the one that reads h0
    p.sub = 1;
    p.sub_blocks = (d.T + kTok - 1) / kTok;
    p.sub_inv = inverse_of(1);
  }
  const unsigned wgs = static_cast<unsigned>(d.Bt) * d.G * p.cpg;
  switch ((d.N + 31) / 32) {
    case 1: launch_nt<1>(p, wgs, stream, trace); break;
    case 2: launch_nt<2>(p, wgs, stream, trace); break;
    case 3: launch_nt<3>(p, wgs, stream, trace); break;
    default: launch_nt<4>(p, wgs, stream, trace); break;
  }
  return hipGetLastError();
}

}  // namespace ssd
