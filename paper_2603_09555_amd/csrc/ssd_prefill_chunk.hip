// Prefill of small plain batches (bf16 io) in two launches instead of four: a workgroup per (batch row, 64-column slice of
// a head, chunk of 256 tokens) and nothing carried from one block of tokens to the next inside it.
//
// With cs_l the inclusive prefix sum of dt*A inside the chunk and S_c the state entering chunk c (Alg. 1; Eq. 3):
//     chunk_states   L_c = sum_s dt_s exp(cs_end - cs_s) x_s (x) B_s          every chunk's own contribution
//     chunk_outputs  S_c = exp(decay of chunk c-1) S_c-1 + L_c-1             summed from S_0 on as the states are loaded
//                    y_l = exp(cs_l) C_l . S_c + sum_s<=l (C_l . B_s) dt_s exp(cs_l - cs_s) x_s + D x_l
// The second is the quadratic form of the chunk on tiles of 32 x 32 tokens, eight rows of tiles for eight waves; waves w
// and w + 4, which share a SIMD, take rows w and 7 - w, nine tiles in all.  The scores never leave the registers: a tile
// of S^T = B C^T comes out of the matrix instruction as the operand that the product with x^T wants, up to the order of
// the contraction index, in which x^T is stored.  The mask is exact: on the diagonal tile exp(cs_l - cs_s), below it
// exp(decay of the row's tile up to l) times exp(decay of the tiles between) times exp(decay behind s in its tile), all
// with exponents that are never positive and are sums of decays, not differences.
//
// Over 256 tokens such a weight may be zero where the recurrence, step by step, never multiplies an infinity by zero; and a
// score of zero times it is undefined for tokens before it, too.  So a wave whose results are not all finite forms them again by
// the recurrence as it stands (recur_states, recur_rows): what is infinite, of which sign, and what is undefined are then
// the recurrence's.  Finite inputs get there only if a sum overflows.  The checks cost a call of one chunk up to 0.2 us; a prompt of
// NaNs, every wave of which then walks, takes 866 us at 2048 tokens x 24 heads and 628 at 250 x 40.
//
// What bounds it: latency.  2048 tokens x 24 heads, 192 + 24 workgroups, 17.8 us (scan kernels 33.8, a launch and a trip of
// the states through memory more).  Where it took 19.9: states 4.6 us from the first workgroup's start (loads 2.0, staging 1.5,
// product 1.1), outputs 10.5 (300 KB of loads to a CU 2.7, staging and the barrier 1.4, tiles 3.5 in the longest row, states
// and their product 2.5, y 0.4), the rest launches.  Matrix instructions are 1.9 us of it.
#include <type_traits>

#include "ssd_split_bf16.hpp"

namespace ssd {
namespace {
using namespace split;

constexpr int kTile = 32;                // tokens per tile
constexpr int kWaves = 8;                // = tiles per chunk
constexpr int kThr = 64 * kWaves;
constexpr int kChunk = kTile * kWaves;   // tokens per workgroup
constexpr int kP = 64, kN = 128;         // headdim columns and state columns per workgroup
constexpr int kSlot = kP * kN;           // floats of a state
constexpr int kMostChunks = 64;
constexpr int kAhead = 3;
constexpr int kXcds = 8, kCus = 256;
constexpr float kLog2e = 1.4426950408889634f;
constexpr uint32_t kNowhere = 0xFFFFFF00u;  // an offset beyond any descriptor

struct ChunkParams {
  const uint8_t *x, *B, *C;  // bf16
  const float *dt, *A, *D, *h0;
  uint8_t *y;
  float *final_state;
  float *slots;   // [batch row][slice][chunks (+ 1, a copy of h0)] states, 16-byte pieces in the order of the
                  // threads; the extra one holds a copy of h0 where final_state shares its memory (keep_h0)
  float *decay;   // [batch row][slice][chunk] log2 of the chunk's total decay
  int T, H, N, G, hpg, pdiv, chunks, slots_per, keep_h0;  // H, hpg count 64-column slices; pdiv slices per head
  int total, per_xcd;
  DtXform dtx;
};

// Chunks of one slice have consecutive numbers and lie on one XCD (see wg_coords in ssd_prefill_mfma.hip).
struct Item {
  int b, h, c, rows;  // rows: tokens of the chunk
};
__device__ __forceinline__ bool item_of(const ChunkParams &p, int per_slice, Item &it) {
  const int id = blockIdx.x, w = (id % kXcds) * p.per_xcd + id / kXcds;
  if (w >= p.total) return false;
  it.c = w % per_slice;
  it.h = (w / per_slice) % p.H;
  it.b = w / (per_slice * p.H);
  it.rows = max(0, min(kChunk, p.T - it.c * kChunk));
  return true;
}

// Rows of 16-byte pieces in LDS without padding: the low three bits of a piece's number are mixed with its row.
//   natural rows (row r for lane r):                       r ^ r/8
//   rows read in the order pi_of_row, written 8 apart:     see f_pi
__device__ __forceinline__ int f_nat(int row) { return (row ^ (row >> 3)) & 7; }
__device__ __forceinline__ int f_pi(int row) {
  return ((row & 3) | ((row >> 2) & 4)) ^ (((row >> 3) & 1) | ((row >> 4) & 2));
}

// A thread's 4 tokens x 8 columns (four 16-byte loads), transposed: column c of it as four consecutive tokens.
__device__ __forceinline__ u32x2 column_of(const u32x4 v[4], int c) {
  const uint32_t sel = (c & 1) ? 0x07060302u : 0x05040100u;
  return u32x2{__builtin_amdgcn_perm(v[1][c >> 1], v[0][c >> 1], sel), __builtin_amdgcn_perm(v[3][c >> 1], v[2][c >> 1], sel)};
}

__device__ __forceinline__ float step_size(const ChunkParams &p, const Item &it, int head, int row) {
  const uint32_t drow = static_cast<uint32_t>(p.H / p.pdiv) * 4;
  const Rsrc rd = make_rsrc(reinterpret_cast<const uint8_t *>(p.dt) + (static_cast<size_t>(it.b) * p.T + static_cast<size_t>(it.c) * kChunk) * drow,
                            static_cast<uint32_t>(it.rows) * drow);
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rd, row * drow + 4 * head, 0, 0));
}

// A state in the order [p][n], from the layout of either kernel through LDS: whole rows go out.
__device__ __forceinline__ int state_piece(int row, int piece) { return row * (kN / 4) + (piece ^ (row & 7)); }
__device__ __forceinline__ void store_state(const ChunkParams &p, size_t bh, const f32x4 *rows) {
  float *const out = p.final_state + bh * kP * p.N;
#pragma unroll
  for (int k = 0; k < kSlot / 4 / kThr; ++k) {
    const int row = static_cast<int>(threadIdx.x >> 5) + kThr / 32 * k, piece = threadIdx.x & 31;
    if (4 * piece < p.N) *reinterpret_cast<f32x4 *>(out + static_cast<size_t>(row) * p.N + 4 * piece) = rows[state_piece(row, piece)];
  }
}

// ---- the recurrence as it stands ----
__device__ __forceinline__ bool all_finite(float seen) { return __builtin_amdgcn_ballot_w64(!(seen < __builtin_inff())) == 0; }
__device__ __forceinline__ float larger(float seen, float v) { return max_or_nan(seen, fabsf(v)); }
// v + S, decayed by 2^d: finite values that decay below fp32's range are zero, infinities stay what they are.  (d is
// -infinity, whose factor is a plain zero, where a single token decays everything away; see chunk_states.)
__device__ __forceinline__ f32x4 chain(f32x4 S, float d, f32x4 v) {
  const bool far = d < -126.f && d > -__builtin_inff();
  const float e = far ? 0x1p-126f : exp2_fast(d), again = far ? 0x1p-126f : 1.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) S[i] = S[i] * e * again * again + v[i];
  return S;
}
// One token: S[i] = dA S[i] + (dt x) B[i] on the columns that exist.
__device__ __forceinline__ f32x4 recur(f32x4 S, float dA, float ux, u32x2 B) {
  const float b[4] = {bf_lo(B.x), bf_hi(B.x), bf_lo(B.y), bf_hi(B.y)};
#pragma unroll
  for (int i = 0; i < 4; ++i) S[i] = fmaf(dA, S[i], ux * b[i]);
  return S;
}
__device__ __forceinline__ float x_at(Rsrc rx, uint32_t at) {
  return __uint_as_float(static_cast<uint32_t>(static_cast<uint16_t>(__builtin_amdgcn_raw_buffer_load_b16(rx, at, 0, 0))) << 16);
}

// ---- L_c and the chunk's total decay; kSingle: the only chunk's, and with h0 the final state ----
struct StatesLds {
  __align__(16) uint8_t sBt[kN * kChunk * 2];  // B^T [n][s]
  __align__(16) uint8_t sXt[kP * kChunk * 2];  // (w x)^T [p][s]
  __align__(16) float s_w[kChunk];
  float s_total[kWaves];
};
template <bool kSingle>
__device__ __forceinline__ void chunk_states(const ChunkParams &p, const Item &it, StatesLds &lds) {
  uint8_t *const sBt = lds.sBt, *const sXt = lds.sXt;
  float *const s_w = lds.s_w, *const s_total = lds.s_total;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, kg = lane >> 5;
  const int head = it.h / p.pdiv, g = it.h / p.hpg;
  const size_t tok = static_cast<size_t>(it.b) * p.T + static_cast<size_t>(it.c) * kChunk;
  const uint32_t xrow = static_cast<uint32_t>(p.H) * (kP * 2), brow = static_cast<uint32_t>(p.G) * p.N * 2;
  const Rsrc rx = make_rsrc(p.x + tok * xrow, static_cast<uint32_t>(it.rows) * xrow);
  const Rsrc rB = make_rsrc(p.B + tok * brow, static_cast<uint32_t>(it.rows) * brow);

  // ---- wave w stages the 32 tokens of tile w: 4 tokens x 8 columns per load group, whole rows side by side ----
  float dtv = step_size(p, it, head, kTile * wave + r);
  const float alog = p.A[head] * kLog2e, bias = p.dtx.bias != nullptr ? p.dtx.bias[head] : 0.f;
  u32x4 vb[2][4], vx[4];
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int s = kTile * wave + 4 * ((lane >> 4) + 4 * k) + i, n0 = 8 * (lane & 15);
      vb[k][i] = buf_load16(rB, n0 < p.N ? s * brow + (g * p.N + n0) * 2 : kNowhere);
    }
#pragma unroll
  for (int i = 0; i < 4; ++i)
    vx[i] = buf_load16(rx, (kTile * wave + 4 * (lane >> 3) + i) * xrow + it.h * (kP * 2) + 16 * (lane & 7));
  const int nt = wave & 3, pt = wave >> 2;  // the wave's tile of the state: 32 state columns x 32 headdim columns
  const size_t bh = static_cast<size_t>(it.b) * p.H + it.h;
  u32x4 vh[4] = {};
  const bool with_h0 = it.c == 0 && p.h0 != nullptr;
  const Rsrc rh = make_rsrc(with_h0 ? p.h0 + bh * kP * p.N : p.dt, with_h0 ? kP * p.N * 4u : 0u);
#pragma unroll
  for (int i4 = 0; i4 < 4; ++i4) {
    const int n0 = 32 * nt + 8 * i4 + 4 * kg;
    vh[i4] = buf_load16(rh, n0 < p.N ? ((32 * pt + r) * p.N + n0) * 4u : kNowhere);
  }

  dtv = dt_apply_branchless(dtv, bias, p.dtx);
  dtv = kTile * wave + r < it.rows ? dtv : 0.f;
  // (-infinity where a token decays everything away: its zero is one of the recurrence, not of the product of many decays)
  const float d = cut_decay(dtv * alog), after = suffix32(d);
  const float total = __builtin_amdgcn_ballot_w64(d <= kCutLog2) != 0 ? -__builtin_inff() : read_lane(after + d, 0);
  if (lane == 0) s_total[wave] = total;
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int u = 8 * wave + (lane >> 4) + 4 * k, n = 8 * (lane & 15) + c;  // u: which four tokens
      *reinterpret_cast<u32x2 *>(sBt + n * (kChunk * 2) + (((u >> 1) ^ f_nat(n)) << 4) + 8 * (u & 1)) = column_of(vb[k], c);
    }
  __syncthreads();  // the tiles' decays
  float behind = 0.f, all = 0.f;
#pragma unroll
  for (int k = 0; k < kWaves; ++k) {
    const float t = s_total[kWaves - 1 - k];
    behind += kWaves - 1 - k > wave ? t : 0.f;
    all += t;
  }
  if (kg == 0) s_w[kTile * wave + r] = dtv * exp2_fast(after + behind);
  // (written and read by this wave)
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const f32x4 w = *reinterpret_cast<const f32x4 *>(&s_w[kTile * wave + 4 * (lane >> 3)]);
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const int u = 8 * wave + (lane >> 3), pc = 8 * (lane & 7) + c;
    const uint32_t a0 = vx[0][c >> 1], a1 = vx[1][c >> 1], a2 = vx[2][c >> 1], a3 = vx[3][c >> 1];
    const u32x2 o = (c & 1) ? u32x2{pack2(w.x * bf_hi(a0), w.y * bf_hi(a1)), pack2(w.z * bf_hi(a2), w.w * bf_hi(a3))}
                            : u32x2{pack2(w.x * bf_lo(a0), w.y * bf_lo(a1)), pack2(w.z * bf_lo(a2), w.w * bf_lo(a3))};
    *reinterpret_cast<u32x2 *>(sXt + pc * (kChunk * 2) + (((u >> 1) ^ f_nat(pc)) << 4) + 8 * (u & 1)) = o;
  }
  __syncthreads();
  const uint8_t *const ab = sBt + (32 * nt + r) * (kChunk * 2), *const ax = sXt + (32 * pt + r) * (kChunk * 2);
  const int fb = f_nat(32 * nt + r), fx = f_nat(32 * pt + r);
  f32x16 acc = {};
#pragma unroll
  for (int q = 0; q < kChunk / 16; ++q) {
    Op a, b;
    a.q = *reinterpret_cast<const u32x4 *>(ab + (((2 * q + kg) ^ fb) << 4));
    b.q = *reinterpret_cast<const u32x4 *>(ax + (((2 * q + kg) ^ fx) << 4));
    acc = mfma(a, b, acc);
  }
  // lane r: headdim column 32 pt + r; element i: state column 32 nt + 8 (i/4) + 4 kg + i % 4
  float *const slot = p.slots + bh * p.slots_per * kSlot + tid * 4;
  const float e_all = exp2_fast(all);
  if constexpr (kSingle) __syncthreads();  // the operands have been read
  f32x4 v[4];
  float seen = 0.f;
#pragma unroll
  for (int i4 = 0; i4 < 4; ++i4) {
    const f32x4 h = __builtin_bit_cast(f32x4, vh[i4]);
    v[i4] = f32x4{acc[4 * i4], acc[4 * i4 + 1], acc[4 * i4 + 2], acc[4 * i4 + 3]};
    if (with_h0) {
      if (!kSingle && p.keep_h0) *reinterpret_cast<f32x4 *>(slot + static_cast<size_t>(p.chunks) * kSlot + i4 * (4 * kThr)) = h;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i4][i] = fmaf(e_all, h[i], v[i4][i]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) seen = larger(seen, v[i4][i]);
  }
  if (!all_finite(seen)) {
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) v[i4] = __builtin_bit_cast(f32x4, vh[i4]);  // (zero but for the first chunk's h0)
    for (int j = 0; j < it.rows; j += kTile) {
      const float dts = dt_apply_branchless(step_size(p, it, head, j + r), bias, p.dtx);
      const int n = min(kTile, it.rows - j);
#pragma clang loop unroll(disable)
      for (int t = 0; t < n; ++t) {
        const float dt_t = read_lane(dts, t), ux = dt_t * x_at(rx, (j + t) * xrow + it.h * (kP * 2) + 2 * (32 * pt + r));
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const int n0 = 32 * nt + 8 * i4 + 4 * kg;
          const u32x2 b = buf_load8(rB, n0 < p.N ? (j + t) * brow + (g * p.N + n0) * 2 : kNowhere);
          v[i4] = n0 < p.N ? recur(v[i4], exp2_fast(dt_t * alog), ux, b) : f32x4{};
        }
      }
    }
  }
#pragma unroll
  for (int i4 = 0; i4 < 4; ++i4) {
    if constexpr (kSingle)
      reinterpret_cast<f32x4 *>(sBt)[state_piece(32 * pt + r, 8 * nt + 2 * i4 + kg)] = v[i4];
    else
      *reinterpret_cast<f32x4 *>(slot + static_cast<size_t>(it.c) * kSlot + i4 * (4 * kThr)) = v[i4];
  }
  if constexpr (kSingle) {
    __syncthreads();
    store_state(p, bh, reinterpret_cast<const f32x4 *>(sBt));
  } else if (tid == 0) {
    p.decay[bh * p.chunks + it.c] = all;
  }
}

// ---- outputs of a chunk; of the one behind the last: the final state ----
struct OutputsLds {
  __align__(16) uint8_t sB[kChunk * kN * 2];         // B [s][n]
  __align__(16) uint8_t sXt[kP * kChunk * 2];        // x^T [p][s], s in the order of the scores
  __align__(16) uint8_t sH[kP * kN * 2];             // the entering state [p][n]
  __align__(16) uint8_t sTurn[kWaves][kTile * 128];  // a wave's own rows on their way
  __align__(16) float s_behind[kChunk], s_cs[kChunk], s_dt[kChunk];
  float s_total[kWaves];
};
// y of the chunk's tile tt by one wave, from the state that enters the chunk on; a lane has headdim column `lane` and all
// state columns.
template <bool kSingle>
__device__ __forceinline__ void recur_rows(const ChunkParams &p, const Item &it, int tt, Rsrc rx, Rsrc rB, Rsrc rC, Rsrc rs, Rsrc ry,
                                           bool from_h0, int oldest, int newest, float chunk_decay) {
  constexpr int kQuads = kN / 4;
  const int lane = threadIdx.x & 63, head = it.h / p.pdiv, g = it.h / p.hpg;
  const uint32_t xrow = static_cast<uint32_t>(p.H) * (kP * 2), brow = static_cast<uint32_t>(p.G) * p.N * 2;
  const float alog = p.A[head] * kLog2e, bias = p.dtx.bias != nullptr ? p.dtx.bias[head] : 0.f, Dh = p.D[head];
  f32x4 S[kQuads];
  const Rsrc rh = make_rsrc(from_h0 ? p.h0 + (static_cast<size_t>(it.b) * p.H + it.h) * kP * p.N : p.dt, from_h0 ? kP * p.N * 4u : 0u);
#pragma unroll
  for (int i = 0; i < kQuads; ++i) S[i] = __builtin_bit_cast(f32x4, buf_load16(rh, 4 * i < p.N ? (lane * p.N + 4 * i) * 4u : kNowhere));
  if (!from_h0) {
#pragma clang loop unroll(disable)
    for (int k = oldest; k <= newest; ++k) {
      const float d = k == oldest ? 0.f : read_lane(chunk_decay, k);
#pragma unroll
      for (int i = 0; i < kQuads; ++i) {
        const uint32_t piece = 64 * (i >> 3) + 32 * (i & 1) + (lane & 31) + 256 * ((i & 6) + (lane >> 5));  // (see chunk_outputs)
        S[i] = chain(S[i], d, __builtin_bit_cast(f32x4, buf_load16(rs, static_cast<uint32_t>(k) * (kSlot * 4) + 16 * piece)));
      }
    }
  }
  for (int j = 0; j <= tt; ++j) {
    const float dts = dt_apply_branchless(step_size(p, it, head, kTile * j + (lane & 31)), bias, p.dtx);
    const int n = min(kTile, it.rows - kTile * j);
#pragma clang loop unroll(disable)
    for (int t = 0; t < n; ++t) {
      const uint32_t row = kTile * j + t, at = row * xrow + it.h * (kP * 2) + 2 * lane, bc = row * brow + g * p.N * 2;
      const float dt_t = read_lane(dts, t), dA = exp2_fast(dt_t * alog), xv = x_at(rx, at), ux = dt_t * xv;
      float part = 0.f;
      int N = p.N;
      asm volatile("" : "+s"(N));  // (or the comparisons are made ahead of the loop and kept in scalar registers)
#pragma unroll
      for (int i = 0; i < kQuads; i += 2) {
        if (4 * i < N) {  // (no product with the columns that do not exist: zero times an infinity)
          const u32x4 b = buf_load16(rB, bc + 8 * i), c = buf_load16(rC, bc + 8 * i);
          S[i] = recur(S[i], dA, ux, u32x2{b.x, b.y});
          S[i + 1] = recur(S[i + 1], dA, ux, u32x2{b.z, b.w});
#pragma unroll
          for (int q = 0; q < 4; ++q) part = fmaf(bf_hi(c[q]), S[i + q / 2][2 * (q & 1) + 1], fmaf(bf_lo(c[q]), S[i + q / 2][2 * (q & 1)], part));
        }
      }
      if (j == tt) __builtin_amdgcn_raw_buffer_store_b16(static_cast<uint16_t>(pack2(fmaf(Dh, xv, part), 0.f)), ry, at, 0, 0);
    }
  }
}

template <bool kSingle>
__device__ __forceinline__ void chunk_outputs(const ChunkParams &p, const Item &it, OutputsLds &lds) {
  uint8_t *const sB = lds.sB, *const sXt = lds.sXt, *const sH = lds.sH;
  float *const s_behind = lds.s_behind, *const s_cs = lds.s_cs, *const s_dt = lds.s_dt, *const s_total = lds.s_total;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, kg = lane >> 5;
  const int tt = wave < 4 ? wave : kWaves + 3 - wave;  // the wave's row of tiles
  const int head = it.h / p.pdiv, g = it.h / p.hpg;
  const size_t tok = static_cast<size_t>(it.b) * p.T + static_cast<size_t>(it.c) * kChunk;
  const uint32_t xrow = static_cast<uint32_t>(p.H) * (kP * 2), brow = static_cast<uint32_t>(p.G) * p.N * 2;
  const Rsrc rx = make_rsrc(p.x + tok * xrow, static_cast<uint32_t>(it.rows) * xrow);
  const Rsrc rB = make_rsrc(p.B + tok * brow, static_cast<uint32_t>(it.rows) * brow);
  const Rsrc rC = make_rsrc(p.C + tok * brow, static_cast<uint32_t>(it.rows) * brow);
  const size_t bh = static_cast<size_t>(it.b) * p.H + it.h;
  const Rsrc rs = make_rsrc(p.slots + bh * p.slots_per * kSlot, kSingle ? 0u : static_cast<uint32_t>(p.slots_per) * (kSlot * 4));

  // ---- everything is requested before anything is waited for ----
  float dtv = step_size(p, it, head, kTile * tt + r);
  const float alog = p.A[head] * kLog2e, bias = p.dtx.bias != nullptr ? p.dtx.bias[head] : 0.f, Dh = p.D[head];
  const float chunk_decay = !kSingle && lane < it.c ? p.decay[bh * p.chunks + lane] : 0.f;
  u32x4 vc[2][4], vb[8], vx[4];
#pragma unroll
  for (int hf = 0; hf < 2; ++hf)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int n0 = 64 * hf + 8 * (lane & 7);
      vc[hf][k] = buf_load16(rC, n0 < p.N ? (kTile * tt + (lane >> 3) + 8 * k) * brow + (g * p.N + n0) * 2 : kNowhere);
    }
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int n0 = 8 * (lane & 15);
    vb[k] = buf_load16(rB, n0 < p.N ? (kTile * wave + (lane >> 4) + 4 * k) * brow + (g * p.N + n0) * 2 : kNowhere);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
    vx[i] = buf_load16(rx, (kTile * wave + 4 * (lane >> 3) + i) * xrow + it.h * (kP * 2) + 16 * (lane & 7));
  u32x4 xr[4];  // the wave's own rows again, for the skip term
#pragma unroll
  for (int k = 0; k < 4; ++k) xr[k] = buf_load16(rx, (kTile * tt + (lane >> 3) + 8 * k) * xrow + it.h * (kP * 2) + 16 * (lane & 7));
  // the states of the chunks before, oldest first: one now, the others kAhead at a time; the first chunk starts from h0 (or its
  // copy, where final_state takes h0's place)
  const bool from_h0 = (kSingle || it.c == 0) && p.h0 != nullptr && !(!kSingle && p.keep_h0);
  const int newest = !kSingle && it.c > 0 ? it.c - 1 : p.h0 == nullptr ? -1 : from_h0 ? 0 : p.chunks, oldest = !kSingle && it.c > 0 ? 0 : max(newest, 0);
  // (piece tid + 256 i of a state: headdim row 32 (i & 1) + r, state columns 32 wave + 8 (i / 2) + 4 kg ..)
  constexpr int kOwn = kSlot / 4 / (kThr / 2);
  const uint32_t vs = static_cast<uint32_t>(tid) * 16;
  const bool folds = wave < 4;
  auto request = [&](int k, u32x4 raw[kOwn]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kOwn; ++i)
      raw[i] = buf_load16(rs, k <= newest ? static_cast<uint32_t>(k) * (kSlot * 4) + i * (kThr / 2 * 16) + vs : kNowhere);
  };
  u32x4 first[kOwn];
  if (folds) {
    if (from_h0) {
      const Rsrc rh = make_rsrc(p.h0 + bh * kP * p.N, kP * p.N * 4u);
#pragma unroll
      for (int i = 0; i < kOwn; ++i) {
        const int n0 = 32 * wave + 8 * (i >> 1) + 4 * kg;
        first[i] = buf_load16(rh, n0 < p.N ? ((32 * (i & 1) + r) * p.N + n0) * 4u : kNowhere);
      }
    } else {
      request(oldest, first);
    }
  }

  // ---- the entering state; lane k holds the decay over chunk k ----
  const float factor = exp2_fast(chunk_decay);
  f32x4 S[kOwn];
  auto fold = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kOwn; ++i) S[i] = __builtin_bit_cast(f32x4, first[i]);
    for (int k0 = oldest + 1; k0 <= newest; k0 += kAhead) {
      u32x4 raw[kAhead][kOwn];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) request(k0 + k, raw[k]);
#pragma unroll
      for (int k = 0; k < kAhead; ++k) {
        const float e = k0 + k <= newest ? read_lane(factor, min(k0 + k, newest)) : 1.f;  // (a state beyond: zero)
#pragma unroll
        for (int i = 0; i < kOwn; ++i) {
          const f32x4 v = __builtin_bit_cast(f32x4, raw[k][i]);
#pragma unroll
          for (int q = 0; q < 4; ++q) S[i][q] = fmaf(e, S[i][q], v[q]);
        }
      }
    }
  };
  if (!kSingle && it.c == p.chunks) {  // the final state
    f32x4 *const rows = reinterpret_cast<f32x4 *>(sB);
    if (folds) {
      fold();
      float seen = 0.f;
#pragma unroll
      for (int i = 0; i < kOwn; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) seen = larger(seen, S[i][q]);
      if (!all_finite(seen)) {
        request(oldest, first);
#pragma unroll
        for (int i = 0; i < kOwn; ++i) S[i] = __builtin_bit_cast(f32x4, first[i]);
#pragma clang loop unroll(disable)
        for (int k = oldest + 1; k <= newest; ++k) {
          request(k, first);
          const float d = read_lane(chunk_decay, k);
#pragma unroll
          for (int i = 0; i < kOwn; ++i) S[i] = chain(S[i], d, __builtin_bit_cast(f32x4, first[i]));
        }
      }
#pragma unroll
      for (int i = 0; i < kOwn; ++i) rows[state_piece(32 * (i & 1) + r, 8 * wave + (i & ~1) + kg)] = S[i];
    }
    __syncthreads();
    store_state(p, bh, rows);
    return;
  }
  // ---- C: a wave's own rows, through its piece of LDS into operand layout ----
  uint8_t *const turn = lds.sTurn[wave];
  Op co[8];
#pragma unroll
  for (int hf = 0; hf < 2; ++hf) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int row = (lane >> 3) + 8 * k;
      *reinterpret_cast<u32x4 *>(turn + row * 128 + (((lane & 7) ^ (row & 7)) << 4)) = vc[hf][k];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int q = 0; q < 4; ++q) co[4 * hf + q].q = *reinterpret_cast<const u32x4 *>(turn + r * 128 + (((2 * q + kg) ^ (r & 7)) << 4));
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  // ---- decays of the wave's tile; lane r = token ----
  dtv = dt_apply_branchless(dtv, bias, p.dtx);
  dtv = kTile * tt + r < it.rows ? dtv : 0.f;
  const float d = cut_decay(dtv * alog), cs = prefix32(d), after = suffix32(d), total = read_lane(after + d, 0);
  if (kg == 0) {
    s_behind[kTile * tt + r] = dtv * exp2_fast(after);
    s_cs[kTile * tt + r] = cs;
    s_dt[kTile * tt + r] = dtv;
  }
  if (lane == 0) s_total[tt] = total;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int s = kTile * wave + (lane >> 4) + 4 * k;
    *reinterpret_cast<u32x4 *>(sB + s * (kN * 2) + (((lane & 15) ^ (s & 7)) << 4)) = vb[k];
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    // tokens 4 a .. 4 a + 3 of a group of 16 go to place 2 (a & 1) + (a >> 1): the scores' order
    const int u = lane >> 3, a = u & 3, chunk = 4 * wave + 2 * (u >> 2) + (a & 1), pc = 8 * (lane & 7) + c;
    *reinterpret_cast<u32x2 *>(sXt + pc * (kChunk * 2) + ((chunk ^ f_pi(pc)) << 4) + 8 * (a >> 1)) = column_of(vx, c);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int row = (lane >> 3) + 8 * k;
    *reinterpret_cast<u32x4 *>(turn + row * 128 + (((lane & 7) ^ (row & 7)) << 4)) = xr[k];
  }
  __syncthreads();

  // ---- Y^T[p][l], lane r = token l of the row of tiles; tile pt: headdim columns 32 pt + 16 kg + element.  (A row of
  //      tiles beyond the sequence is zeros.) ----
  f32x16 Y[2] = {};
  // A software pipeline over the tiles, from the diagonal back: B's operands of the next tile are requested as soon as the
  // scores have read this one's, ahead of the vector work on the scores.  (Left to itself the compiler reads one operand
  // at a time and waits for it: 0.8 us a tile.)
  const uint8_t *const b_row = sB + r * (kN * 2);
  uint32_t x_row[2];  // (of the second 32 columns: the other one, 32 rows on)
#pragma unroll
  for (int u = 0; u < 2; ++u) x_row[u] = pi_of_row(r) * (kChunk * 2) + (((2 * u + kg) ^ f_pi(pi_of_row(r))) << 4);
  Op bo[8];
  auto request_b = [&](int j) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 8; ++q) bo[q].q = *reinterpret_cast<const u32x4 *>(b_row + j * (kTile * kN * 2) + (((2 * q + kg) ^ (r & 7)) << 4));
  };
  float tiles_between = 0.f;
  auto tile = [&](int j, auto diagonal_tag) __attribute__((always_inline)) {
    constexpr bool kDiagonal = decltype(diagonal_tag)::value;
    f32x16 v = {};  // S^T of tile (tt, j): rows s, column l = r
#pragma unroll
    for (int q = 0; q < 8; ++q) v = mfma(bo[q], co[q], v);
    __builtin_amdgcn_sched_barrier(0);
    f32x4 w[4];
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) w[i4] = *reinterpret_cast<const f32x4 *>((kDiagonal ? s_cs : s_behind) + kTile * j + 8 * i4 + 4 * kg);
    f32x4 dt_s[4];
    if constexpr (kDiagonal) {
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) dt_s[i4] = *reinterpret_cast<const f32x4 *>(&s_dt[kTile * j + 8 * i4 + 4 * kg]);
    }
    Op xo[2][2];  // [columns 32 pt ..][16 tokens]
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int pt = 0; pt < 2; ++pt)
        xo[pt][u].q = *reinterpret_cast<const u32x4 *>(sXt + (x_row[u ^ pt] ^ ((j & 1) << 6)) + (j >> 1) * 128 + pt * (32 * kChunk * 2));
    request_b(max(j - 1, 0));
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kDiagonal) {  // (fminf would make an undefined decay, of a head whose A is NaN, one of 2^0)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          v[4 * i4 + i] = 8 * i4 + 4 * kg + i <= r ? v[4 * i4 + i] * (dt_s[i4][i] * exp2_fast(min_or_nan(cs - w[i4][i], 0.f))) : 0.f;
    } else {
      const float e = exp2_fast(tiles_between + cs);
      tiles_between += s_total[j];
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4)
#pragma unroll
        for (int i = 0; i < 4; ++i) v[4 * i4 + i] *= e * w[i4][i];
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      Op sc;
#pragma unroll
      for (int k = 0; k < 4; ++k) sc.u[k] = pack2(v[8 * u + 2 * k], v[8 * u + 2 * k + 1]);
#pragma unroll
      for (int pt = 0; pt < 2; ++pt) Y[pt] = mfma(xo[pt][u], sc, Y[pt]);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  request_b(tt);
  tile(tt, std::true_type{});
  for (int j = tt - 1; j >= 0; --j) tile(j, std::false_type{});
  if (newest >= 0) {  // uniform over the workgroup
    if (folds) {  // (these waves have the short rows of tiles, one to four of them)
      fold();
#pragma unroll
      for (int i = 0; i < kOwn; ++i) {
        const int row = 32 * (i & 1) + r, unit = 4 * wave + (i >> 1);
        *reinterpret_cast<u32x2 *>(sH + row * (kN * 2) + ((unit ^ f_pi(row)) << 4) + 8 * kg) =
            u32x2{pack2(S[i][0], S[i][1]), pack2(S[i][2], S[i][3])};
      }
    }
    __syncthreads();
    f32x16 Z[2] = {};
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int pt = 0; pt < 2; ++pt) {
        const int row = 32 * pt + pi_of_row(r);
        Op a;
        a.q = *reinterpret_cast<const u32x4 *>(sH + row * (kN * 2) + (((2 * q + kg) ^ f_pi(row)) << 4));
        Z[pt] = mfma(a, co[q], Z[pt]);
      }
    float to_tile = 0.f;  // log2 decay from the start of the chunk to the start of the row's tile
    for (int k = 0; k < tt; ++k) to_tile += s_total[k];
    const float e_row = exp2_fast(to_tile + cs);
#pragma unroll
    for (int pt = 0; pt < 2; ++pt)
#pragma unroll
      for (int i = 0; i < 16; ++i) Y[pt][i] = fmaf(e_row, Z[pt][i], Y[pt][i]);
  }

  const Rsrc ry = make_rsrc(p.y + tok * xrow, static_cast<uint32_t>(it.rows) * xrow);
  {
    float seen = 0.f;
#pragma unroll
    for (int pt = 0; pt < 2; ++pt)
#pragma unroll
      for (int i = 0; i < 16; ++i) seen = larger(seen, Y[pt][i]);
    if (!all_finite(kTile * tt + r < it.rows ? seen : 0.f)) {
      recur_rows<kSingle>(p, it, tt, rx, rB, rC, rs, ry, from_h0, oldest, newest, chunk_decay);
      return;
    }
  }
  // ---- y = Y + D x, rounded once, in the place of the x it takes and out as whole rows ----
#pragma unroll
  for (int pt = 0; pt < 2; ++pt)
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      uint8_t *const at = turn + r * 128 + (((4 * pt + 2 * kg + hf) ^ (r & 7)) << 4);
      const u32x4 xv = *reinterpret_cast<const u32x4 *>(at);
      u32x4 o;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        o[k] = pack2(fmaf(Dh, bf_lo(xv[k]), Y[pt][8 * hf + 2 * k]), fmaf(Dh, bf_hi(xv[k]), Y[pt][8 * hf + 2 * k + 1]));
      *reinterpret_cast<u32x4 *>(at) = o;
    }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int row = (lane >> 3) + 8 * k;
    buf_store16(ry, (kTile * tt + row) * xrow + it.h * (kP * 2) + 16 * (lane & 7),
                *reinterpret_cast<const u32x4 *>(turn + row * 128 + (((lane & 7) ^ (row & 7)) << 4)));
  }
}

__global__ __launch_bounds__(kThr, 2) void chunk_states_kernel(const ChunkParams p) {
  __shared__ StatesLds lds;
  Item it;
  if (item_of(p, p.chunks, it)) chunk_states<false>(p, it, lds);
}
__global__ __launch_bounds__(kThr, 2) void chunk_outputs_kernel(const ChunkParams p) {
  __shared__ OutputsLds lds;
  Item it;
  if (item_of(p, p.chunks + 1, it)) chunk_outputs<false>(p, it, lds);
}
// Prompts of one chunk: outputs and final state don't depend on each other and run side by side.
__global__ __launch_bounds__(kThr, 2) void chunk_single_kernel(const ChunkParams p) {
  __shared__ union {
    StatesLds states;
    OutputsLds outputs;
  } lds;
  Item it;
  if (!item_of(p, 2, it)) return;
  const bool outputs = it.c == 0;
  it.c = 0;
  it.rows = p.T;
  if (outputs)
    chunk_outputs<true>(p, it, lds.outputs);
  else
    chunk_states<true>(p, it, lds.states);
}

}  // namespace

int chunk_count(const Dims &d) { return (d.T + kChunk - 1) / kChunk; }

// (one chunk: only a copy of h0, and with it the chunk's state, needs memory)
static size_t chunk_workspace(const Dims &d, bool keep_h0) {
  const size_t rows = static_cast<size_t>(d.Bt) * d.H * (d.P / kP), chunks = chunk_count(d);
  if (chunks == 1 && !keep_h0) return 0;
  return rows * ((chunks + (keep_h0 ? 1 : 0)) * kSlot + chunks) * sizeof(float);
}

static bool overlap(const Dims &d, const float *h0, const float *final_state) {
  const size_t bytes = static_cast<size_t>(d.Bt) * d.H * d.P * d.N * sizeof(float);
  const char *const h = reinterpret_cast<const char *>(h0), *const f = reinterpret_cast<const char *>(final_state);
  return h0 != nullptr && h < f + bytes && f < h + bytes;
}

// Whether the kernels can run the shape in a workspace of that size.
static bool chunk_supported(const Dims &d, size_t workspace_bytes, bool keep_h0) {
  return d.bf16 && d.P % kP == 0 && d.N % 8 == 0 && d.N <= kN && chunk_count(d) <= kMostChunks &&
         static_cast<unsigned long long>(kChunk) * d.H * d.P * 2 <= 0x7fffffffull &&
         static_cast<unsigned long long>(kChunk) * d.H * 4 <= 0x7fffffffull &&
         static_cast<unsigned long long>(kChunk) * d.G * d.N * 2 <= 0x7fffffffull &&
         static_cast<unsigned long long>(d.Bt) * d.H * (d.P / kP) * (chunk_count(d) + 1) <= (1u << 20) &&
         chunk_workspace(d, keep_h0) <= workspace_bytes;
}

// Taken while the second launch -- a workgroup per slice and chunk and one for each slice's final state, one workgroup to a
// CU -- is a round of the chip, from 4 to 18 chunks also a little more.  Of 4700 drawn shapes (10 to 16384 tokens, 1 to 600
// slices) timed against the scan kernels, those of up to 256 workgroups take 0.55 to 1.0 of the time (median 0.7; a few of more
// than 50 chunks, whose states each workgroup chains, up to 1.15), those of up to 320 0.75 to 1.05 with 4 to 18 chunks, 1.02
// to 1.2 with 2 or 3, 0.85 to 1.3 with more; one chunk, one launch of two workgroups per slice, 0.6 to 0.88 up to 256 of them and
// beyond 1.03 to 1.5 (11 x 123 tokens x 14 slices 16.5 us, scan 12.8; 12583 tokens x 6 slices 56.6, 44.0).
bool chunk_chosen(const Dims &d, size_t workspace_bytes, bool h0_aliases_final_state) {
  const Knobs &k = knobs();
  if (k.chunk == 2 || !chunk_supported(d, workspace_bytes, h0_aliases_final_state)) return false;
  if (k.chunk == 1) return true;
  // (knobs of the scan kernels ask for them)
  if (k.seg_chunks > 0 || k.seg_blocks > 0 || k.seg_parts > 0 || k.y_stream >= 0 || k.scan_heads > 0 ||
      k.fold_max_slots != Knobs().fold_max_slots)
    return false;
  const long slices = static_cast<long>(d.Bt) * d.H * (d.P / kP), chunks = chunk_count(d);
  return (chunks + 1) * slices <= (chunks >= 4 && chunks <= 18 ? 320 : kCus);
}
bool chunk_chosen(const Dims &d, size_t workspace_bytes, const float *h0, const float *final_state) {
  return chunk_chosen(d, workspace_bytes, overlap(d, h0, final_state));
}

hipError_t launch_prefill_chunk(const Dims &d, const void *x, const float *dt, const float *A, const void *B, const void *C,
                                const float *D, const float *h0, void *y, float *final_state, void *workspace,
                                hipStream_t stream, KernelTrace *trace) {
  ChunkParams p;
  p.x = static_cast<const uint8_t *>(x);
  p.B = static_cast<const uint8_t *>(B);
  p.C = static_cast<const uint8_t *>(C);
  p.dt = dt;
  p.A = A;
  p.D = D;
  p.h0 = h0;
  p.y = static_cast<uint8_t *>(y);
  p.final_state = final_state;
  p.pdiv = d.P / kP;
  p.T = d.T;
  p.H = d.H * p.pdiv;
  p.N = d.N;
  p.G = d.G;
  p.hpg = d.hpg * p.pdiv;
  p.chunks = chunk_count(d);
  p.keep_h0 = overlap(d, h0, final_state);
  p.slots_per = p.chunks + p.keep_h0;
  p.slots = static_cast<float *>(workspace);
  p.decay = p.slots + static_cast<size_t>(d.Bt) * p.H * p.slots_per * kSlot;
  p.dtx = d.dtx;
  auto grid = [&](int per_slice) {
    p.total = d.Bt * p.H * per_slice;
    p.per_xcd = (p.total + kXcds - 1) / kXcds;
    return dim3(kXcds * p.per_xcd);
  };
  if (p.chunks == 1 && !p.keep_h0) {
    const dim3 g = grid(2);
    hipLaunchKernelGGL(chunk_single_kernel, g, dim3(kThr), 0, stream, p);
    trace_mark(trace, stream, "chunk_single");
    return hipGetLastError();
  }
  const dim3 for_states = grid(p.chunks);
  hipLaunchKernelGGL(chunk_states_kernel, for_states, dim3(kThr), 0, stream, p);
  trace_mark(trace, stream, "chunk_states");
  const dim3 for_outputs = grid(p.chunks + 1);
  hipLaunchKernelGGL(chunk_outputs_kernel, for_outputs, dim3(kThr), 0, stream, p);
  trace_mark(trace, stream, "chunk_outputs");
  return hipGetLastError();
}

}  // namespace ssd
