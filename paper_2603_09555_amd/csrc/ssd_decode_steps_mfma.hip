// Many known decode steps in one launch, on the matrix pipe (bf16 io; dstate 64 or 128; headdim a multiple of 32).
//
// nsteps applications of the step of Alg. 2 to inputs that are all known are a short prefill from a carried state
// (Eq. 3), so they can be evaluated 32 steps at a time as contractions.  With cs_l the inclusive prefix sum of
// dt*A over the block and S the state entering it, per (layer, batch row, head):
//     G[l][s] = C_l . B_s                                                     (s <= l)
//     y[l][p] = exp(cs_l) sum_n C[l][n] S[p][n] + sum_s (G[l][s] dt_s exp(cs_l - cs_s)) x[s][p] + D x[l][p]
//     S'      = exp(cs_31) S + sum_s (dt_s exp(cs_31 - cs_s) x[s][p]) B[s][n]
// B, C and x are bf16 and enter the products exactly; what is fp32 in the recurrence -- the state, the masked
// scores, the weighted input -- is split into three bf16 parts without loss (ssd_split_bf16.hpp), so every product
// is exact and every sum is fp32: the result differs from single steps by the order of fp32 sums.  The decay
// between a step and the end of the block is summed from the end, so the newest inputs, which weigh most, carry the
// smallest exponent error.  The mask takes cs apart into ch + cl (cut_decay, coarse_part), ch exact: its weights are
//     exp(cl_l) (exp(ch_l - ch_s) (dt_s exp(-cl_s))),
// the factor of the row l applied to y as a whole.
//
// The step-by-step kernel (decode_steps_kernel) is bound by the vector ALU, three instructions per state element
// and step.  Here a state element costs one split (11 instructions per two values) and its share of 3 + 3 matrix
// instructions per 32 steps, and the call is bound by reading and writing the state once.
// Measured, 64 layers x 80 heads x 64 x 128, us per call, step-by-step kernel / this one: 9 steps 89 / 68, 16 steps 133 / 72,
// 64 steps 412 / 101 (423 MB that must move: 4.2 TB/s); batch 16: 16 steps 1895 / 975 (5.4 GB and more); one layer: 64
// steps 47 / 10.7.  Final state of 64 steps against 64 bits: 1.5e-7 / 8e-8.  Two waves per SIMD: at three (168 registers)
// the spills cost more than the third wave gives (64 steps 133).
//
// One wave per slice of 32 headdim columns x dstate, four slices of one B/C group per workgroup (they share the
// staged B and C).  The state slice sits in MFMA accumulators: tile nt, element i of lane (r, kg) is state column
// 32 nt + 8 (i/4) + 4 kg + i%4 of headdim column pi(r).  Eight accumulators in a row are, after the split, an A
// operand with the contraction order {4kg..4kg+3, 8+4kg..8+4kg+3} of 16 state columns; C and B lie in LDS with
// their columns in that order.  The same order of tokens turns the masked scores -- G is computed transposed, s
// down the accumulators -- into B operands; x^T and B^T operands come from row-major tiles by transposed reads.
#include "ssd_split_bf16.hpp"

namespace ssd {
namespace {
using namespace split;

constexpr int kTok = 32;      // steps per block
constexpr int kCols = 32;     // headdim columns per wave
constexpr int kWaves = 4;
constexpr int kThr = 64 * kWaves;
constexpr int kXStride = kCols + 8;  // bf16 elements per row of an x tile
constexpr int kTurnStride = 32 + 4;  // floats per row of a state tile on its way through LDS
constexpr size_t kMemCacheBytes = 256ull << 20;
constexpr float kLog2e = 1.4426950408889634f;

struct StepsParams {
  float *state;
  const uint8_t *x, *B, *C;
  const float *dt, *A, *D;
  uint8_t *y;
  size_t npairs, nbc;  // (layer, row, head) triples; (layer, row, group) triples
  int nsteps, Bt, H, P, G, hpg;
  int slots, cpg;      // slices of 32 columns per group; workgroups per group
  DtXform dtx;
};

template <int N>
struct StepsLds {
  static constexpr int kRowStride = N + 8;  // bf16 elements per row of the B and C tiles
  static constexpr int kTile = kTok * kRowStride;
  static constexpr int kX = kTok * kXStride;
  static constexpr int kTiles = (2 * kTile + kWaves * kX) * 2;             // bytes
  static constexpr int kTurn = kWaves * kCols * kTurnStride * 4;           // bytes, in the place of the tiles
  static constexpr int kBytes = kTiles > kTurn ? kTiles : kTurn;
};

// Largest magnitudes of packed bf16 pairs, as bits (an infinity or a NaN has 0x7f80 or more).  x, B and C of 2^24 and more,
// step sizes of 2^40 and a state of 2^60 are left to the recurrence, as are infinities and NaNs: below that no product on
// the way leaves fp32's range that the recurrence's stay inside (a score C.B may, where x is as small as they are large).
constexpr uint32_t kIoLimit = 0x4b80u, kStateLimit = 0x5d800000u;
constexpr float kDtLimit = 0x1p40f;
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t max_bf16(uint32_t seen, uint32_t u) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, seen), __builtin_bit_cast(u16x2, u & 0x7fff7fffu)));
}

// kStream: the state is read and written past the caches (see load_h4 of the single-step kernels for the rule).
template <int N, bool kStream>
__global__ __launch_bounds__(kThr, 2) void decode_steps_mfma_kernel(const StepsParams p) {
  using L = StepsLds<N>;
  constexpr int kNt = kStream ? 2 : 0;  // cache-policy field of the state's loads and stores: nt
  constexpr int NT = N / 32;
  constexpr int kItems = 16 * (N / 8);          // (row pair, 16-byte piece) items of a B or C tile
  constexpr int kPer = 2 * kItems / kThr;       // per thread, B and C together
  static_assert(kPer * kThr == 2 * kItems, "the threads share the tiles evenly");
  __shared__ __align__(16) uint8_t smem[L::kBytes];
  __shared__ __align__(16) float s_ch[kWaves][kTok], s_in[kWaves][kTok], s_w[kWaves][kTok];
  __shared__ int s_odd;
  uint16_t *const sB = reinterpret_cast<uint16_t *>(smem);
  uint16_t *const sC = sB + L::kTile;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, kg = lane >> 5;
  uint16_t *const sX = sC + L::kTile + wave * L::kX;

  const int col = blockIdx.x % p.cpg;
  const size_t bg = blockIdx.x / p.cpg;            // (layer * Bt + row) * G + group
  const int g = static_cast<int>(bg % p.G);
  const size_t lb = bg / p.G;
  const int layer = static_cast<int>(lb / p.Bt);
  const int slot_raw = kWaves * col + wave;
  const bool live = slot_raw < p.slots;            // (a wave without a slice repeats the last one and stores nothing)
  const int slot = live ? slot_raw : p.slots - 1;
  const int per_head = p.P / kCols;
  const int h = g * p.hpg + slot / per_head;
  const int p0 = kCols * (slot % per_head);
  const size_t pair = lb * p.H + h;
  const float Ah = p.A[static_cast<size_t>(layer) * p.H + h];
  const float Dh = p.D[static_cast<size_t>(layer) * p.H + h];
  const float dbias = p.dtx.bias != nullptr ? p.dtx.bias[static_cast<size_t>(layer) * p.H + h] : 0.f;
  const float alog = Ah * kLog2e;

  // ---- addressing: rows (steps) of x / y, of B / C and of dt ----
  const size_t xrow = p.npairs * p.P * 2, brow = p.nbc * N * 2, drow = p.npairs * 4;
  const uint8_t *const xb = p.x + (pair * p.P + p0) * 2;
  uint8_t *const yb = p.y + (pair * p.P + p0) * 2;
  const uint8_t *const Bb = p.B + bg * N * 2, *const Cb = p.C + bg * N * 2;
  const uint8_t *const db = reinterpret_cast<const uint8_t *>(p.dt) + pair * 4;
  const uint32_t xr32 = static_cast<uint32_t>(xrow), br32 = static_cast<uint32_t>(brow), dr32 = static_cast<uint32_t>(drow);
  // descriptor of the rows of block s0 that exist, `width` bytes of each (none: an empty one)
  auto rows_of = [&](const uint8_t *base, size_t row, uint32_t row32, uint32_t width, int s0) {
    const int n = min(kTok, p.nsteps - s0);
    return make_rsrc(base + static_cast<size_t>(s0) * row, n > 0 ? (n - 1) * row32 + width : 0u);
  };

  // ---- data of a block in flight ----
  u32x4 r_bc[kPer][2], r_x[2];
  float r_dt;
  auto load_block = [&](int s0) __attribute__((always_inline)) {
    const Rsrc rB = rows_of(Bb, brow, br32, N * 2, s0), rC = rows_of(Cb, brow, br32, N * 2, s0);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int item = tid + kThr * k, it = item % kItems;
      const uint32_t off = static_cast<uint32_t>(2 * (it / (N / 8))) * br32 + 16 * (it % (N / 8));
      // (whole waves take B or C: kItems is a multiple of 64)
      const bool isC = __builtin_amdgcn_readfirstlane(item / kItems) != 0;
#pragma unroll
      for (int j = 0; j < 2; ++j) r_bc[k][j] = buf_load16(isC ? rC : rB, off + j * br32);
    }
    const Rsrc rx = rows_of(xb, xrow, xr32, 2 * kCols, s0);
#pragma unroll
    for (int k = 0; k < 2; ++k) r_x[k] = buf_load16(rx, static_cast<uint32_t>(16 * k + (lane >> 2)) * xr32 + 16 * (lane & 3));
    r_dt = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rows_of(db, drow, dr32, 4, s0), r * dr32, 0, 0));
  };

  // ---- the state slice: 32 rows of N floats, contiguous; through LDS into the accumulators ----
  float *const st = p.state + (pair * p.P + p0) * N;
  const uint32_t st_off = (lane >> 3) * (N * 4) + 16 * (lane & 7);  // + 8 k rows, + 32 nt columns
  float *const turn = reinterpret_cast<float *>(smem) + wave * (kCols * kTurnStride);
  f32x16 H[NT];
  uint32_t odd = 0;  // largest magnitude of the state, as bits
  {
    const Rsrc rs = make_rsrc(st, kCols * N * 4);
    u32x4 raw[NT][4];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int k = 0; k < 4; ++k) raw[nt][k] = buf_load16<kNt>(rs, st_off + 8 * k * (N * 4) + 128 * nt);
    load_block(0);
    if (tid == 0) s_odd = 0;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
#pragma unroll
        for (int j = 0; j < 4; ++j) odd = max(odd, raw[nt][k][j] & 0x7fffffffu);
        *reinterpret_cast<u32x4 *>(turn + (8 * k + (lane >> 3)) * kTurnStride + 4 * (lane & 7)) = raw[nt][k];
      }
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const f32x4 v = *reinterpret_cast<const f32x4 *>(turn + pi_of_row(r) * kTurnStride + 8 * i4 + 4 * kg);
#pragma unroll
        for (int j = 0; j < 4; ++j) H[nt][4 * i4 + j] = v[j];
      }
    }
  }
  bool any_odd = odd >= kStateLimit || !(fabsf(Ah) < __builtin_inff());

  // LDS addresses of this lane (elements)
  const uint32_t a_row = r * L::kRowStride + 8 * kg;  // row-major operands of the B and C tiles, + 16 kk
  const int tj = lane & 15, t_row = 4 * kg + (tj >> 2), t_half = (lane >> 4) & 1;  // transposed reads: quad tj of the group
  const int quad_n = 8 * (tj & 1) + 4 * ((tj >> 1) & 1);  // where columns 4 (tj & 3) .. of a group of 16 lie in the B tile
  const uint32_t a_bt = t_row * L::kRowStride + 16 * t_half + quad_n;  // + 32 nt columns, + 8 / 16 token rows
  const uint32_t a_xt = t_row * kXStride + 16 * (tj & 1) + 4 * (2 * t_half + ((tj >> 1) & 1));  // column pi(r)'s quad

  for (int s0 = 0; s0 < p.nsteps; s0 += kTok) {
    __syncthreads();  // the previous block's readers (at first: the turning of the state) are done with LDS
    // ---- registers -> LDS ----
    uint32_t seen = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int item = tid + kThr * k, it = item % kItems, ch = it % (N / 8);
      uint16_t *const dst = sB + (item / kItems) * L::kTile + 2 * (it / (N / 8)) * L::kRowStride + 16 * (ch >> 1) + 4 * (ch & 1);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const u32x4 v = r_bc[k][j];
        // the columns of a group of 16 in the order 0-3, 8-11, 4-7, 12-15
        *reinterpret_cast<u32x2 *>(dst + j * L::kRowStride) = u32x2{v.x, v.y};
        *reinterpret_cast<u32x2 *>(dst + j * L::kRowStride + 8) = u32x2{v.z, v.w};
#pragma unroll
        for (int w = 0; w < 4; ++w) seen = max_bf16(seen, v[w]);
      }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      *reinterpret_cast<u32x4 *>(sX + (16 * k + (lane >> 2)) * kXStride + 8 * (lane & 3)) = r_x[k];
#pragma unroll
      for (int w = 0; w < 4; ++w) seen = max_bf16(seen, r_x[k][w]);
    }
    // ---- decays: lane r (both halves) = step s0 + r; steps beyond the last have step size zero ----
    const float dtv = s0 + r < p.nsteps ? dt_apply_biased(r_dt, dbias, p.dtx) : 0.f;
    const float d = cut_decay(dtv * alog), dh = coarse_part(d);
    const float ch = prefix32(dh), cl = prefix32(d - dh);  // from the start of the block, in two parts
    const float after = suffix32(d), total = read_lane(after + d, 0);
    any_odd |= !(fabsf(dtv) < kDtLimit) || (seen & 0xffffu) >= kIoLimit || seen >= kIoLimit << 16;
    if (kg == 0) {
      s_ch[wave][r] = ch;
      s_in[wave][r] = dtv * exp2_fast(-cl);
      s_w[wave][r] = dtv * exp2_fast(after);
    }
    const float el = exp2_fast(ch), el_low = exp2_fast(cl), e_all = exp2_fast(total);
    if (__builtin_amdgcn_ballot_w64(any_odd) != 0 && lane == 0) s_odd = 1;
    load_block(s0 + kTok);
    __syncthreads();
    if (s_odd != 0) break;  // uniform over the workgroup

    // ---- masked scores, transposed: element i of tile column l = r is step s = 8 (i/4) + 4 kg + i%4 ----
    Op gm[2][3];
    {
      f32x16 gt = {};
#pragma unroll
      for (int kk = 0; kk < N / 16; ++kk) {
        Op b, c;
        b.q = *reinterpret_cast<const u32x4 *>(sB + a_row + 16 * kk);
        c.q = *reinterpret_cast<const u32x4 *>(sC + a_row + 16 * kk);
        gt = mfma(b, c, gt);
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        float v[8];
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          const int sb = 16 * q + 8 * hf + 4 * kg;
          const f32x4 ch_s = *reinterpret_cast<const f32x4 *>(&s_ch[wave][sb]);
          const f32x4 in_s = *reinterpret_cast<const f32x4 *>(&s_in[wave][sb]);
#pragma unroll
          for (int j = 0; j < 4; ++j)
            v[4 * hf + j] = sb + j <= r ? gt[8 * q + 4 * hf + j] * (in_s[j] * exp2_fast(ch - ch_s[j])) : 0.f;
        }
        split3(v, gm[q]);
      }
    }
    // ---- Y^T[p][l]: the state's part, scaled by the decay up to step l = r, then the block's own inputs ----
    f32x16 Y = {};
#pragma unroll
    for (int kk = 0; kk < N / 16; ++kk) {
      Op c, hp[3];
      c.q = *reinterpret_cast<const u32x4 *>(sC + a_row + 16 * kk);
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = H[kk >> 1][8 * (kk & 1) + j];
      split3(v, hp);
#pragma unroll
      for (int part = 2; part >= 0; --part) Y = mfma(hp[part], c, Y);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) Y[i] *= el;
    Op xo[2];  // x^T: headdim column pi(r), steps 16 q + {4kg.., 8 + 4kg..}
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      xo[q].h[0] = lds_read_tr(sX + a_xt + 16 * q * kXStride);
      xo[q].h[1] = lds_read_tr(sX + a_xt + (16 * q + 8) * kXStride);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int part = 2; part >= 0; --part) Y = mfma(xo[q], gm[q][part], Y);
    // ---- y: lane (r, kg) holds columns 16 kg .. 16 kg + 15 of step r ----
    {
      const Rsrc ry = make_rsrc(yb + static_cast<size_t>(s0) * xrow,
                                live ? (min(kTok, p.nsteps - s0) - 1) * xr32 + 2 * kCols : 0u);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const u32x4 xv = *reinterpret_cast<const u32x4 *>(sX + r * kXStride + 16 * kg + 8 * c);
        u32x4 o;
#pragma unroll
        for (int w = 0; w < 4; ++w)
          o[w] = pack2(fmaf(el_low, Y[8 * c + 2 * w], Dh * bf_lo(xv[w])), fmaf(el_low, Y[8 * c + 2 * w + 1], Dh * bf_hi(xv[w])));
        buf_store16(ry, static_cast<uint32_t>(r) * xr32 + 32 * kg + 16 * c, o);
      }
    }
    // ---- the state to the end of the block ----
    Op xm[2][3];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      float v[8];
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const f32x4 w = *reinterpret_cast<const f32x4 *>(&s_w[wave][16 * q + 8 * hf + 4 * kg]);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          v[4 * hf + 2 * k] = w[2 * k] * bf_lo(xo[q].h[hf][k]);
          v[4 * hf + 2 * k + 1] = w[2 * k + 1] * bf_hi(xo[q].h[hf][k]);
        }
      }
      split3(v, xm[q]);
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
      for (int i = 0; i < 16; ++i) H[nt][i] *= e_all;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        Op bt;
        bt.h[0] = lds_read_tr(sB + a_bt + 32 * nt + 16 * q * L::kRowStride);
        bt.h[1] = lds_read_tr(sB + a_bt + 32 * nt + (16 * q + 8) * L::kRowStride);
#pragma unroll
        for (int part = 2; part >= 0; --part) H[nt] = mfma(bt, xm[q][part], H[nt]);
      }
    }
  }
  __syncthreads();

  if (s_odd != 0) {
    // An input or the state holds an infinity, a NaN or a value beyond the limits above: a zero of the mask times an
    // infinity would reach steps and rows that the recurrence keeps clear of it.  The workgroup applies the recurrence as it stands, to the state in memory
    // (which nothing has been written to yet): one row at a time, lanes across dstate.
    if (!live) return;
    for (int s = 0; s < p.nsteps; ++s) {
      const float dtv = dt_apply_biased(p.dt[static_cast<size_t>(s) * p.npairs + pair], dbias, p.dtx);
      const float dA = expf(dtv * Ah);
      const size_t xe = (static_cast<size_t>(s) * p.npairs + pair) * p.P + p0, be = (static_cast<size_t>(s) * p.nbc + bg) * N;
      for (int row = 0; row < kCols; ++row) {
        const float xv = IoBf16::load(p.x, xe + row), ux = dtv * xv;
        float part = 0.f;
        for (int n = lane; n < N; n += 64) {
          const float v = fmaf(dA, st[row * N + n], ux * IoBf16::load(p.B, be + n));
          st[row * N + n] = v;
          part = fmaf(IoBf16::load(p.C, be + n), v, part);
        }
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) part += __shfl_xor(part, m, 64);
        if (lane == 0) IoBf16::store(p.y, xe + row, fmaf(Dh, xv, part));
      }
    }
    return;
  }

  // ---- the state back to memory, whole row segments ----
  const Rsrc rs = make_rsrc(st, live ? kCols * N * 4 : 0);
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4)
      *reinterpret_cast<f32x4 *>(turn + pi_of_row(r) * kTurnStride + 8 * i4 + 4 * kg) =
          f32x4{H[nt][4 * i4], H[nt][4 * i4 + 1], H[nt][4 * i4 + 2], H[nt][4 * i4 + 3]};
#pragma unroll
    for (int k = 0; k < 4; ++k)
      buf_store16<kNt>(rs, st_off + 8 * k * (N * 4) + 128 * nt,
                  *reinterpret_cast<const u32x4 *>(turn + (8 * k + (lane >> 3)) * kTurnStride + 4 * (lane & 7)));
  }
}

}  // namespace

// Fewer steps than this are left to decode_steps_kernel, whose state is bit for bit that of single steps: callers that check
// a few drafted tokens may count on it, and eight steps were held to it before this kernel was there.  That, not the time,
// draws the line (64 layers, batch 1: 4 steps 73 us here, 74 there; 8 steps 75 and 93).
constexpr int kMinSteps = 9;
// With one or two slices per group (a B/C group of its own for heads of 32 or 64 columns) half of a workgroup's waves and
// more have none and take up the room of those that do.  A call of more workgroups than run side by side (two per CU) then
// needs this many steps times slices.  us there / here, 24 layers x batch 8: 24 heads and groups x 64 x 128, 9 steps 88 /
// 93, 16 steps 130 / 94; x 64 x 64, 9 steps 44 / 50, 16 steps 69 / 51; 8 heads and groups x 32 x 128, 9 steps 18.5 / 30, 16
// steps 27 / 30, 40 steps 56 / 45.  (headdim 32 with dstate 64 has no such kernel: a launch per step, 142 us for 9.)
constexpr int kMinWork = 22, kFullGrid = 512;

bool decode_steps_mfma_chosen(int nsteps, int nlayers, const Dims &d) {
  const unsigned long long lim = 0xFFFF0000ull;  // 32 rows of a tensor must be addressable with 32-bit byte offsets
  const unsigned long long npairs = static_cast<unsigned long long>(nlayers) * d.Bt * d.H;
  const unsigned long long nbc = static_cast<unsigned long long>(nlayers) * d.Bt * d.G;
  const unsigned long long slots = static_cast<unsigned long long>(d.hpg) * (d.P / kCols);
  const unsigned long long wgs = nbc * ((slots + kWaves - 1) / kWaves);
  if (slots <= kWaves / 2 && wgs > kFullGrid && nsteps * slots < kMinWork && !(d.P == 32 && d.N == 64)) return false;
  return d.bf16 && nsteps >= kMinSteps && (d.N == 64 || d.N == 128) && d.P % kCols == 0 &&
         npairs * d.P * 2 * kTok <= lim && nbc * d.N * 2 * kTok <= lim && npairs * 4 * kTok <= lim && wgs <= 0x7fffffffull;
}

hipError_t launch_decode_steps_mfma(int nsteps, int nlayers, const Dims &d, float *state, const void *x, const float *dt,
                                    const float *A, const void *B, const void *C, const float *D, void *y,
                                    hipStream_t stream) {
  StepsParams p;
  p.state = state;
  p.x = static_cast<const uint8_t *>(x);
  p.B = static_cast<const uint8_t *>(B);
  p.C = static_cast<const uint8_t *>(C);
  p.dt = dt;
  p.A = A;
  p.D = D;
  p.y = static_cast<uint8_t *>(y);
  p.npairs = static_cast<size_t>(nlayers) * d.Bt * d.H;
  p.nbc = static_cast<size_t>(nlayers) * d.Bt * d.G;
  p.nsteps = nsteps;
  p.Bt = d.Bt;
  p.H = d.H;
  p.P = d.P;
  p.G = d.G;
  p.hpg = d.hpg;
  p.slots = d.hpg * (d.P / kCols);
  p.cpg = (p.slots + kWaves - 1) / kWaves;
  p.dtx = d.dtx;
  const dim3 grid(static_cast<unsigned>(p.nbc * p.cpg)), block(kThr);
  const bool stream_state = p.npairs * d.P * d.N * sizeof(float) > kMemCacheBytes;
  if (d.N == 128 && stream_state)
    hipLaunchKernelGGL((decode_steps_mfma_kernel<128, true>), grid, block, 0, stream, p);
  else if (d.N == 128)
    hipLaunchKernelGGL((decode_steps_mfma_kernel<128, false>), grid, block, 0, stream, p);
  else if (stream_state)
    hipLaunchKernelGGL((decode_steps_mfma_kernel<64, true>), grid, block, 0, stream, p);
  else
    hipLaunchKernelGGL((decode_steps_mfma_kernel<64, false>), grid, block, 0, stream, p);
  return hipGetLastError();
}

}  // namespace ssd
