// MFMA prefill for the Mamba-2 head shape (headdim 64 or a multiple of it, dstate 128 -- other state
// sizes are mapped onto it, see "state slices" at the launcher -- bf16 io; any chunk length, any number of
// heads per group).  A head with headdim 64 k is
// processed as k independent heads of 64 columns ("head" below means such a 64-column slice): its
// columns never interact, x, y and the state are laid out exactly as those of k narrower heads, and
// the slices share the head's decay records, A and D.
//
// The chunked algorithm (Alg. 1; Eq. 3) is evaluated on 64-token blocks.  Below the diagonal
// blocks the decay mask of Eq. 3 has rank one per block pair, so the off-diagonal part of the
// masked product equals "C_l . (state entering the block)": a wave walks the blocks of its
// head in order with the fp32 state H (headdim x dstate) resident in MFMA accumulators -- the
// inter-chunk state pass happens in registers with no per-chunk launch -- and only the
// diagonal 64x64 blocks need the mask.  Inside a diagonal block the mask is factorised around
// the middle of the block (c31 = prefix sum at token 31):
//     exp(cs_l - cs_s) = exp(cs_l - c31) * exp(c31 - cs_s)
// The second factor is folded into the input once per token (Xm = dt_s exp(c31 - cs_s) x_s),
// the first one scales output rows, and what remains of the mask -- the causal zero pattern --
// is head independent and baked into G = tril(C B^T), computed once per group.  So the mask is
// never materialised, costs no per-element work per head, and every exponent that is evaluated
// is bounded by the decay of 32 tokens; blocks where that leaves the fp32 range ("steep" blocks, far beyond
// the benchmark's dt*|A| <= 1.6 per token) keep the mask un-factorised, see block_cumsum_block.
// With Ht = exp(c31) * (state entering the block), per block and head:
//     Y^T  = Ht C^T + Xm^T G^T            (state -> output, K = dstate; intra-block, K <= 64)
//     y    = exp(cs_l - c31) o Y + D x     (epilogue)
//     H'   = Ht + B^T Xm                   (chunk-state accumulation, K = 64)
//     Ht_next = exp(c63 - c31) exp(c31_next) H'
// all on v_mfma_f32_32x32x16_bf16 with fp32 accumulation (76 MFMAs per block and head); decay
// arithmetic is fp32.
//
// Work decomposition: one WAVE per (head, half of headdim), four heads of one B/C group per
// workgroup of eight waves, one workgroup per CU (two waves per SIMD).  A wave owns a 128 x 32
// slice of the state and never exchanges data with another wave.  The C, B^T and G tiles are
// staged once per workgroup in double-buffered LDS and shared by the four heads; each wave
// stages its own slice of the scaled input.  Global loads for block j+2 are issued while block
// j+1 is being computed; two barriers per block (tiles of the next block visible; both halves of the
// output rows in LDS).
//
// Kernels (launch order):
//   block_prep     one launch for both preparation steps: per (batch, group, block) G = tril(C B^T)
//                  (diagonal blocks only, bf16) and a transposed copy of B, both shared by all heads of
//                  the group; per (batch, head, block) the prefix sums of dt*A turned into per-token
//                  input factors, per-row output factors and per-block state factors.
//   chunk_scan<true>  ("segment_states") per (batch, 4 or 2 heads, segment): the segment's end state from a
//                  zero start (only the chunk-state accumulation), so that segments can run in parallel.
//   segment_pass   sequential pass over segment end states -> state entering each segment.
//   chunk_scan<false> per (batch, 4 heads, segment): everything above, from the entering state; with two heads per
//                  workgroup it is pair_scan.
// A segment is a whole number of 64-token blocks; with one segment only the first and the last kernel
// run, and with few segments segment_pass does not: the last kernel sums the few states itself.
#include <cmath>
#include <type_traits>

#include "ssd_internal.hpp"

namespace ssd {
namespace {

constexpr int kBlk = 64;   // tokens per block
constexpr int kP = 64;     // headdim
constexpr int kN = 128;    // dstate
constexpr int kThreads = 256;
constexpr int kCStride = kN + 8;     // LDS row strides in bf16 elements (16-byte pad against
constexpr int kBtStride = kBlk + 8;  // bank conflicts of the row-per-lane operand reads)
constexpr int kXStride = kBlk + 8;
constexpr float kLog2e = 1.4426950408889634f;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
// Native vectors (not the HIP struct types: copies of those go through memcpy and may end up in
// scratch memory instead of registers).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x4 mk4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) { return u32x4{a, b, c, d}; }
__device__ __forceinline__ u32x2 mk2(uint32_t a, uint32_t b) { return u32x2{a, b}; }

// One MFMA input operand: 8 bf16 per lane.
union Operand {
  bf16x8 v;
  u32x4 q;
  uint32_t u[4];
};

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {  // two fp32 -> packed bf16, RNE
  f32x2 v = {lo, hi};
  bf16x2 b = __builtin_convertvector(v, bf16x2);
  return __builtin_bit_cast(uint32_t, b);
}
__device__ __forceinline__ float bf_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }
__device__ __forceinline__ float fast_exp2(float v) { return __builtin_amdgcn_exp2f(v); }

// D(32x32) += A(32x16) * B(16x32).  Lane (r = lane%32, kg = lane/32) supplies A[r][8kg..8kg+7] and
// B[8kg..8kg+7][r]; it receives D[(i/4)*8 + 4kg + i%4][r] in element i.
__device__ __forceinline__ f32x16 mfma(const Operand &a, const Operand &b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, b.v, c, 0, 0, 0);
}

// ---- state slices ----------------------------------------------------------------------------------
// The kernels are written for 128 state columns.  A launch works on columns [off, off + valid) of a
// dstate axis of `width` columns (valid <= 128; columns beyond `valid` are zero padding): dstate 64 is
// one padded slice, dstate 256 is two slices, each an SSD of its own with the same x and dt, whose
// outputs add up (everything is linear in the triple B, C, state).
struct NSlice {
  int width, off, valid;
};

// ---- tables of a variable-length call -----------------------------------------------------------
// A packed batch (sequences back to back along the token axis, boundaries in a device array of
// cumulative lengths) is handled as a batch whose rows differ in length: every sequence gets whole
// 64-token blocks of its own (the ragged last block of each is masked by the buffer descriptors, as
// for a plain batch) and one or more segments.  Two tiny kernels turn the boundaries into tables:
//   tok0[q], len[q]      first token and length of sequence q; len[nseq]: blocks per segment
//   blk0[q], item0[q]    number of blocks / segments of the sequences before q (entry nseq: totals)
//   slot0[q]             number of state slots before q: a sequence of several segments has one slot
//                        per segment, a sequence of one segment needs none
//   blk_seq[i]           sequence that block i belongs to
//   item_seq[i]          sequence that entry i of the segment list belongs to
// Blocks and segments are numbered over the whole batch; workspace arrays are indexed by those
// numbers (capacities nb_cap, slot_cap are upper bounds that the host can compute from the token
// count and the number of sequences alone).  Boundaries that are not non-decreasing within
// [0, total] give empty tables: every later kernel then finds nothing to do.

__global__ __launch_bounds__(256) void varlen_scan_kernel(const int32_t *__restrict__ cu, int nseq, int total,
                                                          int blk_len, int seg_blocks, int32_t *__restrict__ tok0,
                                                          int32_t *__restrict__ len, int32_t *__restrict__ blk0,
                                                          int32_t *__restrict__ item0, int32_t *__restrict__ slot0) {
  __shared__ int sblk[256], sitem[256], sslot[256];
  __shared__ int bad;
  const int tid = threadIdx.x;
  const int per = (nseq + 255) / 256;
  const int q0 = min(nseq, tid * per), q1 = min(nseq, q0 + per);
  if (tid == 0) bad = 0;
  __syncthreads();
  int nb = 0, ni = 0, ns = 0;
  bool mine_bad = false;
  for (int q = q0; q < q1; ++q) {
    const int a = cu[q], b = cu[q + 1];
    if (a < 0 || b < a || b > total) mine_bad = true;
    const int n = (b - a + blk_len - 1) / blk_len;
    const int segs = max(1, (n + seg_blocks - 1) / seg_blocks);
    nb += n;
    ni += segs;
    ns += segs > 1 ? segs : 0;
  }
  if (mine_bad) atomicOr(&bad, 1);
  sblk[tid] = nb;
  sitem[tid] = ni;
  sslot[tid] = ns;
  __syncthreads();
  if (tid == 0) {  // exclusive prefix over the 256 partial sums
    len[nseq] = seg_blocks;
    int a = 0, b = 0, c = 0;
    for (int i = 0; i < 256; ++i) {
      const int t = sblk[i], u = sitem[i], v = sslot[i];
      sblk[i] = a;
      sitem[i] = b;
      sslot[i] = c;
      a += t;
      b += u;
      c += v;
    }
    blk0[nseq] = bad ? 0 : a;
    item0[nseq] = bad ? 0 : b;
    slot0[nseq] = bad ? 0 : c;
  }
  __syncthreads();
  int rb = sblk[tid], ri = sitem[tid], rs = sslot[tid];
  for (int q = q0; q < q1; ++q) {
    const int a = cu[q], l = cu[q + 1] - a;
    const int n = (l + blk_len - 1) / blk_len;
    const int segs = max(1, (n + seg_blocks - 1) / seg_blocks);
    tok0[q] = bad ? 0 : a;
    len[q] = bad ? 0 : l;
    blk0[q] = bad ? 0 : rb;
    item0[q] = bad ? 0 : ri;
    slot0[q] = bad ? 0 : rs;
    rb += n;
    ri += segs;
    rs += segs > 1 ? segs : 0;
  }
}

// Largest q in [0, nseq) with first[q] <= i: the sequence that contains block (or segment) i.
__device__ __forceinline__ int owner_of(const int32_t *__restrict__ first, int nseq, int i) {
  int lo = 0, hi = nseq;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (first[mid] <= i) lo = mid; else hi = mid;
  }
  return lo;
}
// Segments are listed with every sequence's non-last segments first (all of them are full length,
// seg_blocks blocks) and the last segment of every sequence after them (any length from empty to
// full), longest first while the batch has at most kSortMax sequences (rank by counting, quadratic
// but tiny): workgroups are dispatched in list order, so the long ones start first and the short
// ones fill the gaps; and the states-only pass, which needs no last segment, takes a prefix of the
// list.  Sequence q has item0[q] - q non-last segments before it.
constexpr int kSortMax = 2048;
__host__ __device__ inline bool list_sorted(int nseq, int seg_blocks) { return nseq <= kSortMax && seg_blocks < 32768; }
__global__ __launch_bounds__(256) void varlen_fill_kernel(const int32_t *__restrict__ blk0,
                                                          const int32_t *__restrict__ item0, int nseq,
                                                          int seg_blocks, int32_t *__restrict__ blk_seq,
                                                          int32_t *__restrict__ item_seq) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < blk0[nseq]) blk_seq[i] = owner_of(blk0, nseq, i);
  const int n_items = item0[nseq], n_full = n_items - nseq;
  if (i < n_full) {
    int lo = 0, hi = nseq;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (item0[mid] - mid <= i) lo = mid; else hi = mid;
    }
    item_seq[i] = lo;
  }
  // (no early return above: the barrier below is reached by every thread)
  __shared__ int16_t last_blocks[kSortMax];  // blocks in the last segment of every sequence (<= seg_blocks)
  const bool sort = list_sorted(nseq, seg_blocks);
  const bool ranks_here = static_cast<int>(blockIdx.x) * 256 < n_items && static_cast<int>(blockIdx.x) * 256 + 256 > n_full;
  if (sort && ranks_here)
    for (int k = threadIdx.x; k < nseq; k += 256)
      last_blocks[k] = static_cast<int16_t>((blk0[k + 1] - blk0[k]) - (item0[k + 1] - item0[k] - 1) * seg_blocks);
  __syncthreads();
  if (i >= n_full && i < n_items) {
    const int q = i - n_full;
    int rank = q;
    if (sort) {
      const int mine = last_blocks[q];
      rank = 0;
      for (int k = 0; k < nseq; ++k) {
        const int other = last_blocks[k];
        rank += (other > mine || (other == mine && k < q)) ? 1 : 0;
      }
    }
    item_seq[n_full + rank] = q;
  }
}

// A reduction over the wave, uniform: rotations inside rows of 16 lanes, then the four rows' results.
template <typename Op>
__device__ __forceinline__ int wave_reduce(int v, Op op) {
  v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, false));  // row_ror:8
  v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x124, 0xf, 0xf, false));
  v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x122, 0xf, 0xf, false));
  v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x121, 0xf, 0xf, false));
  return op(op(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
            op(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// Modelled time (us) of a packed batch of `nseq` sequences, `blocks` blocks in all and `longest` in the longest, cut into
// segments of s blocks, `items` of them.  The scan: the busiest CU's load -- a workgroup's start counts as some blocks --
// and the longest walk; with segments that are not the last of their sequence also the states-only pass, the same way, and
// the chain.  An entry to a workgroup: fitted to 70 drawn batches (2 to 64 sequences, 740 to 29700 tokens, 4 to 102 heads; ragged,
// equal, one or a few long among short ones) at eight lengths each, from the host's shortest on, 7 % rms.  (Four heads to a workgroup, which only a
// test asks for, go by the same.)  A length
// guessed on the host cannot serve both a ragged batch and one long prompt among short ones: the guess of four times the
// mean left 8192 + 63 x 1 tokens x 24 heads uncut, 322 us (now 72; 89 with the length of one sequence).
// Dealt items (see Deal), fitted to 400 batches of more than a round of these (draws, equal lengths, one or a few long among short ones), 1150
// timings at up to eight lengths, 10 % rms.  The deal in rounds is less even than the model has it where a few items are long: of
// lengths within 5 % of the cheapest the shortest is taken, which is 1.1 % behind the fastest timed in the geometric mean, 19 % at worst.
constexpr float kDealtMargin = 1.05f;
__host__ __device__ inline float packed_cost(const SegChoice &c, int s, int blocks, int longest, int nseq, int items) {
  auto both = [](float a, float b) { return sqrtf(a * a + b * b); };
  const float n = static_cast<float>(items), full = static_cast<float>(items - nseq), len = static_cast<float>(s);
  const float walk = s < longest ? len : static_cast<float>(longest), grid = n * c.fill < 1.f ? n * c.fill : 1.f;
  float us;
  if (c.dealt) {
    us = 21.8f + 1.57f * both((blocks + 3.6f * n) * c.fill, walk);
    if (items > nseq) us += 0.0376f * full * c.slices + 0.69f * len * both(1.f, full * c.state_fill);
  } else {
    us = 15.f + (1.13f + 0.24f * grid) * both((blocks + 3.9f * n) * c.fill, walk + 3.9f);
    if (items > nseq) us += 0.0123f * full * c.slices + 0.82f * (len + 6.4f) * both(1.f, full * c.fill);
  }
  return items > c.max_items ? 1.25f * us : us;
}

// Both steps in one workgroup, for batches small enough for it (one thread per sequence; the lists filled in a few
// trips): the scans run across the threads and the searches in LDS.  64 sequences, 16384 tokens: the two kernels above
// take 7.4 + 4.7 us and a launch between them, most of it one thread's serial sum; this one
// 5.6 us (the whole call 185 -> 174; 11 sequences, 763 tokens, 9 heads: 36 -> 30).
// It also chooses the segment length: a wave per candidate.
constexpr int kTableThreads = 1024;
constexpr int kTableBlocks = 16 * kTableThreads;  // most blocks (and list entries) it fills
__global__ __launch_bounds__(kTableThreads) void varlen_tables_kernel(
    const int32_t *__restrict__ cu, int nseq, int total, int blk_len, const SegChoice choice, int32_t *__restrict__ tok0,
    int32_t *__restrict__ len, int32_t *__restrict__ blk0, int32_t *__restrict__ item0, int32_t *__restrict__ slot0,
    int32_t *__restrict__ blk_seq, int32_t *__restrict__ item_seq) {
  constexpr int kWaves = kTableThreads / 64;
  constexpr int kOwn = SegChoice::kMost / kWaves;  // candidates per wave
  __shared__ float s_cost[SegChoice::kMost];
  __shared__ int s_cand[SegChoice::kMost];
  __shared__ int s_blk[kTableThreads + 1], s_item[kTableThreads + 1], s_sum[3][kWaves];
  __shared__ int s_last[kTableThreads];
  __shared__ int s_bad;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) s_bad = 0;
  int mine_k[kOwn];
#pragma unroll
  for (int j = 0; j < kOwn; ++j) mine_k[j] = choice.cand[__builtin_amdgcn_readfirstlane(wave) + kWaves * j];
  __syncthreads();
  int a = 0, l = 0, n = 0;
  if (tid < nseq) {
    a = cu[tid];
    const int b = cu[tid + 1];
    if (a < 0 || b < a || b > total) {
      s_bad = 1;
    } else {
      l = b - a;
      n = (l + blk_len - 1) / blk_len;
    }
    s_last[tid] = n;
  }
  // blocks per segment
  int seg_blocks = choice.cand[0];
  if (choice.count > 1) {
    __syncthreads();
    int longest = 0, blocks = 0;
    for (int q = lane; q < nseq; q += 64) {
      longest = max(longest, s_last[q]);
      blocks += s_last[q];
    }
    longest = wave_reduce(longest, [](int x, int y) { return max(x, y); });
    blocks = wave_reduce(blocks, [](int x, int y) { return x + y; });
#pragma unroll
    for (int j = 0; j < kOwn; ++j) {
      const int s = mine_k[j], k = wave + kWaves * j;
      if (k >= choice.count) break;
      const float inv = 1.f / static_cast<float>(s);
      int items = 0;
      for (int q = lane; q < nseq; q += 64)  // ceil(n / s), at least one (exact: n is at most kTableBlocks)
        items += max(1, static_cast<int>((static_cast<float>(s_last[q] + s) - 0.5f) * inv));
      items = wave_reduce(items, [](int x, int y) { return x + y; });
      if (lane == 0) {
        s_cost[k] = packed_cost(choice, s, blocks, longest, nseq, items);
        s_cand[k] = s;
      }
    }
    __syncthreads();
    // the cheapest, the shortest of equals: a positive float orders like its bits, whose last five give way to the index
    int best = lane < choice.count ? ((__float_as_int(s_cost[lane]) & ~31) | lane) : 0x7fffffff;
    best = wave_reduce(best, [](int x, int y) { return min(x, y); }) & 31;
    if (choice.dealt)  // (the shortest that is about as cheap)
      best = __builtin_ctzll(__builtin_amdgcn_ballot_w64(lane < choice.count && s_cost[lane] <= kDealtMargin * s_cost[best]));
    seg_blocks = s_cand[best];
  }
  const int segs = tid < nseq ? max(1, (n + seg_blocks - 1) / seg_blocks) : 0;
  // exclusive sums over the sequences: blocks, segments, state slots
  const int own[3] = {n, segs, segs > 1 ? segs : 0};
  int sum[3] = {own[0], own[1], own[2]};
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int up = __shfl_up(sum[k], off, 64);
      sum[k] += lane >= off ? up : 0;
    }
  }
  if (lane == 63) {
#pragma unroll
    for (int k = 0; k < 3; ++k) s_sum[k][wave] = sum[k];
  }
  __syncthreads();
  const bool bad = s_bad != 0;
  for (int w = 0; w < wave; ++w) {
#pragma unroll
    for (int k = 0; k < 3; ++k) sum[k] += s_sum[k][w];
  }
  if (tid < nseq) {
    tok0[tid] = bad ? 0 : a;
    len[tid] = bad ? 0 : l;
    blk0[tid] = s_blk[tid] = bad ? 0 : sum[0] - own[0];
    item0[tid] = s_item[tid] = bad ? 0 : sum[1] - own[1];
    slot0[tid] = bad ? 0 : sum[2] - own[2];
    s_last[tid] = n - (segs - 1) * seg_blocks;  // blocks in the last segment
    if (tid == nseq - 1) {
      len[nseq] = seg_blocks;
      blk0[nseq] = s_blk[nseq] = bad ? 0 : sum[0];
      item0[nseq] = s_item[nseq] = bad ? 0 : sum[1];
      slot0[nseq] = bad ? 0 : sum[2];
    }
  }
  __syncthreads();
  const int blocks = s_blk[nseq], n_items = s_item[nseq], n_full = bad ? 0 : n_items - nseq;
  for (int i = tid; i < blocks; i += kTableThreads) blk_seq[i] = owner_of(s_blk, nseq, i);
  for (int i = tid; i < n_full; i += kTableThreads) {
    int lo = 0, hi = nseq;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (s_item[mid] - mid <= i) lo = mid; else hi = mid;
    }
    item_seq[i] = lo;
  }
  if (tid < nseq && !bad) {
    const int mine = s_last[tid];
    int rank = 0;
    for (int k = 0; k < nseq; ++k) {
      const int other = s_last[k];
      rank += (other > mine || (other == mine && k < tid)) ? 1 : 0;
    }
    item_seq[n_full + rank] = tid;
  }
}

// Buffer addressing: a 128-bit descriptor (base, size) in scalar registers plus a 32-bit byte offset
// per lane.  The hardware checks the per-lane offset against the size: loads beyond it return zero
// and stores beyond it are dropped, which is how the ragged last block is handled (a descriptor
// that ends at the last token of the batch row) without clamps or branches.
using Rsrc = __amdgpu_buffer_rsrc_t;
__device__ __forceinline__ Rsrc make_rsrc(const void *base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, static_cast<int>(bytes), 0x00020000);
}
__device__ __forceinline__ u32x4 buf_load16(Rsrc r, uint32_t voff, uint32_t soff) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
}
// kPolicy is the instruction's cache-policy field: 0 = default (write-back through L2 and the memory-side
// cache), kStreamStore = sc0 | nt, a non-temporal store that does not displace what those caches hold.
constexpr int kStreamStore = 3;
constexpr int kYPlain = 0, kYStream = 1, kYAdd = 2;
template <int kPolicy = 0>
__device__ __forceinline__ void buf_store16(Rsrc r, uint32_t voff, u32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, voff, 0, kPolicy);
}

// Memory straight into LDS: the wave's 64 lanes fetch 16 bytes each, from wherever their offsets say, and the 1024 bytes
// land in lane order from the LDS address `to` on (uniform, as is the descriptor; lanes beyond the descriptor write
// zeros).  Nothing passes through registers.  Written as assembly because the compiler, which does not tell the
// LDS buffers apart, would let every later LDS read wait for it: the caller waits itself (vector memory operations
// complete in order), before the barrier that hands the buffer over.  The compiler does not look for hazards inside: a vector
// instruction that writes a scalar register, as the moves to uniform registers and the reload of a spilled one are, is
// followed by five wait states before a vector memory instruction reads it, the write of m0 by one.
__device__ __forceinline__ uint32_t uniform32(uint32_t v) { return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v))); }
__device__ __forceinline__ u32x4 raw_rsrc(const void *base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  return u32x4{uniform32(static_cast<uint32_t>(a)), uniform32(static_cast<uint32_t>(a >> 32)) & 0xFFFFu, uniform32(bytes), 0x00020000u};
}
__device__ __forceinline__ void load_to_lds(u32x4 rsrc, uint32_t voff, uint32_t to) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 4\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
               :: "v"(voff), "s"(rsrc), "s"(uniform32(to)) : "memory", "m0");
}

// Four of them to consecutive places.  The places come from the instructions' offsets, which move the addresses in
// memory as well: voff[k] is to be 1024 k less than the offset that is meant.  (With m0 written before each of them a request
// holds its wave for 95 cycles when the four SIMDs of a CU make them, in pairs behind one write for 45.)
__device__ __forceinline__ void load_to_lds4(u32x4 rsrc, uint32_t v0, uint32_t v1, uint32_t v2, uint32_t v3, uint32_t to) {
  asm volatile("s_mov_b32 m0, %5\n\ts_nop 4\n\tbuffer_load_dwordx4 %0, %4, 0 offen lds\n\tbuffer_load_dwordx4 %1, %4, 0 offen offset:1024 lds\n\t"
               "buffer_load_dwordx4 %2, %4, 0 offen offset:2048 lds\n\tbuffer_load_dwordx4 %3, %4, 0 offen offset:3072 lds"
               :: "v"(v0), "v"(v1), "v"(v2), "v"(v3), "s"(rsrc), "s"(uniform32(to)) : "memory", "m0");
}

// A 64-bit value that is the same in every lane, moved to scalar registers.
__device__ __forceinline__ size_t uniform_size(size_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
  return (static_cast<size_t>(hi) << 32) | lo;
}

// ---- scores_bt: G = tril(C B^T) on the diagonal blocks, and B transposed ------------------------------
// One workgroup per (block, group).  The block covers rows [row0, row0 + 64) of the (tokens, G, N)
// arrays B and C, of which only rows below row_end belong to its sequence; its results go to tile
// number `tile` of Gd (64 l x 64 s, bf16) and of Btr (128 n x 64 s, bf16).  ns: which columns of the
// dstate axis this launch works on (see NSlice); with a slice that is not the whole axis, the slice of C
// is also copied, zero padded to 128 columns, to Cpad (tokens, G, 128), from which the scan then reads it.
// Both tiles are read once, 16 consecutive bytes per thread and whole rows per 16 threads (a lane per
// row, which is what the MFMA operands want, would fetch every 128-byte line of the tiles four times,
// 32 bytes at a time: measured four times slower with many groups), and go through LDS -- B whole, C one
// half of the dstate axis (64 columns) at a time, from the registers that hold the whole tile: the
// workgroup's LDS is what limits how many of these short, latency-bound workgroups a CU holds (six this
// way; four with both tiles whole, which put the launch through two rounds at the benchmark shapes).
//   sB  kBlk rows of kN + 2 elements: the odd dword stride makes the transposed read-back conflict free
//   sC  kBlk rows of 64 + 8 elements, read as operands with 16-byte reads; once the products are done
//       it holds G on its way out (rows of kBlk + 8 elements), so that G too is stored in whole rows
constexpr int kHalfN = kN / 2;
constexpr int kSbStride = kN + 2, kScStride = kHalfN + 8;
constexpr int kGtStride = kBlk + 8;
constexpr int kSbElems = kBlk * kSbStride, kScElems = kBlk * kScStride;
static_assert(kBlk * kGtStride <= kScElems, "G fits where the half tile of C was");
__device__ __forceinline__ void scores_bt_block(uint16_t *sB, uint16_t *sC, size_t row0, size_t row_end, size_t tile,
                                                int g, const uint16_t *__restrict__ B, const uint16_t *__restrict__ C,
                                                uint16_t *__restrict__ Gd, uint16_t *__restrict__ Btr, int G,
                                                const NSlice ns, uint16_t *__restrict__ Cpad) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ws = wave >> 1, wl = wave & 1;
  const int r = lane & 31, kg = lane >> 5;

  // The block's rows of the group's slice of B and of C, addressed as row * row_bytes + 2 * column.  The
  // descriptors end with the slice of the last row that belongs to the sequence, so later rows read as
  // zero; a column beyond the slice is given an offset no descriptor covers.  No load sits behind a
  // branch, so all of them are in flight together.
  const uint32_t row_bytes = static_cast<uint32_t>(G) * ns.width * 2;
  const uint32_t rows_here = row_end > row0 ? static_cast<uint32_t>(row_end - row0 < kBlk ? row_end - row0 : kBlk) : 0;
  // (readfirstlane: 64-bit comparisons are vector instructions, and a descriptor with a part in vector
  // registers is accessed through a loop over the lanes' values)
  const uint32_t span = __builtin_amdgcn_readfirstlane(rows_here ? (rows_here - 1) * row_bytes + static_cast<uint32_t>(ns.valid) * 2 : 0);
  const size_t first = (row0 * G + g) * ns.width + ns.off;
  const Rsrc rB = make_rsrc(B + first, span), rC = make_rsrc(C + first, span);
  constexpr uint32_t kNowhere = 0xFFFFFF00u;
  constexpr int kPieces = kBlk * (kN / 8) / kThreads;
  // thread -> 16-byte piece `ch` of the rows row_first + 16 i
  const int ch = threadIdx.x % (kN / 8), row_first = threadIdx.x / (kN / 8);
  static_assert(kThreads % (kN / 8) == 0, "a thread keeps its piece of the row over its rows");
  constexpr int kRowStep = kThreads / (kN / 8);
  u32x4 vb[kPieces], vc[kPieces];
#pragma unroll
  for (int i = 0; i < kPieces; ++i) {
    const int row = row_first + i * kRowStep;
    const uint32_t off = 8 * ch < ns.valid ? row * row_bytes + ch * 16 : kNowhere;  // columns beyond the slice: zero
    vb[i] = buf_load16(rB, off, 0);
    vc[i] = buf_load16(rC, off, 0);
  }
  if (Cpad != nullptr) {
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      const int row = row_first + i * kRowStep;
      if (row0 + row < row_end) *reinterpret_cast<u32x4 *>(Cpad + ((row0 + row) * G + g) * kN + 8 * ch) = vc[i];
    }
  }
#pragma unroll
  for (int i = 0; i < kPieces; ++i) {
    uint32_t *dst = reinterpret_cast<uint32_t *>(sB + (row_first + i * kRowStep) * kSbStride + 8 * ch);
    dst[0] = vb[i].x;
    dst[1] = vb[i].y;
    dst[2] = vb[i].z;
    dst[3] = vb[i].w;
  }
  // G^T tile (rows s, columns l): lane ends up with four consecutive s for its l.
  f32x16 acc = {};
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    if (half) __syncthreads();  // the first half's operands have been read
    if (ch / (kHalfN / 8) == half) {
#pragma unroll
      for (int i = 0; i < kPieces; ++i)
        *reinterpret_cast<u32x4 *>(sC + (row_first + i * kRowStep) * kScStride + 8 * (ch % (kHalfN / 8))) = vc[i];
    }
    __syncthreads();
    const uint32_t *bp = reinterpret_cast<const uint32_t *>(sB + (32 * ws + r) * kSbStride + kHalfN * half + 8 * kg);
    const uint16_t *cp = sC + (32 * wl + r) * kScStride + 8 * kg;
#pragma unroll
    for (int q = 0; q < kHalfN / 16; ++q) {
      Operand a, c;
      a.q = mk4(bp[8 * q], bp[8 * q + 1], bp[8 * q + 2], bp[8 * q + 3]);
      c.q = *reinterpret_cast<const u32x4 *>(cp + 16 * q);
      acc = mfma(a, c, acc);
    }
  }
  // B^T: the staged block read back n-major
  uint16_t *Bout = Btr + tile * kN * kBlk;
#pragma unroll
  for (int i = 0; i < kN * (kBlk / 8) / kThreads; ++i) {
    const int c8 = threadIdx.x + i * kThreads, n = c8 / (kBlk / 8), s0 = (c8 % (kBlk / 8)) * 8;
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t lo = sB[(s0 + 2 * k) * kSbStride + n], hi = sB[(s0 + 2 * k + 1) * kSbStride + n];
      w[k] = lo | (hi << 16);
    }
    *reinterpret_cast<u32x4 *>(Bout + n * kBlk + s0) = mk4(w[0], w[1], w[2], w[3]);
  }
  __syncthreads();  // every wave has read its operands: sC may take G
  uint16_t *sGt = sC;
  const int l = 32 * wl + r;
#pragma unroll
  for (int i4 = 0; i4 < 4; ++i4) {
    const int s = 32 * ws + i4 * 8 + 4 * kg;
    u32x2 v;  // causal zero pattern: keep s <= l
    v.x = pack2(s + 0 <= l ? acc[4 * i4 + 0] : 0.f, s + 1 <= l ? acc[4 * i4 + 1] : 0.f);
    v.y = pack2(s + 2 <= l ? acc[4 * i4 + 2] : 0.f, s + 3 <= l ? acc[4 * i4 + 3] : 0.f);
    *reinterpret_cast<u32x2 *>(sGt + l * kGtStride + s) = v;
  }
  __syncthreads();
  // G in whole rows
  uint16_t *Gout = Gd + tile * kBlk * kBlk;
#pragma unroll
  for (int i = 0; i < kBlk * (kBlk / 8) / kThreads; ++i) {
    const int ch16 = threadIdx.x + i * kThreads, row = ch16 / (kBlk / 8), piece = ch16 % (kBlk / 8);
    *reinterpret_cast<u32x4 *>(Gout + row * kBlk + 8 * piece) =
        *reinterpret_cast<const u32x4 *>(sGt + row * kGtStride + 8 * piece);
  }
}

// ---- block_cumsum: per (head, block) decay bookkeeping ------------------------------------------
// One workgroup per (block, 16 heads starting at h0).  With cs_s the block-relative inclusive prefix
// sum of dt*A*log2(e) (the "segsum" input) and c31, c63 its values at tokens 31 and 63, every head
// gets one record of kRec floats per block:
//   [0,64)     rowf_l = exp2(cs_l - c31)                   output-row factor of the decay mask
//   [64,128)   f_s    = dt_s * exp2(c31 - cs_s)            input factor of the decay mask
//   [128]      exp2(c63 - c31)     state: middle of the block -> end of the block
//   [129]      c63                 log2 of the block's total decay
//   [130]      exp2(c31)           state: start of the block -> middle of the block
//   [131]      [128] * [130] of the next block: middle of the block -> middle of the next block
// The two mask factors evaluate exponents as large as the decay across half a block.  A block of a head
// whose decay across either half exceeds 2^kSteepExp is STEEP: the factors would leave the fp32 range
// (their product would be wrong by O(1) with nothing non-finite to show for it), so the mask is not
// factorised there -- the full kernel applies exp2(cs_l - cs_s), whose exponent is never positive, to
// the scores of that head in registers (see chunk_scan_kernel) -- and the record holds instead
//   [0,64)     dt_l
//   [64,128)   dt_s * exp2(c63 - cs_s)    input weight relative to the END of the block (never > dt_s)
//   [128]      1     [129] c63     [130] -1 (marks the record)     [131] A * log2(e)
// With these the states-only pass, which multiplies [64,128) by [128] and by the decay of the later
// blocks, needs no change.  No benchmark input is steep (dt <= 0.1, |A| <= 16: 74 at most).
// The block covers rows [row0, row0 + 64) of dt (tokens, H); rows from row_end on are not part of
// the sequence and count as dt = 0 (state-neutral padding).  The caller's dt values pass through
// dt_apply (optional bias, softplus, clamp) as they are read.  dt is transposed through LDS, 64 tokens
// of the block plus the first 32 of the next one (for [131]).  Head h's record goes to record number
// h * rec_stride + rec_off.
constexpr int kRec = 2 * kBlk + 4;
constexpr int kCumHeads = 16;
constexpr float kSteepExp = 96.f;
__device__ __forceinline__ void block_cumsum_block(float (*tile)[kCumHeads + 1], size_t row0, size_t row_end, int h0,
                                                   size_t rec_stride, size_t rec_off, const float *__restrict__ dt,
                                                   const float *__restrict__ A, float *__restrict__ prep, int H,
                                                   const DtXform dtx) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // dt of the block's 64 tokens and of the first 32 of the next block, 16 heads each: six values per
  // thread, requested together (no load sits behind a branch).  The descriptor covers the rows from
  // row0 to the end of the sequence, so later rows read as zero; a head beyond H is given an offset
  // outside it.  Padding must end up as dt = 0 whatever the step-size map makes of a zero.
  constexpr int kTileToks = kBlk + kBlk / 2, kLoads = kTileToks * kCumHeads / kThreads;
  const size_t rows_left = row_end > row0 ? row_end - row0 : 0;
  const Rsrc rdt = make_rsrc(dt + row0 * H, __builtin_amdgcn_readfirstlane(static_cast<uint32_t>((rows_left < kTileToks ? rows_left : kTileToks) * H * 4)));
  constexpr int kPer = kCumHeads / (kThreads / 64);
  float a_head[kPer];  // A of the wave's heads (see below), requested with everything else
#pragma unroll
  for (int k = 0; k < kPer; ++k) a_head[k] = A[min(h0 + wave + k * (kThreads / 64), H - 1)];
  float raw[kLoads], bias[kLoads];
#pragma unroll
  for (int k = 0; k < kLoads; ++k) {
    const int i = threadIdx.x + k * kThreads, tok = i / kCumHeads, hh = i % kCumHeads;
    const bool head_ok = h0 + hh < H;
    raw[k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                           rdt, head_ok ? static_cast<uint32_t>(tok * H + h0 + hh) * 4u : 0xFFFFFF00u, 0, 0));
    bias[k] = dtx.bias != nullptr ? dtx.bias[head_ok ? h0 + hh : H - 1] : 0.f;
  }
#pragma unroll
  for (int k = 0; k < kLoads; ++k) {
    const int i = threadIdx.x + k * kThreads, tok = i / kCumHeads, hh = i % kCumHeads;
    const bool there = static_cast<size_t>(tok) < rows_left && h0 + hh < H;
    tile[tok][hh] = there ? dt_apply_branchless(raw[k], bias[k], dtx) : 0.f;
  }
  __syncthreads();
  // A wave takes the heads wave, wave + 4, wave + 8, wave + 12 of the group of 16.  Their prefix sums
  // are four independent chains of cross-lane steps, written side by side so that the latency of one
  // chain's step is covered by the steps of the others.
  float dtv[kPer], v[kPer], nx[kPer], ah[kPer];
  bool live[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int hh = wave + k * (kThreads / 64);
    live[k] = h0 + hh < H;
    ah[k] = live[k] ? a_head[k] * kLog2e : 0.f;
    dtv[k] = tile[lane][hh];
    v[k] = cut_step(dtv[k], ah[k]) * ah[k];
    // prefix sum at token 31 of the next block: the sum of its first 32 terms
    nx[k] = lane < kBlk / 2 ? cut_step(tile[kBlk + lane][hh], ah[k]) * ah[k] : 0.f;
  }
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const float up = __shfl_up(v[k], off, 64);
      if (lane >= off) v[k] += up;
    }
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) nx[k] += __shfl_xor(nx[k], m, 64);
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const float c0 = __shfl(v[k], 0, 64);
    const float c31 = __shfl(v[k], 31, 64);
    const float c63 = __shfl(v[k], 63, 64);
    if (live[k]) {
      const int h = h0 + wave + k * (kThreads / 64);
      float *rec = prep + (static_cast<size_t>(h) * rec_stride + rec_off) * kRec;
      // (negated test: a NaN prefix sum also takes the steep form, which has no exponent to overflow)
      const bool steep = !(c0 - c31 <= kSteepExp && c31 - c63 <= kSteepExp);
      if (!steep) {
        rec[lane] = fast_exp2(v[k] - c31);
        rec[kBlk + lane] = dtv[k] * fast_exp2(c31 - v[k]);
        if (lane < 4)
          rec[2 * kBlk + lane] = lane == 0   ? fast_exp2(c63 - c31)
                                 : lane == 1 ? c63
                                 : lane == 2 ? fast_exp2(c31)
                                             : fast_exp2(c63 - c31) * fast_exp2(nx[k]);
      } else {
        rec[lane] = dtv[k];
        rec[kBlk + lane] = dtv[k] * fast_exp2(c63 - v[k]);
        if (lane < 4) rec[2 * kBlk + lane] = lane == 0 ? 1.f : lane == 1 ? c63 : lane == 2 ? -1.f : ah[k];
      }
    }
  }
}

// Both preparation steps in one launch (they are independent of each other and each is far too
// small to fill the chip): the first n_scores workgroups compute G and B^T, the others the decay
// records.  NB = blocks per batch row (plain batch) or the block capacity (variable-length batch,
// where workgroups beyond the actual number of blocks have nothing to do).
// grid (n_scores + NB * ceil(H/16) * Bt), n_scores = NB * Bt * G; Bt = 1 for a variable-length batch.
// Workspace tiles are numbered (b * G + g) * NB + block, records (b * H + h) * NB + block.
__global__ __launch_bounds__(kThreads) void block_prep_kernel(const uint16_t *__restrict__ B,
                                                              const uint16_t *__restrict__ C,
                                                              uint16_t *__restrict__ Gd,
                                                              uint16_t *__restrict__ Btr,
                                                              const float *__restrict__ dt,
                                                              const float *__restrict__ A,
                                                              float *__restrict__ prep, int T, int H, int G,
                                                              int NB, int n_scores, const VarPlan vp,
                                                              const NSlice ns, uint16_t *__restrict__ Cpad,
                                                              const DtXform dtx) {
  // score workgroups: the B and C tiles; decay workgroups: the transposed dt (in the same memory)
  __shared__ __align__(16) uint16_t sB[kSbElems];
  __shared__ __align__(16) uint16_t sC[kScElems];
  static_assert(sizeof(float) * (kBlk + kBlk / 2) * (kCumHeads + 1) <= sizeof(uint16_t) * kScElems, "dt tile fits");
  float (*tile)[kCumHeads + 1] = reinterpret_cast<float (*)[kCumHeads + 1]>(sC);
  const int wg = blockIdx.x;
  const bool scores = wg < n_scores;
  const int i = scores ? wg : wg - n_scores;
  // Workgroups that read neighbouring pieces of the same rows of B and C (the groups of a block) or of dt
  // (the sets of 16 heads of a block) have consecutive numbers, so that they run at about the same time.
  const int hgroups = (H + kCumHeads - 1) / kCumHeads;
  const int fan = scores ? G : hgroups;
  const int part = i % fan;          // group, or set of 16 heads
  const int jb = (i / fan) % NB;     // block inside the batch row, or block of the packed batch
  const int b = i / (fan * NB);
  size_t row0, row_end;
  if (vp.tok0 != nullptr) {
    if (jb >= vp.blk0[vp.nseq]) return;
    const int q = vp.blk_seq[jb];
    row0 = static_cast<size_t>(vp.tok0[q]) + static_cast<size_t>(jb - vp.blk0[q]) * kBlk;
    row_end = static_cast<size_t>(vp.tok0[q]) + vp.len[q];
  } else {
    row0 = static_cast<size_t>(b) * T + static_cast<size_t>(jb) * kBlk;
    row_end = static_cast<size_t>(b) * T + T;
  }
  // (the tables are read with vector loads: tell the compiler that the rows are the same for every lane,
  // or every buffer descriptor built from them costs a loop over the lanes' values per access)
  row0 = uniform_size(row0);
  row_end = uniform_size(row_end);
  if (scores)
    scores_bt_block(sB, sC, row0, row_end, (static_cast<size_t>(b) * G + part) * NB + jb, part,
                    B, C, Gd, Btr, G, ns, Cpad);
  else
    block_cumsum_block(tile, row0, row_end, part * kCumHeads, NB, static_cast<size_t>(b) * H * NB + jb, dt, A, prep, H,
                       dtx);
}

// ---- chunk_scan / segment_states ----------------------------------------------------------------
// kPair: with what the two-head scan has besides.  (In the other kernels these members are not there: four heads per workgroup
// with them, and with multiplications instead of their few divisions, 9 x 2912 tokens x 60 heads in four groups 176.7 us, 172.3
// without -- the same loop, another start.)
template <int>
struct Absent {};
template <bool kPair>
struct ScanParamsOf {
  template <int i>
  using PairOnly = std::conditional_t<kPair, uint32_t, Absent<i>>;
  const uint8_t *x;
  const uint8_t *C;
  const float *D;
  const uint8_t *Gd;
  const uint8_t *Btr;
  const float *prep;
  [[no_unique_address]] PairOnly<0> prep_bytes;  // of all decay records
  uint8_t *y;
  const float *h0;         // (sequences, H, P, N) initial states, or nullptr = zeros (read by one-segment sequences)
  const float *Hin;        // state entering each segment of a sequence of several: one slot per segment
  float *final_state;      // (sequences, H, P, N): written by the last segment of each sequence
  float *seg_state;        // states-only: local end state of a segment -> the slot of the NEXT segment
  float *seg_decay;        // states-only: log2 of the segment's total decay, one per slot
  int T, H, G, hpg, NB, seg_blocks, S;  // H, hpg count 64-column slices
  int cpg;                 // workgroups ("head groups of four", or of two) per B/C group: ceil(hpg / 4); the slots of the
                           // last one beyond hpg repeat the group's last slice with every store suppressed
  // The states-only pass may cut every segment into `parts` pieces of `part_blocks` blocks (more,
  // shorter workgroups when the segments alone would leave most of the chip idle); the pass over
  // segment states then chains the pieces, and a sequence has `slots` state slots, of which segment
  // sg of the full scan starts from slot sg * parts.  Plain batches only; parts = 1 otherwise.
  int parts, part_blocks, slots;
  // fold != 0 (plain batches of few segments): no pass over segment states has run.  The first segment
  // starts from h0 itself; segment sg sums the local end states of the pieces before it (slots 1 .. sg
  // parts) and h0, each times the decay of the pieces after it, as it loads them.
  int fold;
  int pdiv, Hrec;          // slices per head (headdim / 64); heads (owners of decay records, A, D)
  NSlice ns;               // columns of h0 / final_state (rows of ns.width floats) this launch works on
  int cols, segs, total, per_xcd;  // workgroup mapping, see wg_coords
  [[no_unique_address]] PairOnly<1> cpg_inv;   // for quotient()
  [[no_unique_address]] PairOnly<2> pdiv_inv;
  [[no_unique_address]] PairOnly<3> cols_inv;
  [[no_unique_address]] PairOnly<4> segs_inv;
  VarPlan vp;              // tok0 == nullptr: plain batch
};
using ScanParams = ScanParamsOf<false>;
using PairParams = ScanParamsOf<true>;
static_assert(sizeof(PairParams) >= sizeof(ScanParams) + 5 * sizeof(uint32_t), "absent members take no room");

// Where a workgroup works: head group `col`, segment `sg` of `S` of sequence `b`, whose `nb` blocks
// start at token `tok0` of the packed token axis (`len` tokens), at workspace tile / record number
// `blk0` (per group / per head: stride `blk_stride`), and whose state slots (one per segment, per
// head: stride `slot_stride`) start at `slot0`.
struct SeqView {
  int col, sg, S, b, nb, seg_blocks;
  size_t tok0, blk0, blk_stride, slot0, slot_stride;
  uint32_t len;
};

// Workgroup -> (head group, segment, sequence).  The chip dispatches consecutive workgroup ids to
// its eight XCDs in turn, and each XCD has its own L2.  The workgroups that share C / B^T / G tiles
// (all head groups of one segment of one sequence) are therefore given ids that are congruent
// modulo 8, so that they run on one XCD and the tiles are fetched into one L2 instead of eight:
// XCD k owns the contiguous range [k * per_xcd, (k + 1) * per_xcd) of the (sequence, segment, head
// group) list, head group fastest.  Ids beyond the list (the grid is rounded up to 8 * per_xcd) idle.
// `last_too`: whether the last segment of a sequence is in the list (not for the states-only pass).
constexpr int kXcds = 8;
template <bool kPair>
__device__ __forceinline__ bool wg_coords_varlen(const ScanParamsOf<kPair> &p, bool last_too, SeqView &v);
template <bool kPair>
__device__ __forceinline__ bool wg_coords(const ScanParamsOf<kPair> &p, bool last_too, SeqView &v) {
  if (p.vp.tok0 != nullptr) return wg_coords_varlen(p, last_too, v);
  const int id = blockIdx.x;
  const int w = (id % kXcds) * p.per_xcd + id / kXcds;
  if (w >= p.total) return false;
  if constexpr (kPair) {
    const int item = quotient(w, p.cols, p.cols_inv);
    v.col = w - item * p.cols;
    v.b = quotient(item, p.segs, p.segs_inv);
    v.sg = item - v.b * p.segs;
  } else {
    v.col = w % p.cols;
    v.sg = (w / p.cols) % p.segs;
    v.b = w / (p.cols * p.segs);
  }
  v.S = p.S;
  v.nb = p.NB;
  v.seg_blocks = p.seg_blocks;
  v.tok0 = static_cast<size_t>(v.b) * p.T;
  v.len = static_cast<uint32_t>(p.T);
  v.blk0 = static_cast<size_t>(v.b) * p.NB;   // times G (tiles) or H (records) in the caller's stride
  v.blk_stride = p.NB;
  v.slot0 = static_cast<size_t>(v.b) * p.slots;
  v.slot_stride = p.slots;
  return true;
}
// Variable-length batch: the list (see varlen_fill_kernel) and with it the split over the XCDs come
// from the device-side tables; the grid was sized for the host's upper bound on its length.
// (The tables don't change while a kernel runs; read as constant memory they come through the scalar cache, where the next
// workgroup finds them: as ordinary loads they cost every workgroup's start 1.1 us.)
__device__ __forceinline__ int table_at(const int32_t *t, int i) {
  return ((const __attribute__((address_space(4))) int32_t *)t)[i];
}
template <bool kPair>
__device__ __forceinline__ bool wg_coords_varlen(const ScanParamsOf<kPair> &p, bool last_too, SeqView &v) {
  const int n_items = table_at(p.vp.item0, p.vp.nseq), seg_blocks = table_at(p.vp.len, p.vp.nseq);
  const int n_full = n_items - p.vp.nseq;
  const int n_list = last_too ? n_items : n_full;
  // The same contiguous split over the XCDs as for a plain batch, so that every XCD gets the same
  // number of workgroups.  The list is sorted by length; for the full pass (whose entries differ in
  // length) it is first dealt into eight hands, hand k holding entries k, k + 8, ..., and the hands
  // are laid end to end: every XCD then works on the same mix of long and short entries, long first.
  // (By the list's actual length: split by its capacity, which would save this trip to memory, four sequences of 2202
  // tokens in 20 segments of a capacity of 24 left some XCDs three rounds of workgroups and others two: 128 -> 153 us.)
  const int total = n_list * p.cols;
  const int per_xcd = (total + kXcds - 1) / kXcds;
  const int id = blockIdx.x;
  if (id / kXcds >= per_xcd) return false;
  const int w = (id % kXcds) * per_xcd + id / kXcds;
  if (w >= total) return false;
  int item;
  if constexpr (kPair) {
    item = quotient(w, p.cols, p.cols_inv);
    v.col = w - item * p.cols;
  } else {
    v.col = w % p.cols;
    item = w / p.cols;
  }
  if (last_too) {
    const int base = n_list / kXcds, rem = n_list % kXcds;  // hands 0..rem-1 hold base + 1 entries
    const int big = rem * (base + 1);
    const int hand = item < big ? item / (base + 1) : rem + (item - big) / base;
    const int pos = item < big ? item % (base + 1) : (item - big) % base;
    item = pos * kXcds + hand;
  }
  const int q = table_at(p.vp.item_seq, item);
  const int first = table_at(p.vp.item0, q);
  v.b = q;
  v.seg_blocks = seg_blocks;
  v.S = table_at(p.vp.item0, q + 1) - first;
  v.sg = item < n_full ? item - (first - q) : v.S - 1;
  v.len = static_cast<uint32_t>(table_at(p.vp.len, q));
  v.nb = static_cast<int>((v.len + kBlk - 1) / kBlk);
  v.tok0 = static_cast<size_t>(table_at(p.vp.tok0, q));
  v.blk0 = static_cast<size_t>(table_at(p.vp.blk0, q));
  v.blk_stride = static_cast<size_t>(p.vp.nb_cap);
  v.slot0 = static_cast<size_t>(table_at(p.vp.slot0, q));
  v.slot_stride = static_cast<size_t>(p.vp.slot_cap);
  return true;
}

constexpr int kHeadsPerWg = 4;
constexpr int kGStride = kBlk + 8;

// Waits until no vector memory operation of the wave is outstanding.  Used once, at the end of a
// loop prologue: the compiler places its waits for the worst case over all paths into a loop, and the
// order in which a prologue happened to request its loads would otherwise dictate (too strict) waits
// to every iteration.  (vmcnt = 0, expcnt and lgkmcnt not waited for.)
__device__ __forceinline__ void wait_all_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// The MFMA writes row m of a 32-row result to lane group kg = (m >> 2) & 1, element 4 (m >> 3) + (m & 3).
// Giving MFMA row m the headdim column pi(m) = 16 kg + element makes every lane own 16 consecutive
// columns of its token: 32 contiguous bytes of y per lane instead of four 8-byte pieces.
__device__ __forceinline__ int swap_row(int m) { return (m & ~12) | (m & 4) << 1 | (m & 8) >> 1; }
__device__ __forceinline__ int pi_of_row(int m) { return 16 * ((m >> 2) & 1) + 4 * (m >> 3) + (m & 3); }

// One wave per (head, half of headdim): the wave owns a 128 x 32 slice of the state (64
// accumulator registers), a 64 x 32 output tile (32) and its input operands (16); with the next
// block's data in flight it stays under 256 registers, so the eight waves of a workgroup run two
// per SIMD and one wave's MFMAs overlap the other's vector work and memory waits.
//
// What bounds the kernel is the memory path (every CU has to pull its share of x and push its share
// of y, and a CU sustains only ~1/256 of the chip's bandwidth), so the loop is arranged to keep
// requests outstanding all the time and to move no byte twice: the skip term D x reads x from a raw
// copy that the staging step leaves in LDS instead of loading it again, the loads of the block after
// next are issued in the middle of an iteration, as soon as their registers are free, and the stores
// of y are spread over the second half.
#ifndef SSD_ROW_STORES
#define SSD_ROW_STORES 1
#endif
// y leaves as whole 128-byte rows (the two waves of a head exchange their halves through LDS, one more
// barrier per block) instead of 64-byte half rows per wave.
constexpr bool kRowStores = SSD_ROW_STORES != 0;
constexpr int kRawStride = 40;                       // raw x rows: 32 columns + 16 bytes, in bf16 elements
constexpr int kGLowStride = 32 + 8;                  // G rows 0..31 keep only columns 0..31 (the rest is masked)
constexpr int kGTile = 32 * kGLowStride + 32 * kGStride;  // elements of a compacted G tile
// HPW = heads per workgroup (two waves each): four, where two waves share a SIMD; in the states-only pass also two, for
// launches that would otherwise leave half of the chip idle (see small_grid).  (The full scan with two heads: pair_walk.)
// kYMode, how y leaves: kYPlain -- ordinary stores; kYStream -- non-temporal stores, so that writing y does not
// evict x, which the states-only pass has just pulled into the memory-side cache, before this kernel reads it
// again (chosen per launch, see stream_y()); kYAdd -- added to what y already holds (the later state slices
// of a dstate above 128: the sum of the slices' outputs is formed where the last one is stored).
// The LDS tiles of a scan workgroup, as pointers that keep their address space across a function call.
typedef __attribute__((address_space(3))) uint16_t lds_u16;
struct LdsTiles {
  lds_u16 *sC, *sBt, *sG, *sXm, *sRaw;
};
template <bool kStatesOnly, int HPW>
struct ScanLds {
  static constexpr int kCElems = kStatesOnly ? 8 : kBlk * kCStride, kCBufs = kStatesOnly ? 1 : 2;
  static constexpr int kBtElems = kN * kBtStride;
  static constexpr int kGElems = kStatesOnly ? 8 : kGTile, kGBufs = kStatesOnly ? 1 : 2;
  static constexpr int kXmElems = kP * kXStride;
  static constexpr int kXmBufs = kStatesOnly ? 2 : 1;  // the states-only pass reads the other wave's half: two copies
  static constexpr int kRawElems = kStatesOnly ? 8 : kBlk * kRawStride, kRawBufs = kStatesOnly ? 1 : 2 * HPW;
};

// The walk of one workgroup over its blocks.  kMixed: the walk may meet steep blocks (see
// block_cumsum_block) and chooses the form block by block; otherwise every block has the common form.
template <bool kStatesOnly, int HPW, int kYMode, bool kMixed>
__device__ __forceinline__ void scan_walk(const ScanParams &p, const SeqView &sv, const LdsTiles lds) {
  static_assert(!(kStatesOnly && kYMode != kYPlain), "the states-only pass writes no y");
  static_assert(!(kStatesOnly && kMixed), "the states-only pass needs no second form");
  constexpr int kThr = 128 * HPW;
  constexpr int kBtPieces = kN * kBlk * 2 / 16 / kThr;  // 16-byte pieces per thread of the B^T tile,
  constexpr int kCPieces = kBlk * kN * 2 / 16 / kThr;   // of the C tile
  constexpr int kGPieces = kBlk * kBlk * 2 / 16 / kThr; // and of the G tile
  constexpr int kPieces = kBtPieces + kCPieces + kGPieces;
  using L = ScanLds<kStatesOnly, HPW>;
  // (generic pointers derived from the address-space pointers: the compiler keeps them LDS accesses)
  uint16_t (*const sC)[L::kCElems] = reinterpret_cast<uint16_t (*)[L::kCElems]>((uint16_t *)lds.sC);
  uint16_t (*const sBt)[L::kBtElems] = reinterpret_cast<uint16_t (*)[L::kBtElems]>((uint16_t *)lds.sBt);  // B^T [n][s]
  uint16_t (*const sG)[L::kGElems] = reinterpret_cast<uint16_t (*)[L::kGElems]>((uint16_t *)lds.sG);
  uint16_t (*const sXm)[L::kXmElems] = reinterpret_cast<uint16_t (*)[L::kXmElems]>((uint16_t *)lds.sXm);  // Xm^T [row][s], per head
  uint16_t (*const sRaw)[L::kRawElems] = reinterpret_cast<uint16_t (*)[L::kRawElems]>((uint16_t *)lds.sRaw);  // x [s][col], per wave

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: addresses derived from it stay scalar
  const int hw = wave >> 1, ph = wave & 1;  // head inside the workgroup, half of headdim
  // Waves w and w + 4 of the workgroup share a SIMD.  Giving one of the two the higher issue priority
  // for the whole kernel lets it run ahead between barriers instead of both contending for the same
  // pipe in the same phase (measured: 3 % on 8 x 4096 tokens x 48 heads, nothing lost elsewhere).
  if (wave >= 4) __builtin_amdgcn_s_setprio(1);
  const int col = sv.col, sg = sv.sg;
  // The heads of a workgroup share one B/C group.  A group whose number of (64-column) slices is not a
  // multiple of four leaves slots of its last workgroup without a slice: those waves repeat the group's last
  // slice -- they take part in the shared staging and the barriers like any other -- and write nothing.
  const int g = col / p.cpg;
  const int slot = (col % p.cpg) * HPW + hw;
  const bool live = slot < p.hpg;
  const int h = g * p.hpg + min(slot, p.hpg - 1);
  // workspace numbering: tiles (b, g, block), records (b, h, block), state slots (b, h, segment) for a
  // plain batch; (g, block), (h, block), (h, segment) with batch-wide block / segment numbers otherwise
  const bool plain = p.vp.tok0 == nullptr;
  const size_t tile0 = plain ? (sv.blk0 * p.G + static_cast<size_t>(g) * sv.blk_stride) : (g * sv.blk_stride + sv.blk0);
  const int hrec = h / p.pdiv;  // the head this slice belongs to
  const size_t rec0 = plain ? (sv.blk0 * p.Hrec + static_cast<size_t>(hrec) * sv.blk_stride) : (hrec * sv.blk_stride + sv.blk0);
  const size_t slot0 = plain ? (sv.slot0 * p.H + static_cast<size_t>(h) * sv.slot_stride) : (h * sv.slot_stride + sv.slot0);
  const size_t bh = static_cast<size_t>(sv.b) * p.H + h;  // row of final_state
  const int r = lane & 31, kg = lane >> 5;
  // (the states-only pass walks a piece of a segment, the full scan a whole segment)
  const int walk = kStatesOnly && plain ? p.part_blocks : sv.seg_blocks;
  const int jb0 = min(sv.nb, sg * walk);
  const int jb1 = min(sv.nb, jb0 + walk);
  const int cg = lane & 3, tg = lane >> 2;  // x staging: columns 8cg..8cg+7 of the half, tokens 4tg..4tg+3
  uint16_t *const myX = sXm[hw] + 32 * ph * kXStride;  // this wave's 32 rows of Xm^T
  uint16_t *const myRaw = sRaw[kStatesOnly ? 0 : wave];

  // ---- addressing: scalar bases, per-lane byte offsets that never change ----
  const uint32_t xrow = static_cast<uint32_t>(p.H) * (kP * 2);   // bytes per token of x / y
  const uint32_t crow = static_cast<uint32_t>(p.G) * (kN * 2);   // bytes per token of C
  const uint32_t xbytes = sv.len * xrow;                         // the sequence's rows of x / y
  const uint32_t cbytes = sv.len > 0 ? sv.len * crow - static_cast<uint32_t>(g) * (kN * 2) : 0;
  const uint8_t *const xb = p.x + sv.tok0 * xrow;
  uint8_t *const yb = p.y + sv.tok0 * xrow;
  const uint8_t *const cb = p.C + (sv.tok0 * p.G + g) * (kN * 2);
  const Rsrc rs_bt = make_rsrc(p.Btr + tile0 * (kN * kBlk * 2), static_cast<uint32_t>(sv.nb) * (kN * kBlk * 2));
  const Rsrc rs_g = make_rsrc(p.Gd + tile0 * (kBlk * kBlk * 2), static_cast<uint32_t>(sv.nb) * (kBlk * kBlk * 2));
  const float *const prep_bh = p.prep + rec0 * kRec;
  const Rsrc rs_prep = make_rsrc(prep_bh, static_cast<uint32_t>(sv.nb) * (kRec * 4));
  // descriptors of x, y and C start at the block and end at the sequence's last token
  auto x_rsrc = [&](int jb) { return make_rsrc(xb + static_cast<size_t>(jb) * kBlk * xrow, xbytes - static_cast<uint32_t>(jb) * kBlk * xrow); };
  auto y_rsrc = [&](int jb) { return make_rsrc(yb + static_cast<size_t>(jb) * kBlk * xrow, live ? xbytes - static_cast<uint32_t>(jb) * kBlk * xrow : 0u); };
  auto c_rsrc = [&](int jb) { return make_rsrc(cb + static_cast<size_t>(jb) * kBlk * crow, cbytes - static_cast<uint32_t>(jb) * kBlk * crow); };
  const uint32_t vt = static_cast<uint32_t>(tid) * 16;  // shared tiles: 16 bytes per thread, tid-major
  const uint32_t xcol = static_cast<uint32_t>(h) * (kP * 2) + 64 * ph;
  uint32_t vx[4], vc[kCPieces];
#pragma unroll
  for (int i = 0; i < 4; ++i) vx[i] = static_cast<uint32_t>(4 * tg + i) * xrow + xcol + 16 * cg;
#pragma unroll
  for (int k = 0; k < kCPieces; ++k) {
    const int c = tid + kThr * k;
    vc[k] = static_cast<uint32_t>(c >> 4) * crow + 16 * (c & 15);
  }
  const uint32_t vf = static_cast<uint32_t>(kBlk + 4 * tg) * 4;  // input factors of this thread's four tokens
  // G: thread -> (row, 16-byte piece); in rows 0..31 only pieces 0..3 are kept (s <= l < 32), the
  // threads of the other pieces duplicate a kept one (same data to the same place)
  uint32_t vg[kGPieces], lds_g[kGPieces];
#pragma unroll
  for (int k = 0; k < kGPieces; ++k) {
    const int g_row = (tid + kThr * k) >> 3, g_pc = (g_row < 32) ? (tid & 3) : (tid & 7);
    vg[k] = static_cast<uint32_t>(g_row * kBlk + 8 * g_pc) * 2;
    lds_g[k] = (g_row < 32 ? g_row * kGLowStride : 32 * kGLowStride + (g_row - 32) * kGStride) + 8 * g_pc;
  }

  // ---- data of a block in flight (registers) ----
  u32x4 r_c[kCPieces], r_bt[kBtPieces], r_g[kGPieces];  // shared tiles: this thread's 16-byte pieces
  // own slice: 4 tokens x 8 columns, and the input factors of the 4 tokens (fp32 bits); two blocks
  // of them are in flight (x comes from HBM and is the stream that must never run dry)
  constexpr int kSets = 2;
  u32x4 r_x[kSets][4];
  u32x4 r_f[kSets];

  // Global loads of block jb, in three portions so that they can be spread over the instruction stream.
  auto load_part = [&](int part, int jb, int set = 0) __attribute__((always_inline)) {
    if (part == 0) {
      const Rsrc rx = x_rsrc(jb);
#pragma unroll
      for (int i = 0; i < 4; ++i) r_x[set][i] = buf_load16(rx, vx[i], 0);
      r_f[set] = buf_load16(rs_prep, vf, jb * (kRec * 4));
    } else if (part == 1) {
#pragma unroll
      for (int k = 0; k < kBtPieces; ++k) r_bt[k] = buf_load16(rs_bt, vt, jb * (kN * kBlk * 2) + k * (kThr * 16));
    } else if (!kStatesOnly) {
      const Rsrc rc = c_rsrc(jb);
#pragma unroll
      for (int k = 0; k < kCPieces; ++k) r_c[k] = buf_load16(rc, vc[k], 0);
#pragma unroll
      for (int k = 0; k < kGPieces; ++k) r_g[k] = buf_load16(rs_g, vg[k], jb * (kBlk * kBlk * 2));
    }
  };

  // LDS destinations of this thread's pieces (fixed)
  uint32_t lds_bt[kBtPieces], lds_c[kCPieces];
#pragma unroll
  for (int k = 0; k < kBtPieces; ++k) {
    const int c = tid + kThr * k;
    lds_bt[k] = (c >> 3) * kBtStride + 8 * (c & 7);
  }
#pragma unroll
  for (int k = 0; k < kCPieces; ++k) {
    const int c = tid + kThr * k;
    lds_c[k] = (c >> 4) * kCStride + 8 * (c & 15);
  }
  // Xm^T: column 8cg + c of the half goes to row pi^-1(8cg + c) = 16 (cg & 1) + 4 (cg >> 1) + 8 (c >> 2) + (c & 3)
  uint16_t *const xm_dst = myX + (16 * (cg & 1) + 4 * (cg >> 1)) * kXStride + 4 * tg;
  uint16_t *const raw_dst = myRaw + (4 * tg) * kRawStride + 8 * cg;

  // Registers -> LDS for the block in flight, in slices.  Slice c < 8 computes column c of the own
  // slice, Xm^T[row][s] = f_s x[s][col] (four tokens per 8-byte write).
  // (xbuf: which copy of Xm^T, for the states-only pass; the full kernel has one)
  auto stage_column = [&](int c, int set = 0, int xbuf = 0) __attribute__((always_inline)) {
    const float f0 = __uint_as_float(r_f[set].x), f1 = __uint_as_float(r_f[set].y),
                f2 = __uint_as_float(r_f[set].z), f3 = __uint_as_float(r_f[set].w);
    const int w = c >> 1;
    const uint32_t a0 = r_x[set][0][w], a1 = r_x[set][1][w], a2 = r_x[set][2][w], a3 = r_x[set][3][w];
    uint16_t *dst = xm_dst + xbuf * (HPW * L::kXmElems) + (8 * (c >> 2) + (c & 3)) * kXStride;
    if (c & 1)
      *reinterpret_cast<u32x2 *>(dst) =
          mk2(pack2(f0 * bf_hi(a0), f1 * bf_hi(a1)), pack2(f2 * bf_hi(a2), f3 * bf_hi(a3)));
    else
      *reinterpret_cast<u32x2 *>(dst) =
          mk2(pack2(f0 * bf_lo(a0), f1 * bf_lo(a1)), pack2(f2 * bf_lo(a2), f3 * bf_lo(a3)));
  };
  auto stage_tile = [&](int piece, int buf) __attribute__((always_inline)) {  // B^T's pieces first, then C's, then G's
    if (piece < kBtPieces) {
      *reinterpret_cast<u32x4 *>(&sBt[buf][lds_bt[piece]]) = r_bt[piece];
    } else if constexpr (!kStatesOnly) {
      const int c = piece - kBtPieces, k = c - kCPieces;
      if (k < 0) {
        *reinterpret_cast<u32x4 *>(&sC[buf][lds_c[c]]) = r_c[c];
      } else {
        *reinterpret_cast<u32x4 *>(&sG[buf][lds_g[k]]) = r_g[k];
      }
    }
  };
  auto stage_raw = [&](int set = 0) __attribute__((always_inline)) {  // the unscaled rows, for the skip term of the block's epilogue
    if constexpr (!kStatesOnly) {
#pragma unroll
      for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4 *>(raw_dst + i * kRawStride) = r_x[set][i];
    }
  };

  // Per-block state factors (record entries 128..131): uniform over the wave, but fetched with
  // ordinary (broadcast) vector loads and requested well ahead of their use.  A scalar load would share
  // its counter with the LDS operations and, returning out of order, turn every LDS wait into a wait
  // for everything including the scalar load's trip to memory.
  auto factor_ptr = [&](int jb) { return prep_bh + static_cast<size_t>(jb) * kRec + 2 * kBlk; };
  // Output-row factors of this lane's two tokens (r, 32 + r): of the current block, and of the next
  // one.  The next block's are requested early in an iteration, BEFORE the stores of y and the loads
  // of x: vector memory operations complete in order, so a small load issued after them could only be
  // waited for together with them.
  float rowf0 = 0.f, rowf1 = 0.f, rowf0n = 0.f, rowf1n = 0.f;
  auto load_rowf = [&](int jb) __attribute__((always_inline)) {
    if constexpr (!kStatesOnly) {
      const float *rec = prep_bh + static_cast<size_t>(jb) * kRec;
      rowf0n = rec[r];
      rowf1n = rec[32 + r];
    }
  };

  // ---- state slice: Hacc[nt][i] = Ht^T[n = 32nt + (i/8)*16 + 8kg + i%8][headdim column 32 ph + pi_of_row(r)]: the full
  //      kernel reads the rows of B^T in the order that leaves eight consecutive state columns in a lane (swap_row), which is how
  //      C's 16-byte pieces hold them.  (The states-only pass reads them as they come: n = 32nt + (i/4)*8 + 4kg + i%4.) ----
  f32x16 Hacc[4];
  u32x4 hraw[16];          // the entering state as loaded (full kernel)
  bool has_state = false;  // uniform over the workgroup
  // Everything the prologue needs from memory -- D, the entering state, the first block factor and (below)
  // the first block -- is requested before any of it is waited for: one trip to memory instead of one each.
  float Dh = kStatesOnly || p.D == nullptr ? 0.f : p.D[hrec];
  if constexpr (!kStatesOnly) {
    // A sequence of one segment starts from h0 itself (this workgroup reads it here and is the only
    // one to write final_state, so the two may share memory); with several segments every segment,
    // the first included, starts from the slot that the pass over segment states has filled.
    // Rows of hrow floats of which hvalid columns exist; no state at all: an empty descriptor, whose
    // loads return zero.
    const float *hbase = nullptr;
    uint32_t hrow = kN, hvalid = kN;
    if (sv.S > 1 && !(p.fold && sg == 0)) {
      hbase = p.Hin + (slot0 + static_cast<size_t>(sg) * p.parts) * (kP * kN);
    } else if (p.h0 != nullptr) {
      hbase = p.h0 + bh * kP * p.ns.width + p.ns.off;
      hrow = static_cast<uint32_t>(p.ns.width);
      hvalid = static_cast<uint32_t>(p.ns.valid);
    }
    const Rsrc rs_h = make_rsrc(hbase != nullptr ? hbase : p.prep, hbase != nullptr ? ((kP - 1) * hrow + hvalid) * 4u : 0u);
    // Requested in whole row segments (16 lanes x 16 bytes = 64 state columns of one headdim column, four
    // columns per instruction); the accumulator layout -- 16-byte pieces of 32 different rows per lane --
    // is reached through LDS below (turn_state), once the first block's loads are on their way as well.
    has_state = hbase != nullptr;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const uint32_t row = 32 * ph + 4 * (k & 7) + (lane >> 4), n0 = 64 * (k >> 3) + 4 * (lane & 15);
      hraw[k] = buf_load16(rs_h, n0 < hvalid ? (row * hrow + n0) * 4u : 0xFFFFFF00u, 0);
    }
  } else {
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
      for (int i = 0; i < 16; ++i) Hacc[nt][i] = 0.f;
  }
  // The accumulators hold the state up to a factor that is applied lazily: `pending` takes the state
  // from where the previous block left it (the middle of that block) to the middle of the current
  // block.  It is multiplied in eight elements at a time, right where those elements are converted
  // to an MFMA operand, so the multiplies hide under the matrix instructions of the same loop.
  float pending = jb0 < jb1 && !kStatesOnly ? factor_ptr(jb0)[2] : 1.f;
  // A steep block (see block_cumsum_block) marks its record with a negative entry there; it starts from
  // the state as it is at the start of the block.  Uniform over the wave, kept in a scalar register.
  bool steep_cur = false;
  if constexpr (kMixed) {
    steep_cur = __builtin_amdgcn_readfirstlane(__float_as_int(pending)) < 0;
    if (steep_cur) pending = 1.f;
  }

  // LDS operand addresses of this lane (element offsets inside a tile)
  const uint32_t a_c = r * kCStride + 8 * kg;    // + 32 rows for the second token half, + 16 kk
  const uint32_t a_g0 = r * kGLowStride + 8 * kg;                     // token r, + 16 q (q < 2)
  const uint32_t a_g1 = 32 * kGLowStride + r * kGStride + 8 * kg;     // token 32 + r, + 16 q
  const uint32_t a_bt = (kStatesOnly ? r : swap_row(r)) * kBtStride + 8 * kg;  // + 32 nt rows, + 16 q
  const uint16_t *const raw_src = myRaw + r * kRawStride + 16 * kg;   // + 32 rows for the second half, + 8 c
  uint16_t *const raw_rw = myRaw + r * kRawStride + 16 * kg;
  // output rows.  Half rows: lane i handles 16 bytes of token i/4 (+16k) of the wave's own half.  Whole
  // rows: the wave handles tokens 32ph + i/8 (+8k), lane i the 16-byte piece i%8 of the 128-byte row --
  // pieces 0..3 come from the tile of the head's first wave, 4..7 from that of its second wave.
  const uint16_t *const raw_dst_row =
      kRowStores && !kStatesOnly
          ? sRaw[kStatesOnly ? 0 : 2 * hw + ((lane & 7) >> 2)] + (32 * ph + (lane >> 3)) * kRawStride + 8 * (lane & 3)
          : myRaw + (lane >> 2) * kRawStride + 8 * (lane & 3);
  const uint32_t vy = kRowStores ? static_cast<uint32_t>(32 * ph + (lane >> 3)) * xrow +
                                       static_cast<uint32_t>(h) * (kP * 2) + 16 * (lane & 7)
                                 : static_cast<uint32_t>(lane >> 2) * xrow + xcol + 16 * (lane & 3);
  constexpr int kRowStep = kRowStores ? 8 : 16;  // tokens between a lane's four pieces
  auto lds16 = [](const uint16_t *ptr) {
    Operand o;
    o.q = *reinterpret_cast<const u32x4 *>(ptr);
    return o;
  };

  float seg_total = 0.f;
  // The loop body below is free of branches around memory operations (block indices are clamped to
  // the segment instead, redundant loads in the last two iterations are harmless): the hardware
  // counts outstanding loads and stores in order, and only with straight-line code can the compiler
  // wait for exactly the older ones and leave the newer ones in flight.
  // It is written as an explicit software pipeline: every group of matrix instructions is preceded by
  // the LDS reads of the NEXT group's operands and accompanied by independent vector work (state
  // scaling and conversion and the staging of the next block in the first phase, the output epilogue
  // in the second); the scheduling fences keep the compiler from undoing that order.
  const int jlast = jb1 - 1;
  if constexpr (kStatesOnly) {
    // ---- states only: the segment's end state from a zero start, H = sum_s w_s x_s (x) B_s with
    //      w_s = dt_s * (decay from token s to the END OF THE SEGMENT).  Taking the weights relative
    //      to the segment end (every exponent <= 0: nothing overflows, what has decayed away
    //      underflows to zero as it should) means the accumulators are never rescaled: per block only
    //      H += B^T Xm.  w_s = f_s * (middle -> end of its block) * exp2(decay of the blocks after it).
    //      The kernel is a pure stream of x (plus the shared B^T tile), so x is requested two blocks
    //      ahead: block k's iteration stages block k+1 from one register set and then refills that set
    //      with block k+3.  Two iterations are written out per loop trip so that the set index is a
    //      compile-time constant. ----
    auto at = [&](int j) { return min(j, jlast); };
    auto load_factors = [&](int j) { return *reinterpret_cast<const f32x2 *>(factor_ptr(j)); };
    // {middle -> end, log2 of the total decay} of the block to be staged next, fetched one iteration
    // before it is used
    f32x2 sf_stage = {1.f, 0.f};
    // The first TWO blocks are requested at once, together with the decays that are summed next: the second
    // block's B^T pieces land in registers of their own until the first block's have gone to LDS, so the
    // prologue costs one trip to memory, not two.
    f32x2 sf_second = {1.f, 0.f};
    u32x4 r_bt_second[kBtPieces];
    if (jb0 < jb1) {
      load_part(0, jb0, 0);
      load_part(1, jb0);
      load_part(0, at(jb0 + 1), 1);
#pragma unroll
      for (int k = 0; k < kBtPieces; ++k)
        r_bt_second[k] = buf_load16(rs_bt, vt, at(jb0 + 1) * (kN * kBlk * 2) + k * (kThr * 16));
      sf_stage = load_factors(jb0);
      sf_second = load_factors(at(jb0 + 1));
    }
    for (int j = jb0; j < jb1; j += 64) {  // the segment's total log2 decay: one lane per block
      float v = j + lane < jb1 ? factor_ptr(j + lane)[1] : 0.f;
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
      seg_total += v;
    }
    float rest = seg_total;  // log2 decay of the blocks after the one being staged
    float ws = 0.f;
    auto next_weight = [&]() __attribute__((always_inline)) {
      rest -= sf_stage.y;
      ws = sf_stage.x * fast_exp2(rest);
    };
    auto weigh = [&](int set) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 4; ++i) r_f[set][i] = __float_as_uint(__uint_as_float(r_f[set][i]) * ws);
    };
    if (jb0 < jb1) {
      next_weight();
      weigh(0);
      sf_stage = sf_second;
#pragma unroll
      for (int c = 0; c < 8; ++c) stage_column(c, 0);
#pragma unroll
      for (int k = 0; k < kBtPieces; ++k) *reinterpret_cast<u32x4 *>(&sBt[0][lds_bt[k]]) = r_bt[k];
#pragma unroll
      for (int k = 0; k < kBtPieces; ++k) r_bt[k] = r_bt_second[k];
      wait_all_loads();  // (everything so far is needed by now: nothing is lost)
      load_part(0, at(jb0 + 2), 0);
    }
    __syncthreads();
    auto body = [&](int par, int jb) __attribute__((always_inline)) {
      const int buf = par, set = par ^ 1;  // block jb sits in LDS buffer `par`; block jb+1 in register set par^1
      const uint16_t *const tBt = sBt[buf];
      next_weight();                          // weight of block jb+1 from the factors fetched an iteration ago
      sf_stage = load_factors(at(jb + 2));    // for the next iteration
      // This pass is bound by its LDS operand reads (without them it takes half the time), so its two
      // waves per head split the state differently from the full kernel: wave `ph` owns state columns
      // [64 ph, 64 ph + 64) for all 64 headdim columns -- two n tiles x two column tiles, 2 + 2 operand
      // reads per group of four matrix instructions where four n tiles x one column tile need 4 + 1.
      // (Staging is unchanged: wave `ph` stages headdim half `ph` of Xm^T; the other half comes from the
      // head's other wave, through the barrier that every block has anyway -- and since that wave may
      // already be staging the next block while this one still reads, Xm^T has two copies in this pass.)
      Operand xo[4][2], bto[4][2];
      const uint16_t *const headX = sXm[buf * HPW + hw];  // block jb's copy; the next block is staged into the other
      auto request = [&](int q) __attribute__((always_inline)) {
#pragma unroll
        for (int pt = 0; pt < 2; ++pt) xo[q][pt] = lds16(headX + (32 * pt + r) * kXStride + 16 * q + 8 * kg);
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) bto[q][nt] = lds16(tBt + a_bt + 32 * (2 * ph + nt) * kBtStride + 16 * q);
      };
      // Hacc[2 pt + nt]: headdim columns 32 pt + pi(r), state columns 32 (2 ph + nt) + row of the element
      auto multiply = [&](int q) __attribute__((always_inline)) {
#pragma unroll
        for (int pt = 0; pt < 2; ++pt)
#pragma unroll
          for (int nt = 0; nt < 2; ++nt) Hacc[2 * pt + nt] = mfma(bto[q][nt], xo[q][pt], Hacc[2 * pt + nt]);
      };
      // The two waves of a SIMD (w and w + 4) take the two halves of an iteration in opposite order: while
      // one reads its operands and keeps the matrix pipe busy, the other stages the next block on the vector
      // ALU.  Both halves only need what the barrier at the end of the previous iteration has published
      // (the matrix half reads LDS copy `buf`, the staging half writes copy `buf ^ 1`), so their order is
      // free; with every wave in the same half at the same time the pipes would take turns idling.
      auto matrix_half = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) request(q);
#pragma unroll
        for (int q = 0; q < 4; ++q) multiply(q);
      };
      const bool matrix_first = wave < 4;
      if (matrix_first) matrix_half();
      __builtin_amdgcn_sched_barrier(0);
      // the next block is staged, then its registers are refilled (tile of block jb+2, x of block jb+3)
      weigh(set);
#pragma unroll
      for (int c = 0; c < 8; ++c) stage_column(c, set, buf ^ 1);
#pragma unroll
      for (int k = 0; k < kBtPieces; ++k) *reinterpret_cast<u32x4 *>(&sBt[buf ^ 1][lds_bt[k]]) = r_bt[k];
      load_part(1, at(jb + 2));
      load_part(0, at(jb + 3), set);
      __builtin_amdgcn_sched_barrier(0);
      if (!matrix_first) matrix_half();
      __syncthreads();
    };
    // pairs of blocks, then the odd one: with the test between the two halves of a pair the compiler
    // would also have to allow for "first half, then first half again", where the set staged at the
    // top has only just been requested, and would wait for the newest loads in every iteration
    int jb = jb0;
    for (; jb + 1 < jb1; jb += 2) {
      body(0, jb);
      body(1, jb + 1);
    }
    if (jb < jb1) body(0, jb);
  }
  if constexpr (!kStatesOnly) {
    auto at = [&](int j) { return min(j, jlast); };
    if (jb0 < jb1) {
      // ---- prologue: block jb0 into LDS buffer 0; blocks jb0+1 and jb0+2 in flight ----
#pragma unroll
      for (int part = 0; part < 3; ++part) load_part(part, jb0, 0);
    }
    // The entering state into the accumulators: every wave turns its 32 x 128 tile, half at a time, through
    // a private piece of LDS (waves 0-3 in what will be the B^T buffers, waves 4-7 in the C buffers; rows of
    // 64 state columns padded by 16 bytes).  The barrier hands those buffers over to the staging below.
    if (has_state) {
      constexpr int kTurnStride = 64 + 4;  // floats
      float *const turn = reinterpret_cast<float *>(wave < 4 ? &sBt[0][0] : &sC[0][0]) + (wave & 3) * (32 * kTurnStride);
#pragma unroll
      for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int k = 0; k < 8; ++k)
          *reinterpret_cast<u32x4 *>(turn + (4 * k + (lane >> 4)) * kTurnStride + 4 * (lane & 15)) = hraw[8 * half + k];
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
          for (int i4 = 0; i4 < 4; ++i4) {
            const f32x4 v = *reinterpret_cast<const f32x4 *>(turn + pi_of_row(r) * kTurnStride + 32 * nt + 16 * (i4 >> 1) + 8 * kg + 4 * (i4 & 1));
            Hacc[2 * half + nt][4 * i4 + 0] = v.x;
            Hacc[2 * half + nt][4 * i4 + 1] = v.y;
            Hacc[2 * half + nt][4 * i4 + 2] = v.z;
            Hacc[2 * half + nt][4 * i4 + 3] = v.w;
          }
      }
      if (p.fold && sg >= 1) {
        // What was loaded is the local end state of the piece that ends where this segment begins; the
        // earlier pieces' (slots sg parts - 1 .. 1) and h0 follow, one at a time through the same registers,
        // each weighted by the decay of everything after it.  (Uniform over the workgroup.)
        float log2_decay = 0.f;
        for (int k = sg * p.parts - 1; k >= 0; --k) {
          log2_decay += p.seg_decay[slot0 + k];
          if (k == 0 && p.h0 == nullptr) break;
          const float *base = k > 0 ? p.Hin + (slot0 + k) * (kP * kN) : p.h0 + bh * kP * p.ns.width + p.ns.off;
          const uint32_t trow = k > 0 ? kN : static_cast<uint32_t>(p.ns.width);
          const uint32_t tvalid = k > 0 ? kN : static_cast<uint32_t>(p.ns.valid);
          const Rsrc rs_t = make_rsrc(base, ((kP - 1) * trow + tvalid) * 4u);
          const float wgt = fast_exp2(log2_decay);
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const uint32_t row = 32 * ph + 4 * (i & 7) + (lane >> 4), n0 = 64 * (i >> 3) + 4 * (lane & 15);
            hraw[i] = buf_load16(rs_t, n0 < tvalid ? (row * trow + n0) * 4u : 0xFFFFFF00u, 0);
          }
#pragma unroll
          for (int half = 0; half < 2; ++half) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
              *reinterpret_cast<u32x4 *>(turn + (4 * i + (lane >> 4)) * kTurnStride + 4 * (lane & 15)) = hraw[8 * half + i];
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
              for (int i4 = 0; i4 < 4; ++i4) {
                const f32x4 v = *reinterpret_cast<const f32x4 *>(turn + pi_of_row(r) * kTurnStride + 32 * nt + 16 * (i4 >> 1) + 8 * kg + 4 * (i4 & 1));
                Hacc[2 * half + nt][4 * i4 + 0] += wgt * v.x;
                Hacc[2 * half + nt][4 * i4 + 1] += wgt * v.y;
                Hacc[2 * half + nt][4 * i4 + 2] += wgt * v.z;
                Hacc[2 * half + nt][4 * i4 + 3] += wgt * v.w;
              }
          }
        }
      }
      __syncthreads();
    } else {
#pragma unroll
      for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int i = 0; i < 16; ++i) Hacc[nt][i] = 0.f;
    }
    if (jb0 < jb1) {
#pragma unroll
      for (int c = 0; c < 8; ++c) stage_column(c, 0);
#pragma unroll
      for (int piece = 0; piece < kPieces; ++piece) stage_tile(piece, 0);
      if constexpr (!kRowStores) stage_raw(0);
      // the following blocks are requested in the order the loop requests blocks (shared tiles, own
      // slices, row factors): the compiler derives its waits from the order of outstanding loads,
      // and they stay exact only if the path into the loop and the path around it agree on it
      load_part(1, at(jb0 + 1));
      load_part(2, at(jb0 + 1));
      load_part(0, at(jb0 + 1), 1);
      if constexpr (!kRowStores) load_part(0, at(jb0 + 2), 0);
      load_rowf(jb0);
    }
    wait_all_loads();
    // Pin the two as "arrived": otherwise the wait for them is placed at their first use inside the
    // loop, where it also waits for every younger load of every iteration.
    asm volatile("" : "+v"(Dh));
    asm volatile("" : "+v"(pending));
    rowf0 = rowf0n;
    rowf1 = rowf1n;
    __syncthreads();

    // One block.  `par` is the parity of the block inside the segment, a compile-time constant (two
    // iterations are written out per loop trip): block jb sits in LDS buffer par, block jb+1 in
    // register set par^1 (it is staged during this iteration, and the set then refilled with block
    // jb+3), block jb+2 in register set par.
    // steep_tag: the block is steep (a compile-time constant per instantiation; the loop below picks the
    // instantiation block by block).  Both forms issue the same memory operations in the same order, so
    // the waits the compiler derives for the common form are not affected by the other.  The steep form
    // differs in four places: the state -> output term is scaled by exp2(cs_l) as soon as it is complete;
    // the masked product takes the raw x and, as its other operand, the scores times
    // dt_s exp2(cs_l - cs_s) -- the un-factorised mask, exponent never positive, applied in registers to
    // this lane's eight scores per operand; the state is taken to the end of the block before the update
    // (whose operand carries end-relative weights, see the record); the output rows need no factor.
    // In a mixed walk the factor owed to the accumulators at the end of the block depends on the form of
    // the next block.
    auto body = [&](int par, int jb, auto steep_tag) __attribute__((always_inline)) {
      constexpr bool kSteep = decltype(steep_tag)::value;
      static_assert(kMixed || !kSteep, "a steep block is only met in the mixed walk");
      float pend_next = 0.f;
      const int buf = par, setA = par ^ 1;
      const bool more = jb < jlast;
      f32x4 fac = {0.f, 0.f, 0.f, 0.f};  // record entries 128..131 of this block
      float nf = 0.f;                    // entry 130 of the next block
      const uint16_t *const tC = sC[buf], *const tG = sG[buf], *const tBt = sBt[buf];
      float dt_t = 0.f, cs_t = 0.f;      // steep: step size and inclusive prefix sum of dt*A*log2(e) of token `lane`
      if constexpr (kSteep) {
        const float alog = factor_ptr(jb)[3];
        dt_t = kg ? rowf1 : rowf0;
        cs_t = cut_step(dt_t, alog) * alog;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const float up = __shfl_up(cs_t, off, 64);
          if (lane >= off) cs_t += up;
        }
      }

      if constexpr (kRowStores) {
        // the raw rows of this block go to LDS only now: until the barrier that ended the previous
        // iteration the other wave of the head was still reading the previous block's y from this
        // tile.  Then the register set is refilled with the block after next.
        stage_raw(par);
        load_part(0, at(jb + 2), par);
      }
      Operand xo[4];  // Xm^T[row r][s = 16q + 8kg ..]
      if constexpr (!kSteep) {
#pragma unroll
        for (int q = 0; q < 4; ++q) xo[q] = lds16(myX + r * kXStride + 16 * q + 8 * kg);
      }
      Operand bto[2][4];  // operands of the state update, double buffered over q
      f32x16 Y[2] = {};

      // ---- phase 1: Y^T[row][l] = sum_n Ht[row][n] C[l][n]  +  sum_{s<=l} Xm[s][row] G[l][s];
      //      alongside, the next block moves from registers to the other LDS buffer, and as soon as
      //      the registers of its shared tiles are free the tiles of block jb+2 are requested ----
      Operand co[2][2], go[2][2];
      co[0][0] = lds16(tC + a_c);
      co[0][1] = lds16(tC + a_c + 32 * kCStride);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        if (kk < 7) {
          co[(kk + 1) & 1][0] = lds16(tC + a_c + 16 * (kk + 1));
          co[(kk + 1) & 1][1] = lds16(tC + a_c + 32 * kCStride + 16 * (kk + 1));
        } else {
          go[0][1] = lds16(tG + a_g1);
          go[0][0] = lds16(tG + a_g0);
        }
        // bf16 copy of a 16-column slice of Ht as an MFMA operand: slice 2nt+u covers n = 32nt + 16u + 8kg + {0..7}
        f32x16 &hv = Hacc[kk >> 1];
        const int u = kk & 1;
        Operand ho;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          hv[8 * u + 2 * k] *= pending;
          hv[8 * u + 2 * k + 1] *= pending;
          ho.u[k] = pack2(hv[8 * u + 2 * k], hv[8 * u + 2 * k + 1]);
        }
        Y[0] = mfma(ho, co[kk & 1][0], Y[0]);
        Y[1] = mfma(ho, co[kk & 1][1], Y[1]);
        constexpr int kPerGroup = kPieces / 5;
        static_assert(kPerGroup * 5 == kPieces, "five groups stage all pieces");
        if (kk < 5) {
#pragma unroll
          for (int k = 0; k < kPerGroup; ++k) stage_tile(kPerGroup * kk + k, buf ^ 1);
        }
        if (kk == 4) {
          load_rowf(at(jb + 1));
          if constexpr (kMixed) {
            fac = *reinterpret_cast<const f32x4 *>(factor_ptr(jb));
            nf = factor_ptr(at(jb + 1))[2];
          } else {
            // to the middle of the next block; after the last block only the way to its end is left
            pend_next = factor_ptr(jb)[more ? 3 : 0];
          }
        }
        if (kk == 5) load_part(1, at(jb + 2));
        if (kk == 6) load_part(2, at(jb + 2));
        // (steep: the state update is the only user of this block's scaled input, which the next block's
        // would overwrite here; it is staged after that update instead)
        if constexpr (!kSteep) stage_column(kk, setA);
        __builtin_amdgcn_sched_barrier(0);
      }
      // the masked product
      u32x4 xe;  // x of the block in output layout (token r + 32lt, columns 32ph + 16kg + 8c ..), read from
                 // the raw copy at the start of the group whose end uses it
      if constexpr (kSteep) {
        const float csl[2] = {__shfl(cs_t, r, 64), __shfl(cs_t, 32 + r, 64)};
        {
          const float s0 = fast_exp2(csl[0]), s1 = fast_exp2(csl[1]);
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            Y[0][i] *= s0;
            Y[1][i] *= s1;
          }
        }
        const uint16_t *const xcol_src = myRaw + pi_of_row(r);  // this lane's column of the raw rows
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float cs_s[8], dt_s[8];
          Operand xr;  // raw x^T[row r][s = 16q + 8kg ..]
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int src = 16 * q + 8 * kg + j;
            cs_s[j] = __shfl(cs_t, src, 64);
            dt_s[j] = __shfl(dt_t, src, 64);
          }
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const uint32_t lo = xcol_src[(16 * q + 8 * kg + 2 * k) * kRawStride];
            const uint32_t hi = xcol_src[(16 * q + 8 * kg + 2 * k + 1) * kRawStride];
            xr.u[k] = lo | (hi << 16);
          }
#pragma unroll
          for (int lt = (q < 2 ? 0 : 1); lt < 2; ++lt) {
            const Operand gq = lds16(lt ? tG + a_g1 + 16 * q : tG + a_g0 + 16 * q);
            Operand gh;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const float w0 = dt_s[2 * k] * fast_exp2(fminf(csl[lt] - cs_s[2 * k], 0.f));
              const float w1 = dt_s[2 * k + 1] * fast_exp2(fminf(csl[lt] - cs_s[2 * k + 1], 0.f));
              gh.u[k] = pack2(bf_lo(gq.u[k]) * w0, bf_hi(gq.u[k]) * w1);
            }
            Y[lt] = mfma(xr, gh, Y[lt]);
          }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) xo[q] = lds16(myX + r * kXStride + 16 * q + 8 * kg);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) bto[0][nt] = lds16(tBt + a_bt + 32 * nt * kBtStride);
        const float e63 = fast_exp2(fac.y);  // the state, so far at the start of the block, to its end
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
          for (int i = 0; i < 16; ++i) Hacc[nt][i] *= e63;
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int q = 0; q < (kSteep ? 0 : 4); ++q) {
        if (q < 3) {
          go[(q + 1) & 1][1] = lds16(tG + a_g1 + 16 * (q + 1));
          if (q + 1 < 2) go[(q + 1) & 1][0] = lds16(tG + a_g0 + 16 * (q + 1));
        } else {
#pragma unroll
          for (int nt = 0; nt < 4; ++nt) bto[0][nt] = lds16(tBt + a_bt + 32 * nt * kBtStride);
        }
        if (q < 2) Y[0] = mfma(xo[q], go[q & 1][0], Y[0]);
        Y[1] = mfma(xo[q], go[q & 1][1], Y[1]);
        __builtin_amdgcn_sched_barrier(0);
      }

      // ---- phase 2: H'^T[n][col] = Ht^T[n][col] + sum_s B^T[n][s] Xm[s][col]; alongside, the output
      //      epilogue of the block (y[l][col] = rowf_l Y + D x; element i of the lane is column
      //      32ph + 16kg + i), one quarter per group ----
      const Rsrc ry = y_rsrc(jb);
      const float rowf[2] = {kSteep ? 1.f : rowf0, kSteep ? 1.f : rowf1};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (q < 3) {
#pragma unroll
          for (int nt = 0; nt < 4; ++nt) bto[(q + 1) & 1][nt] = lds16(tBt + a_bt + 32 * nt * kBtStride + 16 * (q + 1));
        }
        xe = lds16(raw_src + 32 * (q >> 1) * kRawStride + 8 * (q & 1)).q;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) Hacc[nt] = mfma(bto[q & 1][nt], xo[q], Hacc[nt]);
        const int lt = q >> 1, c = q & 1;
        const f32x16 &Yt = Y[lt];
        const u32x4 xv = xe;
        u32x4 o;
#pragma unroll
        for (int w = 0; w < 4; ++w)
          o[w] = pack2(rowf[lt] * Yt[8 * c + 2 * w] + Dh * bf_lo(xv[w]),
                       rowf[lt] * Yt[8 * c + 2 * w + 1] + Dh * bf_hi(xv[w]));
        // the quarter replaces, in place, the x it was computed from: y leaves through the raw copy
        *reinterpret_cast<u32x4 *>(raw_rw + 32 * lt * kRawStride + 8 * c) = o;
        __builtin_amdgcn_sched_barrier(0);
      }

      // ---- y goes out in row layout, read back from LDS: the output layout of the MFMA would give
      //      32-byte pieces, which the memory system handles much worse next to the concurrent reads of
      //      x than 64-byte half rows, and those worse than whole 128-byte rows.  For whole rows the
      //      two waves of a head wait for each other's halves (the barrier below) and each stores the
      //      rows of 32 tokens; the raw rows of the next block then go to LDS at the top of the next
      //      iteration instead of here.  Tokens beyond the sequence are beyond the descriptor and are
      //      dropped. ----
      if constexpr (kSteep) {
#pragma unroll
        for (int c = 0; c < 8; ++c) stage_column(c, setA);
      }
      u32x4 yprev[4];  // kYAdd: what y holds so far, requested before the barrier
      if constexpr (kYMode == kYAdd) {
#pragma unroll
        for (int k = 0; k < 4; ++k) yprev[k] = buf_load16(ry, vy + static_cast<uint32_t>(kRowStep * k) * xrow, 0);
      }
      if constexpr (kRowStores) __syncthreads();  // both halves of every row of y are in LDS
      {
        u32x4 yo[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) yo[k] = *reinterpret_cast<const u32x4 *>(raw_dst_row + kRowStep * k * kRawStride);
        if constexpr (kYMode == kYAdd) {
#pragma unroll
          for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int w = 0; w < 4; ++w)
              yo[k][w] = pack2(bf_lo(yo[k][w]) + bf_lo(yprev[k][w]), bf_hi(yo[k][w]) + bf_hi(yprev[k][w]));
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
          buf_store16<kYMode == kYStream ? kStreamStore : 0>(ry, vy + static_cast<uint32_t>(kRowStep * k) * xrow, yo[k]);
      }
      if constexpr (!kRowStores) {
        stage_raw(setA);
        load_part(0, at(jb + 3), setA);
      }
      // The factor still owed to the accumulators: from the middle of this block (steep: from its end) to
      // the middle of the next block -- to its start if that one is steep; after the last block only the
      // way to its end is left.
      if constexpr (kMixed) {
        const bool next_steep = more && __builtin_amdgcn_readfirstlane(__float_as_int(nf)) < 0;
        if constexpr (kSteep)
          pending = more && !next_steep ? nf : 1.f;
        else
          pending = more && !next_steep ? fac.w : fac.x;
        steep_cur = next_steep;
      } else {
        pending = pend_next;
      }
      rowf0 = rowf0n;
      rowf1 = rowf1n;
      __syncthreads();  // block jb's tiles may be overwritten; block jb+1's tiles are visible
    };
    // pairs of blocks, then the odd one: with the test between the two halves of a pair the compiler
    // would also have to allow for "first half, then first half again", where the set staged at the
    // top has only just been requested, and would wait for the newest loads in every iteration
    if constexpr (!kMixed) {
      int jb = jb0;
      for (; jb + 1 < jb1; jb += 2) {
        body(0, jb, std::false_type{});
        body(1, jb + 1, std::false_type{});
      }
      if (jb < jb1) body(0, jb, std::false_type{});
    } else {
      auto step = [&](int par, int jb) __attribute__((always_inline)) {
        if (steep_cur)
          body(par, jb, std::true_type{});
        else
          body(par, jb, std::false_type{});
      };
      int jb = jb0;
      for (; jb + 1 < jb1; jb += 2) {
        step(0, jb);
        step(1, jb + 1);
      }
      if (jb < jb1) step(0, jb);
    }
  }
  if constexpr (!kStatesOnly) {
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
      for (int i = 0; i < 16; ++i) Hacc[nt][i] *= pending;
  }

  // ---- write the state out (canonical (p, n) layout, four consecutive n per 16-byte store) ----
  if constexpr (kStatesOnly) {
    // (this pass tiles the state differently, see its loop body: tile 2 pt + nt of wave ph)
    // In the accumulators a lane holds 16-byte pieces of 32 different state rows: stored as they are, every
    // store instruction would touch 32 rows, 32 bytes each (measured: 5 us of the pass at 16384 tokens x 80
    // heads, 6.6 of 17 at 2048 x 24).  The wave turns its tile through a private piece of LDS instead -- the
    // tiles there are dead after the loop's last barrier -- half at a time (32 headdim columns x 64 state
    // columns, rows padded by 16 bytes), and stores four whole 256-byte row segments per instruction.  One
    // wave, one piece of LDS, in-order LDS operations: no barrier.
    if (live) {
      constexpr int kTurnStride = 64 + 4;  // floats
      static_assert(2 * HPW * 32 * kTurnStride * sizeof(float) <= L::kXmBufs * HPW * L::kXmElems * sizeof(uint16_t),
                    "the waves' turning tiles fit where Xm^T was");
      float *const turn = reinterpret_cast<float *>(&sXm[0][0]) + wave * (32 * kTurnStride);
      float *slot = p.seg_state + (slot0 + sg + 1) * (kP * kN);
#pragma unroll
      for (int pt = 0; pt < 2; ++pt) {
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
          for (int i4 = 0; i4 < 4; ++i4) {
            const f32x16 &t = Hacc[2 * pt + nt];
            *reinterpret_cast<f32x4 *>(turn + pi_of_row(r) * kTurnStride + 32 * nt + 8 * i4 + 4 * kg) =
                f32x4{t[4 * i4 + 0], t[4 * i4 + 1], t[4 * i4 + 2], t[4 * i4 + 3]};
          }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int row = 4 * k + (lane >> 4), piece = lane & 15;
          *reinterpret_cast<f32x4 *>(slot + static_cast<size_t>(32 * pt + row) * kN + 64 * ph + 4 * piece) =
              *reinterpret_cast<const f32x4 *>(turn + row * kTurnStride + 4 * piece);
        }
      }
      if (lane == 0 && ph == 0) p.seg_decay[slot0 + sg] = seg_total;
    }
  } else if (sg == sv.S - 1 && live) {
    // The same turn for the final state of the full kernel (a wave owns 32 headdim columns x 128 state
    // columns there: two halves of 64 state columns).  Waves 0-3 turn their tiles in what was the B^T
    // buffers, waves 4-7 in the C buffers; every wave is past the loop's last barrier.
    constexpr int kTurnStride = 64 + 4;  // floats
    static_assert(4 * 32 * kTurnStride * sizeof(float) <= 2 * L::kBtElems * sizeof(uint16_t) &&
                      4 * 32 * kTurnStride * sizeof(float) <= L::kCBufs * L::kCElems * sizeof(uint16_t),
                  "four turning tiles fit in either buffer pair");
    float *const turn = reinterpret_cast<float *>(wave < 4 ? &sBt[0][0] : &sC[0][0]) + (wave & 3) * (32 * kTurnStride);
    float *const rows = p.final_state + (bh * kP + 32 * ph) * p.ns.width + p.ns.off;
    const int valid = p.ns.valid;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const f32x16 &t = Hacc[2 * half + nt];
          *reinterpret_cast<f32x4 *>(turn + pi_of_row(r) * kTurnStride + 32 * nt + 16 * (i4 >> 1) + 8 * kg + 4 * (i4 & 1)) =
              f32x4{t[4 * i4 + 0], t[4 * i4 + 1], t[4 * i4 + 2], t[4 * i4 + 3]};
        }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int row = 4 * k + (lane >> 4), n0 = 64 * half + 4 * (lane & 15);
        if (n0 < valid)
          *reinterpret_cast<f32x4 *>(rows + static_cast<size_t>(row) * p.ns.width + n0) =
              *reinterpret_cast<const f32x4 *>(turn + row * kTurnStride + 4 * (lane & 15));
      }
    }
  }
}

// The mixed walk as a function of its own: it is compiled, and its registers are allocated, apart from
// the kernel around the call, so what the rare steep form needs (it spills) costs the common walk nothing.
// (Arguments by value: a reference would make the kernel keep its own copy in private memory, where
// nothing counts as uniform any more.)
template <int kYMode>
__device__ __attribute__((noinline)) void scan_walk_mixed(const ScanParams p, const SeqView sv, const LdsTiles lds) {
  scan_walk<false, kHeadsPerWg, kYMode, true>(p, sv, lds);
}

// Whether the blocks this wave walks in the full scan include a steep one: one lane per block reads the
// marker of its record.
__device__ __forceinline__ bool walk_meets_steep_block(const ScanParams &p, const SeqView &sv) {
  const int lane = threadIdx.x & 63;
  const int slot = (sv.col % p.cpg) * kHeadsPerWg + (static_cast<int>(threadIdx.x) >> 7);
  const int h = (sv.col / p.cpg) * p.hpg + min(slot, p.hpg - 1);
  const int hrec = h / p.pdiv;
  const bool plain = p.vp.tok0 == nullptr;
  const size_t rec0 = plain ? (sv.blk0 * p.Hrec + static_cast<size_t>(hrec) * sv.blk_stride) : (hrec * sv.blk_stride + sv.blk0);
  const int jb0 = min(sv.nb, sv.sg * sv.seg_blocks), jb1 = min(sv.nb, jb0 + sv.seg_blocks);
  const float *marks = p.prep + rec0 * kRec + 2 * kBlk + 2;
  float lowest = 1.f;
  for (int j = jb0; j < jb1; j += 64)
    if (j + lane < jb1) lowest = fminf(lowest, marks[static_cast<size_t>(j + lane) * kRec]);
  return __builtin_amdgcn_ballot_w64(lowest < 0.f) != 0;
}

// ---- the full scan with two heads per workgroup -------------------------------------------------------
// Two waves per head as above; four of these, one to a SIMD, compute, and the other wave of each SIMD feeds them.
//   - Everything a block needs -- the shared tiles, x, the decay record -- travels straight from memory into LDS
//     (load_to_lds) at the feeding waves' request: no registers, no LDS writes, no waits but the feeders' own, one per
//     block.  A wave that makes such a request stands still for 95 cycles (measured with four waves of a CU making one
//     each, 64 vector instructions apart): with the fourteen requests and four stores of a block among its own
//     instructions a computing wave took 4190 cycles a block of 8 x 4096 tokens x 48 heads, with feeders 3660.
//   - The feeders also scale x and turn it for the matrix instructions (3610: now they are what a block waits for) and
//     make their requests in runs of four (see load_to_lds4): 3250.  The same work in waves that load into registers and
//     write LDS themselves takes 5240.  Addresses counted from the item's first block (by time stamps in the feeders, cold
//     inputs, cycles on another scale than the ones above): 2700 -> 2590, of which a feeder works 2430 and a computing
//     wave 2300; 7 x 826 tokens x 23 heads 2750 -> 2680, but 16384 x 80, where 240 workgroups wait for memory, 4080 -> 4190.
//     x loaded into registers three blocks ahead, with requests between quarters of the turn: 8 x 4096
//     x 48 140 us a call instead of 120.
//   - The tiles and the record of the next block arrive during a block, in the buffer of a pair that it does not use.  A
//     block of x goes through one of three buffers: it arrives until the middle of the block before its own, when the feeder that
//     requested it turns it into Xm^T; it serves the skip term of its block and is replaced, in place, by y; and
//     the feeders store y in whole rows in the block after, before they request x into the same place.
//   - So a block has one barrier.
//   - A group of matrix instructions finds its LDS operands two groups ahead of it, and the vector work of a block is
//     spread so that every group has some.
// (The matrix instructions work on architectural registers, see the build flags: with the state in accumulation registers
// a block moved 160 of them, 8 cycles each.)
// LDS, in bytes: [x 3 x 16384][tiles 2 x 38912: C, B^T, G rows 32..63, G rows 0..31][Xm^T 2 x 16384][records 2 x 1024].
struct PairLds {
  static constexpr int kX = 0, kXBuf = 2 * kBlk * kP * 2, kTiles = 3 * kXBuf, kBt = kBlk * kN * 2, kGHigh = 2 * kBt,
                       kGLow = kGHigh + 32 * kBlk * 2, kTileBuf = kGLow + 32 * 32 * 2, kXm = kTiles + 2 * kTileBuf,
                       kXmHead = kP * kBlk * 2, kRec = kXm + 4 * kXmHead, kRecBuf = 1024, kBytes = kRec + 2 * kRecBuf;
};
static_assert(PairLds::kBytes <= 160 * 1024 && PairLds::kTiles % 256 == 0 && PairLds::kTileBuf % 256 == 0 && PairLds::kXm % 256 == 0,
              "fits the LDS of a CU; a row of C, two of B^T and G, four of x and of G's short rows cover the 64 banks");

template <typename T>
using lds_as = __attribute__((address_space(3))) T;
typedef lds_as<uint8_t> lds_u8;

// Where the 16-byte pieces of a row lie.  Sixteen lanes that read the same piece of sixteen consecutive rows (the
// operands of the matrix instructions) have to meet sixteen different places of the 256 bytes that the banks hold:
//   C, 256-byte rows: piece c of row t at place c ^ (t & 15);
//   B^T, G rows 32..63 and Xm^T, 128-byte rows: c ^ (t / 2 & 7) (Xm^T also ^ 4 in its upper half, for the writes);
//   G rows 0..31, 64-byte rows of the 32 columns that matter: c ^ (t / 4 & 3);
//   x, per head two halves of 32 tokens, each two halves ph of 32 columns: of the latter token t's piece c at place 64 (t / 16 & 1) +
//     16 (t & 3) + 4 ((t / 4 & 3) ^ 2 ph) + (c ^ (t & 3)), which also serves the four tokens per lane of the turn and whole rows of y.

// ---- what a workgroup walks: items, an item being two heads of an entry of the segment list ----
// The walk goes from the last block of an item to the first of the next as it goes from block to block: what the next
// item's blocks need is requested while this one's are computed.  A workgroup of its own for every entry pays 5 us for its start, and
// where they are several a CU they end unevenly: 64 ragged sequences, 16384 tokens, 80 heads 173 us with four heads to a
// workgroup (152 of them the scan, 1280 workgroups), dealt 155.6 (136, traced).  What is left is the memory: x, y and a final state
// of 32 KB a sequence and head are 504 MB, 3.7 TB/s; of 5300 cycles a block, ends of items included, a computing wave works
// 2280 and a feeder 3150, two thirds of them until its requests are taken.
struct ItemView {
  uint32_t tok0, len, blk0, slot0, b;  // as in SeqView
  int sg, S, col, nb, jb0, jb1;
};
__device__ __forceinline__ void item_blocks(ItemView &v, int seg_blocks) {
  v.nb = static_cast<int>((v.len + kBlk - 1) / kBlk);
  v.jb0 = min(v.nb, v.sg * seg_blocks);
  v.jb1 = min(v.nb, v.jb0 + seg_blocks);
}

// The item of a workgroup that has one at most: true if it has one.
__device__ __forceinline__ bool one_item(const PairParams &p, int &seg_blocks, ItemView &first) {
  SeqView v;
  if (!wg_coords(p, true, v)) return false;
  seg_blocks = v.seg_blocks;
  first.tok0 = static_cast<uint32_t>(v.tok0);
  first.len = v.len;
  first.blk0 = static_cast<uint32_t>(v.blk0);
  first.slot0 = static_cast<uint32_t>(v.slot0);
  first.b = v.b;
  first.sg = v.sg;
  first.S = v.S;
  first.col = v.col;
  item_blocks(first, seg_blocks);
  return true;
}

// A packed batch of more items than workgroups.  The items, entry by entry and so longest first (but for those that are not the
// last of their sequence, which are first and equal), are dealt in rounds of a workgroup per CU: the first round forth, all later
// ones back, so that who had the longest item gets the shortest of every later round.  (Simulated over 300 drawn batches:
// the last workgroup ends 1.10 times as late as an even share of the work, or its longest item, asks for; dealt forth and back in
// turn 1.13, longest-first to whoever is free, over the whole chip, 1.05, as the hardware does it with every entry bound to
// an XCD 1.42.  A list made to measure by every workgroup comes to 1.05 too, and costs each 12 us: its 8 KB of code run once,
// at the rate at which instructions come from the L2.)  A round's places go XCD by XCD, so that an entry's tiles are fetched into few L2s.
struct Deal {
  int n_full, n_mine, place, seg_blocks;
};
__device__ __forceinline__ Deal deal_of(const PairParams &p) {
  Deal d;
  const int entries = table_at(p.vp.item0, p.vp.nseq), total = entries * p.cols, wgs = gridDim.x;
  d.seg_blocks = table_at(p.vp.len, p.vp.nseq);
  d.n_full = entries - p.vp.nseq;
  const int xcd = blockIdx.x % kXcds, in_xcd = blockIdx.x / kXcds, per_xcd = total < wgs ? (total + kXcds - 1) / kXcds : wgs / kXcds;
  d.place = xcd * per_xcd + in_xcd;
  d.n_mine = in_xcd < per_xcd && d.place < total ? 1 : 0;
  const int back = total - wgs - (wgs - 1 - d.place);  // items from the second round's on
  if (total > wgs && back > 0) d.n_mine += (back + wgs - 1) / wgs;
  return d;
}
// Its item i: entry and column, and (looked up in two steps, each an item ahead of the next) the entry's sequence, the rest.
struct ItemPlace {
  int entry, col, q;
};
__device__ __forceinline__ ItemPlace item_place(const PairParams &p, const Deal &d, int i) {
  const int wgs = gridDim.x;
  const int pos = i == 0 ? d.place : i * wgs + wgs - 1 - d.place;
  ItemPlace at;
  at.entry = quotient(pos, p.cols, p.cols_inv);
  at.col = pos - at.entry * p.cols;
  at.q = table_at(p.vp.item_seq, at.entry);
  return at;
}
__device__ __forceinline__ ItemView item_at(const PairParams &p, const Deal &d, const ItemPlace &at) {
  ItemView v;
  const int first = table_at(p.vp.item0, at.q);
  v.b = at.q;
  v.S = table_at(p.vp.item0, at.q + 1) - first;
  v.sg = at.entry < d.n_full ? at.entry - (first - at.q) : v.S - 1;
  v.col = at.col;
  v.len = table_at(p.vp.len, at.q);
  v.tok0 = table_at(p.vp.tok0, at.q);
  v.blk0 = table_at(p.vp.blk0, at.q);
  v.slot0 = table_at(p.vp.slot0, at.q);
  item_blocks(v, d.seg_blocks);
  return v;
}
// The items in turn.  kList: several, from the deal; otherwise the one.
template <bool kList>
struct Items {
  Deal deal;
  ItemView ahead;        // item `next`
  ItemPlace ahead2 = {};  // and where the one after it is
  int next = 0, n;
  __device__ __forceinline__ Items(const Deal &d, const ItemView &first) : deal(d), ahead(first), n(1) {}
  __device__ __forceinline__ Items(const PairParams &p, const Deal &d, int i) : deal(d), next(i), n(d.n_mine) {
    ahead = item_at(p, d, item_place(p, d, i));
    if (i + 1 < n) ahead2 = item_place(p, d, i + 1);
  }
  __device__ __forceinline__ ItemView take(const PairParams &p) {
    const ItemView v = ahead;
    ++next;
    if constexpr (kList) {
      if (next < n) ahead = item_at(p, deal, ahead2);
      if (next + 1 < n) ahead2 = item_place(p, deal, next + 1);
    }
    return v;
  }
};

// The thread's number, as something that is only known here: what is computed from it stays in the role that needs it,
// instead of being kept in registers through the others (whose spills would wait for all requests under way).
__device__ __forceinline__ int here(unsigned thread) {
  int t = static_cast<int>(thread);
  asm volatile("" : "+v"(t));
  return t;
}
// ... and the lane's in its wave, from nothing that would have to be kept.
__device__ __forceinline__ int lane_here() {
  int t;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(t));
  return t;
}

// The feeding waves, 4..7: feeder w serves head w / 2 and, of x and y, tokens 32 (w & 1) .. + 31.
template <int kYMode, bool kList>
__device__ __forceinline__ void pair_feed(const PairParams &p, Items<kList> items, lds_u8 *const lds) {
  using L = PairLds;
  const uint32_t lds_at = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
  const int tid = here(threadIdx.x) & 255, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hw = wave >> 1, ph = wave & 1;
  const bool plain = p.vp.tok0 == nullptr;
  const uint32_t xrow = static_cast<uint32_t>(p.H) * (kP * 2), crow = static_cast<uint32_t>(p.G) * (kN * 2);

  // ---- what has to be known of a block to request and store what belongs to it ----
  struct Block {
    size_t x_at, c_at;       // bytes from the start of x (and y) to its first row, of C
    uint32_t xb, cb;         // bytes behind these that belong to the sequence; 0: there is no such block
    uint32_t tile;           // of B^T and G
    uint32_t rec0, rec1;     // decay records of the two heads
  };
  bool live = false;  // y of the item's blocks is stored
  auto first_block = [&](const ItemView &v, Block &b) __attribute__((always_inline)) {
    const int g = quotient(v.col, p.cpg, p.cpg_inv), slot = (v.col - g * p.cpg) * 2;
    live = slot + hw < p.hpg;
    const int h0 = g * p.hpg + min(slot, p.hpg - 1), h1 = g * p.hpg + min(slot + 1, p.hpg - 1), h = hw ? h1 : h0;
    const uint32_t tok = v.tok0 + static_cast<uint32_t>(v.jb0) * kBlk, rest = v.len - static_cast<uint32_t>(v.jb0) * kBlk;
    b.x_at = static_cast<size_t>(tok) * xrow + static_cast<uint32_t>(h) * (kP * 2);
    b.c_at = (static_cast<size_t>(tok) * p.G + g) * (kN * 2);
    b.xb = rest * xrow - static_cast<uint32_t>(h) * (kP * 2);
    b.cb = rest * crow - static_cast<uint32_t>(g) * (kN * 2);
    const uint32_t stride = plain ? p.NB : p.vp.nb_cap;
    b.tile = v.blk0 * (plain ? p.G : 1) + g * stride + v.jb0;
    const uint32_t rec = v.blk0 * (plain ? p.Hrec : 1) + v.jb0;
    b.rec0 = rec + quotient(h0, p.pdiv, p.pdiv_inv) * stride;
    b.rec1 = rec + quotient(h1, p.pdiv, p.pdiv_inv) * stride;
  };

  // ---- requests: per-lane offsets that never change, descriptors that start at the block.  Of x and C a wave fetches four
  //      times 1024 bytes to consecutive places (see load_to_lds4) from rows that may be nearer to each other than that: their
  //      descriptors start 3072 bytes earlier, and all that is asked of them lies beyond these ----
  constexpr uint32_t kEarly = 3072;
  uint32_t vx[4], vc[4];  // x: 16 tokens of one half of headdim each, the first half's first
#pragma unroll
  for (int o = 0; o < 4; ++o) {
    const int i = lane >> 4, half = o >> 1, t = 32 * ph + 16 * (o & 1) + 4 * ((lane >> 2 & 3) ^ 2 * half) + i;
    vx[o] = static_cast<uint32_t>(t) * xrow + 64 * half + 16 * ((lane & 3) ^ i) + (kEarly - 1024 * o);
    const int row = 16 * wave + 4 * o + (lane >> 4);
    vc[o] = static_cast<uint32_t>(row) * crow + 16 * ((lane ^ row) & 15) + (kEarly - 1024 * o);
  }
  // B^T: rows 32 wave + 8 k + lane / 8; the places of consecutive k differ by an exchange of the halves of a row
  uint32_t vb[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) vb[k] = static_cast<uint32_t>(32 * wave + (lane >> 3)) * (kBlk * 2) + 16 * ((lane ^ (lane >> 4) ^ 4 * k) & 7);
  const uint32_t vt = static_cast<uint32_t>(32 + (tid >> 3)) * (kBlk * 2) + 16 * ((tid ^ (tid >> 4)) & 7);  // G's upper rows
  // The tenth request of a wave: waves 0 and 1 fetch a half of G's short rows each, waves 2 and 3 (both the same) the record
  // entries that the two heads need next: 32 lanes the input factors of the block after, 32 the output-row factors.
  const bool fetches_g = wave < 2;
  const uint32_t vg = static_cast<uint32_t>(16 * (wave & 1) + (lane >> 2)) * (kBlk * 2) + 16 * ((lane ^ (lane >> 4)) & 3);
  // this wave's ten requests of a block's tiles (and records): C from c (cb bytes), B^T and G number `tile`, and the tenth; `no` block:
  // empty descriptors, which fetch nothing
  auto fetch_nine = [&](const uint8_t *c, uint32_t cb, const uint8_t *bt, const uint8_t *g, int buf, bool no) __attribute__((always_inline)) {
    const uint32_t to = lds_at + L::kTiles + buf * L::kTileBuf;
    load_to_lds4(raw_rsrc(c - kEarly, no ? 0 : cb + kEarly), vc[0], vc[1], vc[2], vc[3], to + wave * 4096);
    load_to_lds4(raw_rsrc(bt, no ? 0 : kN * kBlk * 2), vb[0], vb[1], vb[0], vb[1], to + L::kBt + wave * 4096);
    load_to_lds(raw_rsrc(g, no ? 0 : kBlk * kBlk * 2), vt, to + L::kGHigh + wave * 1024);
  };
  auto fetch_tenth = [&](const uint8_t *g, const uint8_t *rec, uint32_t rec_bytes, uint32_t vr, int buf, bool no) __attribute__((always_inline)) {
    load_to_lds(raw_rsrc(fetches_g ? g : rec, no ? 0 : fetches_g ? kBlk * kBlk * 2u : rec_bytes), vr,
                fetches_g ? lds_at + L::kTiles + buf * L::kTileBuf + L::kGLow + wave * 1024 : lds_at + L::kRec + buf * L::kRecBuf);
  };
  auto fetch_x = [&](const uint8_t *x, uint32_t xb, uint32_t xbuf, bool no) __attribute__((always_inline)) {
    load_to_lds4(raw_rsrc(x - kEarly, no ? 0 : xb + kEarly), vx[0], vx[1], vx[2], vx[3], lds_at + L::kX + xbuf + wave * 4096);
  };

  auto lds16 = [&](uint32_t at) {
    Operand o;
    o.q = *(lds_as<u32x4> *)(lds + at);
    return o;
  };
  // whole rows of y: tokens 32ph + 4 (lane / 8) + k, piece lane % 8, of which 0..3 come from the head's first wave
  const int y_tile = (lane & 7) >> 2;
  auto row_at = [&](int k) {
    return L::kX + wave * 4096 + y_tile * 2048 + (lane >> 5) * 1024 + k * 256 + (((lane >> 3) & 3) ^ 2 * y_tile) * 64 + ((lane & 3) ^ k) * 16;
  };
  const uint32_t vy = static_cast<uint32_t>(32 * ph + 4 * (lane >> 3)) * xrow + 16 * (lane & 7);
  u32x4 yo[4];
  auto read_y = [&](uint32_t xbuf) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < 4; ++k) yo[k] = lds16(row_at(k) + xbuf).q;
  };
  auto add_y = [&](Rsrc ry) __attribute__((always_inline)) {  // kYAdd: to what y holds so far
    u32x4 prev[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) prev[k] = buf_load16(ry, vy + static_cast<uint32_t>(k) * xrow, 0);
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int w = 0; w < 4; ++w)
        yo[k][w] = pack2(bf_lo(yo[k][w]) + bf_lo(prev[k][w]), bf_hi(yo[k][w]) + bf_hi(prev[k][w]));
  };
  auto store_y = [&](Rsrc ry, int k) __attribute__((always_inline)) {
    buf_store16<kYMode == kYStream ? kStreamStore : 0>(ry, vy + static_cast<uint32_t>(k) * xrow, yo[k]);
  };

  // the turn: this lane has tokens 32ph + 4tg + i, columns 8cg + c, which go to row pi^-1 = 16 (cg & 1) + 4 (cg / 2 & 1) + 8 (c / 4) +
  // (c & 3) of their half (cg / 4)
  const int cg = lane & 7, tg = lane >> 3, half = cg >> 2;
  uint32_t a_turn[4], a_xmw[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    a_turn[i] = L::kX + wave * 4096 + half * 2048 + (tg >> 2) * 1024 + i * 256 + ((tg & 3) ^ 2 * half) * 64 + ((cg & 3) ^ i) * 16;
    const int row = 16 * (cg & 1) + 4 * (cg >> 1 & 1) + 8 * (i >> 1) + 2 * (i & 1);  // (of columns 4 (i / 2) + 2 (i & 1) and the next)
    a_xmw[i] = L::kXm + (2 * hw + half) * (L::kXmHead / 2) + row * (kBlk * 2) + 16 * ((4 * ph + (tg >> 1)) ^ (row >> 1 & 7) ^ (row >> 4) * 4) + 8 * (tg & 1);
  }
  // x times the input factors (of the record buffer `rec`) to Xm^T: four tokens per 8-byte write
  u32x4 xr[4], f;
  auto read_turn = [&](uint32_t xbuf, uint32_t rec) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) xr[i] = lds16(a_turn[i] + xbuf).q;
    f = lds16(L::kRec + rec + hw * 256 + ph * 128 + 16 * tg).q;
  };
  auto turn = [&](uint32_t xm) __attribute__((always_inline)) {
    const float f0 = __uint_as_float(f.x), f1 = __uint_as_float(f.y), f2 = __uint_as_float(f.z), f3 = __uint_as_float(f.w);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const uint32_t a0 = xr[0][c >> 1], a1 = xr[1][c >> 1], a2 = xr[2][c >> 1], a3 = xr[3][c >> 1];
      lds_as<u32x2> *const dst = (lds_as<u32x2> *)(lds + a_xmw[c >> 1] + xm + (c & 1) * (kBlk * 2));
      if (c & 1)
        *dst = mk2(pack2(f0 * bf_hi(a0), f1 * bf_hi(a1)), pack2(f2 * bf_hi(a2), f3 * bf_hi(a3)));
      else
        *dst = mk2(pack2(f0 * bf_lo(a0), f1 * bf_lo(a1)), pack2(f2 * bf_lo(a2), f3 * bf_lo(a3)));
    }
  };
  // One block.  y: where that of the block before is stored; tiles: requests the next block's, x: that of the one after.
  uint32_t x_prev = 2 * L::kXBuf, x_cur = 0, x_next = L::kXBuf;  // the buffers of the block before (and then of the one after the next), of this, of the next
  // (The order is held by fences where there are several items, 64 ragged sequences, 16384 tokens, 80 heads 156.7 -> 156.0 us, 16 of
  // them 122.9 -> 120.4; in the walk of one item they cost a block up to 150 cycles: 7 x 826 tokens x 23 heads 29.5, 28.4 without, 8 x
  // 4096 x 48 120.5, 117.4.)
  auto block = [&](uint32_t par, bool first, auto &&y, auto &&tiles, auto &&x) __attribute__((always_inline)) {
    read_y(x_prev);
    if (first) __syncthreads();  // an item's first block: its tiles and Xm^T are visible, the other tile buffer is free of states
    if constexpr (kList) __builtin_amdgcn_sched_barrier(0);  // (requests first: the compiler would put all of the block's addresses before them)
    tiles(par ^ 1);
    if constexpr (kList) __builtin_amdgcn_sched_barrier(0);
    if constexpr (kYMode == kYAdd) add_y(y());
    asm volatile("" : "+v"(yo[0]), "+v"(yo[1]), "+v"(yo[2]), "+v"(yo[3])::"memory");  // (read before x is requested into its place)
    asm volatile("s_waitcnt vmcnt(14)" ::: "memory");  // x of the next block; younger: the stores before, tiles
    read_turn(x_next, par * L::kRecBuf);
    x(x_prev);
    if constexpr (kList) __builtin_amdgcn_sched_barrier(0);
    turn((par ^ 1) * (2 * L::kXmHead));
    if constexpr (kList) __builtin_amdgcn_sched_barrier(0);
    const Rsrc ry = y();
#pragma unroll
    for (int k = 0; k < 4; ++k) store_y(ry, k);
    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");  // the next block's tiles and record; younger: x, stores
    __syncthreads();  // ... and its Xm^T are visible, this block's may be overwritten
    const uint32_t t = x_prev;
    x_prev = x_cur;
    x_cur = x_next;
    x_next = t;
  };
  auto last_y = [&](Rsrc ry) __attribute__((always_inline)) {
    read_y(x_prev);
    if constexpr (kYMode == kYAdd) add_y(ry);
#pragma unroll
    for (int k = 0; k < 4; ++k) store_y(ry, k);
  };
  // ---- prologue: the first block's tiles, input factors and x, the second block's x ----
  auto start = [&](const uint8_t *first_factors, uint32_t bytes, uint32_t vf, auto &&x0, auto &&tiles0, auto &&x1) __attribute__((always_inline)) {
    x0(0);
    // (the factors of the first block, which every feeder fetches for itself: the records come a block behind them)
    load_to_lds(raw_rsrc(first_factors, bytes), vf + kBlk * 4 + 16 * (lane & 15), lds_at + L::kRec + L::kRecBuf);
    tiles0(0);
    x1(L::kXBuf);
    asm volatile("s_waitcnt vmcnt(14)" ::: "memory");  // (tiles and the second block's x)
    read_turn(0, L::kRecBuf);
    turn(0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  };

  if constexpr (!kList) {
    const ItemView v = items.take(p);
    const int jb0 = v.jb0, jlast = v.jb1 - 1;
    if (jb0 > jlast) return;
    Block b;
    first_block(v, b);
    const uint8_t *const xb = p.x + b.x_at, *const cb = p.C + b.c_at, *const btb = p.Btr + static_cast<size_t>(b.tile) * (kN * kBlk * 2),
                  *const gb = p.Gd + static_cast<size_t>(b.tile) * (kBlk * kBlk * 2), *const recb = reinterpret_cast<const uint8_t *>(p.prep + static_cast<size_t>(b.rec0) * kRec);
    uint8_t *const yb = p.y + b.x_at;
    const uint32_t head_step = (b.rec1 - b.rec0) * (kRec * 4), vh = (lane & 16) ? head_step : 0u;
    const uint32_t vr = fetches_g ? vg : vh + (lane < 32 ? (kRec + kBlk) * 4u : 0u) + 16 * (lane & 15);
    auto tiles_of = [&](int rel, int buf, bool no) __attribute__((always_inline)) {
      const uint8_t *const g = gb + static_cast<size_t>(rel) * (kBlk * kBlk * 2);
      fetch_nine(cb + static_cast<size_t>(rel) * kBlk * crow, b.cb - static_cast<uint32_t>(rel) * kBlk * crow, btb + static_cast<size_t>(rel) * (kN * kBlk * 2), g, buf, no);
      fetch_tenth(g, recb + static_cast<size_t>(rel) * (kRec * 4), head_step + static_cast<uint32_t>(v.nb - jb0 - rel) * (kRec * 4), vr, buf, no);
    };
    auto x_of = [&](int rel, uint32_t xbuf, bool no) __attribute__((always_inline)) { fetch_x(xb + static_cast<size_t>(rel) * kBlk * xrow, b.xb - static_cast<uint32_t>(rel) * kBlk * xrow, xbuf, no); };
    auto y_of = [&](int rel, bool no) { return make_rsrc(yb + static_cast<size_t>(rel) * kBlk * xrow, live && !no ? b.xb - static_cast<uint32_t>(rel) * kBlk * xrow : 0u); };
    const int last = jlast - jb0;
    start(recb, head_step + static_cast<uint32_t>(v.nb - jb0) * (kRec * 4), vh, [&](uint32_t to) { x_of(0, to, false); }, [&](int buf) { tiles_of(0, buf, false); },
          [&](uint32_t to) { x_of(min(1, last), to, last == 0); });
    __syncthreads();
    for (int rel = 0; rel <= last; ++rel)
      block(rel & 1, false, [&]() { return y_of(rel - (rel > 0 ? 1 : 0), rel == 0); }, [&](int buf) { tiles_of(rel < last ? rel + 1 : last, buf, rel >= last); },
            [&](uint32_t to) { x_of(rel + 1 < last ? rel + 2 : last, to, rel + 1 >= last); });
    last_y(y_of(last, false));
  } else {
    // the blocks of the items, one after the other; `after` is where the requests have got to
    struct Y {
      size_t at;
      uint32_t bytes;
      bool first;
    };
    Block next = {}, after = {};  // the block whose tiles are requested next (or now), the one whose x is
    int jb = 0, jb1 = 0;
    auto advance = [&]() __attribute__((always_inline)) {  // `after` to the block after it
      Y y;
      y.first = ++jb >= jb1;
      if (y.first) {
        do {
          if (items.next >= items.n) {
            jb = jb1 = 0;
            after.xb = after.cb = 0;
            break;
          }
          const ItemView v = items.take(p);
          jb = v.jb0;
          jb1 = v.jb1;
          if (jb < jb1) first_block(v, after);
        } while (jb >= jb1);
      } else {
        after.x_at += kBlk * xrow;
        after.c_at += kBlk * crow;
        after.xb -= kBlk * xrow;
        after.cb -= kBlk * crow;
        ++after.tile;
        ++after.rec0;
        ++after.rec1;
      }
      y.at = after.x_at;
      y.bytes = live ? after.xb : 0;
      return y;
    };
    // the requests of `after`'s tiles, which becomes `next`, and of the input factors of the one after it
    auto tiles_and_advance = [&](int buf, Y &y) __attribute__((always_inline)) {
      next = after;
      const uint8_t *const g = p.Gd + static_cast<size_t>(next.tile) * (kBlk * kBlk * 2);
      fetch_nine(p.C + next.c_at, next.cb, p.Btr + static_cast<size_t>(next.tile) * (kN * kBlk * 2), g, buf, next.cb == 0);
      __builtin_amdgcn_sched_barrier(0);
      y = advance();
      const uint32_t of_next = (lane & 16 ? next.rec1 : next.rec0) * (kRec * 4), of_after = (lane & 16 ? after.rec1 : after.rec0) * (kRec * 4) + kBlk * 4;
      fetch_tenth(g, reinterpret_cast<const uint8_t *>(p.prep), p.prep_bytes, fetches_g ? vg : (lane < 32 ? of_after : of_next) + 16 * (lane & 15), buf, next.cb == 0);
    };
    auto x_of_after = [&](uint32_t to) __attribute__((always_inline)) { fetch_x(p.x + after.x_at, after.xb, to, after.xb == 0); };
    Y y_before = {0, 0, false}, y_now = advance(), y_next, y_after;
    if (after.xb == 0) return;
    start(reinterpret_cast<const uint8_t *>(p.prep), p.prep_bytes, (lane & 16 ? after.rec1 : after.rec0) * (kRec * 4), x_of_after,
          [&](int buf) { tiles_and_advance(buf, y_next); }, x_of_after);
    bool more = true;  // (whether there is a block to compute)
    for (uint32_t par = 0; more; par ^= 1) {
      block(par, y_now.first, [&]() { return make_rsrc(p.y + y_before.at, y_before.bytes); }, [&](int buf) { tiles_and_advance(buf, y_after); }, x_of_after);
      more = next.xb != 0;
      y_before = y_now;
      y_now = y_next;
      y_next = y_after;
    }
    last_y(make_rsrc(p.y + y_before.at, y_before.bytes));
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (no request may outlive the workgroup's LDS)
}

template <bool kList>
__device__ void pair_walk_mixed(const PairParams p, const Deal deal, const ItemView first, int item, uint32_t parity, uint32_t x_cur, lds_u8 *const lds);

// The computing waves, 0..3: wave w has half w & 1 of headdim of head w / 2.  kMixed: some of the items' blocks may be steep.
// Without kMixed, an item with a steep block is left to pair_walk_mixed, with all that come after it.  kList: there may be several items.
template <bool kMixed, bool kList>
__device__ __forceinline__ void pair_walk(const PairParams &p, Items<kList> items, uint32_t parity, uint32_t x_cur, lds_u8 *const lds) {
  using L = PairLds;
  const int tid = here(threadIdx.x), lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hw = wave >> 1, ph = wave & 1;
  const bool plain = p.vp.tok0 == nullptr;
  const int r = lane & 31, kg = lane >> 5;

  // ---- LDS addresses of this lane, in bytes ----
  auto lds16 = [&](uint32_t at) {
    Operand o;
    o.q = *(lds_as<u32x4> *)(lds + at);
    return o;
  };
  const int br = swap_row(r);
  const uint32_t a_c = L::kTiles + r * (kN * 2) + 16 * (kg ^ (r & 15));                         // ^ 32 kk, + 32 rows
  const uint32_t a_bt = L::kTiles + L::kBt + br * (kBlk * 2) + 16 * (kg ^ (br >> 1 & 7));       // ^ 32 q, + 32 nt rows
  const uint32_t a_g1 = L::kTiles + L::kGHigh + r * (kBlk * 2) + 16 * (kg ^ (r >> 1 & 7));      // token 32 + r, ^ 32 q
  const uint32_t a_g0 = L::kTiles + L::kGLow + r * 64 + 16 * (kg ^ (r >> 2 & 3));               // token r, ^ 32 q (q < 2)
  const uint32_t a_xm = L::kXm + (2 * hw + ph) * (L::kXmHead / 2) + r * (kBlk * 2) + 16 * (kg ^ (r >> 1 & 7) ^ (r >> 4) * 4);  // ^ 32 q
  // x and y in output layout: token r (+ 32: 4096 bytes on), columns 16kg + 8c
  const uint32_t a_out = L::kX + hw * 8192 + ph * 2048 + (r >> 4) * 1024 + (r & 3) * 256 + ((r >> 2 & 3) ^ 2 * ph) * 64;
  auto out_at = [&](int c) { return a_out + 16 * ((2 * kg + c) ^ (r & 3)); };
  // Where a wave turns 32 x 64 elements of its state between the accumulators' layout and whole rows: in the tile buffer
  // that the item's first block, whose tiles have arrived, does not have, before the feeders request the second block's tiles into it.
  constexpr int kTurnStride = 64 + 4;  // floats
  static_assert(4 * 32 * kTurnStride * sizeof(float) <= L::kTileBuf, "four turning tiles fit in a tile buffer");

  // ---- an item: its head, its blocks, where its record and states are ----
  int jb0 = 0, jb1 = 0, jlast = 0, h = 0, hrec = 0;
  bool live = false;
  ItemView v;
  const float *prep_bh = p.prep;
  size_t slot0 = 0, bh = 0;
  auto to_item = [&]() __attribute__((always_inline)) {
    v = items.take(p);
    const int g = quotient(v.col, p.cpg, p.cpg_inv), slot = (v.col - g * p.cpg) * 2 + hw;
    live = slot < p.hpg;
    h = g * p.hpg + min(slot, p.hpg - 1);
    hrec = quotient(h, p.pdiv, p.pdiv_inv);
    const size_t rec0 = plain ? (static_cast<size_t>(v.blk0) * p.Hrec + static_cast<size_t>(hrec) * p.NB) : (static_cast<size_t>(hrec) * p.vp.nb_cap + v.blk0);
    slot0 = plain ? (static_cast<size_t>(v.slot0) * p.H + static_cast<size_t>(h) * p.slots) : (static_cast<size_t>(h) * p.vp.slot_cap + v.slot0);
    bh = static_cast<size_t>(v.b) * p.H + h;
    jb0 = v.jb0;
    jb1 = v.jb1;
    jlast = jb1 - 1;
    prep_bh = p.prep + rec0 * kRec;
  };
  auto factor_ptr = [&](int jb) { return prep_bh + static_cast<size_t>(jb) * kRec + 2 * kBlk; };
  // {middle -> end, log2 of the total decay, start -> middle, middle -> middle of the next block} of 64 blocks, a lane each
  f32x4 facv = {0.f, 0.f, 0.f, 0.f};
  float Dv = 0.f;
  auto request_factors = [&]() __attribute__((always_inline)) {
    Dv = p.D == nullptr ? 0.f : p.D[hrec];
    facv = *reinterpret_cast<const f32x4 *>(jb0 < jb1 ? factor_ptr(min(jb0 + lane_here(), jlast)) : p.prep);
  };
  u32x4 hraw[16];
  auto load_state = [&](const float *base, uint32_t row_floats, uint32_t valid) __attribute__((always_inline)) {
    const Rsrc rs = make_rsrc(base != nullptr ? base : p.prep, base != nullptr ? ((kP - 1) * row_floats + valid) * 4u : 0u);
    const int ln = lane_here();  // (what is computed from it is not kept in registers through the walk)
    const uint32_t n0 = 4 * (ln & 15), at = ((32 * ph + (ln >> 4)) * row_floats + n0) * 4u;
    const uint32_t beyond[2] = {n0 < valid ? 0u : 0xC0000000u, n0 + 64 < valid ? 0u : 0xC0000000u};  // (no descriptor covers these)
#pragma unroll
    for (int k = 0; k < 16; ++k) hraw[k] = buf_load16(rs, (at + 16 * (k & 7) * row_floats + 256 * (k >> 3)) | beyond[k >> 3], 0);
  };
  // ---- state slice: Hacc[nt][i] = Ht^T[n = 32nt + (i/8)*16 + 8kg + i%8][headdim column 32 ph + pi_of_row(r)]: the rows of
  //      B^T are read in the order that leaves eight consecutive state columns in a lane (swap_row), which is how
  //      C's 16-byte pieces hold them ----
  f32x16 Hacc[4] = {};
  auto turn_at = [&]() { return (lds_as<float> *)(lds + L::kTiles + (parity ^ 1) * L::kTileBuf) + wave * (32 * kTurnStride); };
  auto add_state = [&](float wgt, bool first) __attribute__((always_inline)) {
    lds_as<float> *const turn = turn_at();
    const int ln = lane_here();
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int k = 0; k < 8; ++k)
        *(lds_as<u32x4> *)(turn + (4 * k + (ln >> 4)) * kTurnStride + 4 * (ln & 15)) = hraw[8 * half + k];
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const f32x4 v = *(lds_as<f32x4> *)(turn + pi_of_row(ln & 31) * kTurnStride + 32 * nt + 16 * (i4 >> 1) + 8 * (ln >> 5) + 4 * (i4 & 1));
#pragma unroll
          for (int e = 0; e < 4; ++e) Hacc[2 * half + nt][4 * i4 + e] = first ? v[e] : Hacc[2 * half + nt][4 * i4 + e] + wgt * v[e];
        }
    }
  };
  // (a sequence of one segment, and the first of a folded chain, start from h0 itself; see scan_walk)
  bool has_state = false;  // uniform over the workgroup
  auto request_state = [&]() __attribute__((always_inline)) {
    const float *hbase = nullptr;
    uint32_t hrow = kN, hvalid = kN;
    if (v.S > 1 && (kList || !(p.fold && v.sg == 0))) {
      hbase = p.Hin + (slot0 + static_cast<size_t>(v.sg) * p.parts) * (kP * kN);
    } else if (p.h0 != nullptr) {
      hbase = p.h0 + bh * kP * p.ns.width + p.ns.off;
      hrow = static_cast<uint32_t>(p.ns.width);
      hvalid = static_cast<uint32_t>(p.ns.valid);
    }
    has_state = hbase != nullptr;
    if (kList && !has_state) return;
    load_state(hbase, hrow, hvalid);  // (one item: without a branch, at whose end the compiler would wait)
    if constexpr (kList) add_state(1.f, true);
  };
  auto enter_state = [&]() __attribute__((always_inline)) {
    if (!has_state) return;
    add_state(1.f, true);
    if (p.fold && v.sg >= 1) {  // (the earlier pieces' local end states and h0, see scan_walk)
      float log2_decay = 0.f;
      for (int k = v.sg * p.parts - 1; k >= 0; --k) {
        log2_decay += p.seg_decay[slot0 + k];
        if (k == 0 && p.h0 == nullptr) break;
        load_state(k > 0 ? p.Hin + (slot0 + k) * (kP * kN) : p.h0 + bh * kP * p.ns.width + p.ns.off,
                   k > 0 ? kN : static_cast<uint32_t>(p.ns.width), k > 0 ? kN : static_cast<uint32_t>(p.ns.valid));
        add_state(fast_exp2(log2_decay), false);
      }
    }
  };
  float pending = 1.f;  // as in scan_walk: what the accumulators are still owed
  float Dh = 0.f;
  float fac = 0.f;      // of 64 blocks, a lane each: to the middle of the next, of the last block to its end
  bool steep_cur = false;
  auto of_block = [&](float f, int rel) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(f), rel & 63)); };

  // One block; par: the parity of its number in the walk (a compile-time constant), which is that of its buffers but x's.
  auto body = [&](int par, int jb, auto steep_tag) __attribute__((always_inline)) {
    constexpr bool kSteep = decltype(steep_tag)::value;
    static_assert(kMixed || !kSteep, "a steep block is only met in the mixed walk");
    const int rel = jb - jb0;
    const uint32_t tile = par * L::kTileBuf, rec = L::kRec + par * L::kRecBuf, xm = par * (2 * L::kXmHead);
    [[maybe_unused]] const bool more = jb < jlast;

    // ---- phase 1: Y^T[row][l] = sum_n Ht[row][n] C[l][n]  +  sum_{s<=l} Xm[s][row] G[l][s] ----
    Operand co[3][2], go0[2], go1[4], xo[4], bto[2][4], xe[4];
    auto read_c = [&](int kk) __attribute__((always_inline)) {
      co[kk % 3][0] = lds16((a_c ^ (32 * kk)) + tile);
      co[kk % 3][1] = lds16((a_c ^ (32 * kk)) + tile + 32 * kN * 2);
    };
    auto read_bt = [&](int q, int nt) __attribute__((always_inline)) { bto[q & 1][nt] = lds16((a_bt ^ (32 * q)) + tile + 32 * nt * kBlk * 2); };
    read_c(0);
    read_c(1);
#pragma unroll
    for (int q = 0; q < 4; ++q) xo[q] = lds16((a_xm ^ (32 * q)) + xm);
    float rowf[2] = {*(lds_as<float> *)(lds + rec + 512 + hw * 256 + 4 * r), *(lds_as<float> *)(lds + rec + 512 + hw * 256 + 128 + 4 * r)};
    float dt_t = 0.f, cs_t = 0.f;  // steep: step size and inclusive prefix sum of dt*A*log2(e) of token `lane`
    if constexpr (kSteep) {
      const float alog = of_block(facv.w, rel);
      dt_t = kg ? rowf[1] : rowf[0];
      cs_t = cut_step(dt_t, alog) * alog;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const float up = __shfl_up(cs_t, off, 64);
        if (lane >= off) cs_t += up;
      }
    }
    f32x16 Y[2] = {};
    // bf16 copy of a 16-column slice of Ht as a matrix operand, n = 16 kk + 8kg + {0..7}
    Operand ho[2];
    auto convert = [&](int kk) __attribute__((always_inline)) {
      f32x16 &hv = Hacc[kk >> 1];
      const int u = kk & 1;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        hv[8 * u + 2 * k] *= pending;
        hv[8 * u + 2 * k + 1] *= pending;
        ho[kk & 1].u[k] = pack2(hv[8 * u + 2 * k], hv[8 * u + 2 * k + 1]);
      }
    };
    convert(0);
    __builtin_amdgcn_sched_barrier(0);
    // (Behind every matrix instruction stands the vector work that is done while it runs: two in a row make the wave wait
    // 28 cycles for the pipe.)
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      if (kk < 6) {
        read_c(kk + 2);
      } else if (!kSteep) {
        go1[2 * (kk - 6)] = lds16((a_g1 ^ (64 * (kk - 6))) + tile);
        go1[2 * (kk - 6) + 1] = lds16((a_g1 ^ (64 * (kk - 6) + 32)) + tile);
        go0[kk - 6] = lds16((a_g0 ^ (32 * (kk - 6))) + tile);
      }
      Y[0] = mfma(ho[kk & 1], co[kk % 3][0], Y[0]);
      __builtin_amdgcn_sched_barrier(0);
      if (kk < 7) convert(kk + 1);
      __builtin_amdgcn_sched_barrier(0);
      Y[1] = mfma(ho[kk & 1], co[kk % 3][1], Y[1]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- the masked product ----
    if constexpr (kSteep) {
      const float csl[2] = {__shfl(cs_t, r, 64), __shfl(cs_t, 32 + r, 64)};
      const float s0 = fast_exp2(csl[0]), s1 = fast_exp2(csl[1]);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        Y[0][i] *= s0;
        Y[1][i] *= s1;
      }
      const int col = pi_of_row(r);  // this lane's column of the raw rows
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float cs_s[8], dt_s[8];
        Operand xs;  // raw x^T[row r][s = 16q + 8kg ..]
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int src = 16 * q + 8 * kg + j;
          cs_s[j] = __shfl(cs_t, src, 64);
          dt_s[j] = __shfl(dt_t, src, 64);
        }
        auto raw_at = [&](int t) {
          return static_cast<uint32_t>(*(lds_as<uint16_t> *)(
              lds + L::kX + x_cur + hw * 8192 + (t >> 5) * 4096 + ph * 2048 + (t >> 4 & 1) * 1024 + (t & 3) * 256 + ((t >> 2 & 3) ^ 2 * ph) * 64 + ((col >> 3) ^ (t & 3)) * 16 + (col & 7) * 2));
        };
#pragma unroll
        for (int k = 0; k < 4; ++k) xs.u[k] = raw_at(16 * q + 8 * kg + 2 * k) | raw_at(16 * q + 8 * kg + 2 * k + 1) << 16;
#pragma unroll
        for (int lt = (q < 2 ? 0 : 1); lt < 2; ++lt) {
          const Operand gq = lds16(lt ? (a_g1 ^ (32 * q)) + tile : (a_g0 ^ (32 * q)) + tile);
          Operand gh;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float w0 = dt_s[2 * k] * fast_exp2(fminf(csl[lt] - cs_s[2 * k], 0.f));
            const float w1 = dt_s[2 * k + 1] * fast_exp2(fminf(csl[lt] - cs_s[2 * k + 1], 0.f));
            gh.u[k] = pack2(bf_lo(gq.u[k]) * w0, bf_hi(gq.u[k]) * w1);
          }
          Y[lt] = mfma(xs, gh, Y[lt]);
        }
      }
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) read_bt(0, nt);
#pragma unroll
      for (int q = 0; q < 4; ++q) xe[q] = lds16(out_at(q & 1) + x_cur + (q >> 1) * 4096);
      const float e63 = fast_exp2(of_block(facv.y, rel));  // the state, so far at the start of the block, to its end
#pragma unroll
      for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int i = 0; i < 16; ++i) Hacc[nt][i] *= e63;
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int q = 0; q < (kSteep ? 0 : 4); ++q) {
      if (q < 2) {
        read_bt(0, 2 * q);
        read_bt(0, 2 * q + 1);
      } else {
        xe[2 * (q - 2)] = lds16(out_at(0) + x_cur + (q - 2) * 4096);
        xe[2 * (q - 2) + 1] = lds16(out_at(1) + x_cur + (q - 2) * 4096);
      }
      Y[1] = mfma(xo[q], go1[q], Y[1]);
      if (q < 2) Y[0] = mfma(xo[q], go0[q], Y[0]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- phase 2: H'^T[n][col] = Ht^T[n][col] + sum_s B^T[n][s] Xm[s][col]; alongside, the output
    //      epilogue of the block (y[l][col] = rowf_l Y + D x; element i of the lane is column
    //      32ph + 16kg + i), one quarter per group ----
    if constexpr (kSteep) rowf[0] = rowf[1] = 1.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (q < 3) {
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) read_bt(q + 1, nt);
      }
      const int lt = q >> 1, c = q & 1;
      u32x4 o;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        Hacc[w] = mfma(bto[q & 1][w], xo[q], Hacc[w]);
        __builtin_amdgcn_sched_barrier(0);
        o[w] = pack2(rowf[lt] * Y[lt][8 * c + 2 * w] + Dh * bf_lo(xe[q].u[w]), rowf[lt] * Y[lt][8 * c + 2 * w + 1] + Dh * bf_hi(xe[q].u[w]));
        __builtin_amdgcn_sched_barrier(0);
      }
      // the quarter replaces, in place, the x it was computed from
      *(lds_as<u32x4> *)(lds + out_at(c) + x_cur + lt * 4096) = o;
      __builtin_amdgcn_sched_barrier(0);
    }
    // as in scan_walk: from the middle of this block (steep: from its end) to the middle of the next, to its start
    // if that one is steep; after the last block only the way to its end is left
    if constexpr (kMixed) {
      const float to_next = of_block(facv.w, rel), to_end = of_block(facv.x, rel);
      const float nf = (rel & 63) < 63 ? of_block(facv.z, rel + 1) : __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(factor_ptr(more ? jb + 1 : jlast)[2])));
      const bool next_steep = more && __float_as_int(nf) < 0;
      if constexpr (kSteep)
        pending = more && !next_steep ? nf : 1.f;
      else
        pending = more && !next_steep ? to_next : to_end;
      steep_cur = next_steep;
    } else {
      pending = of_block(fac, rel);
    }
    x_cur = x_cur == 2 * L::kXBuf ? 0 : x_cur + L::kXBuf;
    __syncthreads();  // the next block's tiles are visible, this block's may be overwritten, its y read
  };
  auto step = [&](int par, int jb) __attribute__((always_inline)) {
    if constexpr (kMixed) {
      if (steep_cur) {
        body(par, jb, std::true_type{});
        return;
      }
    }
    body(par, jb, std::false_type{});
  };
  // ---- the final state, four consecutive n per 16-byte store ----
  auto store_state = [&](float *const rows) __attribute__((always_inline)) {
    lds_as<float> *const turn = turn_at();
    const int ln = lane_here();
    // (by descriptor, so that the number of stores, behind which what the next item needs is waited for, is known)
    const Rsrc rs = make_rsrc(rows, (31u * p.ns.width + p.ns.valid) * 4u);
    const uint32_t n0 = 4 * (ln & 15), at = ((ln >> 4) * static_cast<uint32_t>(p.ns.width) + n0) * 4u;
    const uint32_t beyond[2] = {n0 < static_cast<uint32_t>(p.ns.valid) ? 0u : 0xC0000000u, n0 + 64 < static_cast<uint32_t>(p.ns.valid) ? 0u : 0xC0000000u};
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const f32x16 &t = Hacc[2 * half + nt];
          *(lds_as<f32x4> *)(turn + pi_of_row(ln & 31) * kTurnStride + 32 * nt + 16 * (i4 >> 1) + 8 * (ln >> 5) + 4 * (i4 & 1)) =
              f32x4{t[4 * i4 + 0], t[4 * i4 + 1], t[4 * i4 + 2], t[4 * i4 + 3]} * pending;
        }
#pragma unroll
      for (int k = 0; k < 8; ++k)
        buf_store16(rs, (at + 16 * k * static_cast<uint32_t>(p.ns.width) + 256 * half) | beyond[half], *(lds_as<u32x4> *)(turn + (4 * k + (ln >> 4)) * kTurnStride + 4 * (ln & 15)));
    }
  };

  to_item();
  if constexpr (!kList) request_state();
  request_factors();
  for (;;) {
    if constexpr (!kMixed) {  // a block of the item is steep (its record's entry 130 is negative): the rest of the walk is mixed
      float lowest = jb0 < jb1 ? facv.z : 1.f;
      for (int j = jb0 + 64; j < jb1; j += 64)
        if (j + lane < jb1) lowest = fminf(lowest, factor_ptr(j + lane)[2]);
      if (__builtin_amdgcn_ballot_w64(lowest < 0.f) != 0) {
        pair_walk_mixed<kList>(p, items.deal, v, items.next - 1, parity, x_cur, lds);
        __builtin_amdgcn_endpgm();  // (so that nothing has to be kept over the call)
      }
    }
    if constexpr (kList) {
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) Hacc[nt] = f32x16{};
      request_state();
    } else {
      enter_state();
    }
    Dh = Dv;
    pending = 1.f;
    if (jb0 < jb1) {
      pending = of_block(facv.z, 0);
      if constexpr (kMixed) {
        steep_cur = __float_as_int(pending) < 0;
        if (steep_cur) pending = 1.f;
      }
      __syncthreads();  // the first block's tiles are visible; the feeders may request the second's
    }
    for (int first = jb0; first < jb1; first += 64) {
      if (first > jb0) facv = *reinterpret_cast<const f32x4 *>(factor_ptr(min(first + lane_here(), jlast)));
      const int last = min(first + 64, jb1);
      if constexpr (!kMixed) {
        fac = first + lane_here() < jlast ? facv.w : facv.x;
        asm volatile("" : "+v"(fac));
      }
      int jb = first;
      if (kList && parity != 0) step(1, jb++);  // (otherwise every walk of 64 starts in the first buffer)
      for (; jb + 1 < last; jb += 2) {
        step(0, jb);
        step(1, jb + 1);
      }
      parity = 0;
      if (jb < last) {
        step(0, jb);
        parity = 1;
      }
    }
    // ---- its last state, and what the next item needs from memory ----
    const bool stores = v.sg == v.S - 1 && live;
    float *const rows = p.final_state + (bh * kP + 32 * ph) * p.ns.width + p.ns.off;
    const bool more = kList && items.next < items.n;
    if (more) {
      to_item();
      request_factors();
    }
    // (the factors' arrival is waited for here, where the stores behind their request can be counted)
    if (stores) {
      store_state(rows);
      asm volatile("" : "+v"(facv), "+v"(Dv)::"memory");
    } else {
      asm volatile("" : "+v"(facv), "+v"(Dv)::"memory");
    }
    if (!more) return;
  }
}

template <bool kList>
__device__ __attribute__((noinline)) void pair_walk_mixed(const PairParams p, const Deal deal, const ItemView first, int item, uint32_t parity, uint32_t x_cur,
                                                          lds_u8 *const lds) {
  const Deal d = {static_cast<int>(uniform32(deal.n_full)), static_cast<int>(uniform32(deal.n_mine)), static_cast<int>(uniform32(deal.place)),
                  static_cast<int>(uniform32(deal.seg_blocks))};
  if constexpr (kList)
    pair_walk<true, true>(p, Items<true>(p, d, uniform32(item)), uniform32(parity), uniform32(x_cur), lds);
  else
    pair_walk<true, false>(p, Items<false>(d, first), 0, 0, lds);
}

template <bool kStatesOnly, int HPW, int kYMode = kYPlain>
__global__ __launch_bounds__(128 * HPW) __attribute__((amdgpu_waves_per_eu(2, 2))) void chunk_scan_kernel(const ScanParams p) {
  static_assert(kStatesOnly || HPW == kHeadsPerWg, "the full scan with two heads is pair_scan_kernel");
  using L = ScanLds<kStatesOnly, HPW>;
  __shared__ __align__(16) uint16_t sC[L::kCBufs][L::kCElems];
  __shared__ __align__(16) uint16_t sBt[2][L::kBtElems];
  __shared__ __align__(16) uint16_t sG[L::kGBufs][L::kGElems];
  __shared__ __align__(16) uint16_t sXm[L::kXmBufs * HPW][L::kXmElems];
  __shared__ __align__(16) uint16_t sRaw[L::kRawBufs][L::kRawElems];
  SeqView sv;
  if (!wg_coords(p, !kStatesOnly, sv)) return;  // uniform over the workgroup
  const LdsTiles lds = {(lds_u16 *)&sC[0][0], (lds_u16 *)&sBt[0][0], (lds_u16 *)&sG[0][0], (lds_u16 *)&sXm[0][0],
                        (lds_u16 *)&sRaw[0][0]};
  if constexpr (!kStatesOnly) {
    // Waves of one workgroup may take different walks: both stage the same shared tiles and meet at the
    // same barriers, block for block.
    if (walk_meets_steep_block(p, sv)) {
      scan_walk_mixed<kYMode>(p, sv, lds);
      return;
    }
  }
  scan_walk<kStatesOnly, HPW, kYMode, false>(p, sv, lds);
}

// kList: a packed batch, as many workgroups as CUs, each with the items that it is dealt; otherwise an item each.
// (the two roles, and the two walks, pass the same barriers, block for block; waves of one workgroup may take different walks)
template <int kYMode, bool kList>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void pair_scan_kernel(const PairParams p) {
  __shared__ __align__(1024) uint8_t lds_bytes[PairLds::kBytes];
  lds_u8 *const lds = (lds_u8 *)lds_bytes;
  const bool feeds = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x)) >= 256;  // (uniform, and known to be)
  auto run = [&](const Items<kList> &items) __attribute__((always_inline)) {
    if (feeds)
      pair_feed<kYMode, kList>(p, items, lds);
    else
      pair_walk<false, kList>(p, items, 0, 0, lds);
  };
  if constexpr (kList) {
    const Deal deal = deal_of(p);
    if (deal.n_mine > 0) run(Items<true>(p, deal, 0));
  } else {
    ItemView first;
    Deal deal = {0, 1, 0, 0};
    if (one_item(p, deal.seg_blocks, first)) run(Items<false>(deal, first));
  }
}

// ---- segment_pass: slot[0] = h0; slot[sg] = exp2(decay[sg-1]) * slot[sg-1] + local[sg-1] --------
// grid (P*N/1024, rows), four consecutive state elements per thread; a row is a (sequence, head), of a packed batch a
// (non-last segment, head).  seg_state slot sg (sg >= 1)
// holds the local end state of segment sg-1 on entry and the state entering segment sg on exit.
// The chain over segments is serial, but the loads do not depend on it: they are issued eight
// segments at a time (sixteen measured slower) before the chain consumes them, so the kernel pays a few memory round trips
// instead of one per segment.
__global__ __launch_bounds__(kThreads) void segment_pass_kernel(float *__restrict__ seg_state,
                                                                const float *__restrict__ seg_decay,
                                                                const float *__restrict__ h0, int S_plain, int H,
                                                                size_t rows, const VarPlan vp, const NSlice ns) {
  constexpr int kAhead = 8;
  const int e = (blockIdx.x * kThreads + threadIdx.x) * 4;
  if (vp.tok0 != nullptr) rows = static_cast<size_t>(max(0, vp.item0[vp.nseq] - vp.nseq)) * H;  // (none if rejected)
  for (size_t row = blockIdx.y; row < rows; row += gridDim.y) {
  int S = S_plain;
  size_t bh = row, slot0 = row * S_plain;  // (sequence, head); its first slot
  if (vp.tok0 != nullptr) {
    // one row per head and non-last segment of the list; the row of a sequence's first segment does its chain
    const int i = static_cast<int>(row / H), h = static_cast<int>(row % H);
    const int q = vp.item_seq[i];
    const int first = vp.item0[q];
    if (i != first - q) continue;
    S = vp.item0[q + 1] - first;
    bh = static_cast<size_t>(q) * H + h;
    slot0 = static_cast<size_t>(h) * vp.slot_cap + vp.slot0[q];
  }
  if (S < 2) continue;  // a single segment starts from h0 itself
  f32x4 run = {0.f, 0.f, 0.f, 0.f};
  if (h0 && e % kN < ns.valid)  // h0 rows hold ns.width columns, of which this launch owns a slice
    run = *reinterpret_cast<const f32x4 *>(h0 + (bh * kP + e / kN) * ns.width + ns.off + e % kN);
  float *sp = seg_state + slot0 * (kP * kN) + e;
  const float *dp = seg_decay + slot0;
  *reinterpret_cast<f32x4 *>(sp) = run;
  for (int s0 = 1; s0 < S; s0 += kAhead) {
    f32x4 v[kAhead];
    float d[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      const int sg = min(s0 + k, S - 1);  // clamped: the surplus loads of the last group are not used
      v[k] = *reinterpret_cast<const f32x4 *>(sp + static_cast<size_t>(sg) * kP * kN);
      d[k] = dp[sg - 1];
    }
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      if (s0 + k < S) {
        const float f = fast_exp2(d[k]);
        run = f32x4{f * run.x + v[k].x, f * run.y + v[k].y, f * run.z + v[k].z, f * run.w + v[k].w};
        *reinterpret_cast<f32x4 *>(sp + static_cast<size_t>(s0 + k) * kP * kN) = run;
      }
    }
  }
  }
}

// Blocks per segment.  A segment is any whole number of 64-token blocks; the number of segments, and
// with it the workspace, is bounded by max_segments (plain batch) or by one segment per chunk (packed
// batch).  The
// choice minimises a small cost model fitted to measurements on MI355X (microseconds): one workgroup
// per CU is resident, workgroups run in rounds of 256, a workgroup walks its blocks (plus a prologue
// worth about two) at a per-block time that grows with the number of workgroups competing for
// memory, and more than one segment costs the states pass (same structure, cheaper blocks), the
// serial pass over segment states (traffic proportional to segments x sequences) and two launches.
// The constants are a least-squares fit to 31 timed (shape, segment length) points of the three
// bf16 benchmark shapes (residual 5 us rms).
// The test-only knobs (see Knobs) force chunks or blocks per segment, and pieces per segment in the
// states-only pass.
constexpr int kNumCUs = 256;
double rounds_time(long wgs, double blocks, double t_idle, double t_busy) {
  double t = 0.0;
  for (long left = wgs; left > 0; left -= kNumCUs) {
    const double n = static_cast<double>(left < kNumCUs ? left : kNumCUs);
    const double load = n / kNumCUs;
    t += (blocks + 1.9) * (t_idle + (t_busy - t_idle) * load);
  }
  return t;
}
// Most segments a plain batch may be cut into (the workspace holds one state slot per segment and
// head): one per chunk, or -- short prompts, few heads -- one per block as long as that does not
// exceed what fills the chip several times over; and never more than fill the chip four times over
// (at least 64), which keeps the workspace of a very long prompt small: the choice below would not
// take more anyway.
// Workgroups of four head slots per batch row and segment: every B/C group has ceil(slices per group / 4).
int head_groups(const Dims &d, int heads = kHeadsPerWg) { return d.G * ((d.hpg * (d.P / kP) + heads - 1) / heads); }
int max_segments(const Dims &d) {
  const int nblocks = (d.T + kBlk - 1) / kBlk;
  const long groups = static_cast<long>(d.Bt) * head_groups(d);
  long by_fill = (8L * kNumCUs + groups - 1) / groups;
  if (by_fill > 64) by_fill = 64;
  if (by_fill > nblocks) by_fill = nblocks;
  long most = (4L * kNumCUs + groups - 1) / groups;
  if (most < 64) most = 64;
  long s = d.Nc > by_fill ? d.Nc : by_fill;
  if (s > most) s = most;
  return static_cast<int>(s);
}
// Modelled time of the states-only pass plus the chain over state slots when each of the S - 1
// segments it covers is cut into k pieces (see ScanParams::parts); the best k among the divisors of
// the segment length, at most max_slots slots.  max_parts = 1: segments are not cut.
double states_cost(long groups, double seqs, int S, int seg_blocks, int max_slots, int max_parts, int *parts) {
  double best = 0.0;
  *parts = 1;
  for (int k = 1; k <= max_parts && k <= seg_blocks; ++k) {
    if (seg_blocks % k != 0 || (k > 1 && (S - 1) * k + 1 > max_slots)) continue;
    const double cost = rounds_time(groups * (S - 1) * k, seg_blocks / k, 1.16, 1.16) + 0.0261 * ((S - 1) * k + 1) * seqs;
    if (k == 1 || cost < best) {
      best = cost;
      *parts = k;
    }
  }
  return best;
}

// min_blocks: the shortest segment allowed (packed batches size their tables for whole chunks).
constexpr double kColdXBytes = 144.0 * 1024 * 1024;  // x above this does not survive in the memory-side cache
int choose_seg_blocks(const Dims &d, int min_blocks, int max_slots, int max_parts) {
  const int chunk_blocks = d.L / kBlk;
  const int nblocks = (d.T + kBlk - 1) / kBlk;
  if (const int k = knobs().seg_chunks; k >= 1) return (k > d.Nc ? d.Nc : k) * chunk_blocks;
  if (const int k = knobs().seg_blocks; k >= min_blocks && k >= 1) return k;
  const int slices = d.H * (d.P / kP);
  const long groups = static_cast<long>(d.Bt) * head_groups(d);
  const double seqs = static_cast<double>(d.Bt) * slices;
  const int hi = nblocks > min_blocks ? nblocks : min_blocks;
  int best_blocks = hi;
  double best = 0.0;
  bool have = false;
  // The states pass leaves the x it has read -- every segment but the last of each sequence -- in the
  // memory-side cache, where the full scan finds it again; the last segment's x comes from HBM if the
  // tensor is too large to have stayed there from whoever wrote it, at a measured 1.25 times the per-block
  // time.  Segments somewhat longer than the count needs, leaving a shorter last one, even that out (8 x
  // 4096 tokens x 48 heads: 168 us with 32 + 32 blocks, 161 with 36 + 28).
  const double x_bytes = static_cast<double>(d.Bt) * d.T * d.H * d.P * 2.0;
  const double cold = x_bytes > kColdXBytes ? 1.25 : 1.0;
  for (int cand = min_blocks; cand <= hi; ++cand) {
    const long segs = (nblocks + cand - 1) / cand;
    const double last = static_cast<double>(nblocks - (segs - 1) * cand);
    const double walk = segs > 1 && cold * last > cand ? cold * last : cand;  // the longest walk, in warm blocks
    double cost = rounds_time(groups * segs, walk, 2.57, 3.35);
    int parts;
    if (segs > 1) {
      cost += states_cost(groups, seqs, static_cast<int>(segs), cand, max_slots, max_parts, &parts) + 3.1 + 7.0;
      // a short chain over state slots is summed by the full scan itself (see ScanParams::fold): no pass over
      // segment states and its launch, one more trip to memory per slot beyond the first instead (the net
      // saving measured on six shapes of 24 to 384 sequences: 2 to 11 us)
      if ((segs - 1) * parts <= knobs().fold_max_slots) cost -= 1.5 + 0.025 * seqs;
    }
    if (!have || cost < best) {
      have = true;
      best = cost;
      best_blocks = cand;
    }
  }
  return best_blocks;
}

// A launch whose workgroups number at most one per CU when they take two heads each takes two: its computing waves have
// their SIMD's vector unit almost to themselves and are fed by others (see pair_walk), which is worth more than the shared tiles
// that are then fetched twice as often.  (Of the states-only pass alone the same holds: on 45 drawn shapes grids of up to
// 256 take 0.82 to 1.01 of the time of four heads; it loses at 16384 tokens x 80 heads, 35.8 -> 40.0 us.)
bool small_grid(long wgs_of_two) { return wgs_of_two <= kNumCUs; }

// Blocks per segment of a plain batch with two heads per workgroup, all in one round, and the pieces its states-only pass
// cuts a segment into; 0 where the sequences alone are more than a round.  Microseconds of a whole call, fitted to 90
// drawn shapes (300 to 18400 tokens, 2 to 163 slices, batches of up to 12) at the lengths that give 1 to 24 segments (611 timings,
// 4.6 % rms): the choice is 0.8 % behind the fastest of the timed lengths and takes 0.80 of the time of four heads
// with their own choice, 1.04 at worst (of 411 others 0.81; six 2 % slower and more, 5 x 3182 tokens x 40 heads with dstate 256 207
// us to 185, 3 x 9977 x 45 340 to 322; to ask both models would cost up to 39 % elsewhere).  Beyond a round four heads are as fast or faster (968 tokens x 141 heads in
// batches of 12: 150.9 us, two heads 157.7; 2328 x 139 in batches of 4: 130.5, two heads in two rounds 133.8).
// 8 x 4096 tokens x 48 heads 161 -> 130 us (one segment instead of two; 123 with y streamed), 2016 x 59 in batches of 6 100 -> 70.
int two_head_blocks(const Dims &d, int min_blocks, int max_slots, int *parts) {
  const int nblocks = (d.T + kBlk - 1) / kBlk;
  const long groups2 = static_cast<long>(d.Bt) * head_groups(d, 2), groups4 = static_cast<long>(d.Bt) * head_groups(d);
  const double seqs = static_cast<double>(d.Bt) * d.H * (d.P / kP);
  int best = 0;
  double best_us = 0.0;
  for (int cand = min_blocks > 2 ? min_blocks : nblocks < 2 ? 1 : 2; cand <= nblocks; ++cand) {
    const int S = (nblocks + cand - 1) / cand;
    if (!small_grid(groups2 * S)) continue;
    if (cand > min_blocks && best != 0 && S == (nblocks + cand - 2) / (cand - 1)) continue;  // (as many segments, and longer)
    const double load = static_cast<double>(groups2 * S) / kNumCUs;
    double us = 11.0 + (1.11 + 1.04 * load) * cand;
    int k = 1;
    if (S > 1) {
      (void)states_cost(groups4, seqs, S, cand, max_slots, 8, &k);
      const int slots = (S - 1) * k;
      us += 3.93 + 0.72 * (cand / k) * static_cast<double>((groups2 * slots + kNumCUs - 1) / kNumCUs);
      us += slots <= knobs().fold_max_slots ? (0.66 + 0.0119 * seqs) * slots : 3.94 + 0.0184 * slots * seqs;
    }
    if (best == 0 || us < best_us) {
      best = cand;
      best_us = us;
      *parts = k;
    }
  }
  return best;
}

// Workspace.  Plain batch: rows = Bt sequences of NB blocks each.  Variable-length batch: one "row" whose
// NB is the block capacity ceil(total / 64) + nseq (every sequence may end in a partial block), whose
// segment list holds at most NB / (blocks per chunk) + nseq + 1 entries (a segment is at least a
// chunk, and every sequence has at least one segment) and whose state slots -- needed only by
// sequences of several segments, which are longer than a segment and so cannot be many -- number at
// most min(that, 4 ceil(total / 64) / (blocks per chunk) + 4); then the int32 tables of VarPlan.
struct Layout {
  int NB, S_max, items_max;
  size_t off_G, off_Bt, off_prep, off_state, off_decay, off_tables, off_Cpad, total;
};

Layout make_layout(const Dims &d, bool varlen) {
  Layout w;
  const int rows = varlen ? 1 : d.Bt;
  const int nseq = varlen ? d.Bt : 0;
  w.NB = (d.T + kBlk - 1) / kBlk + nseq;
  const int cb = d.L / kBlk;  // a segment is at least one chunk
  w.items_max = varlen ? w.NB / cb + nseq + 1 : max_segments(d);
  w.S_max = w.items_max;      // state slots per head
  if (varlen) {
    const long tight = 4L * ((d.T + kBlk - 1) / kBlk) / cb + 4;
    if (tight < w.S_max) w.S_max = static_cast<int>(tight);
  }
  const size_t BG = static_cast<size_t>(rows) * d.G, BH = static_cast<size_t>(rows) * d.H;
  const size_t BHs = BH * (d.P / kP);  // 64-column slices
  size_t off = 0;
  w.off_G = off;
  off += round_up(BG * w.NB * kBlk * kBlk * sizeof(uint16_t), 256);
  w.off_Bt = off;
  off += round_up(BG * w.NB * kN * kBlk * sizeof(uint16_t), 256);
  w.off_prep = off;
  off += round_up(BH * w.NB * kRec * sizeof(float), 256);
  w.off_state = off;
  off += round_up(BHs * w.S_max * kP * kN * sizeof(float), 256);
  w.off_decay = off;
  off += round_up(BHs * w.S_max * sizeof(float), 256);
  w.off_tables = off;
  if (varlen) off += round_up((5 * (static_cast<size_t>(nseq) + 1) + w.NB + w.items_max) * sizeof(int32_t), 256);
  // dstate other than 128: a 128-column copy of the slice of C in work
  const size_t tokens = static_cast<size_t>(rows) * d.T;
  w.off_Cpad = off;
  if (d.N != kN) off += round_up(tokens * d.G * kN * sizeof(uint16_t), 256);
  w.total = off;
  return w;
}

bool shape_ok(const Dims &d, unsigned long long tokens, unsigned long long nb) {
  // one sequence of x, C and the per-head block records must be addressable with 32-bit byte offsets
  const unsigned long long lim = 0xFFFF0000ull;
  return d.bf16 && d.P % kP == 0 && d.P <= 16 * kP && d.N % 8 == 0 && d.N <= 4 * kN && d.Bt <= 65535 && d.H <= 65535 &&
         tokens * d.H * (static_cast<unsigned long long>(d.P) * 2) <= lim &&
         tokens * d.G * (static_cast<unsigned long long>(d.N > kN ? d.N : kN) * 2) <= lim &&
         nb * (kN * kBlk * 2) <= lim;
}

// Whether the full kernel writes y with non-temporal stores.  The 256 MiB memory-side cache (Infinity Cache)
// holds x when the kernel starts -- the states-only pass has just read it, or the producer (the convolution)
// has just written it -- unless the y written meanwhile pushes it out before it is read.  Once x takes more
// than a quarter of that cache, x and y no longer fit side by side and y is streamed past the caches.
// Measured (prefill alone, back to back; us with ordinary / non-temporal stores): x of 64-96 MiB 80 / 79, 62 / 62,
// 88 / 88 (no difference: below a quarter of the cache the consumer of y is better off finding it cached);
// 128 MiB 122 / 110 (two passes over x) and 109 / 97 (one); 160 MiB 151 / 131; 192 MiB 178 / 171 and 175 / 153;
// 256 MiB 220 / 211; 320 MiB 278 / 281 (nothing left to protect, nothing lost).  With a dstate above 128 the
// later state slices read y back to add to it, but they read x twice more: the first slice streams y all the
// same (dstate 256: 333 -> 307 us).  With two heads per workgroup (ordinary / non-temporal): the same inputs again and again,
// 16384 tokens x 80 heads in six segments 144 / 123, 3 packed sequences of 24001 x 63 201 / 181, 8 x 4096 x 48 in one 129 / 119;
// inputs that come cold 145 / 148, 208 / 201 and 127 / 121; x just written by the convolution, as a layer finds it, 146 / 146,
// 207 / 194 and 137 / 123, the pair 213 / 199, 298 / 264 and 225 / 192.  The y_stream knob overrides (tests, tuning).
constexpr unsigned long long kMemCacheBytes = 256ull << 20;
bool stream_y(const Dims &d, int rows) {
  if (knobs().y_stream >= 0) return knobs().y_stream != 0;
  const unsigned long long x_bytes = 2ull * rows * d.T * d.H * d.P;
  return 4 * x_bytes > kMemCacheBytes;
}

// Entries of a packed batch's list of segments, at most: those that are not the last of their sequence (each is
// seg_blocks whole blocks with a token behind them); all of them.
int full_items(const Dims &d, const Layout &w, int seg_blocks) { return (w.NB - d.Bt - 1) / seg_blocks; }
int list_items(const Dims &d, const Layout &w, int seg_blocks) { return d.Bt + full_items(d, w, seg_blocks); }

// Whether items can be dealt: that walk addresses the decay records by 32-bit offsets.
bool deal_possible(const Layout &w) { return w.off_state - w.off_prep < 0xFFFF0000ull; }
bool packed_uncut(const Dims &d, const SlicePlan &pl);
bool packed_dealt(const Dims &d, int seg_blocks);
bool dealt_states_two(const Dims &d);
// How a call is cut up: blocks per segment, segments per sequence (0 for a packed batch, where the
// device-side tables hold them per sequence), pieces per segment of the states-only pass, and whether the
// full scan sums the chain over state slots itself (ScanParams::fold).
SlicePlan plan_slice(const Dims &d, bool varlen, bool h0_aliases_final_state) {
  const Layout w = make_layout(d, varlen);
  Dims one = d;  // the segment length of a packed batch is chosen as for one sequence of all its tokens
  if (varlen) one.Bt = 1;
  SlicePlan pl;
  const Knobs &kn = knobs();
  pl.two = 0;
  pl.state_heads = kn.scan_heads == 2 ? 2 : kHeadsPerWg;
  pl.heads = pl.state_heads;
  // two heads per workgroup (see small_grid)
  const bool may_choose = kn.scan_heads == 0 && kn.seg_chunks == 0 && kn.seg_blocks == 0 && kn.seg_parts == 0;
  const bool may_two = kn.scan_heads == 0;
  int two_parts = 1;
  const int two = !varlen && may_choose && may_two ? two_head_blocks(d, (w.NB + w.S_max - 1) / w.S_max, w.S_max, &two_parts) : 0;
  // shortest segment: a chunk for a packed batch; what the state slots allow for a plain one
  pl.seg_blocks = two > 0 ? two : choose_seg_blocks(one, varlen ? d.L / kBlk : (w.NB + w.S_max - 1) / w.S_max, w.S_max, varlen ? 1 : 8);
  if (!varlen && (w.NB + pl.seg_blocks - 1) / pl.seg_blocks > w.S_max) pl.seg_blocks = (w.NB + w.S_max - 1) / w.S_max;
  pl.segments = varlen ? 0 : (w.NB + pl.seg_blocks - 1) / pl.seg_blocks;
  // pieces per segment for the states-only pass (see ScanParams): the split with the least modelled
  // time of that pass plus the longer chain over state slots, among the divisors of the segment length
  pl.parts = 1;
  if (two > 0) {
    pl.two = 1;
    pl.parts = two_parts;
  } else if (!varlen && pl.segments > 1) {
    const long groups = static_cast<long>(d.Bt) * head_groups(d);
    const double seqs = static_cast<double>(d.Bt) * d.H * (d.P / kP);
    (void)states_cost(groups, seqs, pl.segments, pl.seg_blocks, w.S_max, 8, &pl.parts);
    if (const int k = knobs().seg_parts; k >= 1 && pl.seg_blocks % k == 0 && (pl.segments - 1) * k + 1 <= w.S_max) pl.parts = k;
  }
  const int seqs = varlen ? 1 : d.Bt;
  // (the lengths of several sequences are known on the device only; see segment_choice)
  pl.from_lengths = varlen && d.Bt > 1 && d.Bt <= kTableThreads && w.NB <= kTableBlocks && list_items(d, w, pl.seg_blocks) <= kTableBlocks &&
                    kn.seg_chunks == 0 && kn.seg_blocks == 0 && full_items(d, w, pl.seg_blocks) > 0;
  pl.listed = varlen && deal_possible(w) && (kn.deal == 1 || (may_two && kn.deal == 0 && packed_dealt(d, pl.seg_blocks)));
  if (pl.listed) pl.heads = 2;
  if (pl.from_lengths) {
    // (what is not dealt comes to 1.75 rounds of workgroups of two heads at most, but for records of 4 GiB; see packed_dealt)
    if (may_two) pl.heads = 2;
    if (may_two && (!pl.listed || dealt_states_two(d))) pl.state_heads = 2;
    if (packed_uncut(d, pl)) {
      pl.from_lengths = false;
      pl.seg_blocks = w.NB - d.Bt;
    }
  }
  if (!pl.from_lengths && may_two) {  // (packed batch of one segment length: by the most entries that the lists can have)
    const long full = varlen ? full_items(d, w, pl.seg_blocks) : static_cast<long>(pl.segments - 1) * pl.parts;
    const long all = varlen ? list_items(d, w, pl.seg_blocks) : pl.segments;
    if (small_grid(all * seqs * head_groups(d, 2))) pl.heads = 2;
    if (small_grid(full * seqs * head_groups(d, 2))) pl.state_heads = 2;
  }
  // A short chain over state slots is a sum of few terms (and h0), which the later segments' workgroups form
  // as they load their state -- one launch and one round trip of every state through memory less (8 x 4096
  // tokens x 48 heads: 162 -> 152 us).  Not when h0 and final_state share memory: the last segment might
  // store the final state before the first has read h0.
  pl.fold = !varlen && pl.segments >= 2 && (pl.segments - 1) * pl.parts <= knobs().fold_max_slots && !h0_aliases_final_state ? 1 : 0;
  return pl;
}

// What the device may choose the segment length of a packed batch from: lengths from that of one sequence of all the tokens
// -- the shortest that pays, and what grids and tables are sized for -- to all the tokens, 13 % apart and more.
SegChoice segment_choice(const Dims &d, const SlicePlan &pl) {
  SegChoice c = {};
  const int nblocks = (d.T + kBlk - 1) / kBlk;
  c.cand[0] = pl.seg_blocks;
  c.count = 1;
  if (!pl.from_lengths) return c;
  const double ratio = fmax(1.13, pow(static_cast<double>(nblocks) / pl.seg_blocks, 1.0 / 20));
  while (c.count < SegChoice::kMost && c.cand[c.count - 1] < nblocks) {
    const int last = c.cand[c.count - 1], next = static_cast<int>(last * ratio + 0.5);
    c.cand[c.count++] = next > last ? (next < nblocks ? next : nblocks) : last + 1;
  }
  c.dealt = pl.listed;
  const int groups = head_groups(d, pl.heads);
  c.max_items = pl.heads == 2 && !pl.listed ? kNumCUs / groups : 0x7fffffff;
  c.state_fill = static_cast<float>(head_groups(d, pl.state_heads)) / kNumCUs;
  c.fill = static_cast<float>(groups) / kNumCUs;
  c.slices = static_cast<float>(d.H) * (d.P / kP);
  return c;
}

// Whether the scan's workgroups are dealt items (see Deal), by what the sequences alone come to in rounds of two-head
// workgroups.  Up to a round there is nothing to even out.  Beyond, of 420 drawn batches of up to four rounds (microseconds, an entry to a
// workgroup over dealt; ragged, equal lengths, one or a few long ones among short): entries of more than 16 workgroups 1.03 to
// 1.05 for ragged ones up to two rounds and 1.15 to 1.22 beyond 32, more of both after; smaller ones 0.94 to 0.97 up to 1.75
// rounds (27 ragged sequences, 3923 tokens x 20 heads in four groups, dstate 256: 72.9, dealt 80.0), 1.01 to 1.14 after.  What is lost: equal lengths
// up to 1.75 rounds 0.92 to 0.98, which four heads to a workgroup serve in one; a few items beside which all others are short
// 0.85 at worst, because everyone is dealt as many (56 sequences, 5005 tokens, 7 of them 554 long, x 74 heads 92, dealt 103).
// Only a sorted list is dealt: of one in the caller's order, 2500 sequences x 8 heads with a long one in every 64, the same
// workgroups got all the long ones (430 us, dealt 639).
bool packed_dealt(const Dims &d, int seg_blocks) {
  const int groups2 = head_groups(d, 2);
  return list_sorted(d.Bt, seg_blocks) && 4l * d.Bt * groups2 > (groups2 > 16 ? 4 : 7) * kNumCUs;
}

// Whether the states-only pass of a dealt batch has two heads per workgroup.  They are faster if its entries -- the segments that
// are not the last of their sequence, which only the device knows -- come to a round of them (of 160 dealt batches with long
// sequences among short ones 78 are 1.01 to 1.09 times as fast as with four), and slower beyond (38 of them 0.91 to 0.99).  They are expected to be
// few up to ten blocks a CU, and up to three rounds of small entries.  By this rule the 160 are 1.014 times as fast as with four
// heads throughout (1.010 with two throughout, 28 of them slower than with four).
bool dealt_states_two(const Dims &d) {
  const int groups2 = head_groups(d, 2), nblocks = (d.T + kBlk - 1) / kBlk;
  return static_cast<long>(nblocks) * groups2 < 10 * kNumCUs || (groups2 <= kNumCUs / 8 && static_cast<long>(d.Bt) * groups2 <= 3 * kNumCUs);
}

// Whether a short packed batch is left uncut, whatever its lengths: cutting it, or the chance of it, costs the launches of
// the states pass and the chain (8 us), which is a quarter of such a call and more.  So it is where the worst mix -- one
// sequence and a token for each of the others -- is at most a tenth slower uncut by the model.  Up to 20 blocks, where
// the model is good to that: of 240 drawn batches 40, 31 to 43 us each, are 3 to 10 us faster for it and none is slower.
bool packed_uncut(const Dims &d, const SlicePlan &pl) {
  const int nblocks = (d.T + kBlk - 1) / kBlk;
  if (nblocks > 20) return false;
  const SegChoice c = segment_choice(d, pl);
  const int blocks = nblocks + d.Bt - 1;
  float best = 0.f, uncut = 0.f;
  for (int k = 0; k < c.count; ++k) {
    const int s = c.cand[k];
    uncut = packed_cost(c, s, blocks, nblocks, d.Bt, d.Bt - 1 + (nblocks + s - 1) / s);  // (the last candidate: no cut)
    if (k == 0 || uncut < best) best = uncut;
  }
  return uncut - 8.f <= 1.1f * best;
}

// The workgroups of a pass: `heads` head slices each, `segs` segments per sequence, `items` in all.
template <bool kPair>
void map_to(ScanParamsOf<kPair> &p, int heads, int segs, int items) {
  p.cpg = (p.hpg + heads - 1) / heads;
  p.cols = p.G * p.cpg;
  p.segs = segs;
  p.total = p.cols * items;
  p.per_xcd = (p.total + kXcds - 1) / kXcds;
  if constexpr (kPair) {
    p.cpg_inv = inverse_of(p.cpg);
    p.pdiv_inv = inverse_of(p.pdiv);
    p.cols_inv = inverse_of(p.cols);
    p.segs_inv = inverse_of(segs > 0 ? segs : 1);
  }
}

// d: plain batch (cu == nullptr), or Bt = number of sequences and T = total tokens of a packed batch.
// One state slice ns (see NSlice): y and final_state columns of that slice are written.
hipError_t launch_slice(const Dims &d, const NSlice ns, const int32_t *cu, const void *x, const float *dt,
                        const float *A, const void *B, const void *C, const float *D, const float *h0, void *y,
                        bool add_to_y, float *final_state, void *workspace, hipStream_t stream, KernelTrace *trace) {
  const bool varlen = cu != nullptr;
  const Layout w = make_layout(d, varlen);
  char *ws = static_cast<char *>(workspace);
  uint16_t *Gd = reinterpret_cast<uint16_t *>(ws + w.off_G);
  uint16_t *Btr = reinterpret_cast<uint16_t *>(ws + w.off_Bt);
  float *prep = reinterpret_cast<float *>(ws + w.off_prep);
  float *seg_state = reinterpret_cast<float *>(ws + w.off_state);
  float *seg_decay = reinterpret_cast<float *>(ws + w.off_decay);
  uint16_t *Cpad = d.N != kN ? reinterpret_cast<uint16_t *>(ws + w.off_Cpad) : nullptr;
  const int rows = varlen ? 1 : d.Bt;
  const size_t state_bytes = static_cast<size_t>(d.Bt) * d.H * d.P * ns.width * sizeof(float);
  const bool h0_aliases = h0 != nullptr && final_state != nullptr &&
                          reinterpret_cast<const char *>(h0) < reinterpret_cast<const char *>(final_state) + state_bytes &&
                          reinterpret_cast<const char *>(final_state) < reinterpret_cast<const char *>(h0) + state_bytes;
  const SlicePlan pl = plan_slice(d, varlen, h0_aliases);
  const int seg_blocks = pl.seg_blocks;

  VarPlan vp = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0, 0, 0};
  int S = (w.NB + seg_blocks - 1) / seg_blocks;  // plain batch: segments per sequence
  int items = S * d.Bt;                          // segments of the whole batch (varlen: upper bound)
  if (varlen) {
    int32_t *t = reinterpret_cast<int32_t *>(ws + w.off_tables);
    const int n1 = d.Bt + 1;
    int32_t *tok0 = t, *len = t + n1, *blk0 = t + 2 * n1, *item0 = t + 3 * n1, *slot0 = t + 4 * n1,
            *blk_seq = t + 5 * n1, *item_seq = blk_seq + w.NB;
    items = list_items(d, w, seg_blocks);
    S = 0;  // per sequence, from the tables
    vp = VarPlan{tok0, len, blk0, item0, slot0, blk_seq, item_seq, d.Bt, w.NB, w.S_max};
    if (!add_to_y) {  // (a later state slice finds the tables of the first)
      launch_varlen_tables(cu, d.T, kBlk, segment_choice(d, pl), items, vp, stream);
      trace_mark(trace, stream, "varlen_tables");
    }
  }

  const int n_scores = w.NB * rows * d.G;
  // (the decay records depend on dt and A alone: the first state slice has left them in the workspace)
  const int n_cumsum = add_to_y ? 0 : w.NB * ((d.H + kCumHeads - 1) / kCumHeads) * rows;
  hipLaunchKernelGGL(block_prep_kernel, dim3(n_scores + n_cumsum), dim3(kThreads), 0, stream,
                     static_cast<const uint16_t *>(B), static_cast<const uint16_t *>(C), Gd, Btr, dt, A, prep,
                     d.T, d.H, d.G, w.NB, n_scores, vp, ns, Cpad, d.dtx);
  trace_mark(trace, stream, "block_prep");

  const int pdiv = d.P / kP, Hs = d.H * pdiv, parts = pl.parts;
  auto fill = [&](auto &p) {
    p.x = static_cast<const uint8_t *>(x);
    p.C = Cpad != nullptr ? reinterpret_cast<const uint8_t *>(Cpad) : static_cast<const uint8_t *>(C);
    p.D = D;
    p.ns = ns;
    p.Gd = reinterpret_cast<const uint8_t *>(Gd);
    p.Btr = reinterpret_cast<const uint8_t *>(Btr);
    p.prep = prep;
    p.y = static_cast<uint8_t *>(y);
    p.h0 = h0;
    p.Hin = seg_state;
    p.final_state = final_state;
    p.seg_state = seg_state;
    p.seg_decay = seg_decay;
    p.T = d.T;
    p.H = Hs;
    p.pdiv = pdiv;
    p.Hrec = d.H;
    p.G = d.G;
    p.hpg = d.hpg * pdiv;
    p.NB = w.NB;
    p.seg_blocks = seg_blocks;
    p.S = S;
    p.parts = parts;
    p.part_blocks = seg_blocks / parts;
    p.slots = (S - 1) * parts + 1;
    p.vp = vp;
    p.fold = pl.fold;
  };
  // no states pass if no sequence can have more than one segment
  const int full_cap = varlen ? full_items(d, w, seg_blocks) : 0;
  if (varlen ? full_cap > 0 : S > 1) {
    // (which sequences of a packed batch have more than one segment is known on the device only: the workgroups of
    // entries that are last segments, or none, leave at once)
    ScanParams p;
    fill(p);
    map_to(p, pl.state_heads, (S - 1) * parts, varlen ? full_cap : (S - 1) * parts * d.Bt);
    const dim3 grid(kXcds * p.per_xcd), block(128 * pl.state_heads);
    if (pl.state_heads == 2)
      hipLaunchKernelGGL((chunk_scan_kernel<true, 2>), grid, block, 0, stream, p);
    else
      hipLaunchKernelGGL((chunk_scan_kernel<true, kHeadsPerWg>), grid, block, 0, stream, p);
    trace_mark(trace, stream, "segment_states");
    const size_t rows_bh = static_cast<size_t>(varlen ? full_cap : d.Bt) * Hs;
    const size_t most_rows = varlen ? 512 : 65535;  // (packed: most rows hold no chain, and there may be none at all)
    if (!p.fold)
      hipLaunchKernelGGL(segment_pass_kernel, dim3(kP * kN / (4 * kThreads), rows_bh > most_rows ? most_rows : rows_bh),
                         dim3(kThreads), 0, stream, seg_state, seg_decay, h0, p.slots, Hs, rows_bh, vp, ns);
    if (!p.fold) trace_mark(trace, stream, "segment_pass");
  }
  const int scan_items = varlen ? items : S * d.Bt;
  if (pl.heads == 2) {
    PairParams p;
    fill(p);
    p.prep_bytes = static_cast<uint32_t>(w.off_state - w.off_prep);
    map_to(p, 2, S, scan_items);
    auto *const kernel = add_to_y ? (pl.listed ? pair_scan_kernel<kYAdd, true> : pair_scan_kernel<kYAdd, false>)
                         : stream_y(d, rows) ? (pl.listed ? pair_scan_kernel<kYStream, true> : pair_scan_kernel<kYStream, false>)
                                             : (pl.listed ? pair_scan_kernel<kYPlain, true> : pair_scan_kernel<kYPlain, false>);
    hipLaunchKernelGGL(kernel, dim3(pl.listed ? kNumCUs : kXcds * p.per_xcd), dim3(512), 0, stream, p);
  } else {
    ScanParams p;
    fill(p);
    map_to(p, kHeadsPerWg, S, scan_items);
    auto *const kernel = add_to_y              ? chunk_scan_kernel<false, kHeadsPerWg, kYAdd>
                         : stream_y(d, rows) ? chunk_scan_kernel<false, kHeadsPerWg, kYStream>
                                             : chunk_scan_kernel<false, kHeadsPerWg, kYPlain>;
    hipLaunchKernelGGL(kernel, dim3(kXcds * p.per_xcd), dim3(128 * kHeadsPerWg), 0, stream, p);
  }
  trace_mark(trace, stream, "chunk_scan");
  return hipGetLastError();
}

// All state slices: the first writes y (with the skip term D x), every later one adds its output, without the
// skip term, to y where it stores it (the sum is formed in fp32 from the bf16 values and rounded once more:
// y carries up to 1.5 bf16 ulp with two slices instead of 0.5).
hipError_t launch(const Dims &d, const int32_t *cu, const void *x, const float *dt, const float *A, const void *B,
                  const void *C, const float *D, const float *h0, void *y, float *final_state, void *workspace,
                  hipStream_t stream, KernelTrace *trace) {
  for (int off = 0; off < d.N; off += kN) {
    const NSlice ns = {d.N, off, d.N - off < kN ? d.N - off : kN};
    const hipError_t e = launch_slice(d, ns, cu, x, dt, A, B, C, off == 0 ? D : nullptr, h0, y, off > 0, final_state,
                                      workspace, stream, off == 0 ? trace : nullptr);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

}  // namespace

// Tables of a packed batch for blocks of blk_len tokens (the MFMA kernels: 64; the generic kernels:
// one chunk).  vp names the table arrays (device, int32: tok0, len,
// blk0, item0, slot0 of nseq + 1 entries each, blk_seq of nb_cap, item_seq of item_cap entries).
void launch_varlen_tables(const int32_t *cu, int total, int blk_len, const SegChoice &choice, int item_cap, const VarPlan &vp,
                          hipStream_t stream) {
  const int cap = vp.nb_cap > item_cap ? vp.nb_cap : item_cap;
  if (vp.nseq <= kTableThreads && cap <= kTableBlocks) {
    hipLaunchKernelGGL(varlen_tables_kernel, dim3(1), dim3(kTableThreads), 0, stream, cu, vp.nseq, total, blk_len, choice,
                       const_cast<int32_t *>(vp.tok0), const_cast<int32_t *>(vp.len), const_cast<int32_t *>(vp.blk0),
                       const_cast<int32_t *>(vp.item0), const_cast<int32_t *>(vp.slot0),
                       const_cast<int32_t *>(vp.blk_seq), const_cast<int32_t *>(vp.item_seq));
    return;
  }
  const int seg_blocks = choice.cand[0];
  hipLaunchKernelGGL(varlen_scan_kernel, dim3(1), dim3(256), 0, stream, cu, vp.nseq, total, blk_len, seg_blocks,
                     const_cast<int32_t *>(vp.tok0), const_cast<int32_t *>(vp.len), const_cast<int32_t *>(vp.blk0),
                     const_cast<int32_t *>(vp.item0), const_cast<int32_t *>(vp.slot0));
  hipLaunchKernelGGL(varlen_fill_kernel, dim3((cap + 255) / 256), dim3(256), 0, stream, vp.blk0, vp.item0, vp.nseq,
                     seg_blocks, const_cast<int32_t *>(vp.blk_seq), const_cast<int32_t *>(vp.item_seq));
}

// The kernels work on 64-token blocks whatever the chunk length is (results do not depend on it); the chunk
// only bounds the number of segments, for which it counts as the next multiple of 64.
static Dims with_block_chunk(const Dims &d_in) {
  Dims d = d_in;
  d.L = (d.L + kBlk - 1) / kBlk * kBlk;
  d.Nc = (d.T + d.L - 1) / d.L;
  return d;
}

bool mfma_supported(const Dims &d) {
  return shape_ok(d, static_cast<unsigned long long>(d.T), (static_cast<unsigned long long>(d.T) + kBlk - 1) / kBlk);
}

size_t mfma_workspace_bytes(const Dims &d) { return make_layout(with_block_chunk(d), false).total; }

SlicePlan mfma_plan(const Dims &d, bool h0_aliases_final_state) {
  return plan_slice(with_block_chunk(d), false, h0_aliases_final_state);
}

SlicePlan mfma_varlen_plan(const Dims &d_in, const int32_t *cu) {
  const Dims d = with_block_chunk(d_in);
  SlicePlan pl = plan_slice(d, true, false);
  const SegChoice c = segment_choice(d, pl);
  pl.shortest = pl.seg_blocks;
  float cost[SegChoice::kMost], best = 0.f;
  int items[SegChoice::kMost];
  for (int k = 0; k < c.count; ++k) {
    int longest = 0, blocks = 0;
    items[k] = 0;
    for (int q = 0; q < d.Bt; ++q) {
      const int n = (cu[q + 1] - cu[q] + kBlk - 1) / kBlk;
      items[k] += n > c.cand[k] ? (n + c.cand[k] - 1) / c.cand[k] : 1;
      longest = n > longest ? n : longest;
      blocks += n;
    }
    cost[k] = c.count > 1 ? packed_cost(c, c.cand[k], blocks, longest, d.Bt, items[k]) : 0.f;
    if (k == 0 || cost[k] < best) best = cost[k];
  }
  int k = 0;
  while (cost[k] > (c.dealt ? kDealtMargin : 1.f) * best) ++k;
  pl.seg_blocks = c.cand[k];
  pl.segments = items[k];
  return pl;
}

hipError_t launch_prefill_mfma(const Dims &d, const void *x, const float *dt, const float *A, const void *B,
                               const void *C, const float *D, const float *h0, void *y, float *final_state,
                               void *workspace, hipStream_t stream, KernelTrace *trace) {
  return launch(with_block_chunk(d), nullptr, x, dt, A, B, C, D, h0, y, final_state, workspace, stream, trace);
}

// Packed variable-length batch: d.Bt sequences, d.T tokens in total, boundaries in the device array cu.
bool mfma_varlen_supported(const Dims &d) {
  const unsigned long long nb = (static_cast<unsigned long long>(d.T) + kBlk - 1) / kBlk + d.Bt;
  return shape_ok(d, static_cast<unsigned long long>(d.T), nb) && nb <= 0x7fffffffull / 64;
}

size_t mfma_varlen_workspace_bytes(const Dims &d) { return make_layout(with_block_chunk(d), true).total; }

hipError_t launch_prefill_mfma_varlen(const Dims &d, const int32_t *cu_seqlens, const void *x, const float *dt,
                                      const float *A, const void *B, const void *C, const float *D, const float *h0,
                                      void *y, float *final_state, void *workspace, hipStream_t stream,
                                      KernelTrace *trace) {
  return launch(with_block_chunk(d), cu_seqlens, x, dt, A, B, C, D, h0, y, final_state, workspace, stream, trace);
}

}  // namespace ssd
