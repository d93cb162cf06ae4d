// Internal declarations shared by the translation units of the SSD library.
// Nothing here is part of the C ABI (see include/ssd.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "ssd.h"

namespace ssd {

// n / d of scalars by a multiplication with (2^32 - 1) / d, which falls short by one at most.  The start of every workgroup is
// a few such divisions, of 20 to 30 dependent instructions otherwise.
__device__ __forceinline__ int quotient(int n, int d, uint32_t inv) {
  const int q = static_cast<int>(__umulhi(static_cast<uint32_t>(n), inv));
  return q + (n - q * d >= d ? 1 : 0);
}
inline uint32_t inverse_of(int d) { return 0xFFFFFFFFu / static_cast<uint32_t>(d); }

// Optional map from the caller's dt values to the step size (section "Mapping SSD onto JAX
// primitives" lists softplus and clip among the elementwise neighbours that must fuse with the
// decay computation): dt = clamp(softplus(raw + bias[h]), lo, hi).  Default: dt is used as given.
struct DtXform {
  const float *bias = nullptr;  // (nheads) -- decode: (nlayers, nheads) --, device; nullptr = none
  int softplus = 0;
  float lo = 0.f, hi = 0.f;     // clamp to [lo, hi] if hi > 0
  bool identity() const { return bias == nullptr && softplus == 0 && !(hi > 0.f); }
};
// (bias already fetched: kernels that apply the map step after step read it once)
__device__ __forceinline__ float dt_apply_biased(float v, float bias, const DtXform &t) {
  v += bias;
  if (t.softplus) v = v > 20.f ? v : log1pf(expf(v));
  if (t.hi > 0.f) v = fminf(fmaxf(v, t.lo), t.hi);
  return v;
}
__device__ __forceinline__ float dt_apply(float v, int h, const DtXform &t) {
  return dt_apply_biased(v, t.bias != nullptr ? t.bias[h] : 0.f, t);
}
// The same map without a branch (hardware exp2, log2 and reciprocal), for code whose loads must not wait at a join:
// softplus(v) = max(v, 0) + log(1 + e), e = exp(-|v|).  Small step sizes keep their relative accuracy -- 2e-7 from
// v = -80 to 20, where log1pf(expf(v)) has 1.2e-7 --: what the product with log2(e) rounds away comes back as a factor of
// e, and what 1 + e rounds away, which is most of a small e, as the first term of the logarithm's series.
__device__ __forceinline__ float dt_apply_branchless(float v, float bias, const DtXform &t) {
  v += bias;
  const float a = -fabsf(v), p = a * 1.44269502f;
  const float low = fmaf(a, 1.92596303e-8f, fmaf(a, 1.44269502f, -p));  // 1.44269502 + 1.926e-8 = log2(e)
  const float e2 = __builtin_amdgcn_exp2f(p);
  const float e = fmaf(e2, a > -128.f ? low * 0.693147182f : 0.f, e2);
  const float u = 1.f + e;
  const float sp = fmaxf(v, 0.f) + fmaf(0.693147182f, __builtin_amdgcn_logf(u), (e - (u - 1.f)) * __builtin_amdgcn_rcpf(u));
  v = t.softplus ? sp : v;
  const float cl = fminf(fmaxf(v, t.lo), t.hi);
  return t.hi > 0.f ? cl : v;
}

// The log2 decay of a token, cut off at 2^-160, which is zero in fp32 either way.  The decay between two tokens is a
// difference of prefix sums: with a token of dt |A| = 1e6 in them, uncut, it is off by a per cent and more for all tokens
// behind.  (A NaN stays.)
constexpr float kCutLog2 = -160.f;
__device__ __forceinline__ float cut_decay(float d) { return d < kCutLog2 ? kCutLog2 : d; }
// The same on the step size, whose product with alog = A log2(e) may then join the first sum (one rounding less).
__device__ __forceinline__ float cut_step(float dt, float alog) {
  return dt * alog < kCutLog2 ? kCutLog2 * __builtin_amdgcn_rcpf(alog) : dt;
}

// Validated problem dimensions (host side).
struct Dims {
  int Bt, T, H, P, N, G, L;
  int Nc;     // number of chunks, ceil(T / L)
  int hpg;    // heads per B/C group
  bool bf16;  // io dtype of x, B, C, y
  DtXform dtx;  // step-size map of the *_dt entry points (identity otherwise)
};

// ---- bf16 <-> fp32 (bf16 = upper half of the fp32 pattern, round-to-nearest-even) ----
__device__ __forceinline__ float bf16_bits_to_f32(uint16_t v) {
  return __uint_as_float(static_cast<uint32_t>(v) << 16);
}
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return static_cast<uint16_t>((u >> 16) | 0x0040u);  // quiet NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(u >> 16);
}

// Element access for the two io dtypes.
struct IoF32 {
  using type = float;
  static __device__ __forceinline__ float load(const void *p, size_t i) {
    return static_cast<const float *>(p)[i];
  }
  static __device__ __forceinline__ void store(void *p, size_t i, float v) {
    static_cast<float *>(p)[i] = v;
  }
};
struct IoBf16 {
  using type = uint16_t;
  static __device__ __forceinline__ float load(const void *p, size_t i) {
    return bf16_bits_to_f32(static_cast<const uint16_t *>(p)[i]);
  }
  static __device__ __forceinline__ void store(void *p, size_t i, float v) {
    static_cast<uint16_t *>(p)[i] = f32_to_bf16_bits(v);
  }
};

// Optional per-kernel timing (used only by the measurement library): an event is recorded on the
// launch stream after every kernel of a prefill call.
struct KernelTrace {
  static constexpr int kMax = 8;
  int n = 0;
  hipEvent_t ev[kMax + 1];
  const char *names[kMax];
};
inline void trace_mark(KernelTrace *t, hipStream_t s, const char *name) {
  if (t && t->n < KernelTrace::kMax) {
    (void)hipEventRecord(t->ev[t->n + 1], s);
    t->names[t->n++] = name;
  }
}

// Process-wide overrides of choices the library otherwise makes by itself; set only through the
// test-only entry points of include/ssd_testing.h (nothing reads the environment).
struct Knobs {
  int force_generic = 0;   // 1: every prefill takes the generic fp32 kernels
  int seg_chunks = 0;      // > 0: chunks per segment of the MFMA prefill
  int seg_blocks = 0;      // > 0: 64-token blocks per segment (if seg_chunks is not set); split fp32: 32-token blocks
  int seg_parts = 0;       // > 0: pieces per segment in the states-only pass; split fp32: workgroups per segment
  int y_stream = -1;       // 0 / 1: ordinary / non-temporal stores of y in the full scan
  int decode_stream = -1;  // 0 / 1: ordinary / non-temporal accesses to the decode state
  int force_mfma_f32 = 0;  // 1: fp32 io takes the fp32 MFMA kernel whenever the shape is eligible
  int f32_segments = 0;    // > 0: time segments per sequence in the fp32 MFMA kernel
  int scan_heads = 0;      // 2 / 4: head slices per workgroup in the bf16 scan; 0: library's choice
  int deal = 0;            // packed bf16 batches: 1 items dealt to the scan's workgroups, 2 an entry each; 0: library's choice
  int split_images = 0;    // fp32 prefill on split operands: 2 no images of blocks; 0: library's choice
  int chunk = 0;           // bf16 prefill by chunk kernels: 1 wherever they can run, 2 never; 0: library's choice
  int fold_max_slots = 3;  // most state slots a segment sums by itself instead of a pass over segment states (0: never)
};
Knobs &knobs();

// ---- launchers (each returns the first HIP error it sees) ----
hipError_t launch_decode(int nlayers, const Dims &d, float *state, const void *x, const float *dt,
                         const float *A, const void *B, const void *C, const float *D, void *y,
                         hipStream_t stream);

hipError_t launch_decode_steps(int nsteps, int nlayers, const Dims &d, float *state, const void *x,
                               const float *dt, const float *A, const void *B, const void *C, const float *D,
                               void *y, hipStream_t stream);

// Several steps as contractions over blocks of 32 steps (bf16 io); see ssd_decode_steps_mfma.hip.
bool decode_steps_mfma_chosen(int nsteps, int nlayers, const Dims &d);
hipError_t launch_decode_steps_mfma(int nsteps, int nlayers, const Dims &d, float *state, const void *x, const float *dt,
                                    const float *A, const void *B, const void *C, const float *D, void *y,
                                    hipStream_t stream);

size_t generic_workspace_bytes(const Dims &d);
hipError_t launch_prefill_generic(const Dims &d, const void *x, const float *dt, const float *A,
                                  const void *B, const void *C, const float *D, const float *h0,
                                  void *y, float *final_state, void *workspace, hipStream_t stream,
                                  KernelTrace *trace = nullptr);

// How the bf16 MFMA prefill cuts a call up (for the launcher and for the test-only plan query).
struct SlicePlan {
  int seg_blocks, segments, parts, fold;
  int heads, state_heads;  // head slices per workgroup: full scan, states-only pass
  bool listed = false;     // packed batch: the full scan's workgroups walk lists of two-head items (pair_list)
  int two = 0;             // the segments are those chosen for two heads per workgroup (two_head_blocks)
  // packed batch: the device chooses the segment length from the sequences' lengths (seg_blocks is the shortest it may)
  bool from_lengths = false;
  int shortest = 0;  // (of mfma_varlen_plan, where seg_blocks is the choice)
};
SlicePlan mfma_plan(const Dims &d, bool h0_aliases_final_state);
// ... and a packed batch of these boundaries (host array): seg_blocks as the device chooses it, segments of the whole batch.
SlicePlan mfma_varlen_plan(const Dims &d, const int32_t *cu_host);
int mfma_f32_time_segments(const Dims &d);
bool mfma_supported(const Dims &d);
size_t mfma_workspace_bytes(const Dims &d);
hipError_t launch_prefill_mfma(const Dims &d, const void *x, const float *dt, const float *A,
                               const void *B, const void *C, const float *D, const float *h0,
                               void *y, float *final_state, void *workspace, hipStream_t stream,
                               KernelTrace *trace = nullptr);

// Small bf16 prompts, a workgroup per (64-column slice, chunk of 256 tokens); see ssd_prefill_chunk.hip.
int chunk_count(const Dims &d);
bool chunk_chosen(const Dims &d, size_t workspace_bytes, bool h0_aliases_final_state);
bool chunk_chosen(const Dims &d, size_t workspace_bytes, const float *h0, const float *final_state);
hipError_t launch_prefill_chunk(const Dims &d, const void *x, const float *dt, const float *A, const void *B, const void *C,
                                const float *D, const float *h0, void *y, float *final_state, void *workspace,
                                hipStream_t stream, KernelTrace *trace = nullptr);

// fp32 io on fp32 MFMA (one launch, no workspace); see ssd_prefill_mfma_f32.hip.
bool mfma_f32_supported(const Dims &d, bool whenever_eligible);  // false: only where it is expected to win
hipError_t launch_prefill_mfma_f32(const Dims &d, const void *x, const float *dt, const float *A, const void *B,
                                   const void *C, const float *D, const float *h0, void *y, float *final_state,
                                   hipStream_t stream, KernelTrace *trace = nullptr);

// fp32 io on bf16 MFMA with split operands; see ssd_prefill_split_f32.hip.  split_f32_chosen: whether it is expected
// to be the fastest of the three families for the shape.
bool split_f32_supported(const Dims &d);
double f32_other_us(const Dims &d);  // modelled time of the faster of the two other families
bool split_f32_chosen(const Dims &d);
void split_f32_plan(const Dims &d, int *seg_blocks, int *segments, int *parts, int *images, int *states_in_y);
hipError_t launch_prefill_split_f32(const Dims &d, const void *x, const float *dt, const float *A, const void *B,
                                    const void *C, const float *D, const float *h0, void *y, float *final_state,
                                    void *workspace, hipStream_t stream, KernelTrace *trace = nullptr);

// Device-side tables of a packed variable-length batch (all int32; see ssd_prefill_mfma.hip, "tables of a
// variable-length call").  tok0 == nullptr: plain batch.
struct VarPlan {
  const int32_t *tok0, *len, *blk0, *item0, *slot0, *blk_seq, *item_seq;
  int nseq, nb_cap, slot_cap;
};
// Blocks per segment of a packed batch: one of the first `count` candidates (ascending), chosen on the device from the
// lengths; see packed_cost in ssd_prefill_mfma.hip.
struct SegChoice {
  static constexpr int kMost = 32;
  int cand[kMost];
  int count, max_items;  // list entries that still run side by side
  float fill, slices;    // share of the chip that one entry's workgroups take; 64-column slices of all heads
  bool dealt;            // the scan's workgroups are dealt items (then fill is an entry's share of a round of these)
  float state_fill;      // the states-only pass's fill
};
void launch_varlen_tables(const int32_t *cu, int total, int blk_len, const SegChoice &choice, int item_cap, const VarPlan &vp,
                          hipStream_t stream);
size_t generic_varlen_workspace_bytes(const Dims &d);
hipError_t launch_prefill_generic_varlen(const Dims &d, const int32_t *cu_seqlens, const void *x, const float *dt,
                                         const float *A, const void *B, const void *C, const float *D,
                                         const float *h0, void *y, float *final_state, void *workspace,
                                         hipStream_t stream);

// Packed variable-length batch (d.Bt sequences, d.T tokens in total, cu_seqlens on the device).
bool mfma_varlen_supported(const Dims &d);
size_t mfma_varlen_workspace_bytes(const Dims &d);
hipError_t launch_prefill_mfma_varlen(const Dims &d, const int32_t *cu_seqlens, const void *x, const float *dt,
                                      const float *A, const void *B, const void *C, const float *D, const float *h0,
                                      void *y, float *final_state, void *workspace, hipStream_t stream,
                                      KernelTrace *trace = nullptr);

// Depthwise causal convolution (channels-last); z / width: up to three dense outputs by channel range.
hipError_t launch_conv_prefill(int Bt, int T, int ksize, bool bf16, const void *u, const float *w, const float *bias,
                               const void *state_in, void *const z[3], const int width[3], void *state_out, int act,
                               hipStream_t stream);
hipError_t launch_conv_step(int Bt, int ksize, bool bf16, void *state, const void *u, const float *w, const float *bias,
                            void *const z[3], const int width[3], int act, hipStream_t stream);

// ssd_prefill with an event recorded after every kernel (the measurement library's ssd_prefill_profile).
ssd_status prefill_traced(const ssd_shape *shape, const void *x, const float *dt, const float *A, const void *B,
                          const void *C, const float *D, const float *h0, void *y, float *final_state,
                          void *workspace, size_t workspace_bytes_given, void *hip_stream, KernelTrace *trace);

inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

}  // namespace ssd
