/*
 * ssd_testing.h -- test-only entry points of libssd_hip.so.
 *
 * The library chooses by itself which kernel family runs a prefill, how a prompt is
 * cut into segments and whether outputs and states stream past the caches.  Tests
 * and tuning runs need to force those choices (to reach every code path at small
 * sizes, to compare both cache policies bit for bit); these calls do that.  The
 * settings are process-wide and not synchronised: set them from one thread while no
 * call of the library is in flight, and reset them afterwards.  Nothing in the
 * library reads the environment.  Workspace sizes (ssd_prefill_workspace_bytes,
 * ssd_prefill_varlen_workspace_bytes) do not depend on any knob.
 */
#ifndef SSD_TESTING_H_
#define SSD_TESTING_H_

#include "ssd.h"

#ifdef __cplusplus
extern "C" {
#endif

typedef enum {
  SSD_KNOB_FORCE_GENERIC = 0, /* 1: every prefill runs on the generic fp32 kernels; 0: default */
  SSD_KNOB_SEG_CHUNKS = 1,    /* k > 0: k chunks per segment in the MFMA prefill; 0: library's choice */
  SSD_KNOB_SEG_BLOCKS = 2,    /* k > 0: k 64-token blocks per segment (when SEG_CHUNKS is 0); 0: default.  fp32 io
                                 (unless knob 0, 6 or 7 is set): split operands, segments of about k 32-token blocks */
  SSD_KNOB_SEG_PARTS = 3,     /* k > 0: pieces per segment in the states-only pass, if k divides the
                                 segment length and the state slots suffice; 0: default.  fp32 io with
                                 SEG_BLOCKS: workgroups that share a sequence of one segment */
  SSD_KNOB_Y_STREAM = 4,      /* 0 / 1: ordinary / non-temporal stores of y in the full scan; -1: default */
  SSD_KNOB_DECODE_STREAM = 5, /* 0 / 1: ordinary / non-temporal accesses to the decode state; -1: default */
  SSD_KNOB_FORCE_MFMA_F32 = 6, /* 1: fp32 io runs on the fp32 MFMA kernel whenever the shape is eligible (headdim
                                 a multiple of 32, dstate a multiple of 8 up to 128), also where the library
                                 expects the generic kernels to be faster; 0: default */
  SSD_KNOB_F32_SEGMENTS = 7,   /* k > 0: the fp32 MFMA kernel cuts every sequence into k time segments (at most
                                 one per 64-token block); 0: library's choice */
  SSD_KNOB_FOLD_MAX_SLOTS = 8, /* k >= 0: a plain batch whose chain over segment-state slots, (segments - 1) x
                                 pieces, is at most k long runs no separate pass over those states -- every
                                 segment of the full scan sums the slots before it as it loads them; 0: never.
                                 Default 3.  Reset with ssd_testing_reset_knobs */
  SSD_KNOB_SCAN_HEADS = 9,     /* 2 / 4: head slices per workgroup in both passes of the bf16 MFMA prefill; any other
                                 value: library's choice */
  SSD_KNOB_CHUNK = 10,         /* bf16 prefill of a plain batch by the chunk kernels: 1 wherever they can run, 2 never; 0:
                                 library's choice */
  SSD_KNOB_DEAL = 11,          /* packed bf16 batches: 1 the full scan's workgroups are dealt items of two heads, however few
                                 these are, unless the decay records take 4 GiB; 2 they take an entry each; 0: library's choice */
  SSD_KNOB_SPLIT_IMAGES = 12   /* fp32 io on split operands: 2 no images of blocks; 0: library's choice */
} ssd_knob;

/* Sets one knob.  Errors: SSD_ERR_SHAPE for an unknown knob. */
SSD_API ssd_status ssd_testing_set_knob(int32_t knob, int32_t value);

/* All knobs back to the library's own choices. */
SSD_API void ssd_testing_reset_knobs(void);

/* How ssd_prefill would run a shape under the current knobs (host arithmetic only: no GPU call, nothing
 * launched), if not on the chunk kernels (ssd_testing_prefill_chunks).  plan[0]: kernel family, 0 generic fp32 kernels,
 * 1 bf16 MFMA, 2 fp32 MFMA.  For the bf16 MFMA family (per state slice of 128 columns): plan[1] 64-token blocks per segment, plan[2] segments
 * per sequence, plan[3] pieces per segment in the states-only pass, plan[4] 1 if the full scan sums the
 * chain over segment states itself and no separate pass runs (h0_aliases_final_state != 0: as for a call
 * whose h0 and final_state share memory, which rules that out), plan[6] and plan[7] head slices per
 * workgroup of the full scan and of the states-only pass.  For the fp32 MFMA family: plan[5] time
 * segments per sequence on fp32 MFMA, or 0 on split operands, and then plan[1] 32-token blocks in the longest
 * segment, plan[2] segments, plan[3] workgroups that share one, plan[6] 1 if images of the blocks are made for all heads,
 * plan[7] 1 if the states between the launches lie in y.  The other entries are zero.
 * Errors: SSD_ERR_NULL; the shape errors of ssd_prefill. */
SSD_API ssd_status ssd_testing_prefill_plan(const ssd_shape *shape, int32_t h0_aliases_final_state,
                                            int32_t plan[8]);

/* The same plan where its segments are chosen for one round of workgroups of two heads; plan[0] 0 (and all others) for
 * any other shape. */
SSD_API ssd_status ssd_testing_prefill_pair_plan(const ssd_shape *shape, int32_t h0_aliases_final_state, int32_t plan[8]);

/* Chunks per sequence if ssd_prefill would run a shape on the bf16 chunk kernels (a workgroup per 64 headdim columns and
 * chunk of 256 tokens) under the current knobs, else 0: it then runs as ssd_testing_prefill_plan says. */
SSD_API int32_t ssd_testing_prefill_chunks(const ssd_shape *shape, int32_t h0_aliases_final_state);

/* How ssd_prefill_varlen would cut up a packed batch of these boundaries (a HOST array here) under the current knobs, on
 * the bf16 MFMA kernels.  plan[1] 64-token blocks per segment, which the device chooses from the boundaries, plan[2]
 * segments of the whole batch, plan[3] the shortest segment it may choose, plan[4] 1 if there is a choice, plan[5] 1 if
 * the full scan's workgroups are dealt items of two heads, plan[6] and plan[7] as above; plan[0] and all others 0 for a
 * call that runs on the generic kernels.
 * Errors: SSD_ERR_NULL; the shape errors of ssd_prefill_varlen; SSD_ERR_SHAPE for boundaries it would reject. */
SSD_API ssd_status ssd_testing_varlen_plan(const ssd_shape *shape, const int32_t *cu_seqlens, int32_t plan[8]);

#ifdef __cplusplus
}
#endif
#endif /* SSD_TESTING_H_ */
