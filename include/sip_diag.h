/*
 * sip_diag.h -- measurement and diagnostic entry points of the MI355X batched token sampler.
 *
 * Nothing here is needed to sample: these calls time the library's kernels, measure what the
 * memory system gives a bare read in the streaming kernel's launch shape, and report launch
 * shapes.  They live in the same shared library as the entry points of sip.h.
 */
#ifndef SIP_DIAG_H_
#define SIP_DIAG_H_

#include "sip.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Profiling aid.  Arms a one-shot hook on the calling host thread: the next sampling call made
 * by this thread that takes the single-pass path launches its three kernels with the given
 * hipEvent_t handles (created by the caller with timing enabled) attached to the kernel
 * dispatches themselves: `stream_start` / `stream_stop` take the begin and end time stamps of
 * the streaming kernel -- the one pass over the logits, Sec. 5.1's dense row-wise work --,
 * `finish_*` those of the finishing kernel (one workgroup per row on the list the pass left) and
 * `rescue_*` those of the kernel behind it that takes the rows the list did not settle, so that a
 * caller reads each kernel's duration with hipEventElapsedTime without any extra packet between
 * them.  Any pointer may be NULL; all NULL disarms.  No effect on results.
 */
void sip_profile_kernel_events(void* stream_start, void* stream_stop, void* finish_start, void* finish_stop,
                               void* rescue_start, void* rescue_stop);

/*
 * Measurement aid: enqueue a bare streaming read of `bytes` bytes (a multiple of 16 is read) at
 * `src` (device, 16-byte aligned) in the launch shape of the streaming kernel -- `workgroups`
 * workgroups of 512 threads, each on one contiguous piece, 16-byte loads -- that only adds up
 * what it reads.  What this takes is what the memory system gives a kernel of that shape on
 * this machine: the figure the streaming kernel's time is set against beside the published
 * peak.  `workspace`: device, at least 4 * workgroups bytes (one partial sum per workgroup is
 * written).  start_event / stop_event: hipEvent_t handles that take the dispatch's own begin
 * and end time stamps, or NULL.
 */
sip_status sip_probe_read(const void* src, size_t bytes, int32_t workgroups, void* workspace,
                          size_t workspace_bytes, void* start_event, void* stop_event, void* hip_stream);

/*
 * Diagnostic, HOST only: into how many chunks the streaming kernel (stream_kernel) cuts a row of this
 * shape, in the calls that launch it; t_shards = 0 for logits in one matrix, else V = t_shards * V_shard.
 * 0 = no chunks: rows are held in registers or take the exact multi-pass path, -1 = invalid arguments.  A
 * row's chunks are whole units of 1024 elements, dealt out evenly (to each vocabulary piece, if there are
 * pieces); none is empty.  (sip_call_route() says which calls launch it, and how the others cut a row;
 * the workspace holds the chunks either way.  A call with millions of history tokens may cut its rows
 * into fewer where the workspace would else exceed sip_noalloc_scratch_bytes().)
 */
int32_t sip_plan_chunks(int32_t B, int32_t V, sip_dtype dtype, int32_t t_shards);

/* Kernels of a call ("Kernels of a call" in sip.h), one value for each way. */
typedef enum sip_route {
  SIP_ROUTE_EXACT = 0,          /* exact_kernel */
  SIP_ROUTE_RESIDENT = 1,       /* resident_kernel */
  SIP_ROUTE_CHUNKS_ALONE = 2,   /* chunk_rescue_kernel */
  SIP_ROUTE_ROW_FUSED = 3,      /* row_rescue_kernel */
  SIP_ROUTE_ROW = 4,            /* row_kernel, rescue_kernel */
  SIP_ROUTE_CHUNKS_FUSED = 5,   /* stream_kernel, finish_rescue_kernel */
  SIP_ROUTE_CHUNKS = 6          /* stream_kernel, finish_kernel, rescue_kernel */
} sip_route;

/*
 * Diagnostic, HOST only: the sip_route of a call with these arguments, or -1 where they are invalid.  on_state: whether it
 * is on a device-resident state; params: only which of its arrays are there counts, NULL = none; hist_nnz:
 * history tokens, and prompt tokens, of all rows (on a state slots * L_max); compute_units: of the device, 0 = 256.  *chunks
 * (unless NULL): how many chunks each row is cut into, 1 where a workgroup has whole rows.
 */
int32_t sip_call_route(int32_t B, int32_t V, sip_dtype dtype, int32_t t_shards, int32_t on_state, const sip_params* params,
                       int64_t hist_nnz, int32_t k_logprobs, int32_t compute_units, int32_t* chunks);

#ifdef __cplusplus
}
#endif
#endif /* SIP_DIAG_H_ */
