/*
 * kvq_prof.h -- switches of the measurement build of the library (libkvq_prof.so: the same
 * sources compiled with -DKVQ_PROFILE).  They exist for benchmarks and tests only; the library
 * proper (libkvq.so, include/kvq.h) has none of them, and the kernels it launches are the ones
 * the measurement build launches while every switch is off.
 * All switches are process-global and not thread-safe.
 */
#ifndef KVQ_PROF_H
#define KVQ_PROF_H

#include "kvq.h"

#ifdef __cplusplus
extern "C" {
#endif

/* While `before` and `after` (hipEvent_t handles
 * created by the caller) are set, every paged_decode_attn call records `before` on its stream
 * immediately ahead of its split kernel (the kernel that streams the K/V codes) and `after`
 * immediately behind it, so that a benchmark can time that kernel alone.  Pass NULL, NULL to
 * switch the hook off (the initial state).  Process-global and not thread-safe. */
void kvq_profile_split_events(void* before, void* after);

/* While switched on, paged_decode_attn launches a
 * read-only twin of its streaming kernel (same work split, addresses, load instructions and
 * software pipeline, the arithmetic replaced by an XOR of the loaded words) and skips the
 * reduce; `out` is not written and the workspace is scribbled on.  Its duration is the
 * read ceiling of this access pattern on the machine at hand.  Process-global; off initially. */
void kvq_profile_read_ceiling(int on);

/* While switched on, paged_decode_attn launches only
 * its streaming kernel and skips the reduce (`out` is then incomplete), so that a run of calls
 * is a run of back-to-back streaming kernels that two events can bracket.  Off initially. */
void kvq_profile_skip_reduce(int on);

/* 0 makes paged_decode_attn use its streaming kernels also where it otherwise takes the kernel
 * that shares the dequantization among 128 rows: from 128 query rows per kv head on, and from 33
 * on where that is faster; and its flat list of groups also where each (sequence, kv head) otherwise gets a
 * workgroup of its own.  On initially.  Process-global. */
void kvq_profile_prefill_kernel(int on);

/* What paged_decode_attn (or, with shared_prefix_tokens, paged_decode_attn_prefix) would launch for
 * these host-side arguments; batch >= 1.  Host only.  plan_out: [0] 1 if the call goes to the
 * many-row kernel (2 where long contexts go to the one of 256 rows a workgroup), [1] cuts that kernel (the
 * one of 128 rows) may make in the contexts of the batch, [2] wavefronts of the streaming
 * kernel, [3] 64-token groups of the shared prefix that the prefix kernel takes, [4] rows of a row
 * group, and the reduce's [5] grid in x, [6] grid in y and [7] threads per workgroup ([2] and [5] to [7]
 * where the flat list is used). */
int kvq_profile_plan(const kvq_cache_desc_t* desc, int32_t batch, int32_t q_len, int32_t num_q_heads,
                     int32_t max_seq_len, int32_t chunk_tokens, int32_t shared_prefix_tokens,
                     int64_t plan_out[8]);

/* Where kvq_profile_plan says 2: wide_out [0] 64-token groups that the contexts of the batch have together where
 * they go to the kernel of 256 rows a workgroup (0 in other calls), [1] cuts it may make ([1] of
 * kvq_profile_plan are the other kernel's), [2] groups that the shortest has there.  Host only. */
int kvq_profile_wide(const kvq_cache_desc_t* desc, int32_t batch, int32_t q_len, int32_t num_q_heads,
                     int32_t max_seq_len, int64_t wide_out[3]);

/* Pieces that the prefix kernel would cut a shared prefix into, 0 where the call does without that kernel (where
 * plan_out[3] of kvq_profile_plan is 0).  Host only. */
int kvq_profile_prefix_pieces(const kvq_cache_desc_t* desc, int32_t batch, int32_t q_len, int32_t num_q_heads,
                              int32_t max_seq_len, int32_t chunk_tokens, int32_t shared_prefix_tokens);

/* Whether the call goes to the many-row kernel of group-scaled int4 (which kvq_profile_plan's many_rows does
 * not count).  Host only. */
int kvq_profile_group_rows(const kvq_cache_desc_t* desc, int32_t batch, int32_t q_len, int32_t num_q_heads,
                           int32_t max_seq_len, int32_t chunk_tokens);

/* Wavefronts of the workgroup that each (sequence, kv head, row group) would get, 0 where the call goes over
 * the flat list of groups (or to a many-row kernel).  Host only. */
int kvq_profile_pair_waves(const kvq_cache_desc_t* desc, int32_t batch, int32_t q_len, int32_t num_q_heads,
                           int32_t max_seq_len, int32_t chunk_tokens);

/* While `buf` (device, 16 x uint64 per launched
 * wavefront, i.e. 16 * 8 * (number of wavefronts) bytes) is registered, every wavefront of the
 * streaming kernel stores in buf[16*w + k]: the shader clock at entry (k = 0), after its first
 * loads are issued (2), after its steady loop (3), after its last group (4) and after its
 * results are stored (5); its hardware placement XCC_ID << 32 | HW_ID (1); the constant
 * 100 MHz clock at entry (6) and exit (7); and the shader clock when the sequence lengths have
 * arrived (8), when the wavefront's range is worked out (9) and when its first block-table
 * entries have arrived (10).  Slots 11-15 are not written.
 * Pass NULL to switch off (the initial state).  Process-global. */
void kvq_profile_wave_clock(void* buf);

#ifdef __cplusplus
}
#endif
#endif /* KVQ_PROF_H */
