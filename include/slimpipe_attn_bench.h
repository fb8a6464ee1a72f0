/*
 * slimpipe_attn_bench.h - measurement aids of libslimpipe_attn (not part of the paper's method, not needed to
 * use the library): per-kernel event timing, the kernels and cuts a call would take, and the sustained rate of the matrix instruction on this GPU.
 * Used by bench.py and the tests.  Same conventions as slimpipe_attn.h (status codes, device pointers, streams).
 */
#ifndef SLIMPIPE_ATTN_BENCH_H
#define SLIMPIPE_ATTN_BENCH_H

#include <stddef.h>
#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/* Per-kernel timing.  While enabled, the kernels of every entry point but slimpipe_attn_bwd_noalloc (and but the
 * one-workgroup kernel that clears the forward's counters) are bracketed by HIP events recorded on the caller's stream; the
 * launches are the same as without it.  slimpipe_attn_profile_read waits for the recorded events, adds up the elapsed time per
 * kernel kind since the last read and clears the records.  The records are process-wide and guarded by a mutex:
 * enabling the switch serialises the launches of concurrent host threads.  Both arrays of slimpipe_attn_profile_read have
 * SLIMPIPE_KERNEL_KINDS entries. */
enum {
  SLIMPIPE_KERNEL_FWD = 0, SLIMPIPE_KERNEL_DELTA = 1, SLIMPIPE_KERNEL_DQ = 2, SLIMPIPE_KERNEL_DKDV = 3,
  SLIMPIPE_KERNEL_MERGE = 4, SLIMPIPE_KERNEL_FINALIZE = 5, SLIMPIPE_KERNEL_DKDV_REDUCE = 6,
  SLIMPIPE_KERNEL_DQ_REDUCE = 7,
  SLIMPIPE_KERNEL_BWD_BOTH = 8,       /* dq and dk/dv items of a small backward call in one launch */
  SLIMPIPE_KERNEL_BOTH_REDUCE = 9,    /* the reduce of both, for such a call */
  SLIMPIPE_KERNEL_KINDS = 10
};
int slimpipe_attn_profile_enable(int enable);
int slimpipe_attn_profile_read(double total_ms[SLIMPIPE_KERNEL_KINDS], int64_t launches[SLIMPIPE_KERNEL_KINDS]);

/* How slimpipe_attn_bwd (n_chunks = 1) or slimpipe_attn_bwd_chunked would cut a call into work items with a workspace of
 * workspace_bytes (slimpipe_attn_bwd_noalloc: the two row statistics + 256 bytes).  For the smallest calls, which go through a kernel of 32-row and
 * 32-key items (slimpipe_attn_call_path says which), these are the cuts without it.  Host code only, nothing is launched. */
typedef struct slimpipe_bwd_plan {
  int32_t one_launch;      /* dq and dk/dv items in one launch */
  int32_t dq_first;        /* in that launch the dq items come first */
  int32_t dkdv_split;      /* chunks of a key tile's query stream */
  int32_t dq_ranges;       /* key ranges of a query block */
  int64_t dkdv_items, dq_items;
  int32_t compute_units;   /* of the current device (256 where no device can be asked) */
  int32_t dq_by_xcd;       /* the dq items that share keys are dealt to one XCD */
} slimpipe_bwd_plan;
int slimpipe_attn_bwd_plan(const slimpipe_attn_params* p, int32_t n_chunks, size_t workspace_bytes, slimpipe_bwd_plan* plan);

/* Which kernels slimpipe_attn_fwd / slimpipe_attn_bwd (n_chunks = 1) or their chunked variants take for a call with a workspace
 * of workspace_bytes (0, forward only: none).  Host code only, nothing is launched. */
typedef struct slimpipe_call_path {
  int32_t small;           /* workgroups of 32 rows (backward: and of 32 keys) whose waves share out the other side */
  int32_t ranges;          /* key ranges the forward, or dq, is cut into */
  int32_t dq_tile_keys;    /* backward: keys of a tile of the dq items */
  int32_t dkdv_tile_rows;  /* backward: query rows of a tile of the dk/dv items */
} slimpipe_call_path;
int slimpipe_attn_call_path(const slimpipe_attn_params* p, int is_bwd, int32_t n_chunks, size_t workspace_bytes, slimpipe_call_path* path);

/* How the kernel of 32-row and 32-key items would do a backward call that takes it (slimpipe_attn_call_path: small), for gradients that do
 * not lie over out or lse (there own_statistics is 0).  All zero for other calls.  Host code only, nothing is launched. */
typedef struct slimpipe_small_bwd_plan {
  int32_t small;           /* the call takes that kernel */
  int32_t key_blocks;      /* blocks of 32 keys a dk/dv item owns (1 or 2) */
  int32_t own_statistics;  /* no delta kernel ahead of it: the items work out the row statistics themselves */
  int32_t dq_first;        /* the dq items come first */
} slimpipe_small_bwd_plan;
int slimpipe_attn_small_bwd_plan(const slimpipe_attn_params* p, int32_t n_chunks, size_t workspace_bytes, slimpipe_small_bwd_plan* plan);

/* The rate, in TFLOP/s, at which this GPU sustains a pure stream of the bf16 MFMA instruction the attention
 * kernels use, with constant operands (random_operands == 0) or with random ones (!= 0), under which the chip
 * is power limited and clocks lower.  Runs two short kernels (about 20 ms each) on the stream and waits for them.
 * sink: device pointer to at least one float (never written in practice). */
int slimpipe_attn_mfma_rate(int random_operands, float* sink, double* tflops, void* hip_stream);

/* How evenly the XCDs of the GPU run the same work.  Launches `workgroups` workgroups of 8 waves that each issue 4 * iters
 * bf16 matrix instructions on random operands and writes, per workgroup, its start and end time (ticks of the constant
 * 100 MHz wall clock) and the XCD it ran on into the three DEVICE arrays (workgroups entries each).  Waits for the kernel.
 * The hardware hands workgroups to the XCDs round-robin whatever their speed, so a launch of equal workgroups ends when
 * the slowest XCD ends; bench.py reports the per-XCD times as `xcd_spread`. */
int slimpipe_attn_xcd_rate(int32_t iters, int32_t workgroups, int64_t* t_start, int64_t* t_end, uint32_t* xcc, void* hip_stream);

/* What float32 atomic adds into dq would cost a backward kernel that computes the scores once (key-stationary, dK/dV
 * in registers, dQ added into memory).  Launches key_tiles * heads workgroups of 8 waves; each walks the s_q /
 * rows_per_step query tiles of one head and per tile adds 1.0f to a rows_per_step x 128 block of dq
 * ([s_q, heads, 128] float32, device, zero before the call) as eight 32 x 32 MFMA C tiles with head_dim along the
 * lanes (rows_per_step = 32: two waves per tile add to the same 32 rows; 64: each wave its own 32 rows), with
 * filler_mfma (multiple of 4) matrix instructions per wave and step in between, and with_atomics = 0 leaving the
 * adds out.  placement 0: consecutive workgroups share a head; 1: workgroup w takes head w % heads and counts in
 * *xcc_mismatch (device, zero before the call) the workgroups whose XCD differs from w % 8.  rotate != 0 shifts the
 * start tile by the workgroup's key tile.  Afterwards every element of dq holds key_tiles * (64 / rows_per_step).
 * Waits for the kernel; *ms = its duration. */
int slimpipe_attn_dq_atomic_probe(float* dq, int32_t s_q, int32_t heads, int32_t key_tiles, int32_t rows_per_step,
                                  int32_t placement, int32_t rotate, int32_t filler_mfma, int32_t with_atomics,
                                  uint32_t* xcc_mismatch, double* ms, void* hip_stream);

#ifdef __cplusplus
}
#endif
#endif /* SLIMPIPE_ATTN_BENCH_H */
