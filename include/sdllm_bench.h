/*
 * sdllm_bench.h - measurement and test aids exported by libsdllm.so next to the product API of sdllm.h.
 * Nothing here is part of the method; benchmarks use it to find what the memory system delivers, tests to see
 * which kernel a call runs.
 */
#ifndef SDLLM_BENCH_H
#define SDLLM_BENCH_H

#include <stddef.h>
#include <stdint.h>

#include "sdllm.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Reads `bytes` bytes at `src` once with the memory access pattern of the block-attention kernel
 * of Alg. 3 (cache_state 2; non-temporal 16-byte loads, one 512-thread workgroup per contiguous chunk)
 * and discards them.  Timing it gives the bandwidth the memory system delivers for that pattern,
 * the practical ceiling for sdllm_sparse_attn.  `src` must be 16-byte aligned device memory; `sink`
 * is 4 bytes of device memory (may be NULL); `stream` a hipStream_t (NULL = default stream).
 * Returns SDLLM_OK (0), SDLLM_ERR_INVALID_ARG (-1) or SDLLM_ERR_HIP (-4) as in sdllm.h.
 */
int32_t sdllm_stream_read_probe(const void* src, size_t bytes, void* sink, void* stream);

/* Attention calls, by what is attended */
#define SDLLM_CALL_SPARSE 0 /* sdllm_sparse_attn with n_cached keys, or sdllm_block_step, state 2 */
#define SDLLM_CALL_FULL 1   /* sdllm_block_step, state 0 */
#define SDLLM_CALL_UPDATE 2 /* sdllm_block_step, state 1: its dense rows */
#define SDLLM_CALL_DENSE 3  /* sdllm_dense_attn */

#define SDLLM_KERNEL_GENERAL 0     /* any type, head_dim and row count */
#define SDLLM_KERNEL_PER_HEAD 1    /* bf16, head_dim 128, 32 rows: one workgroup per query head and key split */
#define SDLLM_KERNEL_SHARED_TILE 2 /* the same rows, K/V tiles shared by the query heads of a KV head */
#define SDLLM_KERNEL_STREAM 3      /* as PER_HEAD, tiles fetched straight into LDS */
#define SDLLM_KERNEL_DENSE 4       /* bf16, head_dim 128, all rows of a sequence */

typedef struct sdllm_launch_plan {
  int32_t kernel;        /* SDLLM_KERNEL_* */
  int32_t key_splits;    /* workgroups that share a head's keys; merged by a second launch if more than one */
  int32_t waves;         /* per workgroup (SHARED_TILE: query heads per KV head) */
  int32_t touches_ahead; /* STREAM: 1 if the heads of a group bring tiles into L2 for each other */
  int32_t key_groups;    /* DENSE: groups of waves that share a row block's keys, but for a last round with more (sdllm_dense_tail_groups) */
} sdllm_launch_plan_t;

/* How an attention call of this shape is launched (n_cached: SDLLM_CALL_SPARSE only), given all the workspace it asks
 * for, unless sdllm_burst_splits gives it to another kernel.  Host only; the pointers are host pointers. */
int32_t sdllm_launch_plan(const sdllm_shape_t* shape, int32_t call, int32_t n_cached, sdllm_launch_plan_t* plan);

/* Small calls of SDLLM_CALL_SPARSE and SDLLM_CALL_FULL run a kernel that fetches all tiles of a workgroup at once, ahead of what
 * sdllm_launch_plan says: *splits is the number of workgroups that share a head's keys then, 0 for a call that it does not take.  A
 * workspace with less room takes fewer, and the plan of sdllm_launch_plan if there is no room for those that it needs at least, or
 * if it is not aligned to 16 bytes; less than that plan needs is refused either way.
 * Host only. */
int32_t sdllm_burst_splits(const sdllm_shape_t* shape, int32_t call, int32_t n_cached, int32_t* splits);

/* SDLLM_CALL_DENSE on SDLLM_KERNEL_DENSE: *groups is the key groups of the launch that the workgroups of a last, small round are, 0 for a
 * call (or a shape) without such a launch.  Host only. */
int32_t sdllm_dense_tail_groups(const sdllm_shape_t* shape, int32_t* groups);

/* Which kernels reduce the columns of the scoring: those for blocks of 32 query rows, the same with the blocks of 32 rows of a head (rows that
 * are not there among them) as heads, or the general one.  The dense launch of a cache-update step of SDLLM_COLUMNS_32 may leave the
 * scores by itself.  Host only. */
#define SDLLM_COLUMNS_GENERAL 0
#define SDLLM_COLUMNS_32 1
#define SDLLM_COLUMNS_BLOCKS 2
int32_t sdllm_column_kernel(const sdllm_shape_t* shape, int32_t* kernel);

#ifdef __cplusplus
}
#endif
#endif /* SDLLM_BENCH_H */
