/*
 * shiftattn_probe.h - measurement and test aids exported by libshiftattn.so.
 *
 * Not part of the attention path and not part of the product interface (shiftattn.h): host queries
 * that name the launch a prefill or projection call takes, and, for benchmark reports, four kernels that show what the chip attains on the resources the path's kernels are priced against, to print
 * beside the datasheet peaks.  Each call validates its arguments, enqueues one kernel on `stream`
 * (a hipStream_t as void*) and returns SHIFTATTN_OK or a negative code of shiftattn.h; the caller
 * times it.  All buffer pointers are device pointers, 16-byte aligned.
 *
 * ceiling_mfma_bf16: every wavefront of a chip-filling grid issues iters x 32 independent
 *   16x16x32 bf16 MFMAs (the form that sustains the higher rate at the chip's power limit) on the
 *   operand values found in `operands` (2 KiB = 128 lanes x 8 bf16; random values give the clock
 *   real data gives).  *flops (host) receives the flops of the launch.  sink: 4 bytes, never
 *   written in practice.
 * ceiling_mfma_bf16_fresh: the same loop (iters x 64 MFMAs per wavefront) with operands that differ
 *   from one MFMA to the next, as in a product of real matrices: `operands` holds eight A and eight
 *   B fragments per lane (16 KiB = 16 x 64 lanes x 8 bf16), MFMA m takes A fragment m % 8 and B
 *   fragment (m / 8) % 8.  Inputs that toggle cost power, which the chip gives up in clock: the
 *   rate a GEMM-shaped kernel can be held against.
 * ceiling_hbm_read: streams `bytes` (rounded down to 16 KiB) of `src` through every wavefront
 *   with 16-byte non-temporal loads.  *bytes_read (host) receives the bytes requested.
 * ceiling_hbm_copy: copies `bytes` (rounded down to 16 KiB) from src to dst with 16-byte
 *   non-temporal loads and stores, 16 KiB in flight per wavefront: a read + write stream with no
 *   index arithmetic.  *bytes_copied (host) receives the bytes copied (as many are read as written).
 *
 * prefill_plan: host only, nothing is enqueued.  What shiftattn_prefill (num_decode_seqs = 0), or
 *   shiftattn_mixed for its chunks, launches for a batch of these sizes with the workspace that its
 *   size query names, under the options as they are set; a test that aims at a kernel can then say so.
 *   Arguments as for shiftattn_mixed_workspace_bytes.
 * proj_plan: host only, nothing is enqueued.  What a projection of `rows` (>= 1; T_pad for qkv_proj_pack, T for
 *   unpack_o_proj) token rows with an [n_features][k] weight matrix launches when it is given a workspace of
 *   workspace_bytes, under the options as they are set.  fp8: the operands are FP8 codes.
 */
#ifndef SHIFTATTN_PROBE_H
#define SHIFTATTN_PROBE_H

#include <stddef.h>
#include <stdint.h>

#include "shiftattn.h"

#ifdef __cplusplus
extern "C" {
#endif

typedef struct {
    int32_t tile_columns;     /* (token, query head) pairs of a workgroup's tile: 128 or 256; 0: a kernel without such tiles */
    int32_t wave_columns;     /* of them per wavefront: 32, or 64 (tiles of 128 then have two groups of wavefronts) */
    int32_t key_ranges;       /* ranges that a tile's keys are split into; 1: no merge launch for them */
    int32_t tiles_per_wg;     /* 1, or 2: heaviest with lightest */
    int32_t decode_wgs;       /* workgroups of the same launch that take the decode rows; 0: the rows have a launch of their own */
} shiftattn_prefill_plan_t;

int shiftattn_prefill_plan(int32_t num_prefill_seqs, int32_t total_prefill_q, int32_t max_q_len, int32_t max_prefill_seq_len,
                           int32_t num_decode_seqs, int32_t max_decode_seq_len, const shiftattn_attn *a,
                           shiftattn_prefill_plan_t *plan);

typedef struct {
    int32_t streams;          /* 1: the weight-streaming kernel, which takes the call in workgroups of eight or four wavefronts; 0: the tiled kernel */
    int32_t k_ranges;         /* workgroups that share a block of features or an output tile of the last token rows; 1: no workspace is used */
    int32_t token_pieces;     /* streaming kernel: pieces of eight token rows and of eight features that a workgroup multiplies */
    int32_t feature_pieces;
    int32_t lead_tiles;       /* tiled kernel: token tiles of a launch of their own in front (0: none), and their features x token rows */
    int32_t lead_features, lead_tokens;
    int32_t tile_features, tile_tokens;   /* ... and those of the tiles behind them */
} shiftattn_proj_plan_t;

int shiftattn_proj_plan(int32_t rows, int32_t n_features, int32_t k, int32_t fp8, size_t workspace_bytes, shiftattn_proj_plan_t *plan);
int shiftattn_ceiling_mfma_bf16(const void *operands, void *sink, int32_t iters, int64_t *flops, void *stream);
int shiftattn_ceiling_mfma_bf16_fresh(const void *operands, void *sink, int32_t iters, int64_t *flops, void *stream);
int shiftattn_ceiling_hbm_read(const void *src, size_t bytes, void *sink, int64_t *bytes_read, void *stream);
int shiftattn_ceiling_hbm_copy(const void *src, void *dst, size_t bytes, int64_t *bytes_copied, void *stream);

#ifdef __cplusplus
}
#endif
#endif /* SHIFTATTN_PROBE_H */
