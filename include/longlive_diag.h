/*
 * longlive_diag.h - diagnostics and tuning knobs of the MI355X (gfx950) LongLive library.
 *
 * Nothing in this header is part of the method: these calls exist to benchmark the library's own kernel variants
 * against each other and to measure what the GPU's matrix pipe sustains, so that the attention kernel's rate can be
 * read against the rate a pure stream of matrix instructions reaches on the same chip in the same run.
 * Conventions (status codes, device/host pointers, streams) are those of longlive.h.
 */
#ifndef LONGLIVE_DIAG_H
#define LONGLIVE_DIAG_H

#include "longlive.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Attention kernel variant: 0 = default for the shape, otherwise a variant id listed by
 * ll_attn_variant_name.  Process-wide tuning knob for benchmarking. */
ll_status ll_set_attn_variant(int variant);
const char* ll_attn_variant_name(int variant); /* NULL when `variant` does not exist */

/* Into how many groups (1, 2, 4 or 8) the default bf16 kernels deal the keys of a launch's tiles, for n_chunks chunks of
 * rows[i] query rows over kblocks[i] blocks of 32 keys each (host arrays).  A chunk in the cache counts as a launch of its
 * own, with the key set of a full window; a clip or a prompt as the launch it is.  No GPU needed. */
ll_status ll_attn_key_groups(int head_dim, int heads, int n_chunks, const int* rows, const int* kblocks, int* groups);

/* What a streamed chunk of `rows` query rows takes whose key set has `kblocks` blocks of 32 keys (fp8 != 0, the 8-bit cache: 64)
 * once the window is full: its tiles' keys are dealt to `splits` workgroups (1: not split), in each of them to `groups`
 * groups of waves (bf16, not split: ll_attn_key_groups' answer; 8-bit: a tile has 256 / groups rows and its waves all walk
 * all keys of the split).  No GPU needed. */
ll_status ll_attn_split(int head_dim, int fp8, int heads, int rows, int kblocks, int* groups, int* splits);
/* What one launch of n_chunks chunks (24 at most) of rows[i] query rows over kblocks[i] blocks of keys takes (host arrays).  No GPU
 * needed.
 *   ll_attn_key_groups_fp8: a launch of a re-prefill of an 8-bit cache (blocks of 64 keys), all of whose chunks would have splits
 *     when streamed (ll_attn_split): 4 where its tiles have 64 rows and their keys dealt to four groups of waves, else 1.
 *   ll_attn_clip_tail: a clip's forward pass (blocks of 32 keys; the latest chunk is the first): how many tiles per head, from the
 *     end of the list, go out in a launch of their own with their keys dealt to `splits` workgroups; 0 and 1 where none do. */
ll_status ll_attn_key_groups_fp8(int head_dim, int heads, int n_chunks, const int* rows, const int* kblocks, int* groups);
ll_status ll_attn_clip_tail(int head_dim, int heads, int n_chunks, const int* rows, const int* kblocks, int* tiles, int* splits);
/* The partial results of split tiles wait for their merge in 512 slots that all calls on a GPU share; a workgroup that finds
 * no slot free leaves its tile to the merge, where one workgroup then computes the tile's shares one after another, with the
 * same result.  This call takes the free ones among slots [first, first + n) out of use on the current device (hold != 0), or
 * gives back those it took (hold == 0), so that this path can be tested.  Waits for the device before and after. */
ll_status ll_hold_split_slots(int first, int n, int hold);
/* How many of these slots, and of the spaces in which merges compute such tiles, are taken on the current device once it is idle
 * (waits for it): 0, but for slots held by the call above. */
ll_status ll_split_slots_taken(int* taken);

/* Diagnostic, not part of the method: the dense bf16 MFMA rate this GPU sustains when every wave issues nothing
 * but 32x32x16 MFMAs (two waves per SIMD, `workgroups` workgroups of 8 waves, iters * 16 MFMAs per wave), and the
 * core clock it settles at while doing so.  random_operands != 0 fills the operand registers with random bf16
 * mantissas and signs, 0 with the constant 1.0: under a full matrix load the chip is power-limited and the clock
 * depends on how many operand bits toggle, so the two differ by about a third.  bench.py reports the attention
 * kernel's rate next to the random-operand figure.
 *   dev_scratch: device, at least workgroups * 2048 + 16 bytes, contents overwritten.
 *   The kernel runs twice on `stream` (the first run lets the clock settle, the second is timed with events);
 *   the call returns after the stream has finished.  tflops, clock_ghz: host. */
ll_status ll_probe_mfma_rate(void* dev_scratch, size_t scratch_bytes, int workgroups, int iters,
                             int random_operands, double* tflops, double* clock_ghz, void* stream);
/* The same loop with company: `per_mfma` (1 or 2) instructions of kind `companion` issued behind every MFMA, on
 * registers no MFMA touches: 0 none, 1 v_add_f32, 2 v_exp_f32, 3 v_cvt_pk_bf16_f32, 4 v_dot2c_f32_bf16,
 * 5 v_max3_f32, 6 ds_read_b128 (64 KB of LDS, conflict-free), 7 no companion but 16x16x32 MFMAs (twice as many,
 * the same flops).  The drop against companion 0 is what that instruction costs the matrix pipe in issue slots and,
 * with random operands, in power.  tflops counts the MFMA flops only.  Other arguments as above.
 * Companions 8 to 11 run fp8 MFMAs instead (32x32x64, E4M3 operands, four times the flops per instruction; per_mfma
 * is ignored): 8 alone, 9 with what the 8-bit attention kernel issues per MFMA (4 v_exp_f32, 4 v_add_f32,
 * 2 v_cvt_pk_fp8_f32, 2 v_max3_f32, 2 ds_read_b128), 10 with the vector part of that only, 11 with the LDS part only. */
ll_status ll_probe_mfma_mix(void* dev_scratch, size_t scratch_bytes, int workgroups, int iters, int random_operands,
                            int companion, int per_mfma, double* tflops, double* clock_ghz, void* stream);

#ifdef __cplusplus
}
#endif
#endif /* LONGLIVE_DIAG_H */
