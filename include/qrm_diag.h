/*
 * qrm_diag.h - diagnostic entry points of libqrm, for benchmarks and tests only.
 *
 * Nothing here is part of the detection path (Section 4.3 of the paper); a production caller needs
 * include/qrm.h alone.  The calls exist so that measurements and tests can be made through the same
 * C ABI as everything else, without environment variables read inside the hot path.
 */
#ifndef QRM_DIAG_H
#define QRM_DIAG_H

#include "qrm.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Flags of qrm_diag_set_flags; none of them changes what a call computes. */
#define QRM_DIAG_NO_FUSED_PAIRS 1   /* run every convolution block as a launch of its own (A/B timing; the two
                                       schedules round differently, both within the tolerance) */
#define QRM_DIAG_POISON_WORKSPACE 2 /* fill every newly allocated workspace with 0xFF bytes (NaN as bf16 and as
                                       fp32): a kernel that reads workspace bytes no kernel wrote shows in the
                                       results; bits 8..15 of the flags, when not zero, give another fill byte */

#define QRM_DIAG_FUSE_ALWAYS 4      /* run the fused schedule on wide tiles (more than 64 columns) also when a launch
                                       has too few images to fill the compute units that way (tests of that path on
                                       small batches) */

#define QRM_DIAG_CHAIN_ALWAYS 8     /* all blocks in one launch for every batch that such a launch takes, */
#define QRM_DIAG_NO_CHAIN 16        /* or for none (A/B timing, tests; a launch per block gives the same bits) */

/* Sets the context's diagnostic flags (0 = production behaviour).  Affects calls made afterwards. */
QRM_API qrm_status qrm_diag_set_flags(qrm_ctx *ctx, int32_t flags);

/*
 * For tests of what happens when the workgroups of an all-blocks launch do not hear from each other.  _patience: how often a wait
 * looks before it gives up, 0 = once, below zero = the usual number.  _count: sets the number of items that are done of `image` in the
 * first block to `value`, in what such launches keep beside the workspace of `stream` (or, with `shared` not 0, beside that of
 * qrm_detect_static): with all ones the number that the launch waits for never comes up.  _left_over: all of that as a call leaves it
 * whose all-blocks launch has run and whose next one has failed: every word `value`, and marked.  Both synchronise the device.
 */
QRM_API qrm_status qrm_diag_chain_patience(qrm_ctx *ctx, int32_t looks);
QRM_API qrm_status qrm_diag_chain_count(qrm_ctx *ctx, void *stream, int32_t shared, int32_t image, uint32_t value);
QRM_API qrm_status qrm_diag_chain_left_over(qrm_ctx *ctx, void *stream, int32_t shared, uint32_t value);

/*
 * Whether n_img tiles of h x w go through `blocks` blocks of `channels` in one launch on num_cu compute units: *fits such a launch takes
 * them, *taken it does so by the rule.  Host code, no device needed.
 */
QRM_API qrm_status qrm_diag_chain_rule(int32_t channels, int32_t blocks, int32_t n_img, int32_t h, int32_t w, int32_t num_cu,
                                       int32_t *fits, int32_t *taken);

/*
 * The rate the matrix pipes sustain when nothing else runs - eight wavefronts per compute unit issuing the bf16
 * 32x32x16 matrix instruction back to back for a few milliseconds - on operands of the given kind: data = 0
 * zeros, 1 one constant, 2 random (one side small normal values like weights, the other half zeros and half
 * positive like activations after a ReLU).  The part's clock follows its power budget and the power of a matrix
 * instruction follows its data, so the third figure, not the published peak, is what a convolution on real
 * activations can approach.  *tflops receives 10^12 FLOP/s.
 * Allocates and frees a small device buffer; synchronises the device's default stream.
 */
QRM_API qrm_status qrm_diag_matrix_rate(qrm_ctx *ctx, int32_t data, double *tflops);

/*
 * How a fused launch (64 channels, two blocks; `last`: the second one is the network's last) deals the row pairs of
 * n_img tiles of h x w to num_cu compute units: *part = 1 runs that begin and end inside images, 0 whole images per
 * workgroup; *per = pieces per workgroup (row pairs; with `last` four of them); *cost = cost of the longest
 * workgroup: eight for each of its steps, one for each row pair that either block multiplies in them.  Host code, no device needed.
 */
QRM_API qrm_status qrm_diag_pair_split(int32_t n_img, int32_t h, int32_t w, int32_t last, int32_t num_cu, int32_t *part,
                                       int32_t *per, int32_t *cost);

/*
 * The schedule of n_img tiles of h x w, w > 64, on num_cu compute units (64 channels): *fused = 1 two blocks per launch,
 * 0 one; *single_us / *fused_us: what eight blocks are estimated to take either way.  Host code, no device needed.
 */
QRM_API qrm_status qrm_diag_wide_schedule(int32_t n_img, int32_t h, int32_t w, int32_t num_cu, int32_t *fused,
                                          double *single_us, double *fused_us);

/*
 * *row_pairs = row pairs behind one line of the sums that the last fused launch (64 channels) on n_img tiles of h x w leaves for the
 * head: 1 in launches of few tiles, 4 otherwise; *bytes = what a stream's workspace takes for a call of that many tiles
 * through n_blocks blocks of 64 channels without a final ReLU (no code).  Host code, no device needed.
 */
QRM_API qrm_status qrm_diag_last_lines(int32_t n_img, int32_t h, int32_t w, int32_t n_blocks, int32_t num_cu, int32_t *row_pairs,
                                       int64_t *bytes);

/*
 * How qrm_detect_host brings its chunks in (page-locked images of H x W, a network of `channels` and n_blocks without a
 * final ReLU, `used` staging buffers in use): *first / *rest = 1 the first / the later chunks as tiles, 0 as whole images;
 * *lent = compute units the kernels leave to the gather of the next chunk.  Host code, no device needed.
 */
QRM_API qrm_status qrm_diag_host_plan(int32_t channels, int32_t n_blocks, int32_t H, int32_t W, int32_t tile, int32_t chunk_images,
                                      int32_t used, int32_t num_cu, int32_t *first, int32_t *rest, int32_t *lent);

/* How many strips (workgroups) qrm_preprocess cuts each of N windows of T x T into.  Host code, no device needed. */
QRM_API qrm_status qrm_diag_preprocess_strips(int64_t N, int32_t T, int32_t *strips);

/* Lanes that decode one word of a code (n symbols, k of them message) in a launch of N words.  Host code, no device needed. */
QRM_API qrm_status qrm_diag_rs_lanes(int32_t n, int32_t k, int64_t N, int32_t *lanes);

#ifdef __cplusplus
}
#endif
#endif /* QRM_DIAG_H */
