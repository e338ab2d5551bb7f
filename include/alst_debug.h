/*
 * alst_debug.h -- benchmarking and testing aids of libalst.  None of them is part of the method
 * (no counterpart in the paper) and no product code needs them: the timers serve the benchmark,
 * the block mapping, the chunks, the choice of launches and the matrix-instruction rate serve the tests and the roofline context.
 */
#ifndef ALST_DEBUG_H
#define ALST_DEBUG_H

#include "alst.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Benchmarking aid (no counterpart in the paper).  While enabled, every launch of a block GEMM and
 * each group of small kernels between them is bracketed by a pair of HIP events on the launch
 * stream.  alst_profile_read() waits for the recorded events, writes per kind the summed
 * milliseconds and the number of spans into the HOST arrays ms_total[8] and spans[8], and
 * forgets the spans.  A logits or dHidden launch may cover several of the caller's tiles and counts as
 * that many spans, so for these ms_total / spans is the time per tile.  Kinds: 0 logits GEMM, 1 dHidden
 * GEMM, 2 dW GEMM, 3 the small kernels of a cross-entropy chunk; 4 the projection GEMMs of the tiled MLP (alst_mlp.h), 5 its weight-gradient
 * GEMMs, 6 its small kernels; 7 unused.  Short calls make both kinds of
 * gradients in one launch, which counts as dHidden (kind 1), or as weight gradients (kind 5).  The recorded spans are process-wide state behind a lock:
 * calls from several host threads are safe, and their spans land in one list.
 */
int alst_profile_enable(int on);
int alst_profile_read(double* ms_total, int64_t* spans);

/*
 * Testing aid (no counterpart in the paper; host arithmetic only, no device is touched).  The block
 * GEMM launches deal their workgroups round-robin to the 8 XCDs of the chip and give the 32
 * workgroups resident on one XCD a compact run of output blocks; a launch may hold several
 * products ("parts") whose blocks are numbered through.  For a launch of `parts` products of
 * tiles_r x tiles_c blocks this returns the number of workgroups and writes, for workgroup `bid`,
 * the part and block it computes (part = -1: the workgroup leaves at once), evaluated with the
 * same functions the kernels use (one part: in the order for a long contraction, several: in
 * that for weight gradients; for a launch of whole blocks; a last round of at most 128 blocks is
 * dealt out as twice as many halves).  A negative return value is minus an alst_status.
 */
int alst_debug_block_tile(int tiles_r, int tiles_c, int parts, int bid, int* part, int* tr, int* tc);

/*
 * Testing aid (no counterpart in the paper; host arithmetic only, no device is touched): the rows per
 * launch that a layer call works in.  op 0: alst_tiled_mlp_forward, 1: alst_tiled_mlp_backward (K = hidden, M =
 * intermediate size), 2: the y launches of alst_tiled_linear_forward, 3: the dx launches of
 * alst_tiled_linear_backward.  A negative return value is minus an alst_status.
 */
int64_t alst_debug_chunk_rows(int op, int64_t N, int64_t K, int64_t M, int64_t tile);

/*
 * Testing aid (no counterpart in the paper; host arithmetic only, no device is touched): what the launches of a layer
 * call's last chunk of rows run on (op, K, M: as above).  The library chooses its launches with the same functions.
 */
typedef struct {
    int64_t rows;                        /* of the chunk */
    int transposed;                      /* backward: against the weights transposed, not as they are */
    int gated_columns, gated_chained;    /* MLP, gate and up: columns of the small blocks (64 rows), 0: 256 x 256, one a
                                            workgroup or (chained) on persistent workgroups that walk chains of them */
    int product_columns, product_chained;        /* y; backward: dx */
    int wgrad_columns;                   /* the weight gradients of the group (linear layer: the first) */
    int together;                        /* dx and they are one launch */
} alst_debug_layer_info;
int alst_debug_layer(int op, int64_t N, int64_t K, int64_t M, int64_t tile, uint32_t flags, alst_debug_layer_info* info);

/*
 * Testing aid (no counterpart in the paper; host arithmetic only, no device is touched): chunk number
 * `chunk` of the launches of a cross-entropy call that computes gradients, and what the device makes of it if
 * `dense` of its rows are there (rows with a valid label, numbered densely through the sequence).  The library
 * chooses its launches with the same functions.
 */
typedef struct {
    int64_t first, rows;             /* dense rows first .. first + rows - 1, as far as they exist */
    int64_t group0;                  /* first dense row of its dW group */
    int64_t dhidden_blocks;          /* output blocks of dHidden over all ranges, for `dense` rows */
    int64_t dhidden_grid;            /* workgroups of the dHidden launch */
    int64_t dw_blocks;               /* output blocks of dW (0: the chunk does not complete its group) */
    int64_t dw_grid;                 /* workgroups of the dW launch (0: none, or its blocks are in the dHidden launch) */
    int64_t gather_grid;             /* workgroups of the launch that gathers the rows (first chunk: zeroes, transposes W) */
    int64_t largest_grid;            /* workgroups of the chunk's largest launch */
    int ranges;                      /* ranges dHidden's contraction is cut into, for `dense` rows */
    int added_up;                    /* whether the launch that adds partial products up is made */
    int in_stash;                    /* the partial products lie in stash rows not reached yet */
    int logits_columns, dhidden_columns, dw_columns;      /* of the small blocks (64 rows) a product runs on, 0: 256 x 256 */
    int logits_chained;              /* the logits run on persistent workgroups that walk chains of blocks */
    int together;                    /* dHidden and dW are one launch */
    int numbered_by_gather;          /* the gathering launch numbers the rows too */
    int transposed_apart;            /* W is transposed by launches of its own (first chunk) */
} alst_debug_ce_chunk_info;
int alst_debug_ce_chunk(int64_t N, int64_t H, int64_t V, int64_t tile, uint32_t flags, int64_t chunk, int64_t dense,
                        alst_debug_ce_chunk_info* info);

/*
 * Benchmarking aid (no counterpart in the paper): the sustained rate, in TFLOP/s, of the bf16
 * matrix instructions the block GEMMs are built on, measured on the current device with a loop that
 * touches no memory (one wavefront per SIMD of every compute unit, iters * 2^21 flop each).
 * It is the ceiling the GEMM kernels can be compared with besides the published peak: the clock
 * under matrix load depends on the power drawn, hence on the operand bits and the instruction form.
 * data bit 0: 0 = small-integer operands, 1 = random operands in [-1, 1); data bit 1: 0 =
 * v_mfma_f32_32x32x16_bf16 (the cores with a k-major operand), 1 = v_mfma_f32_16x16x32_bf16 (the
 * k-contiguous core).  scratch: device, 256 * 256 floats, overwritten; tflops: HOST double.
 * 1 <= iters <= 2^22; any other data is ALST_ERR_SHAPE.  Synchronises `stream`.
 */
int alst_debug_mfma_rate(int data, int iters, float* scratch, double* tflops, void* stream);

#ifdef __cplusplus
}
#endif
#endif /* ALST_DEBUG_H */
