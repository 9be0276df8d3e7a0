/*
 * bwta_tuning.h -- benchmark and tuning hooks of libbwta.so.  Not part of the layer's contract
 * (bwta.h): nothing here changes a result, only which kernel instance computes it.  The settings
 * are process-wide atomics; a launch uses the values it reads when it is enqueued.
 */
#ifndef BWTA_TUNING_H
#define BWTA_TUNING_H

#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/* bwta_linear with its arguments in one block of memory, for callers whose foreign-function calls cost by
 * the argument (the Python binding: 15 conversions took longer than everything else on the host side of a
 * small layer).  size = sizeof(bwta_linear_args): a block of another layout is refused with
 * BWTA_ERR_UNSUPPORTED, NULL with BWTA_ERR_NULL; everything else is bwta_linear's.  The block may have any
 * alignment and is not kept. */
typedef struct bwta_linear_args {
    const void *A;
    int64_t lda;
    const void *s_a;
    const uint32_t *wsign;
    const void *s_w;
    void *out;
    int64_t ldo;
    void *workspace;
    uint64_t workspace_bytes;
    void *stream;
    int32_t a_scale_mode, w_scale_mode, M, N, K, size;
} bwta_linear_args;
int bwta_linear_call(const void *args);

/* Which family AUTO resolves to for a shape: BWTA_PATH_POPC, BWTA_PATH_MFMA or BWTA_PATH_FP4. */
int bwta_auto_path(int M, int N, int K);
/* Which contraction kernel a product of this shape is dispatched to under the current path setting
 * (a pure host function: nothing is launched).  operand = 0: canonical planes with a workspace
 * (bwta_gemm); BWTA_PREPARED_PLANES or BWTA_PREPARED_FP4: bwta_gemm_prepared with that format;
 * BWTA_OPERAND_FP16: bwta_linear on fp16 rows that its results do not overlap, one of the
 * BWTA_KERNEL_LINEAR_* where ternarisation, product and epilogue are one launch, else the product
 * kernel behind the ternarise launch.
 * Prepared planes never resolve to BWTA_KERNEL_GEMM_FP4: that kernel needs scratch for its
 * fragments and bwta_gemm_prepared has none.  0 for a non-positive dimension or an unknown operand. */
enum {
    BWTA_KERNEL_GEMV_POPC = 1,    /* decode, wave64 popcount            */
    BWTA_KERNEL_GEMV_FP4 = 2,     /* decode, FP4 matrix cores           */
    BWTA_KERNEL_GEMM_FP4 = 3,     /* tiled, FP4 matrix cores            */
    BWTA_KERNEL_GEMM_MFMA_I8 = 4, /* tiled, int8 matrix cores (planes)  */
    BWTA_KERNEL_GEMM_POPC = 5,    /* tiled, wave64 popcount (planes)    */
    BWTA_KERNEL_LINEAR_FUSED = 6, /* whole linear, all of a short K     */
    BWTA_KERNEL_LINEAR_STRIP = 7, /* whole linear, K in slabs           */
    BWTA_KERNEL_LINEAR_ONE = 8,   /* whole linear, one token            */
    BWTA_KERNEL_LINEAR_ROWS = 9   /* whole linear, strips of 16 tokens, all of K at once: few tokens, narrow matrices */
};
enum { BWTA_OPERAND_FP16 = 3 };
int bwta_planned_kernel(int operand, int M, int N, int K);
/* 1 where bwta_planned_kernel answers BWTA_KERNEL_LINEAR_ROWS for BWTA_OPERAND_FP16, else 0. */
int bwta_planned_rows(int M, int N, int K);
/* How many kernels bwta_linear launches for a shape under the current settings, given results that do
 * not overlap the activations (a call that works in place always takes two): 1 where ternarisation,
 * product and epilogue run as one kernel (bwta_planned_kernel says which), else 2.  Informational
 * (benchmarks label their timings with it); 0 for a non-positive dimension. */
int bwta_linear_launches(int M, int N, int K);
/* Tuning hook for benchmark sweeps: force the FP4 kernel's per-wavefront tile (22, 21, 12, 11, 13
 * = blocks of 32 rows x 32 columns per wavefront; 23 = 22 at three wavefronts per SIMD; 222 = 22
 * with K split over two groups of wavefronts; 243, 223, 323 = the kernel that stages both operands
 * through LDS with direct loads, as 128 x 256 tiles of 8 wavefronts, 128 x 128 tiles of 4, or
 * 128 x 256 tiles of 4 wavefronts of 64 tokens x 128 channels; 422, 521, 611 = the kernel of 16 x 16 blocks,
 * fp16 results only, as 128 x 256 tiles, 128 x 128 with K split over two groups of wavefronts, 64 x 128 with
 * K split over four), the popcount decode kernel's row split (1000 + 16 *
 * lanes per row (8, 16, 32) + chunks per lane; ignored where the registers cannot hold it) or the
 * matrix-core decode kernel's work split (2000 + 1024 * ring depth (2..4) + 64 * chunks per
 * wavefront (1..4) + tiles per workgroup (rounded up to a multiple of the ring depth, fewer if LDS
 * does not hold their partials)), or where bwta_linear runs as a single launch (900 never, 901
 * wherever the one-launch kernel can run, 900 + R the same with R channel splits per token
 * strip); 0 restores the built-in choices.  Results do not depend on it. */
int bwta_set_tile(int tile);
/* How a product (BWTA_KERNEL_GEMM_FP4) of fp16 results alone runs under the current settings: bwta_planned_wide says
 * which tile of the kernel of 16 x 16 blocks (422, 521, 611) takes the shape in bwta_gemm and bwta_linear, and
 * bwta_planned_wide_prepared in bwta_gemm_prepared; 0 if none does; then bwta_planned_tile says which of the other tiles.  0 for a non-positive dimension.  A product with int32 results runs on 128 x 128 tiles (22)
 * whatever these answer, except that a tile of the LDS kernel (223, 243, 323) forced by bwta_set_tile takes it too. */
int bwta_planned_wide(int M, int N, int K);
int bwta_planned_wide_prepared(int M, int N, int K);
int bwta_planned_tile(int M, int N, int K);
/* How many blocks of channel tiles a workgroup of the matrix-core decode kernel (BWTA_KERNEL_GEMV_FP4) walks one after the
 * other in a launch of `count` problems of one shape: 1, 2, 4 or 8; 0 where another kernel takes the shape. */
int bwta_planned_decode_blocks(int M, int N, int K, int count);
#ifdef __cplusplus
}
#endif
#endif /* BWTA_TUNING_H */
