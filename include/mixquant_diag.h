/*
 * mixquant_diag.h -- diagnostics exported by libmixquant next to the C ABI of mixquant.h.
 * Nothing here is part of the method; the benchmark uses it to state a measured roof beside the
 * published peak.
 */
#ifndef MIXQUANT_DIAG_H
#define MIXQUANT_DIAG_H

#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Enqueue a loop of `iters` x 8 independent FP16 MFMAs
 * (32x32x16) per wave on pseudo-random register operands, one wave per SIMD on 256 compute
 * units, with no memory traffic.  Timing it gives the matrix rate the chip sustains under its
 * power management for realistic operand toggling, the measured roof quoted beside the
 * published peak.  scratch_dev: at least one float of device memory (practically never
 * written).  *flop_out (host pointer, may be NULL) receives the flop count of the launch.
 * 1 <= iters <= 2^20.
 */
int mq_mfma_probe(float *scratch_dev, int iters, void *stream, double *flop_out);

/*
 * What the entry points of mixquant.h launch for a problem, so that a test can state which kernel, tile or
 * number of K slabs it is about.  Host functions, no GPU access: `cus` is the number of compute units
 * to plan for (256 on an MI355X).
 *
 * A product is one launch, or two that cover the first rows or columns of Y and the others; the second
 * pass of a product cut into K slabs is not counted.  Each launch: the kernel, its workgroups' tile
 * (bm rows x bn columns of Y) and waves, the number of K slabs (1: none, no workspace is touched), and
 * the part of Y that it covers.  (The same for either output type, so that the BF16 output is the rounded
 * FP32 output bit for bit.)  Returns the number of launches (0 for an empty Y), or minus an
 * mq_status.
 */
typedef enum {
    MQ_KERNEL_SIMPLE = 0,      /* any K: one thread per output */
    MQ_KERNEL_FP4_DIRECT = 1,
    MQ_KERNEL_FP4_SMALL = 2,
    MQ_KERNEL_BF16_RING = 3,
    MQ_KERNEL_BF16_STAGE = 4,
    MQ_KERNEL_BF16_D2L = 5,
    MQ_KERNEL_BF16_SHORT = 6
} mq_kernel;
typedef struct {
    int kernel, bm, bn, waves, slabs;
    int64_t rows, cols;
} mq_launch;
int mq_gemm_launches(int64_t M, int64_t N, int64_t K, int layout, int64_t workspace_bytes, int cus, mq_launch out[2]);
int mq_bf16_gemm_launches(int64_t M, int64_t N, int64_t K, int64_t workspace_bytes, int cus, mq_launch out[2]);

/* Rows per workgroup of the quantizers with K-step-major output (K % 64 == 0): source 0 nvfp4_quantize,
 * 1 nvfp4_quantize_silu_mul, 2 nvfp4_quantize_rmsnorm.  Minus an mq_status for bad arguments. */
int mq_quantize_rows(int source, int64_t rows, int64_t K);

#ifdef __cplusplus
}
#endif
#endif /* MIXQUANT_DIAG_H */
