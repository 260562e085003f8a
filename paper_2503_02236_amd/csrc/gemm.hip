// VQ-gemm for gfx950: Y[m][n] = scale[n] * sum_k W[n][k] X[m][k], W held as VQ codes, contraction on the fp16 matrix
// cores with fp32 accumulation.  Operation: VQ-LLM (arXiv 2503.02236) Sec. III-C "VQ-gemm"; dequantization of Sec. II-A.
// This file chooses between the two ways: dequantize once and multiply densely (dequant.hip, gemm_dense.hip), or look
// entries up inside the product (gemm_skinny.hip).
#include "vq_common.h"

namespace vq {

// Large M: dequantize once into the workspace (fp16 [N][K]) and run the dense matrix-core kernel.
// Small M: few M tiles would not reuse the dequantized weights, so the fused kernel looks them up directly (and for a
// small product of more than 256 tokens, whose workspace then stays unused).
static bool gemm_two_stage(const vq_weight_t *w, int M) { return M > 256 && w->K > 0 && w->K % 64 == 0; }

size_t gemm_workspace(const vq_weight_t *w, int M) {
    return gemm_two_stage(w, M) ? (size_t)w->N * w->K * sizeof(half_t) : 0;
}

int launch_gemm(const vq_weight_t *w, const void *X, int M, void *Y, void *ws, hipStream_t s) {
    const half_t *Xp = (const half_t *)X;
    half_t *Yp = (half_t *)Y;
    if (M <= 256 ? M > 16 && gemm_skinny_supported(w) : gemm_skinny_wins(w, M)) return launch_gemm_skinny(w, X, M, Y, s);
    if (gemm_two_stage(w, M)) {
        int st = launch_dequant(w, ws, /*out_fp32=*/0, s);
        if (st != VQ_OK) return st;
        return launch_gemm_dense(Xp, (const half_t *)ws, (const half_t *)w->scale, Yp, M, w->N, w->K, s);
    }
    // any other configuration: 16 tokens at a time through the generic row kernel
    for (int m = 0; m < M; m += 16) {
        int bs = M - m < 16 ? M - m : 16;
        int st = launch_gemv_rows(w, Xp + (size_t)m * w->K, bs, Yp + (size_t)m * w->N, s);
        if (st != VQ_OK) return st;
    }
    return VQ_OK;
}

}  // namespace vq
