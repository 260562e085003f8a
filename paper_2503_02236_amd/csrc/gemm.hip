// VQ-gemm for gfx950: Y[m][n] = scale[n] * sum_k W[n][k] X[m][k], W held as VQ codes, contraction on the fp16 matrix
// cores with fp32 accumulation.  Operation: VQ-LLM (arXiv 2503.02236) Sec. III-C "VQ-gemm"; dequantization of Sec. II-A.
// This file chooses between the two ways: dequantize once and multiply densely (dequant.hip, gemm_tiles.hip; gemm_dense.hip
// for a very long K), or look entries up inside the product (gemm_skinny.hip).
#include "vq_common.h"

namespace vq {

// Large M: dequantize once into the workspace (fp16 [N][K]) and run the dense matrix-core kernel.
// Small M: few M tiles would not reuse the dequantized weights, so the fused kernel looks them up directly (and for a
// small product of more than 256 tokens, whose workspace then stays unused).
static bool gemm_two_stage(const vq_weight_t *w, int M) { return M > 256 && w->K > 0 && w->K % 64 == 0; }

size_t gemm_workspace(const vq_weight_t *w, int M) {
    return gemm_two_stage(w, M) ? (size_t)w->N * w->K * sizeof(half_t) : 0;
}

// One pass over the codes.  More than 256 tokens: where that is faster than the two stages, and always where these do not
// exist (K % 64 != 0): what is left then is 16 tokens a launch, each of which reads all codes (K = 4128, N = 4096, two 12-bit
// codebooks, 2048 tokens: 953 us that way, 223 in one pass).
bool gemm_one_pass(const vq_weight_t *w, int M) {
    if (M <= 16 || !gemm_skinny_supported(w)) return false;
    return M <= 256 || !gemm_two_stage(w, M) || gemm_skinny_wins(w, M);
}

int launch_gemm(const vq_weight_t *w, const void *X, int M, void *Y, void *ws, hipStream_t s) {
    const half_t *Xp = (const half_t *)X;
    half_t *Yp = (half_t *)Y;
    if (gemm_one_pass(w, M)) return launch_gemm_skinny(w, X, M, Y, s);
    if (gemm_two_stage(w, M)) {
        if (gemm_tiles_fits(w->K)) {
            int pick;
            gemm_tiles_time(M, w->N, w->K, &pick);
            const int st = launch_dequant_ordered(w, (half_t *)ws, s);
            return st != VQ_OK ? st : launch_gemm_tiles(Xp, (const half_t *)ws, (const half_t *)w->scale, Yp, M, w->N, w->K, pick, s);
        }
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
