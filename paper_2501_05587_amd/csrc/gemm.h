// Dense products C[m][n] = alpha * sum_k A(m,k) B(n,k) on MFMA with FP32
// accumulation, used by the learned feature map and the feature-space Lloyd
// iterations.  Internal to the library.
#pragma once

#include "kkm_common.h"

namespace kkm {

enum GemmOp { GEMM_BF16 = 0, GEMM_F32 = 1 };
enum GemmEpi {
    EPI_STORE = 0,      // C = alpha * acc
    EPI_BIAS = 1,       // C = alpha * acc + bias[n]
    EPI_BIAS_GELU = 2,  // Z = alpha * acc + bias[n]; C = Z (if C), C2 = GELU(Z)
    EPI_GELU_BWD = 3,   // C = alpha * acc * GELU'(Zp[m][n])
    EPI_LOSS = 4        // C = alpha * acc - Kb[m][n]; per-workgroup sum of C^2 (FP64)
};

struct GemmArgs {
    const float *A;
    int64_t lda;
    const float *B;
    int64_t ldb;
    int64_t M, N, K;
    float alpha;
    float *C;
    int64_t ldc;
    const float *bias;
    float *C2;
    int64_t ldc2;
    const float *Zp;
    int64_t ldz;
    const float *Kb;
    int64_t ldkb;
    double *part;  // [gridDim.x * gridDim.y]
};

// a_kcontig: A(m,k) = A[m*lda + k], else A[k*lda + m]; likewise b_kcontig for B(n,k).
kkm_status gemm_launch(GemmOp op, bool a_kcontig, bool b_kcontig, GemmEpi epi, const GemmArgs &g,
                       hipStream_t stream);

// GELU and its derivative.
__device__ __forceinline__ float gelu(float z) {
    return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
}
__device__ __forceinline__ float gelu_grad(float z) {
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) +
           z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// Adam (bias-corrected); omb1 = 1 - beta1 and omb2 = 1 - beta2 are formed in
// double on the host, c1 = 1 - beta1^t, c2 = 1 - beta2^t.
struct AdamArgs {
    float lr, b1, b2, omb1, omb2, eps, c1, c2;
};
__device__ __forceinline__ void adam_one(float &p, float &mo, float &ve, float gi, const AdamArgs &a) {
    // the fused products spelled out: every kernel that updates rounds alike
    const float m = fmaf(a.omb1, gi, a.b1 * mo);
    const float v = fmaf(gi, a.omb2 * gi, a.b2 * ve);
    mo = m;
    ve = v;
    p -= a.lr * (m / a.c1) / (sqrtf(v / a.c2) + a.eps);
}

// ---------------------------------------------------------------- one training step of a small batch

constexpr int64_t kSmallBatch = 256;  // its most rows

// Kernel values of the batch, computed in the step's first launch (XB's rows
// against each other, FP32; kernel < 0: KB is already in place).
struct BatchKernel {
    int32_t kernel;
    float gamma, coef0;  // Gaussian: gamma log2(e)
    int32_t degree;
};

// The network and the batch of one step: parameters th (offsets o*), XB [B,
// ldx], KB [B, ldkb] (written when kern.kernel >= 0), the activations and
// gradients kept in the workspace, part [ceil(B / 16)].  Adam on th / am / av
// when `adam` is given, else the gradient goes to grad.
struct TrainStep {
    int64_t B, d, h1, h2, out;
    int64_t oW1, ob1, oW2, ob2, oW3, ob3;
    float *th, *am, *av, *grad;
    const float *XB;
    int64_t ldx;
    float *KB;
    int64_t ldkb;
    BatchKernel kern;
    float *Z1, *H1, *Z2, *H2, *Phi, *dPhi, *dZ2, *dZ1;
    double *part, *loss;
};
kkm_status train_step_small(const TrainStep &t, const AdamArgs *adam, hipStream_t stream);

inline int64_t gemm_tiles(int64_t M, int64_t N) { return ((M + 63) / 64) * ((N + 63) / 64); }

}  // namespace kkm
