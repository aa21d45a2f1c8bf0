// fp32 contractions of the LSTM (gemm_f32.hip): host interface.
#pragma once
#include "common.h"

namespace ver {

constexpr int F32_GROUP_MAX = 4;
struct F32Problem {
    const float* A; const float* B; float* C; const float* bias;
    int lda, ldb, ldc, Mr, Nc, K, unperm_h;
    int tiles_n, tile_first;   // column tiles; first tile of the problem in the launch
};
struct F32GroupArgs { F32Problem p[F32_GROUP_MAX]; int n, tiles; };

// Up to four contractions in one launch, all with the contraction index contiguous (K-major: C = A[Mr, K] B[Nc, K]^T + bias)
// or all with it outermost (K-minor: C = A[K, Mr]^T B[K, Nc]).  Leading dimensions, Nc and (K-minor) Mr are multiples
// of 4; unperm_h > 0 stores output row m at row (m % 4) * unperm_h + m / 4.
struct F32Gemm {
    F32GroupArgs a{};
    bool k_minor;
    explicit F32Gemm(bool k_minor_) : k_minor(k_minor_) {}
    // False if an operand is beyond the kernel's 32-bit byte offsets (or the launch is full): not added.
    bool add(const float* A, int lda, const float* B, int ldb, float* C, int ldc, int Mr, int Nc, int K, const float* bias, int unperm_h);
    void launch(hipStream_t s);
};

}  // namespace ver
