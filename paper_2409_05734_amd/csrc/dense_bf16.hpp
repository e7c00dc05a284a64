// Dense i.i.d. model on many signals: the two real products on bf16 matrix
// cores with FP32's accuracy (dense_bf16.hip): launch interface.
#pragma once
#include <hip/hip_runtime.h>

namespace sr {

// Both operands are taken times this, so the partials come out times its square.
constexpr float kBf16Scale = 65536.f;

// One product.  G = 1: C (m x q) = At . Bx, reduction over 2n; G = 2: C^T
// (q x 2n) = Br^T . At, reduction over m; q = 64 per tile of 32 signals.
// Partial s of the S splits goes where the FP32 products put theirs:
// G = 1 split[(s m + i) q_ld + q], G = 2 split[(s q_ld + q) 2n + j].
struct Bf16Gemm {
  const float* A;          // m x 2n floats
  int m, n, nb;
  const float2* src;       // signals (nb x n) or residuals (nb x m)
  const float* src_scale;  // per-signal factor, nullable
  void* pack;              // bf16_pack_bytes
  float* split;
  int q_ld;
};

// Reduction splits of a product (its S partials; steps of 32 apiece).
int bf16_splits(int G, int m, int n, int nb, int* steps);
size_t bf16_pack_bytes(int m, int n, int nb);
hipError_t launch_bf16_gemm(int G, const Bf16Gemm& a, hipStream_t st);

}  // namespace sr
