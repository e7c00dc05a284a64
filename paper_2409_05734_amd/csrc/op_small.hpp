// One application of A or A^H to small 2D grids in one launch (op_small.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "plan.hpp"

namespace sr {

struct OpSmallArgs {
  const float2* in;   // A: signals; A^H: residuals
  float2* z;          // A: z (nullable); A^H: the signals out
  float* y;           // A: |z|^2 (nullable)
  const float2* eph;  // exp(i theta_1) of problem 0, layers of M1 M2 one after another
  const float2* tw0;  // twiddles of M1 and M2 (default thread shape)
  const float2* tw1;
  int L, N1, N2, o1, o2, W1, W2, c1, c2;
  float s_one;  // 1/sqrt(M1 M2)
  int s_x, s_m, s_th;  // elements from one problem's signal, measurements, phases to the next's
};

// Whether the kernel is built for this problem's grid.
bool op_small_supported(const Geo& g);
hipError_t launch_op_small(int M1, int M2, bool adjoint, const OpSmallArgs& a, int problems, hipStream_t s);

}  // namespace sr
