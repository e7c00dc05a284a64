// Dense i.i.d. model on a few signals (dense_rows.hip): launch interface.
#pragma once
#include <hip/hip_runtime.h>

namespace sr {

enum RowsMode : int {
  ROWS_FWD = 0,   // z = A x (and |z|^2)
  ROWS_ADJ = 1,   // partials of A^H r, r given
  ROWS_GD = 2,    // z = A x, r = (|z|^2 - y) z or the Poisson residual, partials of A^H r
  ROWS_SPEC = 3   // z = A x / ||x||, r = T(y / mean(y)) z, partials of A^H r
};

struct RowsArgs {
  const float* A;        // m x 2n floats
  int m, n, nb;
  int rows;              // rows per workgroup (a multiple of the batch)
  const float2* x;       // nb x n
  const float2* r;       // ROWS_ADJ: nb x m
  float2* z_out;         // ROWS_FWD: nb x m, nullable
  float* y_out;          // ROWS_FWD: |z|^2, nullable
  const float* y;        // nb x m
  const double* ysum;    // ROWS_SPEC: sum(y) per signal
  float lam;
  int loss;
  float loss_eps;
  float* loss_part;      // ROWS_GD: [signal][workgroup], nullable
  int loss_ld;
  const float* norm_part;  // ROWS_SPEC: squared-norm partials of x, [signal][norm_ld], norm_cnt of them
  int norm_ld, norm_cnt;
  float* inv;            // ROWS_SPEC: 1/||x_p|| out
  float2* part;          // partials of A^H r, [workgroup][signal][n]
};

enum RowsEpi : int { ROWS_STORE = 0, ROWS_UPDATE_GD = 1, ROWS_UPDATE_SPEC = 2 };

// Work split of one shape: T threads a workgroup, J column pairs a thread
// (n <= 2 T J), R rows a batch, NB signal slots, G workgroups of `rows` rows.
struct RowsShape {
  int T, J, R, NB, G, rows;
};

// Whether the row kernels take this shape, and its split.
bool rows_shape(int m, int n, int nb, RowsShape* s);
inline int rows_update_groups(int n) { return (n + 15) / 16; }
// Products over A's rows (mode ROWS_*), and the sum of the partials with the
// update `epi` (ROWS_STORE / ROWS_UPDATE_*).
hipError_t launch_rows(int mode, const RowsShape& s, const RowsArgs& a, hipStream_t st);
hipError_t launch_rows_update(int epi, const RowsShape& s, const RowsArgs& a, float2* x, float step, float* norm_part,
                              int norm_ld, unsigned* nf, hipStream_t st);

}  // namespace sr
