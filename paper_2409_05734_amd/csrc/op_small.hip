// One application of A (or A^H) to problems on small 2D grids, a workgroup
// each, in one launch.
//
// The pass kernels take L + 1 launches an application, and on a grid of a few
// thousand points there is little else than the latency of a launch and of a
// trip through memory.  Here the grid stays in one workgroup: eight elements a
// thread in registers, the stages of a transform and the changes between
// columns and rows exchanged through the same two LDS buffers in turn, in the
// order and arithmetic of the pass schedule ([U D_1 F_0] [F_1 D_2 F_1] ...
// [F_a]).  What is left is the kernel's own chain (loads, then 2 L + 1
// exchanges of a barrier each and the transforms' arithmetic).
//
// A and A^H as a caller queues them, passes -> here: 64 x 64, L = 1, 2, 3: 19.4,
// 26.7, 33.9 -> 10.2, 13.5, 17.1 us; 32 x 32, L = 2: 26.3 -> 10.3 us; each call
// waited for: 30.7 -> 26.4 us (64 x 64, L = 2).  Problems of one shape are as
// many workgroups: 512 of 64 x 64, 41.6 -> 25.8 us.
//
// The rule (op_small_supported): lengths of one thread shape with eight
// elements and a pad every eight, so that both directions have the same threads
// and buffers, and at most 4096 points.  Twice that is one workgroup of 1024
// threads whose chain is as long as the launches (128 x 64, L = 2, queued 27.0
// -> 24.9 us, waited for 30.5 -> 37.8 us).
#include "op_small.hpp"

#include "fft_core.hpp"
#include "lds_limit.hpp"

namespace sr {

namespace {

template <int M1, int M2, bool ADJ>
__global__ void __launch_bounds__(M1 * M2 / 8) op_small_kernel(const OpSmallArgs a) {
  using TC = Tile<M1, M2, true>;   // along axis 0: all columns
  using TR = Tile<M2, M1, false>;  // along axis 1: all rows
  static_assert(TC::E == 8 && TR::E == 8 && TC::PADSHIFT == 3 && TR::PADSHIFT == 3, "eight elements a thread");
  static_assert(TC::BUF == TR::BUF, "both directions alternate between the same two buffers");
  constexpr int LDX = TR::LD;
  extern __shared__ float2 lds[];
  const int tc = TC::thread_t(), bc = TC::thread_b(), tr = TR::thread_t(), br = TR::thread_b();
  const int mg = M1 * M2;
  const float2* in = a.in + (long long)blockIdx.x * (ADJ ? a.s_m : a.s_x);
  const float2* eph = a.eph + (long long)blockIdx.x * a.s_th;
  typename TC::Twiddles wc;
  typename TR::Twiddles wr;
  TC::load_twiddles(wc, a.tw0, tc);
  TR::load_twiddles(wr, a.tw1, tr);
  int ph = 0;  // LDS buffer of the next exchange, whichever kind it is
  float2 v[8];

  // grid row and column of element j in either layout
  auto row_c = [&](int j) { return TC::elem(tc, j); };
  auto col_r = [&](int j) { return TR::elem(tr, j); };
  auto to_rows = [&]() {
    float2* x = lds + ph * TC::BUF;
#pragma unroll
    for (int j = 0; j < 8; ++j) x[row_c(j) * LDX + bc] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = x[br * LDX + col_r(j)];
    ph ^= 1;
  };
  auto to_cols = [&]() {
    float2* x = lds + ph * TC::BUF;
#pragma unroll
    for (int j = 0; j < 8; ++j) x[br * LDX + col_r(j)] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = x[row_c(j) * LDX + bc];
    ph ^= 1;
  };
  // the diagonal of layer l at this thread's elements
  auto load_diag = [&](float2(&d)[8], int l, bool cols) {
    const float2* e = eph + (long long)(l - 1) * mg;
#pragma unroll
    for (int j = 0; j < 8; ++j) d[j] = cols ? e[row_c(j) * M2 + bc] : e[br * M2 + col_r(j)];
  };
  // measurement at (row i, column c): its index, or -1 outside the window
  auto meas = [&](int i, int c) {
    const int r = i - a.c1, q = c - a.c2;
    return (unsigned)r < (unsigned)a.W1 && (unsigned)q < (unsigned)a.W2 ? r * a.W2 + q : -1;
  };
  auto supp = [&](int i, int c) {
    const int r = i - a.o1, q = c - a.o2;
    return (unsigned)r < (unsigned)a.N1 && (unsigned)q < (unsigned)a.N2 ? r * a.N2 + q : -1;
  };
  auto fft_cols = [&]() { TC::template fft<ADJ>(v, lds, ph, wc, tc, bc); };
  auto fft_rows = [&]() { TR::template fft<ADJ>(v, lds, ph, wr, tr, br); };
  // one middle pass: transform, diagonal with 1/N for both transforms, transform
  auto mid = [&](float2(&d)[8], bool cols) {
    if (cols) fft_cols();
    else fft_rows();
    const float s = cols ? 1.f / M1 : 1.f / M2;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = ADJ ? cmulc(v[j], cscale(d[j], s)) : cmul(v[j], cscale(d[j], s));
    if (cols) fft_cols();
    else fft_rows();
  };

  const int L = a.L;
  const bool last_cols = (L % 2) == 0;  // axis of the pass next to the measurements (pass L + 1)
  // the two single transforms of the first and last pass (axis 0 next to the
  // signal, the last pass's axis next to the measurements)
  const float s_one = last_cols ? 1.f / M1 : a.s_one;
  float2 d[8], dn[8];
  if constexpr (!ADJ) {
    load_diag(d, 1, true);
    if (L >= 2) load_diag(dn, 2, false);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int e = supp(row_c(j), bc);
      v[j] = e >= 0 ? cmul(in[e], cscale(d[j], s_one)) : make_float2(0.f, 0.f);
    }
    fft_cols();
    for (int k = 2; k <= L; ++k) {
      const bool cols = (k % 2) == 1;
#pragma unroll
      for (int j = 0; j < 8; ++j) d[j] = dn[j];
      if (k < L) load_diag(dn, k + 1, !cols);
      if (cols) to_cols();
      else to_rows();
      mid(d, cols);
    }
    if (last_cols) {
      to_cols();
      fft_cols();
    } else {
      to_rows();
      fft_rows();
    }
    float2* z = a.z ? a.z + (long long)blockIdx.x * a.s_m : nullptr;
    float* y = a.y ? a.y + (long long)blockIdx.x * a.s_m : nullptr;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int e = last_cols ? meas(row_c(j), bc) : meas(br, col_r(j));
      if (e >= 0) {
        if (z) z[e] = v[j];
        if (y) y[e] = cabs2(v[j]);
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int e = last_cols ? meas(row_c(j), bc) : meas(br, col_r(j));
      v[j] = e >= 0 ? in[e] : make_float2(0.f, 0.f);
    }
    load_diag(d, L, L == 1 || (L % 2) == 1);
    if (last_cols) fft_cols();
    else fft_rows();
    for (int k = L; k >= 2; --k) {
      const bool cols = (k % 2) == 1;
      load_diag(dn, k - 1, !cols);
      if (cols) to_cols();
      else to_rows();
      mid(d, cols);
#pragma unroll
      for (int j = 0; j < 8; ++j) d[j] = dn[j];
    }
    to_cols();
    fft_cols();
    float2* x = a.z + (long long)blockIdx.x * a.s_x;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int e = supp(row_c(j), bc);
      if (e >= 0) x[e] = cmulc(v[j], cscale(d[j], s_one));
    }
  }
}

template <int M1, int M2, bool ADJ>
hipError_t go(const OpSmallArgs& a, int problems, hipStream_t s) {
  constexpr size_t lds = 2 * sizeof(float2) * (size_t)Tile<M1, M2, true>::BUF;
  auto kern = op_small_kernel<M1, M2, ADJ>;
  if (lds > 65536) {
    static LdsLimit limit;  // (one per instantiation)
    if (hipError_t e = limit.raise((const void*)kern, lds); e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3(problems), dim3(M1 * M2 / 8), lds, s, a);
  return hipGetLastError();
}

#define SR_SMALL_GRIDS(X) X(32, 32) X(32, 64) X(32, 128) X(64, 32) X(64, 64) X(128, 32)

}  // namespace

bool op_small_supported(const Geo& g) {
  if (g.ndim != 2) return false;
#define SR_CASE(p, q) \
  if (g.M1 == p && g.M2 == q) return true;
  SR_SMALL_GRIDS(SR_CASE)
#undef SR_CASE
  return false;
}

hipError_t launch_op_small(int M1, int M2, bool adjoint, const OpSmallArgs& a, int problems, hipStream_t s) {
#define SR_CASE(p, q) \
  if (M1 == p && M2 == q) return adjoint ? go<p, q, true>(a, problems, s) : go<p, q, false>(a, problems, s);
  SR_SMALL_GRIDS(SR_CASE)
#undef SR_CASE
  return hipErrorInvalidValue;
}

}  // namespace sr
