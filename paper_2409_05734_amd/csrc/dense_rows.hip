// Dense i.i.d. model (section II-A) on a few signals: A x and A^H r on the
// vector units, one read of A for both where a solver applies them in turn.
//
// With one to four signals the 64-column matrix-core tiles of dense.hip work
// mostly on padding, and each of A X and A^H R streams A once.  A workgroup
// here takes a run of A's rows; for each small batch of rows it forms z = A x
// (x lives in registers, a column slice per thread), applies the solver's
// weight to z, and adds conj(a) r of the same rows, still in registers, to its
// partial of A^H r.  A second kernel sums the workgroups' partials in index
// order and applies the update.  A GD or power iteration then reads A once.
//
// Bound by the stream of A from HBM: the next batch of rows is loaded into a
// second register set before the current one is reduced, so 64 to 128 KB per
// CU are in flight across the two barriers of a batch.  16384 x 4096, one
// signal: A x 90 us, A^H r 92 us, a GD iteration 98 us (5.5 TB/s), against
// 133, 151 and 279 us on the matrix-core path (two products over A with their
// packing and epilogue kernels, four launches more).
#include "dense_rows.hpp"

#include <algorithm>

#include "fft_core.hpp"
#include "loss.hpp"

namespace sr {

namespace {

typedef float rows_f4 __attribute__((ext_vector_type(4)));

// Sum V values (a power of two) over the wave: halving exchanges leave one
// value per lane group, value index lane / (64 / V), with V - 1 + log2(64/V)
// shuffles instead of 6 V.  Fixed order.
template <int V>
__device__ __forceinline__ float wave_sum_many(float (&v)[V], int lane) {
  int mask = 32;
#pragma unroll
  for (int h = V / 2; h >= 1; h /= 2, mask /= 2) {
    const bool up = (lane & mask) != 0;
#pragma unroll
    for (int i = 0; i < h; ++i) {
      // (values first: a choice between the elements themselves is an index
      // that the compiler searches the registers for, 1754 instructions a kernel
      // of four signals against 413; A x of 20000 x 100 74 -> 17 us)
      const float lo = v[i], hi = v[i + h];
      v[i] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, mask);
    }
  }
  for (; mask >= 1; mask /= 2) v[0] += __shfl_xor(v[0], mask);
  return v[0];
}

// T threads hold n <= 2 T J columns, thread t the complex pairs 2 (t + T j);
// R rows per batch, NB signal slots.  grid.x: workgroups of `rows` rows each,
// grid.y: groups of NB signals.
template <int MODE, int NB, int T, int J, int R>
__global__ void __launch_bounds__(T) dense_rows_kernel(const RowsArgs a) {
  constexpr int V = 2 * R * NB;  // sums per batch: (row, signal, re/im)
  constexpr int W = T / 64;
  static_assert(V <= 64 && (V & (V - 1)) == 0, "one wave finishes the sums");
  constexpr bool DOT = MODE != ROWS_ADJ;
  constexpr bool BACK = MODE != ROWS_FWD;
  __shared__ float red[2][W][V];
  __shared__ float rs[V];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int p0 = blockIdx.y * NB;          // this group's first signal
  const int np = min(NB, a.nb - p0);       // and how many it has
  const int row_lo = blockIdx.x * a.rows;
  const int row_hi = min(a.m, row_lo + a.rows);
  const int lda = 2 * a.n;

  rows_f4 xr[DOT ? NB : 1][J];
  rows_f4 acc[BACK ? NB : 1][J];
  if constexpr (DOT) {
    float sc[NB];
#pragma unroll
    for (int p = 0; p < NB; ++p) sc[p] = 1.f;
    if constexpr (MODE == ROWS_SPEC) {
      __shared__ double nred[W > 1 ? W : 1];
      for (int p = 0; p < np; ++p) {
        double s = 0.0;
        for (int i = tid; i < a.norm_cnt; i += T) s += (double)a.norm_part[(long long)(p0 + p) * a.norm_ld + i];
        const float iv = (float)(1.0 / sqrt(block_sum_t<T, double>(s, nred)));
#pragma unroll
        for (int q = 0; q < NB; ++q)
          if (q == p) sc[q] = iv;
        if (blockIdx.x == 0 && tid == 0) a.inv[p0 + p] = iv;
      }
    }
#pragma unroll
    for (int p = 0; p < NB; ++p)
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int k = 2 * (tid + T * j);
        float2 u = make_float2(0.f, 0.f), v = u;
        if (p < np && k < a.n) {
          u = a.x[(long long)(p0 + p) * a.n + k];
          v = a.x[(long long)(p0 + p) * a.n + k + 1];
        }
        xr[p][j] = rows_f4{u.x * sc[p], u.y * sc[p], v.x * sc[p], v.y * sc[p]};
      }
  }
  if constexpr (BACK) {
#pragma unroll
    for (int p = 0; p < NB; ++p)
#pragma unroll
      for (int j = 0; j < J; ++j) acc[p][j] = rows_f4{0.f, 0.f, 0.f, 0.f};
  }

  rows_f4 cur[R][J], nxt[R][J];
  auto load = [&](rows_f4(&d)[R][J], int row0) {
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int k = 2 * (tid + T * j);
        d[i][j] = rows_f4{0.f, 0.f, 0.f, 0.f};
        if (row0 + i < row_hi && k < a.n)
          d[i][j] = *reinterpret_cast<const rows_f4*>(a.A + (long long)(row0 + i) * lda + 2 * k);
      }
  };

  // the thread that finishes sum v = (row i, signal p, component c)
  const int vi = tid / (2 * NB), vp = (tid / 2) % NB;
  float loss = 0.f;
  float ybar = 0.f;
  if constexpr (MODE == ROWS_SPEC)
    if (tid < V && vp < np) ybar = (float)(a.ysum[p0 + vp] / (double)a.m);

  load(cur, row_lo);
  int par = 0;
  for (int row0 = row_lo; row0 < row_hi; row0 += R, par ^= 1) {
    load(nxt, row0 + R);  // (past the last row: zeros, no access)
    if constexpr (DOT) {
      const bool mine = tid < V && vp < np && row0 + vi < row_hi;
      float yv = 0.f;
      if constexpr (MODE != ROWS_FWD)
        if (mine) yv = a.y[(long long)(p0 + vp) * a.m + row0 + vi];
      float v[V];
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int p = 0; p < NB; ++p) {
          float re = 0.f, im = 0.f;
#pragma unroll
          for (int j = 0; j < J; ++j) {
            const rows_f4 c = cur[i][j], x = xr[p][j];
            re += c[0] * x[0];
            re -= c[1] * x[1];
            im += c[0] * x[1];
            im += c[1] * x[0];
            re += c[2] * x[2];
            re -= c[3] * x[3];
            im += c[2] * x[3];
            im += c[3] * x[2];
          }
          v[(i * NB + p) * 2] = re;
          v[(i * NB + p) * 2 + 1] = im;
        }
      const float s = wave_sum_many<V>(v, lane);
      if ((lane & (64 / V - 1)) == 0) red[par][wave][lane / (64 / V)] = s;
      __syncthreads();
      if (tid < V) {
        float t = red[par][0][tid];
#pragma unroll
        for (int w = 1; w < W; ++w) t += red[par][w][tid];
        const float o = __shfl_xor(t, 1);  // the other component
        const float z2 = t * t + o * o;
        if constexpr (MODE == ROWS_FWD) {
          if (mine) {
            const long long e = (long long)(p0 + vp) * a.m + row0 + vi;
            if (a.z_out) reinterpret_cast<float*>(a.z_out)[2 * e + (tid & 1)] = t;
            if (a.y_out && (tid & 1) == 0) a.y_out[e] = z2;
          }
        } else {
          float w;
          if constexpr (MODE == ROWS_SPEC) {
            w = a.lam;
            if (yv > 0.f) w = fmaxf(1.f - ybar / yv, a.lam);
          } else if (a.loss == LOSS_POISSON) {
            w = poisson_weight(z2, yv, a.loss_eps);
            if (mine) loss += poisson_term(z2, yv, a.loss_eps);
          } else {
            w = z2 - yv;
            if (mine) loss += w * w;
          }
          rs[tid] = mine ? t * w : 0.f;
        }
      }
      if constexpr (BACK) __syncthreads();
    }
    if constexpr (BACK) {
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int p = 0; p < NB; ++p) {
          float rr = 0.f, ri = 0.f;
          if constexpr (MODE == ROWS_ADJ) {
            if (p < np && row0 + i < row_hi) {
              const float2 q = a.r[(long long)(p0 + p) * a.m + row0 + i];
              rr = q.x;
              ri = q.y;
            }
          } else {
            rr = rs[(i * NB + p) * 2];
            ri = rs[(i * NB + p) * 2 + 1];
          }
#pragma unroll
          for (int j = 0; j < J; ++j) {
            const rows_f4 c = cur[i][j];
            acc[p][j][0] += c[0] * rr;
            acc[p][j][0] += c[1] * ri;
            acc[p][j][1] += c[0] * ri;
            acc[p][j][1] -= c[1] * rr;
            acc[p][j][2] += c[2] * rr;
            acc[p][j][2] += c[3] * ri;
            acc[p][j][3] += c[2] * ri;
            acc[p][j][3] -= c[3] * rr;
          }
        }
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int j = 0; j < J; ++j) cur[i][j] = nxt[i][j];
  }

  if constexpr (BACK) {
#pragma unroll
    for (int p = 0; p < NB; ++p)
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int k = 2 * (tid + T * j);
        if (p < np && k < a.n) {
          float2* o = a.part + ((long long)blockIdx.x * a.nb + p0 + p) * a.n + k;
          o[0] = make_float2(acc[p][j][0], acc[p][j][1]);
          o[1] = make_float2(acc[p][j][2], acc[p][j][3]);
        }
      }
  }
  if constexpr (MODE == ROWS_GD) {
    // this workgroup's loss: each signal's rows are on the threads
    // 2 (i NB + p) of the first wave (the odd threads hold the same values)
    if (a.loss_part != nullptr && tid < V) {
#pragma unroll
      for (int o = V / 2; o >= 2 * NB; o /= 2) loss += __shfl_xor(loss, o);
      if (tid < 2 * NB && (tid & 1) == 0 && vp < np) a.loss_part[(long long)(p0 + vp) * a.loss_ld + blockIdx.x] = loss;
    }
  }
}

// g_pk = sum over the G workgroups of part[g][p][k], in index order within
// sixteen interleaved groups, then the groups in order; EPI applies the update
// (0: x = step g; 1: GD; 2: power iteration with squared-norm partials).
// grid (n / 16 rounded up, nb), 256 threads: 16 columns x 16 groups, so that
// even one signal's 4096 columns put a workgroup on every CU (8 MB of partials
// at 256 workgroups).
template <int EPI>
__global__ void __launch_bounds__(256) dense_rows_update_kernel(const float2* __restrict__ part, int G, int n, int nb,
                                                                float2* __restrict__ x, float step, float lam,
                                                                const float* __restrict__ inv, float* norm_part,
                                                                int norm_ld, unsigned* nf) {
  __shared__ float2 s[16][17];
  const int kk = threadIdx.x & 15, gg = threadIdx.x >> 4;
  const int p = blockIdx.y;
  const int k = blockIdx.x * 16 + kk;
  float2 t = make_float2(0.f, 0.f);
  if (k < n) {
    const float2* q = part + (long long)p * n + k;
    const long long ld = (long long)nb * n;
#pragma unroll 8
    for (int g = gg; g < G; g += 16) t = cadd(t, q[(long long)g * ld]);
  }
  s[gg][kk] = t;
  __syncthreads();
  if (threadIdx.x >= 16) return;
  float2 g = s[0][kk];
#pragma unroll
  for (int i = 1; i < 16; ++i) g = cadd(g, s[i][kk]);
  bool bad = false;
  float nrm = 0.f;
  if (k < n) {
    const long long o = (long long)p * n + k;
    float2 nx;
    if constexpr (EPI == ROWS_STORE) {
      nx = cscale(g, step);
    } else if constexpr (EPI == ROWS_UPDATE_GD) {
      const float2 xo = x[o];
      nx = make_float2(xo.x - step * g.x, xo.y - step * g.y);
      bad = !finite2(nx);
    } else {
      const float2 uo = x[o];
      const float c = 2.f * lam * inv[p];
      nx = make_float2(step * g.x - c * uo.x, step * g.y - c * uo.y);
      nrm = cabs2(nx);
      bad = !finite2(nx);
    }
    x[o] = nx;
  }
  if constexpr (EPI != ROWS_STORE) flag_nonfinite(nf, bad);
  if constexpr (EPI == ROWS_UPDATE_SPEC) {
#pragma unroll
    for (int o = 8; o >= 1; o /= 2) nrm += __shfl_xor(nrm, o, 16);
    if (kk == 0) norm_part[(long long)p * norm_ld + blockIdx.x] = nrm;
  }
}

}  // namespace

namespace {
constexpr int kSmallBatch = 8;
constexpr long long kSmallProduct = 1LL << 22;

// Rows per batch: as many as the registers hold twice beside the signals and
// the partial sums (128 VGPRs at 1024 threads; one row more spills).
constexpr int batch_rows(int T, int J, int NB) {
  return NB == 1 ? (T == 1024 && J == 2 ? 2 : 4) : NB == 2 ? 2 : (T == 1024 ? 1 : 2);
}
}  // namespace

// One to four signals of up to 4096 entries: x and the partial sums of A^H r
// fit a workgroup's registers (16 values each per thread and signal at 1024
// threads).  One GD iteration on 16384 x 4096: 98 / 106 / 142 us for 1 / 2 / 4
// signals against 279-285 us on the matrix cores.  Up to eight go in two
// groups of four where the whole product is small (kSmallProduct) and launches
// and latency, not arithmetic, set the time: 1000 x 258 x 8 12 us against 33.
// The line was drawn when the sums still took twice as long (then 4096 x 1024 x
// 8 53 against 47, and 1000 x 258 x 16, in four groups, 27 against 31 with its A x
// alone no faster).  Longer signals and larger batches stay on the matrix cores.
bool rows_shape(int m, int n, int nb, RowsShape* s) {
  if (nb < 1 || n < 1 || n > 4096) return false;
  if (nb > 4 && (nb > kSmallBatch || (long long)m * n * nb > kSmallProduct)) return false;
  s->NB = nb <= 2 ? nb : 4;
  s->T = n <= 256 ? 64 : n <= 1024 ? 256 : 1024;
  s->J = n <= s->T * 2 ? 1 : 2;
  s->R = batch_rows(s->T, s->J, s->NB);
  // Workgroups: 1024 threads are one a CU.  Smaller ones do little between the
  // loads of one batch and the next, so tall matrices take more of them, some
  // ten rows apiece for one wave and twenty for four (three signals, 512 -> the
  // count here, A x and a GD iteration: 100000 x 100 72.6 and 115 -> 23.7 and 43
  // us, 20000 x 100 16.9 and 27.2 -> 7.0 and 21.0, 100000 x 512 115 and 153 -> 86
  // and 98); fewer rows apiece cost more in partials to sum (2000 x 100 10.4 ->
  // 12.2, 6000 x 512 17.2 -> 18.7), and so do more of the longest signals of four
  // waves (20000 x 1000 42.6 -> 46.0).  A batch's groups share the count (and the
  // partial-sum buffers, which hold 2 m values).
  const int want = s->T == 1024 ? 256
                   : s->T == 64 ? std::clamp(m / 10, 512, 2048)
                   : s->J == 1 ? std::clamp(m / 20, 512, 1024)
                               : 512;
  const int cap = std::max(1, std::min(want, 2 * m / nb));
  const int batches = (m + s->R - 1) / s->R;
  const int per = (batches + cap - 1) / cap;
  s->rows = per * s->R;
  s->G = (m + s->rows - 1) / s->rows;
  return true;
}

namespace {
template <int MODE, int NB, int T, int J>
hipError_t go_threads(const RowsShape& s, const RowsArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((dense_rows_kernel<MODE, NB, T, J, batch_rows(T, J, NB)>), dim3(s.G, (a.nb + NB - 1) / NB), dim3(T), 0,
                     st, a);
  return hipGetLastError();
}

template <int MODE, int NB>
hipError_t go_shape(const RowsShape& s, const RowsArgs& a, hipStream_t st) {
  if (s.T == 64) return s.J == 1 ? go_threads<MODE, NB, 64, 1>(s, a, st) : go_threads<MODE, NB, 64, 2>(s, a, st);
  if (s.T == 256) return s.J == 1 ? go_threads<MODE, NB, 256, 1>(s, a, st) : go_threads<MODE, NB, 256, 2>(s, a, st);
  return s.J == 1 ? go_threads<MODE, NB, 1024, 1>(s, a, st) : go_threads<MODE, NB, 1024, 2>(s, a, st);
}

template <int MODE>
hipError_t go_mode(const RowsShape& s, const RowsArgs& a, hipStream_t st) {
  return s.NB == 1 ? go_shape<MODE, 1>(s, a, st) : s.NB == 2 ? go_shape<MODE, 2>(s, a, st) : go_shape<MODE, 4>(s, a, st);
}
}  // namespace

hipError_t launch_rows(int mode, const RowsShape& s, const RowsArgs& a, hipStream_t st) {
  switch (mode) {
    case ROWS_FWD: return go_mode<ROWS_FWD>(s, a, st);
    case ROWS_ADJ: return go_mode<ROWS_ADJ>(s, a, st);
    case ROWS_GD: return go_mode<ROWS_GD>(s, a, st);
    case ROWS_SPEC: return go_mode<ROWS_SPEC>(s, a, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_rows_update(int epi, const RowsShape& s, const RowsArgs& a, float2* x, float step, float* norm_part,
                              int norm_ld, unsigned* nf, hipStream_t st) {
  const dim3 g(rows_update_groups(a.n), a.nb), b(256);
  switch (epi) {
    case ROWS_STORE:
      hipLaunchKernelGGL((dense_rows_update_kernel<ROWS_STORE>), g, b, 0, st, a.part, s.G, a.n, a.nb, x, step, a.lam,
                         a.inv, norm_part, norm_ld, nf);
      break;
    case ROWS_UPDATE_GD:
      hipLaunchKernelGGL((dense_rows_update_kernel<ROWS_UPDATE_GD>), g, b, 0, st, a.part, s.G, a.n, a.nb, x, step,
                         a.lam, a.inv, norm_part, norm_ld, nf);
      break;
    case ROWS_UPDATE_SPEC:
      hipLaunchKernelGGL((dense_rows_update_kernel<ROWS_UPDATE_SPEC>), g, b, 0, st, a.part, s.G, a.n, a.nb, x, step,
                         a.lam, a.inv, norm_part, norm_ld, nf);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace sr
