// The dense model's real products (see dense.hip) on v_mfma_f32_16x16x32_bf16
// with FP32's accuracy.
//
// Each FP32 operand is the sum of three bf16 numbers (its rounding to bf16,
// the rounding of what that leaves, and the rest, which eight bits hold
// exactly); the six products of parts whose orders add up to at most two are
// accumulated in FP32.  The parts left out are below 2^-25 of a product, under
// the rounding of an FP32 product, and a step adds 32 products with one
// rounding, so the error is below that of the FP32 products, which add four at
// a time.
//
// FP32 matrix cores take 109 us for 16384 x 4096 x 32 at their peak, about
// what A's 537 MB take from HBM (106 us), and reach 0.7 of it; six bf16
// products take 41 us at theirs, which leaves the stream of A as the bound.
// A goes from memory to the registers that the matrix cores read, with no LDS
// in between, since both products let a lane load what its fragments hold:
// eight entries of a row (A X; two groups of four, so that a load covers 64
// consecutive bytes of each row), or four consecutive columns of eight rows
// (A^H R, whose four columns go to four column-permuted tiles).  It is split
// there.  The small operand is split once by a pack kernel, in fragment order,
// and staged through LDS for the workgroup's four waves.  A wave holds a 64 x
// 64 tile; two workgroups a CU, from reduction splits where the tiles are
// fewer.  The row tiles of A X start at steps of their own: rows lie a power
// of two of bytes apart in the shapes of use, and all tiles at one column would
// meet on the same few memory channels (the product alone 155 us then).
//
// Measured (16384 x 4096 on 32 signals, A X and A^H R): the products 123 to 137
// and 122 us, 3.9 to 4.4 TB/s of A; with packing and epilogue 141 to 144 and 127
// to 130 us; the library's FP32 product 158 and 171 us, dense_mm_kernel 212 and
// 230 us.  Error against 64 bits 5.1e-7 and 5.3e-7; the library 1.6e-6 and
// 2.3e-6, dense_mm_kernel 8.1e-7 and 8.1e-7.
#include "dense_bf16.hpp"

#include <algorithm>

#include "fft_core.hpp"

namespace sr {

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));

constexpr int kStep = 32;             // reduction per step (one fragment)
constexpr int kFragBytes = 64 * 16;   // one fragment: 16 bytes a lane
constexpr int kStepBytes = 12 * kFragBytes;  // small operand per step: 4 tiles of 16 x 3 parts

// 2^16 v = p[0] + p[1] + p[2], eight entries at a time.  (The matrix cores take
// bf16 denormals as zeros: without the factor the parts of entries below 2^-110
// would lose bits.)
__device__ __forceinline__ void split8(const float (&v)[8], b8 (&p)[3]) {
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    v2f r = {v[e] * kBf16Scale, v[e + 1] * kBf16Scale};
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const b2 h = __builtin_convertvector(r, b2);
      p[s][e] = h[0];
      p[s][e + 1] = h[1];
      if (s < 2) {
        r[0] -= (float)h[0];
        r[1] -= (float)h[1];
      }
    }
  }
}

// Fragments of the small operand: pack[((tile * steps + ks) * 4 + t16) * 3 +
// part][lane] = its entries (k = 32 ks + 8 (lane / 16) + e, q = 16 t16 + lane
// % 16), e = 0..7.  One thread per (tile, ks, t16, lane).
template <int G>
__global__ void __launch_bounds__(256) bf16_pack_kernel(const Bf16Gemm a, int steps, int tiles) {
  const long long id = blockIdx.x * 256ll + threadIdx.x;
  const int lane = (int)(id & 63), t16 = (int)(id >> 6) & 3;
  const long long ts = id >> 8;
  const int ks = (int)(ts % steps), tile = (int)(ts / steps);
  if (tile >= tiles) return;
  const int K = G == 1 ? 2 * a.n : a.m;
  const int q = 16 * t16 + (lane & 15), p = tile * 32 + q / 2, c = q & 1;
  const int k0 = ks * kStep + 8 * (lane >> 4);
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = 0.f;
  if (p < a.nb) {
    const float sc = a.src_scale != nullptr ? a.src_scale[p] : 1.f;
    if constexpr (G == 1) {
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const int k = ks * kStep + 16 * (e >> 2) + 4 * (lane >> 4) + (e & 3);
        if (k < K) {
          const float2 x = cscale(a.src[(long long)p * a.n + k / 2], sc);
          v[e] = c ? x.y : x.x;
          v[e + 1] = c ? x.x : -x.y;
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (k0 + e < K) {
          const float2 r = cscale(a.src[(long long)p * a.m + k0 + e], sc);
          v[e] = c ? r.y : r.x;
        }
      }
    }
  }
  b8 s[3];
  split8(v, s);
  b8* out = reinterpret_cast<b8*>(a.pack) + (ts * 4 + t16) * 3 * 64 + lane;
#pragma unroll
  for (int i = 0; i < 3; ++i) out[i * 64] = s[i];
}

// grid: x = (big tiles of 256) x S, splits fastest; y = signal tiles.
template <int G>
__global__ void __launch_bounds__(256, 2) bf16_gemm_kernel(const Bf16Gemm a, int S, int steps, int all_steps) {
  __shared__ __attribute__((aligned(16))) unsigned char bs[2][kStepBytes];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, l16 = lane & 15;
  const int s = blockIdx.x % S;
  const int o0 = (blockIdx.x / S) * 256 + wave * 64;  // the wave's first row (G 1) or column (G 2) of A
  const int lda = 2 * a.n;
  const int M = G == 1 ? a.m : lda, K = G == 1 ? lda : a.m;
  const int ks0 = s * steps, ks1 = min(all_steps, ks0 + steps);
  const unsigned char* pk = (const unsigned char*)a.pack + ((long long)blockIdx.y * all_steps) * kStepBytes;

  f4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};

  // this lane's part of A for one step: G 1: rows o0 + 16 t + l16, entries
  // 32 ks + 8 g + 0..7; G 2: rows 32 ks + 8 g + e, columns o0 + 4 l16 + 0..3
  f4 cur[8], nxt[8];
  auto load_a = [&](f4(&d)[8], int ks) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int row = G == 1 ? o0 + 16 * (u >> 1) + l16 : ks * kStep + 8 * g + u;
      const int col = G == 1 ? ks * kStep + 16 * (u & 1) + 4 * g : o0 + 4 * l16;
      d[u] = f4{0.f, 0.f, 0.f, 0.f};
      if (row < a.m && col < lda && ks < ks1) d[u] = *reinterpret_cast<const f4*>(a.A + (long long)row * lda + col);
    }
  };
  f4 breg[3];
  auto load_b = [&](int ks) {
    if (ks < ks1) {
#pragma unroll
      for (int u = 0; u < 3; ++u)
        breg[u] = *reinterpret_cast<const f4*>(pk + (long long)ks * kStepBytes + (u * 256 + tid) * 16);
    }
  };
  auto store_b = [&](int buf) {
#pragma unroll
    for (int u = 0; u < 3; ++u) *reinterpret_cast<f4*>(&bs[buf][(u * 256 + tid) * 16]) = breg[u];
  };

  if (ks0 < ks1) {
    // the steps in turn, from a start of the row tile's own
    const int cnt = ks1 - ks0, rot = G == 1 ? (int)((blockIdx.x / S) % cnt) : 0;
    auto at = [&](int j) { return j < cnt ? ks0 + (j + rot < cnt ? j + rot : j + rot - cnt) : ks1; };
    load_b(at(0));
    load_a(cur, at(0));
    store_b(0);
    load_b(at(1));
    __syncthreads();
    int buf = 0;
    for (int j = 0; j < cnt; ++j, buf ^= 1) {
      load_a(nxt, at(j + 1));
      b8 bf[4][3];
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int p = 0; p < 3; ++p)
          bf[t][p] = *reinterpret_cast<const b8*>(&bs[buf][(t * 3 + p) * kFragBytes + lane * 16]);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = G == 1 ? cur[2 * t + (e >> 2)][e & 3] : cur[e][t];
        b8 af[3];
        split8(v, af);
        // smallest products first
#pragma unroll
        for (int o = 2; o >= 0; --o)
#pragma unroll
          for (int i = 0; i <= o; ++i)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              if constexpr (G == 1)
                acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf[u][o - i], acc[t][u], 0, 0, 0);
              else
                acc[u][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[u][o - i], af[i], acc[u][t], 0, 0, 0);
            }
      }
      store_b(buf ^ 1);
      load_b(at(j + 2));
      __syncthreads();
#pragma unroll
      for (int u = 0; u < 8; ++u) cur[u] = nxt[u];
    }
  }

  // D[4 g + r][l16] of each 16 x 16 tile
  const int q0 = 64 * blockIdx.y;
  if constexpr (G == 1) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = o0 + 16 * t + 4 * g + r;
        if (row < M) {
#pragma unroll
          for (int u = 0; u < 4; ++u)
            a.split[((long long)s * a.m + row) * a.q_ld + q0 + 16 * u + l16] = acc[t][u][r];
        }
      }
  } else {
    const int col = o0 + 4 * l16;
    if (col < M) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          *reinterpret_cast<f4*>(&a.split[((long long)s * a.q_ld + q0 + 16 * u + 4 * g + r) * lda + col]) =
              f4{acc[u][0][r], acc[u][1][r], acc[u][2][r], acc[u][3][r]};
    }
  }
}

constexpr int kTargetGroups = 512;  // two workgroups per CU
constexpr int kMaxSplits = 16;      // the epilogues sum at most this many partials

int steps_of(int G, int m, int n) { return ((G == 1 ? 2 * n : m) + kStep - 1) / kStep; }
int signal_tiles(int nb) { return (nb + 31) / 32; }

}  // namespace

int bf16_splits(int G, int m, int n, int nb, int* steps) {
  const int all = steps_of(G, m, n);
  const int tiles = ((G == 1 ? m : 2 * n) + 255) / 256 * signal_tiles(nb);
  // rounded down: a few workgroups past the last full round cost a whole one
  // (12913 x 2780 x 24, A X: 51 tiles in 11 splits 109 us, in 8 89 us)
  const int want = std::max(1, std::min(std::min(all, kMaxSplits), kTargetGroups / tiles));
  *steps = (all + want - 1) / want;
  return (all + *steps - 1) / *steps;
}

size_t bf16_pack_bytes(int m, int n, int nb) {
  return (size_t)signal_tiles(nb) * (size_t)std::max(steps_of(1, m, n), steps_of(2, m, n)) * kStepBytes;
}

hipError_t launch_bf16_gemm(int G, const Bf16Gemm& a, hipStream_t st) {
  int steps;
  const int S = bf16_splits(G, a.m, a.n, a.nb, &steps);
  const int all = steps_of(G, a.m, a.n), tiles = signal_tiles(a.nb);
  const int big = ((G == 1 ? a.m : 2 * a.n) + 255) / 256;
  const dim3 pg((unsigned)((long long)all * tiles)), gg((unsigned)(big * S), (unsigned)tiles), b(256);
  if (G == 1) {
    hipLaunchKernelGGL((bf16_pack_kernel<1>), pg, b, 0, st, a, all, tiles);
    hipLaunchKernelGGL((bf16_gemm_kernel<1>), gg, b, 0, st, a, S, steps, all);
  } else {
    hipLaunchKernelGGL((bf16_pack_kernel<2>), pg, b, 0, st, a, all, tiles);
    hipLaunchKernelGGL((bf16_gemm_kernel<2>), gg, b, 0, st, a, S, steps, all);
  }
  return hipGetLastError();
}

}  // namespace sr
