// Device-side FFT core for gfx950: complex helpers, radix butterflies and a
// register/LDS Stockham transform over a tile of B independent length-N
// transforms.
//
// Layout contract ("canonical" register layout): the ACT = N/E active threads
// of one transform each hold E elements; thread t holds elements k = t + j*ACT,
// j = 0..E-1.  (A transform is allocated TPT threads; TPT = ACT except for the
// split shapes of the lengths with a factor of three.)  Both the input and the output of `Tile::fft` use this layout,
// so that pointwise work between two transforms (phase diagonals, epilogues)
// happens in registers, and global loads/stores along a contiguous axis are
// coalesced.
//
// Each radix-R Stockham stage (span p = product of the previous radices)
// takes inputs at i + r*N/R, i = t + q*TPT, multiplies by the twiddles
// w^(r*k) with k = i mod p and w = exp(-+2 pi i/(p R)), applies the R-point
// DFT and writes output r to (i div p)*p*R + k + r*p.  Intermediate stages
// exchange through LDS (ping-pong buffers, one barrier per stage); the last
// stage's outputs land back in canonical order.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>
#include <stdint.h>

namespace sr {

// ----------------------------------------------------------- complex helpers
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// a * conj(b)
__device__ __forceinline__ float2 cmulc(float2 a, float2 b) {
  return make_float2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
__device__ __forceinline__ float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
__device__ __forceinline__ float cabs2(float2 a) { return a.x * a.x + a.y * a.y; }
__device__ __forceinline__ float2 cconj(float2 a) { return make_float2(a.x, -a.y); }
// multiply by -i (forward quarter turn) or +i (inverse quarter turn)
template <bool INV>
__device__ __forceinline__ float2 quarter(float2 a) {
  return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}
// e^{i theta} scaled by s, with an optional conjugate
template <bool CONJ>
__device__ __forceinline__ float2 phase(float theta, float s) {
  float sn, cs;
  sincosf(theta, &sn, &cs);
  return make_float2(cs * s, CONJ ? -sn * s : sn * s);
}

// e^{i theta} from the hardware sine and cosine, which take their argument in
// turns: theta / (2 pi) reduced to [0, 1) first.  Absolute error about 5e-7
// (against 7e-8 for sincosf) for a few instructions instead of a full range
// reduction; used where the pass kernels evaluate the phase diagonals on the
// fly (the exp(i theta) tables are filled with sincosf).
__device__ __forceinline__ float2 phase_turns(float theta) {
  const float r = __builtin_amdgcn_fractf(theta * 0.159154943091895335768883763372514362f);
  return make_float2(__builtin_amdgcn_cosf(r), __builtin_amdgcn_sinf(r));
}

// e^{i theta} from polynomials, close to sincosf's accuracy (3.6e-8 rms, 1.5e-7
// at most over [0, 2 pi); sincosf 2.1e-8 rms): theta less the nearest multiple
// of pi (in two parts, so that the difference keeps its last bits), sine and
// cosine on [-pi/2, pi/2] by polynomials of least maximum absolute error there
// (the leading terms x and 1 - z/2 fixed, the other four coefficients by
// reweighted least squares; 4.6e-9 and 4e-10, with the coefficients rounded to
// float 1.5e-8 and 6.3e-9), and the sign of the multiple.  About twice the issue time of the hardware pair; for kernels
// where a table's memory traffic costs more than that.  The error stays there
// up to kPhasePolyMax (1.7e-7 at most); from some 10^6 on the multiple itself
// loses bits (2.8e-6 at 4 x 10^6, no phase at all at 10^8).
constexpr float kPhasePolyMax = 131072.f;
__device__ __forceinline__ float2 phase_poly(float theta) {
  constexpr double kPi = 3.141592653589793238462643383279502884;
  constexpr float kHi = (float)kPi, kLo = (float)(kPi - (double)kHi);
  const float q = __builtin_rintf(theta * (float)(1.0 / kPi));
  const float x = __builtin_fmaf(q, -kLo, __builtin_fmaf(q, -kHi, theta));
  const float z = x * x;
  float s = __builtin_fmaf(z, 2.59990315e-06f, -1.98065478e-04f);
  s = __builtin_fmaf(z, s, 8.33301619e-03f);
  s = __builtin_fmaf(z, s, -1.66666567e-01f);
  s = __builtin_fmaf(x * z, s, x);
  float c = __builtin_fmaf(z, -2.61924839e-07f, 2.47692405e-05f);
  c = __builtin_fmaf(z, c, -1.38885679e-03f);
  c = __builtin_fmaf(z, c, 4.16666567e-02f);
  c = __builtin_fmaf(z, c, -0.5f);
  c = __builtin_fmaf(z, c, 1.f);
  const unsigned sign = (unsigned)(int)q << 31;
  return make_float2(__builtin_bit_cast(float, __builtin_bit_cast(unsigned, c) ^ sign),
                     __builtin_bit_cast(float, __builtin_bit_cast(unsigned, s) ^ sign));
}

// Deterministic workgroup sum: a fixed shuffle tree inside each wave, lane
// 0's total broadcast to the wave, then the wave totals added in wave order.
// Every thread gets the same value.  NTHREADS equals blockDim.x and is a whole
// number of waves, or a power of two below one; `red` holds at least NTHREADS /
// 64 values.
template <int NTHREADS, class V>
__device__ __forceinline__ V block_sum_t(V v, V* red) {
  constexpr int W = NTHREADS < 64 ? NTHREADS : 64;
  constexpr int NW = NTHREADS / W;
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) v += __shfl_down(v, o, W);
  v = __shfl(v, 0, W);
  if constexpr (NW == 1) {
    return v;
  } else {
    __syncthreads();  // `red` may still be read by an earlier call
    if ((threadIdx.x & (W - 1)) == 0) red[threadIdx.x / W] = v;
    __syncthreads();
    V s = red[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) s += red[i];
    return s;
  }
}

// Sum of part[0..n) over one wavefront, in every lane: strided per-lane sums in
// index order, then block_sum_t's tree, so the order is fixed.  The reductions
// of per-workgroup partials use it; one thread adding them in turn waits for
// each load (14.5 us for 384 partials, 2.5 us this way).
template <class V>
__device__ __forceinline__ double wave_sum_of(const V* __restrict__ part, int n) {
  double acc = 0.0;
  for (int i = threadIdx.x & 63; i < n; i += 64) acc += (double)part[i];
  return block_sum_t<64, double>(acc, nullptr);
}

template <int NTHREADS>
__device__ __forceinline__ float block_sum(float v, float* red) {
  return block_sum_t<NTHREADS, float>(v, red);
}

// Workgroup index -> tile index such that consecutive tiles run on the same
// XCD.  Workgroups are dispatched to the 8 XCDs round-robin (bid mod 8), each
// with its own L2; tiles that share cache lines (adjacent column tiles) then
// hit the same L2 instead of each XCD fetching the full line.  Bijective on
// [0, G) for any G.
constexpr int kNumXcd = 8;
__device__ __forceinline__ int xcd_tile(int bid, int G) {
  const int q = G / kNumXcd, r = G % kNumXcd, x = bid % kNumXcd, l = bid / kNumXcd;
  return x < r ? x * (q + 1) + l : r * (q + 1) + (x - r) * q + l;
}

// ------------------------------------------------------- buffer memory ops
// Global loads and stores through buffer resources.  A lane whose element
// lies outside its window passes an offset past the resource's range, so the
// hardware returns zero (loads) or drops the write (stores) without a branch;
// offsets are 32-bit byte offsets from a wave-uniform base (every buffer a
// pass touches spans well under 2 GiB).
using Rsrc = __amdgpu_buffer_rsrc_t;
constexpr unsigned kOob = 0x80000000u;  // byte offset past every resource
__device__ __forceinline__ Rsrc rsrc(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, 0x7fffffff, 0x00020000);
}
// Each access takes a lane offset and a scalar offset (added by the memory
// pipeline, outside the range check), so that a thread's elements at a fixed
// stride share one lane offset and cost no address arithmetic apiece.
__device__ __forceinline__ float2 ld2(Rsrc r, unsigned off, unsigned soff) {
  const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 0);
  return make_float2(__builtin_bit_cast(float, (unsigned)v[0]), __builtin_bit_cast(float, (unsigned)v[1]));
}
__device__ __forceinline__ float ld1(Rsrc r, unsigned off, unsigned soff) {
  return __builtin_bit_cast(float, (unsigned)__builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0));
}
__device__ __forceinline__ void st2(Rsrc r, unsigned off, unsigned soff, float2 x) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  u32x2 v;
  v[0] = __builtin_bit_cast(unsigned, x.x);
  v[1] = __builtin_bit_cast(unsigned, x.y);
  __builtin_amdgcn_raw_buffer_store_b64(v, r, off, soff, 0);
}
__device__ __forceinline__ void st1(Rsrc r, unsigned off, unsigned soff, float x) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), r, off, soff, 0);
}

// ------------------------------------------------------- non-finite values
// True unless v is NaN or +-Inf (the comparison fails for NaN).
__device__ __forceinline__ bool finite2(float2 v) {
  return fabsf(v.x) <= 3.402823466e38f && fabsf(v.y) <= 3.402823466e38f;
}

// Raise the non-finite flag from the lanes that met one: a vector store of
// the same value from every such lane (no read-modify-write needed).
__device__ __forceinline__ void flag_nonfinite(unsigned* nf, bool bad) {
  if (nf != nullptr && bad)
    __builtin_amdgcn_raw_buffer_store_b32(1u, __builtin_amdgcn_make_buffer_rsrc(nf, (short)0, 4, 0x00020000), 0u, 0, 0);
}

// --------------------------------------------------------------- butterflies
// In-place R-point DFT, y_k = sum_j u_j w^(jk), w = exp(-2 pi i/R) (forward)
// or exp(+2 pi i/R) (INV).  No scaling.
template <int R, bool INV>
struct Dft;

template <bool INV>
struct Dft<2, INV> {
  __device__ __forceinline__ static void run(float2* u) {
    float2 a = u[0], b = u[1];
    u[0] = cadd(a, b);
    u[1] = csub(a, b);
  }
};

template <bool INV>
struct Dft<3, INV> {
  __device__ __forceinline__ static void run(float2* u) {
    const float h = 0.866025403784438646763723170752936183f;  // sqrt(3)/2
    float2 s = cadd(u[1], u[2]);
    float2 d = csub(u[1], u[2]);
    float2 m = make_float2(u[0].x - 0.5f * s.x, u[0].y - 0.5f * s.y);
    float2 q = cscale(quarter<INV>(d), h);  // -+ i sqrt(3)/2 (u1 - u2)
    u[0] = cadd(u[0], s);
    u[1] = cadd(m, q);
    u[2] = csub(m, q);
  }
};

template <bool INV>
struct Dft<4, INV> {
  __device__ __forceinline__ static void run(float2* u) {
    float2 t0 = cadd(u[0], u[2]);
    float2 t1 = csub(u[0], u[2]);
    float2 t2 = cadd(u[1], u[3]);
    float2 t3 = quarter<INV>(csub(u[1], u[3]));
    u[0] = cadd(t0, t2);
    u[2] = csub(t0, t2);
    u[1] = cadd(t1, t3);
    u[3] = csub(t1, t3);
  }
};

template <bool INV>
struct Dft<8, INV> {
  __device__ __forceinline__ static void run(float2* u) {
    const float c = 0.707106781186547524400844362104849039f;  // sqrt(2)/2
    float2 e[4] = {u[0], u[2], u[4], u[6]};
    float2 o[4] = {u[1], u[3], u[5], u[7]};
    Dft<4, INV>::run(e);
    Dft<4, INV>::run(o);
    // w8^1 = (c, -+c), w8^2 = -+i, w8^3 = (-c, -+c)
    float2 o1 = INV ? make_float2(c * (o[1].x - o[1].y), c * (o[1].x + o[1].y))
                    : make_float2(c * (o[1].x + o[1].y), c * (o[1].y - o[1].x));
    float2 o2 = quarter<INV>(o[2]);
    float2 o3 = INV ? make_float2(-c * (o[3].x + o[3].y), c * (o[3].x - o[3].y))
                    : make_float2(c * (o[3].y - o[3].x), -c * (o[3].x + o[3].y));
    u[0] = cadd(e[0], o[0]);
    u[4] = csub(e[0], o[0]);
    u[1] = cadd(e[1], o1);
    u[5] = csub(e[1], o1);
    u[2] = cadd(e[2], o2);
    u[6] = csub(e[2], o2);
    u[3] = cadd(e[3], o3);
    u[7] = csub(e[3], o3);
  }
};

// 16 = 4 x 4: index n = 4 n1 + n2 in, k = k1 + 4 k2 out; four 4-point DFTs
// over n1, the twiddles w16^(n2 k1), four 4-point DFTs over n2.
template <bool INV>
struct Dft<16, INV> {
  __device__ __forceinline__ static void run(float2* u) {
    const float c1 = 0.923879532511286756128183189396788933f;  // cos(pi/8)
    const float s1 = 0.382683432365089771728459984030398866f;  // sin(pi/8)
    const float h = 0.707106781186547524400844362104849039f;   // cos(pi/4)
    float2 a[4][4];
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2) {
      float2 t[4] = {u[n2], u[4 + n2], u[8 + n2], u[12 + n2]};
      Dft<4, INV>::run(t);
#pragma unroll
      for (int k1 = 0; k1 < 4; ++k1) a[n2][k1] = t[k1];
    }
    // forward w16^j = (cos(2 pi j/16), -sin(2 pi j/16)); the inverse conjugates
    auto tw = [](float2 v, float re, float im) { return INV ? cmulc(v, make_float2(re, im)) : cmul(v, make_float2(re, im)); };
    a[1][1] = tw(a[1][1], c1, -s1);  // j = 1
    a[1][2] = tw(a[1][2], h, -h);    // j = 2
    a[1][3] = tw(a[1][3], s1, -c1);  // j = 3
    a[2][1] = tw(a[2][1], h, -h);    // j = 2
    a[2][2] = quarter<INV>(a[2][2]); // j = 4
    a[2][3] = tw(a[2][3], -h, -h);   // j = 6
    a[3][1] = tw(a[3][1], s1, -c1);  // j = 3
    a[3][2] = tw(a[3][2], -h, -h);   // j = 6
    a[3][3] = tw(a[3][3], -c1, s1);  // j = 9
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) {
      float2 t[4] = {a[0][k1], a[1][k1], a[2][k1], a[3][k1]};
      Dft<4, INV>::run(t);
#pragma unroll
      for (int k2 = 0; k2 < 4; ++k2) u[k1 + 4 * k2] = t[k2];
    }
  }
};

// 6 = 2 x 3 with coprime factors, so no twiddles between them: index
// n = 3 n1 + 2 n2 (mod 6) in, k = 3 k1 + 4 k2 (mod 6) out (the Chinese
// remainder map); three 2-point DFTs over n1, two 3-point DFTs over n2.
template <bool INV>
struct Dft<6, INV> {
  __device__ __forceinline__ static void run(float2* u) {
    float2 a[3][2];
#pragma unroll
    for (int n2 = 0; n2 < 3; ++n2) {
      const float2 x = u[(2 * n2) % 6], y = u[(3 + 2 * n2) % 6];
      a[n2][0] = cadd(x, y);
      a[n2][1] = csub(x, y);
    }
#pragma unroll
    for (int k1 = 0; k1 < 2; ++k1) {
      float2 t[3] = {a[0][k1], a[1][k1], a[2][k1]};
      Dft<3, INV>::run(t);
#pragma unroll
      for (int k2 = 0; k2 < 3; ++k2) u[(3 * k1 + 4 * k2) % 6] = t[k2];
    }
  }
};

// 12 = 3 x 4 with coprime factors, so no twiddles between them: index
// n = 4 n1 + 3 n2 (mod 12) in, k = 4 k1 + 9 k2 (mod 12) out (the Chinese
// remainder map); four 3-point DFTs over n1, three 4-point DFTs over n2.
template <bool INV>
struct Dft<12, INV> {
  __device__ __forceinline__ static void run(float2* u) {
    float2 a[4][3];
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2) {
      float2 t[3] = {u[(3 * n2) % 12], u[(4 + 3 * n2) % 12], u[(8 + 3 * n2) % 12]};
      Dft<3, INV>::run(t);
#pragma unroll
      for (int k1 = 0; k1 < 3; ++k1) a[n2][k1] = t[k1];
    }
#pragma unroll
    for (int k1 = 0; k1 < 3; ++k1) {
      float2 t[4] = {a[0][k1], a[1][k1], a[2][k1], a[3][k1]};
      Dft<4, INV>::run(t);
#pragma unroll
      for (int k2 = 0; k2 < 4; ++k2) u[(4 * k1 + 9 * k2) % 12] = t[k2];
    }
  }
};

// ------------------------------------------------------------- radix lists
template <int... Rs>
struct RadixList {
  static constexpr int count = sizeof...(Rs);
  static constexpr int values[count] = {Rs...};
  static constexpr int product() {
    int p = 1;
    for (int i = 0; i < count; ++i) p *= values[i];
    return p;
  }
  static constexpr int span(int s) {  // product of the first s radices
    int p = 1;
    for (int i = 0; i < s; ++i) p *= values[i];
    return p;
  }
};

// Factorisation and elements-per-thread for each supported length.
template <int N>
struct FftShape;
template <> struct FftShape<16>   { static constexpr int E = 4;  using R = RadixList<4, 4>; };
template <> struct FftShape<32>   { static constexpr int E = 8;  using R = RadixList<8, 4>; };
template <> struct FftShape<64>   { static constexpr int E = 8;  using R = RadixList<8, 8>; };
template <> struct FftShape<128>  { static constexpr int E = 8;  using R = RadixList<8, 4, 4>; };
template <> struct FftShape<256>  { static constexpr int E = 8;  using R = RadixList<8, 8, 4>; };
template <> struct FftShape<512>  { static constexpr int E = 8;  using R = RadixList<8, 8, 8>; };
template <> struct FftShape<1024> { static constexpr int E = 8;  using R = RadixList<8, 8, 4, 4>; };
template <> struct FftShape<2048> { static constexpr int E = 8;  using R = RadixList<8, 8, 8, 4>; };
template <> struct FftShape<4096> { static constexpr int E = 8;  using R = RadixList<8, 8, 8, 8>; };
template <> struct FftShape<24>   { static constexpr int E = 12; using R = RadixList<3, 4, 2>; };
template <> struct FftShape<48>   { static constexpr int E = 12; using R = RadixList<3, 4, 4>; };
template <> struct FftShape<96>   { static constexpr int E = 12; using R = RadixList<12, 4, 2>; };
template <> struct FftShape<192>  { static constexpr int E = 12; using R = RadixList<12, 4, 4>; };
template <> struct FftShape<384>  { static constexpr int E = 12; using R = RadixList<12, 4, 4, 2>; };
template <> struct FftShape<768>  { static constexpr int E = 12; using R = RadixList<12, 4, 4, 4>; };

// Narrow variant of the power-of-two lengths: four elements per thread
// (radix-4 stages, one radix-2 stage for odd powers), i.e. twice the threads
// per transform.  It costs more LDS exchanges but halves each wave's serial
// arithmetic, which pays when a pass has too few transforms to give every
// SIMD of the chip a wave of the default shape.
template <int N>
struct FftNarrow;
template <> struct FftNarrow<64>   { using R = RadixList<4, 4, 4>; };
template <> struct FftNarrow<128>  { using R = RadixList<4, 4, 4, 2>; };
template <> struct FftNarrow<256>  { using R = RadixList<4, 4, 4, 4>; };
template <> struct FftNarrow<512>  { using R = RadixList<4, 4, 4, 4, 2>; };
template <> struct FftNarrow<1024> { using R = RadixList<4, 4, 4, 4, 4>; };
// Split shapes of the lengths with a factor of three: N/8 threads hold eight
// elements each for the loads, the stores and the first and last stages, and
// the stage between them, whose radix takes the factor of three, spreads its
// butterflies over the power of two of threads (T) that the transform is
// allocated.  Three stages, and as few registers as the powers of two: twelve
// elements per thread throughout take four or five stages, half the threads
// and up to 36 twiddles each, and a length of 384 or 768 then has as few
// waves and as long a chain a wave as a power of two twice as long (768 x 384
// grid, [F D F] row pass: 8.3 us in radices 3, 4, 4, 4, 2 with twelve
// elements, 4.6 us this way).
template <int N> struct FftSplit { static constexpr bool value = false; };
template <> struct FftSplit<96>  { static constexpr bool value = true; static constexpr int T = 16;  using R = RadixList<8, 3, 4>; };
template <> struct FftSplit<192> { static constexpr bool value = true; static constexpr int T = 32;  using R = RadixList<8, 3, 8>; };
template <> struct FftSplit<384> { static constexpr bool value = true; static constexpr int T = 64;  using R = RadixList<8, 6, 8>; };
template <> struct FftSplit<768> { static constexpr bool value = true; static constexpr int T = 128; using R = RadixList<8, 12, 8>; };

// Wide thread shape: sixteen elements per thread with radix-16 stages, for
// column tiles of eight 2048-point transforms in 1024 threads.
template <int N> struct FftWide;
template <> struct FftWide<2048> { using R = RadixList<16, 16, 8>; };
template <int N> struct HasWide { static constexpr bool value = false; };
template <> struct HasWide<2048> { static constexpr bool value = true; };
template <int N> struct HasNarrow { static constexpr bool value = false; };
template <> struct HasNarrow<64> { static constexpr bool value = true; };
template <> struct HasNarrow<128> { static constexpr bool value = true; };
template <> struct HasNarrow<256> { static constexpr bool value = true; };
template <> struct HasNarrow<512> { static constexpr bool value = true; };
template <> struct HasNarrow<1024> { static constexpr bool value = true; };

// ------------------------------------------------------------------- tile
// A tile of B transforms of length N.  COL selects the thread mapping used for
// column-mode tiles: lane = t*B + b (consecutive lanes walk the batch, which is
// the contiguous direction in memory) with LDS layout [k][b]; otherwise
// lane = b*TPT + t with LDS layout [b][k + pad].  DB: ping-pong LDS buffers
// (one barrier per stage) or a single buffer (half the LDS, two barriers per
// stage) -- the single buffer lets two large column tiles share a CU.
template <int N, int B, bool COL, bool DB = true, int E_ = FftShape<N>::E, class RL = typename FftShape<N>::R,
          int T_ = N / E_>
struct Tile {
  static constexpr int E = E_;
  static constexpr int TPT = T_;     // threads allocated to one transform
  static constexpr int ACT = N / E;  // threads that hold elements of it
  static constexpr int THREADS = TPT * B;
  // One pad slot every R0 elements for radix-8- or radix-4-first lengths:
  // the stage-0 scatter (stride R0) would otherwise put lanes on one LDS
  // bank pair.  Radix-12-first lengths take one every 32, which spreads both
  // that scatter and the later stages' reads (768 points as rows: 208 LDS
  // cycles a wave for all exchanges by bank count, 248 without pads, 264 and
  // 288 with one every 4 or 8).
  static constexpr int PADSHIFT = RL::values[0] == 16   ? 4
                                  : RL::values[0] == 12 ? 5
                                  : RL::values[0] == 8  ? 3
                                  : (RL::values[0] == 4 && E_ == 4) ? 2 : 0;
  static constexpr int NP = PADSHIFT ? N + (N >> PADSHIFT) : N;  // padded transform length
  static constexpr int LD = NP;               // row-mode LDS stride
  static constexpr int BUF = B * NP;          // complex elements per LDS buffer
  static constexpr int NBUF = DB ? 2 : 1;     // LDS buffers (elements: NBUF * BUF)
  static_assert(N % E == 0, "E must divide N");
  static_assert(RL::product() == N, "radix list must multiply to N");

  __device__ __forceinline__ static int padk(int k) { return PADSHIFT ? k + (k >> PADSHIFT) : k; }
  __device__ __forceinline__ static int lidx(int b, int k) { return COL ? (padk(k) * B + b) : (b * LD + padk(k)); }
  // lidx(b, k + C) from at = lidx(b, k), for a constant C.  Where C is a whole
  // number of pad periods the sum is a constant too, which goes into the LDS
  // instruction (SHIFTS).  That saves instructions, but of accesses at constant
  // distances the compiler merges two into one, which makes rows of 128 to 1024
  // and of 4096 points wait longer for their exchanges than they save: 1000
  // one-dimensional solves of 1024 points 850 us with, 780 us without; 60 GD
  // iterations on 1024 x 1024 2380 and 2303, 16 of 512 x 512 3246 and 3209 (one
  // 512 x 512 by itself, 200 iterations, 3673 and 3695: a wave to a SIMD pays
  // for the instructions instead).
  // Columns (2048 x 2048, 129 -> 122 us an iteration), rows of 2048 points and the
  // split shapes (768 x 384, 1314 us without, 1283 with) gain, short rows are as
  // fast either way.
  static constexpr bool SHIFTS = COL || N % 3 == 0 || N <= 64 || N == 2048;
  template <int C>
  static constexpr bool shifts_whole() {
    return SHIFTS && (PADSHIFT == 0 || C % (1 << PADSHIFT) == 0);
  }
  template <int C>
  static constexpr int shift_of() {
    return (PADSHIFT ? C + (C >> PADSHIFT) : C) * (COL ? B : 1);
  }
  __device__ __forceinline__ static int thread_t() { return COL ? (int)(threadIdx.x / B) : (int)(threadIdx.x % TPT); }
  __device__ __forceinline__ static int thread_b() { return COL ? (int)(threadIdx.x % B) : (int)(threadIdx.x / TPT); }
  __device__ __forceinline__ static int elem(int t, int j) { return t + j * ACT; }
  // Whether thread t holds elements (the callers give the others zeros and
  // drop their results).
  __device__ __forceinline__ static bool holds(int t) { return ACT == TPT || t < ACT; }

  // Stage S: butterflies per thread, and the threads that have them.  The
  // first and last stages work on the canonical layout, the others on what
  // the exchanges through LDS hand them.
  static constexpr bool canonical(int S) { return S == 0 || S + 1 == RL::count; }
  static constexpr int stage_q(int S) {
    return canonical(S) ? E / RL::values[S] : (N / RL::values[S] + TPT - 1) / TPT;
  }
  static constexpr int stage_act(int S) { return N / RL::values[S] / stage_q(S); }

  // Twiddle factors this thread needs, preloaded into registers once
  // (stages >= 1; stage 0 has span 1 and no twiddles).  Forward and inverse
  // transforms of the same length share them (the inverse conjugates).
  static constexpr int tw_offset(int S) {
    int c = 0;
    for (int s = 1; s < S && s < RL::count; ++s) c += stage_q(s) * (RL::values[s] - 1);
    return c;
  }
  static constexpr int NTW = tw_offset(RL::count) > 0 ? tw_offset(RL::count) : 1;
  // The sixteen-element shape reads each stage's twiddles from the table at
  // that stage instead (its 29 would not fit in registers beside the data).
  static constexpr bool LAZY_TW = E_ >= 16;
  struct TableTw {
    Rsrc r;  // the table
    int t;   // this thread
  };
  using Twiddles = typename std::conditional<LAZY_TW, TableTw, float2[NTW]>::type;

  // tw: this shape's thread-order twiddle table, entry i * TPT + t = twiddle
  // slot i of thread t (so each load instruction reads consecutive entries),
  // values exp(-2 pi i e/N) rounded from float64 (see for_each_twiddle).
  __device__ __forceinline__ static void load_twiddles(Twiddles& w, const float2* __restrict__ tw, int t) {
    const Rsrc r = rsrc(tw);
    if constexpr (LAZY_TW) {
      w.r = r;
      w.t = t;
    } else {
#pragma unroll
      for (int i = 0; i < NTW; ++i) w[i] = ld2(r, (unsigned)t * 8u, (unsigned)(i * TPT * 8));
    }
  }

  // This thread's twiddle slot i.
  __device__ __forceinline__ static float2 twiddle(const Twiddles& w, int i) {
    if constexpr (LAZY_TW) return ld2(w.r, (unsigned)w.t * 8u, (unsigned)(i * TPT * 8));
    else return w[i];
  }

  // Host: calls f(slot, t, e) for every twiddle slot of every thread, where
  // slot i of thread t holds exp(-2 pi i e/N).  Stage S >= 1 (span P, radix R)
  // multiplies input r of butterfly q by w^(r k), k = (t + q TPT) mod P,
  // w = exp(-2 pi i/(P R)), i.e. e = r k N/(P R).
  template <class F>
  static void for_each_twiddle(F&& f) {
    twiddle_stage<1>(f);
  }

  // Forward (INV=false) or inverse (INV=true) unscaled DFT of the B transforms.
  // v: canonical registers in, canonical registers out.  lds: two buffers of
  // BUF elements; `phase` selects which buffer the first exchange writes and
  // is advanced so that consecutive transforms keep alternating buffers.
  template <bool INV>
  __device__ __forceinline__ static void fft(float2 (&v)[E], float2* lds, int& phase, const Twiddles& w, int t,
                                             int b) {
    stage<INV, 0>(v, lds, phase, w, t, b);
  }

 private:
  template <int S, class F>
  static void twiddle_stage(F& f) {
    if constexpr (S < RL::count) {
      constexpr int R = RL::values[S];
      constexpr int P = RL::span(S);
      constexpr int Q = stage_q(S);
      constexpr int A = stage_act(S);
      constexpr int STRIDE = N / (P * R);
      for (int t = 0; t < A; ++t)
        for (int q = 0; q < Q; ++q) {
          const int k = (t + q * A) % P;
          for (int r = 1; r < R; ++r) f(tw_offset(S) + q * (R - 1) + (r - 1), t, r * k * STRIDE);
        }
      twiddle_stage<S + 1>(f);
    }
  }

  // Fence between the LDS writes of one stage and the reads of the next: a
  // workgroup barrier, or, when the whole tile is one wavefront, only a
  // wavefront-scope fence (the LDS operations of one wavefront complete in
  // issue order, so nothing waits on other waves).
  __device__ __forceinline__ static void xsync() {
    if constexpr (THREADS <= 64) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
      __syncthreads();
    }
  }

  // x[j] = element t + q A + r N/R, j = q + r Q; `at` points to element t
  template <int R, int Q, int A, int... J>
  __device__ __forceinline__ static void read_stage(float2* x, const float2* at, const float2* src, int t, int b,
                                                    std::integer_sequence<int, J...>) {
    ((x[J] = read_one<(J % Q) * A + (J / Q) * (N / R)>(at, src, t, b)), ...);
  }
  template <int C>
  __device__ __forceinline__ static float2 read_one(const float2* at, const float2* src, int t, int b) {
    if constexpr (shifts_whole<C>()) return at[shift_of<C>()];
    else return src[lidx(b, t + C)];
  }
  // element base + r P <- u[r]; `at` points to element base (a multiple of R
  // where P = 1, so that a pad period of R holds all R outputs)
  template <int R, int P, int... J>
  __device__ __forceinline__ static void write_stage(const float2* u, float2* at, float2* dst, int base, int b,
                                                     std::integer_sequence<int, J...>) {
    (write_one<R, P, J>(u[J], at, dst, base, b), ...);
  }
  template <int R, int P, int J>
  __device__ __forceinline__ static void write_one(float2 u, float2* at, float2* dst, int base, int b) {
    if constexpr (SHIFTS && P == 1 && PADSHIFT && R == (1 << PADSHIFT)) at[J * (COL ? B : 1)] = u;
    else if constexpr (shifts_whole<J * P>()) at[shift_of<J * P>()] = u;
    else dst[lidx(b, base + J * P)] = u;
  }

  template <bool INV, int S>
  __device__ __forceinline__ static void stage(float2 (&v)[E], float2* lds, int& phase, const Twiddles& w, int t,
                                               int b) {
    if constexpr (S < RL::count) {
      constexpr int R = RL::values[S];
      constexpr int P = RL::span(S);
      constexpr int Q = stage_q(S);    // butterflies per thread in this stage
      constexpr int A = stage_act(S);  // threads that have them
      constexpr bool LAST = S + 1 == RL::count;
      static_assert(N % (R * Q) == 0 && A <= TPT, "a stage's butterflies divide evenly over its threads");
      static_assert(!canonical(S) || (E % R == 0 && A == ACT), "the outer stages keep the canonical layout");
      const bool mine = A == TPT || t < A;
      // this stage's twiddles (from registers, or loaded from the table now,
      // in flight across the exchange below)
      constexpr int NS = S > 0 ? Q * (R - 1) : 1;
      float2 ws[NS];
      if constexpr (S > 0) {
#pragma unroll
        for (int i = 0; i < NS; ++i) ws[i] = twiddle(w, tw_offset(S) + i);
      }
      // butterfly q's input r sits at i + r N/R, i = t + q A (for the outer
      // stages that is canonical element q + r Q)
      float2 x[Q * R];
      if constexpr (S > 0) {
        xsync();
        const float2* src = DB ? lds + (phase ^ 1) * BUF : lds;
        if (mine) {
          read_stage<R, Q, A>(x, src + lidx(b, t), src, t, b, std::make_integer_sequence<int, Q * R>{});
        } else {
#pragma unroll
          for (int j = 0; j < Q * R; ++j) x[j] = make_float2(0.f, 0.f);
        }
      } else {
#pragma unroll
        for (int j = 0; j < E; ++j) x[j] = v[j];
      }
      // single buffer: every thread must be done reading it (this stage's
      // loads, or an earlier transform's) before anyone overwrites it
      if constexpr (!DB && !LAST) xsync();
      float2* dst = DB ? lds + phase * BUF : lds;
      const int base0 = (t / P) * P * R + t % P;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        float2 u[R];
#pragma unroll
        for (int r = 0; r < R; ++r) u[r] = x[q + r * Q];
        if constexpr (S > 0) {
#pragma unroll
          for (int r = 1; r < R; ++r) {
            const float2 tf = ws[q * (R - 1) + (r - 1)];
            u[r] = INV ? cmulc(u[r], tf) : cmul(u[r], tf);
          }
        }
        Dft<R, INV>::run(u);
        if constexpr (!LAST) {
          if (mine) {
            // butterfly q's outputs sit at base + r P; q A further butterflies
            // move the base by q A R where A is a multiple of P
            const int i = t + q * A;
            const int base = A % P == 0 ? base0 + q * A * R : (i / P) * P * R + i % P;
            write_stage<R, P>(u, dst + lidx(b, base), dst, base, b, std::make_integer_sequence<int, R>{});
          }
        } else {
#pragma unroll
          for (int r = 0; r < R; ++r) v[q + r * Q] = u[r];
        }
      }
      if constexpr (!LAST) phase ^= 1;
      stage<INV, S + 1>(v, lds, phase, w, t, b);
    }
  }
};

// Tile of shape variant EV: 0 = the length's default shape (the split shape
// where the length has one), 1 = narrow, 2 = wide.
template <int N, int B, bool COL, bool DB, bool SPLIT>
struct TileDefault {
  using type = Tile<N, B, COL, DB>;
};
template <int N, int B, bool COL, bool DB>
struct TileDefault<N, B, COL, DB, true> {
  using type = Tile<N, B, COL, DB, 8, typename FftSplit<N>::R, FftSplit<N>::T>;
};
template <int N, int B, bool COL, bool DB, int EV>
struct TileSel {
  using type = typename TileDefault<N, B, COL, DB, FftSplit<N>::value>::type;
};
template <int N, int B, bool COL, bool DB>
struct TileSel<N, B, COL, DB, 1> {
  using type = Tile<N, B, COL, DB, 4, typename FftNarrow<N>::R>;
};
template <int N, int B, bool COL, bool DB>
struct TileSel<N, B, COL, DB, 2> {
  using type = Tile<N, B, COL, DB, 16, typename FftWide<N>::R>;
};
template <int N, int B, bool COL, bool DB = true, int EV = 0>
using TileV = typename TileSel<N, B, COL, DB, EV>::type;

}  // namespace sr
