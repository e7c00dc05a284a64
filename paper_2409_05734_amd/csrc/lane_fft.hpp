// One-element-per-lane transforms for the one-dimensional kernels.
#pragma once
#include "fft_core.hpp"

namespace sr {

// A transform of N = 64 W points on W waves, an element a lane: a 64-point
// transform inside each wave, exchanged between lanes by DPP and the permlane
// swaps, and a W-point one across the waves through LDS.
//
// A 1D solve is a chain of dependent transforms on one workgroup, so its time
// is a wave's own issue and the exchanges it waits for.  Four elements a lane
// on one wave (256 points) issue four times the arithmetic a lane and go
// through LDS three times a transform (0.49 us each); here a lane has a quarter
// of it and there is one exchange, whose write also undoes the order that the
// 64-point transform leaves (the layout: elem): 0.33 us.  The W-point transform
// has each wave form its own output from all W inputs, so its reads grow as
// W^2: up to twelve waves.
template <int N> struct HasLane { static constexpr bool value = false; };
template <> struct HasLane<64>  { static constexpr bool value = true; };
template <> struct HasLane<128> { static constexpr bool value = true; };
template <> struct HasLane<192> { static constexpr bool value = true; };
template <> struct HasLane<256> { static constexpr bool value = true; };
template <> struct HasLane<384> { static constexpr bool value = true; };
template <> struct HasLane<512> { static constexpr bool value = true; };
template <> struct HasLane<768> { static constexpr bool value = true; };

// One radix-2 step between lanes l and l ^ D (in index, see lane_index): v + v'
// where the lane's bit D is clear, v' - v where it is set; s = +1 or -1 there.
template <int D>
__device__ __forceinline__ float2 lane_butterfly(float2 v, float s) {
  if constexpr (D == 32 || D == 16) {
    // Swapping row halves between the real and the imaginary register puts a
    // pair's two real parts side by side in the one lane and its two imaginary
    // parts in the other; after the sum and the difference, the same swap puts
    // things back.
    const auto swap = [=](float& a, float& b) {
      typedef unsigned u2 __attribute__((ext_vector_type(2)));
      u2 r;
      if constexpr (D == 32) r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
      else r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
      a = __uint_as_float(r[0]);
      b = __uint_as_float(r[1]);
    };
    float a = v.x, b = v.y;
    swap(a, b);
    float sum = a + b, dif = a - b;
    swap(sum, dif);
    return make_float2(sum, dif);
  } else {
    // 8: rotate the row by 8; 4: mirror the half row (lane ^ 7); 2, 1: within the quad
    constexpr int ctrl = D == 8 ? 0x128 : D == 4 ? 0x141 : D == 2 ? 0x4E : 0xB1;
    const auto other = [=](float x) {
      return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), ctrl, 0xf, 0xf, true));
    };
    return make_float2(__builtin_fmaf(s, v.x, other(v.x)), __builtin_fmaf(s, v.y, other(v.y)));
  }
}

template <int N_>
struct LaneTile {
  static constexpr int N = N_, W = N_ / 64;
  static constexpr int E = 1, TPT = N, ACT = N, THREADS = N, NBUF = 2;
  // a pad every 32: a wave's elements lie W apart
  static constexpr int BUF = N + N / 32;
  static constexpr int NTW = 3 + W - 1;
  static_assert(N % 64 == 0 && THREADS <= 1024, "whole waves");

  struct Twiddles {
    float2 t1, t2, t3;            // after the W-point sum, after the first (times 1/sqrt(N)) and second pair of steps
    float2 c[W > 1 ? W - 1 : 1];  // the sum's factors
    float s[4];                // signs of the steps 8, 4, 2, 1
    int wr, rd;                // this thread's place to write, and to read from
    bool q0, q1, q2;           // a quarter turn before the steps 16, 4, 1
  };

  // Index within the wave's 64 points: the lane, its two lowest bits reversed
  // in direction where bit 2 is set, so that flipping index bit 2 is a mirror
  // of the half row.
  __device__ __host__ __forceinline__ static int lane_index(int lane) { return lane ^ ((lane & 4) ? 3 : 0); }
  // The element that thread t holds: bit-reversed within its wave, whose number
  // is the element's residue mod W.
  __device__ __host__ __forceinline__ static int elem(int t, int) {
    const int l = lane_index(t & 63);
    const int r = ((l >> 5) & 1) | ((l >> 3) & 2) | ((l >> 1) & 4) | ((l << 1) & 8) | ((l << 3) & 16) | ((l << 5) & 32);
    return (t >> 6) + W * r;
  }

  // Host: f(slot, t, e) for every twiddle exp(-2 pi i e / N), slots in the
  // order of Twiddles.
  template <class F>
  static void for_each_twiddle(F&& f) {
    for (int t = 0; t < N; ++t) {
      const int l = lane_index(t & 63), w = t >> 6;
      const auto bit = [&](int b) { return (l >> b) & 1; };
      f(0, t, l * w % N);
      f(1, t, W * (l & 15) * (bit(5) + 2 * bit(4)) % N);
      f(2, t, 4 * W * (l & 3) * (bit(3) + 2 * bit(2)) % N);
      for (int j = 1; j < W; ++j) f(2 + j, t, 64 * j * w % N);
    }
  }

  __device__ __forceinline__ static void load_twiddles(Twiddles& w, const float2* __restrict__ tw, int t) {
    w.t1 = tw[t];
    w.t2 = cscale(tw[N + t], rsqrtf((float)N));
    w.t3 = tw[2 * N + t];
#pragma unroll
    for (int j = 1; j < W; ++j) w.c[j - 1] = tw[(2 + j) * N + t];
    const int l = lane_index(t & 63);
#pragma unroll
    for (int i = 0; i < 4; ++i) w.s[i] = (l >> (3 - i)) & 1 ? -1.f : 1.f;
    const int k = elem(t, 0);
    w.wr = k + (k >> 5);
    w.rd = l + (l >> 5);
    w.q0 = (l & 48) == 48;
    w.q1 = (l & 12) == 12;
    w.q2 = (l & 3) == 3;
  }

  // (unitary: t2 holds the scale)
  template <bool INV>
  __device__ __forceinline__ static void fft(float2 (&v)[1], float2* lds, int& phase, const Twiddles& w, int t, int) {
    float2* x = lds + phase * BUF;
    phase ^= 1;
    x[w.wr] = v[0];
    if constexpr (THREADS <= 64) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
      __syncthreads();
    }
    x += w.rd;
    float2 o[W];
#pragma unroll
    for (int j = 0; j < W; ++j) o[j] = x[66 * j];
    float2 y = sum<INV, W>(o, w);
    if constexpr (W > 1) y = turn<INV>(y, w.t1);
    y = pair<INV, 32, 16>(y, 0.f, 0.f, w.q0);
    y = turn<INV>(y, w.t2);
    y = pair<INV, 8, 4>(y, w.s[0], w.s[1], w.q1);
    y = turn<INV>(y, w.t3);
    y = pair<INV, 2, 1>(y, w.s[2], w.s[3], w.q2);
    v[0] = y;
  }

 private:
  template <bool INV>
  __device__ __forceinline__ static float2 turn(float2 y, float2 t) {
    return INV ? cmulc(y, t) : cmul(y, t);
  }
  // this wave's output of the W-point transform, as sums of the halves'
  // outputs while the count is even: H inputs are left, W/H steps of W/H apart
  template <bool INV, int H>
  __device__ __forceinline__ static float2 sum(float2 (&o)[W], const Twiddles& w) {
    if constexpr (H == 1) {
      return o[0];
    } else if constexpr (H % 2 == 0) {
      const float2 c = w.c[H / 2 - 1];
#pragma unroll
      for (int j = 0; j < H / 2; ++j) {
        if constexpr (H == W) {  // a sign
          o[j].x = __builtin_fmaf(c.x, o[j + H / 2].x, o[j].x);
          o[j].y = __builtin_fmaf(c.x, o[j + H / 2].y, o[j].y);
        } else {
          o[j] = cfma<INV>(o[j + H / 2], c, o[j]);
        }
      }
      return sum<INV, H / 2>(o, w);
    } else {
      float2 y = o[0];
#pragma unroll
      for (int j = 1; j < H; ++j) y = cfma<INV>(o[j], w.c[j - 1], y);
      return y;
    }
  }
  // y + a c (conj(c) if INV)
  template <bool INV>
  __device__ __forceinline__ static float2 cfma(float2 a, float2 c, float2 y) {
    y.x = __builtin_fmaf(a.x, c.x, y.x);
    y.y = __builtin_fmaf(a.y, c.x, y.y);
    y.x = __builtin_fmaf(INV ? a.y : -a.y, c.y, y.x);
    y.y = __builtin_fmaf(INV ? -a.x : a.x, c.y, y.y);
    return y;
  }
  // two radix-2 steps, i.e. a radix-4 one across four lanes
  template <bool INV, int D0, int D1>
  __device__ __forceinline__ static float2 pair(float2 y, float s0, float s1, bool q) {
    y = lane_butterfly<D0>(y, s0);
    const float2 r = quarter<INV>(y);
    y.x = q ? r.x : y.x;
    y.y = q ? r.y : y.y;
    return lane_butterfly<D1>(y, s1);
  }
};

}  // namespace sr
