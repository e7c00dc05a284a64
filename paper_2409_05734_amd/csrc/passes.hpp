// Fused FFT pass kernels for the 2D structured operator.
//
// The 2D unitary DFT factors into commuting axis transforms F = F_1 F_0.
// Layer l of A = F D_L ... F D_1 U applies its two axis transforms in the
// order (0,1) when l is odd and (1,0) when l is even, so consecutive
// transforms along the same axis meet and fuse with the phase diagonal
// between them.  One pass = one read and one write of the m-grid:
//
//   forward : [U D_1 F_0] [F_1 D_2 F_1] [F_0 D_3 F_0] ... [F_a -> z, |z|^2]
//   adjoint : [F_a^H] ... [F_0^H D_3^* F_0^H] [F_1^H D_2^* F_1^H] [F_0^H D_1^* U^H]
//   GD/spectral iteration: forward passes, a turnaround pass
//   [F_a -> residual or spectral weight -> F_a^H], then the adjoint passes,
//   the last of which also applies the solver update.
//
// Column-mode passes (transforms along axis 0) read and write tiles of B
// adjacent columns; row-mode passes tiles of B rows.  Passes next to the
// zero-padded support only touch the N_2 support columns ("compact" buffers).
#pragma once
#include "fft_core.hpp"
#include "loss.hpp"

namespace sr {

enum PreOp : int {
  PRE_NONE = 0,
  PRE_PHASE = 1,
  PRE_PHASE_STEP = 2  // D_1 U (step x): the reverse GD step's first pass on the scaled cotangent
};
enum MidOp : int {
  MID_NONE = 0,
  MID_PHASE = 1,            // v <- D v
  MID_PHASE_CONJ = 2,       // v <- D^* v
  MID_GD = 3,               // v <- (|v|^2 - y) v, loss partials
  MID_SPEC = 4,             // v <- T(y) v
  MID_STORE = 5,            // z <- v, |z|^2
  // reverse-mode variants (value u after the first transform; save/gth per layer)
  MID_PHASE_SAVE = 6,       // u <- D v, save <- u                  (forward recompute)
  MID_PHASE_CONJ_GT = 7,    // gth += Im(v conj(save)), v <- D^* v   (forward VJP)
  MID_PHASE_CONJ_SAVE = 8,  // q <- D^* v, save <- q                (adjoint recompute)
  MID_PHASE_GT = 9,         // gth += Im(conj(v) save), v <- D v     (adjoint VJP)
  MID_GD_POIS = 10,         // v <- (1 - y/(|v|^2 + eps)) v, Poisson loss partials
  // turnarounds of the reverse GD step and of the intensities' reverse
  MID_STEP = 11,            // save <- z, v <- (|z|^2 - y) z
  MID_STEP_BAR = 12,        // v <- (2|z|^2 - y) v + z^2 conj(v), gy -= Re(conj(v) z), z = save
  MID_INT_BAR = 13          // v <- 2 y v (y: the cotangent of the intensities)
};
// The reverse-mode mid operations (phase diagonal with a saved intermediate).
constexpr bool mid_rev_phase(int mid) { return mid >= MID_PHASE_SAVE && mid <= MID_PHASE_GT; }

enum PostOp : int {
  POST_STORE = 0,
  POST_PHASE_CONJ_STORE = 1,
  POST_GD = 2,            // x <- x - step g
  POST_SPEC = 3,          // u <- s (step g - 2 lambda u), s = 1/||u|| (deferred normalisation)
  POST_PHASE_CONJ_GT = 4,  // gth_1 += Im(v conj(D_1 U x)), then D_1^* and crop
  // the next iteration's first pass fused behind the update: the new iterate,
  // still in registers, is padded, multiplied by D_1 and transformed along
  // axis 0 into out2 (the compact buffer the next row pass reads)
  POST_GD_FWD = 5,
  POST_SPEC_FWD = 6,
  POST_GTV = 7  // gth_1 += Im(conj(step xin) D_1^* v) on the support, nothing stored
};

struct PassArgs {
  // input buffer: element (transform b, position k) for k in [in_lo, in_hi)
  // row mode: in[b*in_ld + k - in_lo]; column mode: in[(k - in_lo)*in_ld + b]
  const float2* in;
  long long in_ld;
  int in_lo, in_hi;
  // output buffer with the same addressing over the window [out_lo, out_hi)
  float2* out;
  long long out_ld;
  int out_lo, out_hi;
  int ntr;            // number of transforms (rows or columns) in this pass
  int tr_lo;          // grid coordinate of transform 0 on the other axis
  long long grid_ld;  // M2, row stride of the full measurement grid
  const float2* tw;   // thread-order twiddle table of the default thread shape
  const float2* tw_n; // ... of the length's narrow or wide thread shape (where it has one)
  const float* th_pre;
  const float* th_mid;
  const float* th_post;
  // optional precomputed exp(i theta) tables for the same diagonals; when
  // set they replace the phases (one 8-byte load instead of sincos)
  const float2* ep_pre;
  const float2* ep_mid;
  const float2* ep_post;
  float scale_pre, scale_mid, scale_out;
  // epilogues
  const float* y;        // measurements on the window (MID_GD, MID_GD_POIS, MID_SPEC)
  const double* ysum;    // sum(y) (MID_SPEC)
  float inv_m;           // 1/m
  float lam;             // spectral threshold lambda
  float2* z_out;         // MID_STORE: z = A x on the grid (nullable)
  float* y_out;          // MID_STORE: |z|^2 on the grid (nullable)
  float* part_out;       // per-workgroup partial sums (loss or squared norm), nullable
  const float* part_in;  // squared-norm partials of the previous iterate (spectral), nullable
  int npart;
  // solver updates (POST_GD, POST_SPEC)
  float step;            // GD: eta/m; spectral: 1/(m c)
  float two_lam;         // spectral: 2 lambda
  // reverse mode
  float2* save;          // per-layer intermediate on the grid (written or read)
  float* gth;            // phase-cotangent accumulator of this pass's diagonal (grid layout)
  const float2* xin;     // POST_PHASE_CONJ_GT: the signal x (crop layout = output layout)
  float2* out2;          // POST_*_FWD: compact output of the fused forward transform
  long long out2_ld;
  // measurement window: grid rows [win_lo0, win_hi0) x columns [win_lo1,
  // win_hi1), stored row-major with row length win_ld.  y, z_out, y_out (and
  // the input of the adjoint's first pass) live on the window; the residual
  // and the spectral weight are zero outside it.
  int win_lo0, win_hi0, win_lo1, win_hi1;
  long long win_ld;
  int crop;  // nonzero when the window is smaller than the grid (host: picks the window-aware kernels)
  float loss_eps;  // Poisson loss guard (MID_GD_POIS)
  // stacked problems: one launch runs this pass for `stack` problems of one
  // geometry; ntr counts the transforms of all of them, ntr_p those of one,
  // and problem s's data sits s * s_<buffer> elements after problem 0's
  int stack, ntr_p;
  int s_in, s_out, s_out2, s_win, s_th, s_save, s_gth, s_xin;
  const float* step_v;  // GD update of a stack: each problem's step (nullable: `step` for all)
  // POLY kernels: phases of larger magnitude are read from the tables (ep_*),
  // where the polynomials' argument reduction would lose bits
  float th_poly_max;
  // non-finite flag (nullable): the final update of a solve (POST_GD,
  // POST_SPEC) stores 1 here when an updated iterate entry is NaN or Inf
  unsigned* nf;
  // reverse GD step
  float* gy;          // MID_STEP_BAR: cotangents of y, accumulated (nullable)
  const float2* xadd; // POST_PHASE_CONJ_GT: added to the output (nullable)
  int s_xadd;
  int gth_set;        // phase cotangents: write them rather than add (the first term into scratch)
};

// 1/sqrt of the sum of the previous iterate's squared-norm partials: strided
// per-thread sums, then a fixed-order workgroup reduction in float64, so
// every thread (and every workgroup of the pass) gets the same value.
template <int NTHREADS>
__device__ __forceinline__ float inv_norm_from_partials(const float* part, int n) {
  __shared__ double redd[NTHREADS / 64 > 0 ? NTHREADS / 64 : 1];
  double acc = 0.0;
  for (int i = (int)threadIdx.x; i < n; i += NTHREADS) acc += (double)part[i];
  return (float)(1.0 / sqrt(block_sum_t<NTHREADS, double>(acc, redd)));
}

// One tile (B transforms) of a fused pass.  `lds` holds 2*B*N complex
// elements, `red` one float per thread.  part_in/npart/part_out override the
// partial-sum pointers of `a` (persistent kernels alternate them per
// iteration); partial sums are written at index `tile`.  TAB selects the
// phase source: exp(i theta) tables (ep_*) or the phases themselves (th_*),
// evaluated with the hardware's sine and cosine or (POLY) with polynomials,
// and read from the tables after all by a thread with a phase past th_poly_max.
//
// Every global load the tile needs (input, phases, measurements, twiddles,
// the previous iterate) is issued up front, so a pass costs one memory
// round trip plus its arithmetic, not one round trip per stage.  Loads and
// stores go through buffer resources: lanes outside a window (the zero-padded
// rows/columns, transforms past ntr) read zeros and drop their writes.
template <int N, int B, bool COL, int PRE, int MID, bool FFT2, bool INV1, bool INV2, int POST, bool DB = true,
          int EV = 0, bool TAB = false, bool WIN = false, bool POLY = false>
__device__ __forceinline__ void pass_tile(const PassArgs& a, int tile, float2* lds, float* red, const float* part_in,
                                          int npart, float* part_out) {
  using T = TileV<N, B, COL, DB, EV>;
  constexpr int E = T::E;
  constexpr bool MID_PH = (MID == MID_PHASE || MID == MID_PHASE_CONJ || mid_rev_phase(MID));
  constexpr bool PRE_PH = (PRE != PRE_NONE);
  constexpr bool MID_SAVED = (MID == MID_PHASE_CONJ_GT || MID == MID_PHASE_GT);
  constexpr bool MID_Y = (MID == MID_GD || MID == MID_GD_POIS || MID == MID_SPEC || MID == MID_STEP ||
                          MID == MID_STEP_BAR || MID == MID_INT_BAR);
  constexpr bool POST_PH = (POST != POST_STORE);
  constexpr bool POST_X = (POST == POST_GD || POST == POST_SPEC || POST == POST_GD_FWD || POST == POST_SPEC_FWD);
  constexpr bool POST_FWD = (POST == POST_GD_FWD || POST == POST_SPEC_FWD);
  constexpr bool POST_IS_GD = (POST == POST_GD || POST == POST_GD_FWD);
  constexpr bool POST_IS_SPEC = (POST == POST_SPEC || POST == POST_SPEC_FWD);
  const int t = T::thread_t();
  const int bl = T::thread_b();
  const int tb = tile * B + bl;  // transform index (over every problem of a stack)
  const bool active = tb < a.ntr && T::holds(t);
  int b = tb, sp = 0;            // this lane's transform within its problem, and the problem
  if (a.stack > 1) {
    sp = tb / a.ntr_p;
    b = tb - sp * a.ntr_p;
  }
  const int gb = a.tr_lo + b;  // grid coordinate of this transform
  const int gld = (int)a.grid_ld, ild = (int)a.in_ld, old = (int)a.out_ld;
  // the lane's problem's offset in each buffer (zero without a stack)
  const int o_in = sp * a.s_in, o_out = sp * a.s_out, o_out2 = sp * a.s_out2, o_win = sp * a.s_win;
  const int o_th = sp * a.s_th, o_sv = sp * a.s_save, o_gt = sp * a.s_gth, o_xin = sp * a.s_xin;

  // ---- addressing.  Element j of this lane sits j steps after element 0 in
  // every buffer (ACT rows or columns each), so an access takes the lane's
  // offset of element 0 and the scalar offset of j steps.  What does not vary
  // over the lanes (a window's start) goes into the buffer's base, which keeps
  // lane offsets non-negative.  A window that covers the whole transform (all
  // but the passes next to the support, and trimmed measurements) needs no
  // test per element: the lane is in or out.
  // (2048 x 2048 grid, 1024 x 1024 signal: vector instructions a thread of the
  // two column passes 858 -> 700 and 811 -> 646, their longest shape 126 -> 97
  // registers; a GD iteration, L = 3, 129 -> 122 us.)
  constexpr int ACT = T::ACT;
  const int g_lane = COL ? t * gld + gb : gb * gld + t, g_step = COL ? ACT * gld : ACT;      // grid
  const int i_lane = COL ? t * ild + b : b * ild + t, i_step = COL ? ACT * ild : ACT;        // input buffer
  const int u_lane = COL ? t * old + b : b * old + t, u_step = COL ? ACT * old : ACT;        // output buffer
  const int i_cut = COL ? a.in_lo * ild : a.in_lo, u_cut = COL ? a.out_lo * old : a.out_lo;  // their windows' starts
  const bool in_full = a.in_lo <= 0 && a.in_hi >= N, out_full = a.out_lo <= 0 && a.out_hi >= N;
  const int in_len = active ? a.in_hi - a.in_lo : 0, out_len = active ? a.out_hi - a.out_lo : 0;
  auto in_win = [&](int j) { return (unsigned)(t - a.in_lo + j * ACT) < (unsigned)in_len; };
  auto out_win = [&](int j) { return (unsigned)(t - a.out_lo + j * ACT) < (unsigned)out_len; };
  // lane offset of an element of B bytes, past the range where !ok
  auto off = [](bool ok, int lane, unsigned bytes) -> unsigned { return ok ? (unsigned)lane * bytes : kOob; };
  // measurement window: membership and index of element j of this transform
  // (the transform's own coordinate is tested once).  Kernels built without
  // WIN take the window to be the whole grid (no trimming).
  const int wld = (int)a.win_ld;
  const bool m_lane =
      WIN ? active && (COL ? (gb >= a.win_lo1 && gb < a.win_hi1) : (gb >= a.win_lo0 && gb < a.win_hi0)) : active;
  const int m_klo = COL ? a.win_lo0 : a.win_lo1;
  const int m_len = m_lane ? (COL ? a.win_hi0 : a.win_hi1) - m_klo : 0;
  const int m_off = o_win + (WIN ? (COL ? t * wld + gb : gb * wld + t) : g_lane);
  const int m_step = WIN ? (COL ? ACT * wld : ACT) : g_step;
  const int m_cut = WIN ? a.win_lo0 * wld + a.win_lo1 : 0;
  auto m_in = [&](int j) { return WIN ? (unsigned)(t - m_klo + j * ACT) < (unsigned)m_len : active; };
  // the adjoint's first pass ([F_a^H] alone) reads its input on the window
  constexpr bool IN_WIN = WIN && (PRE == PRE_NONE && MID == MID_NONE && !FFT2 && INV1 && POST == POST_STORE);

  // ---- issue every global load
  float2 v[E];
  float2 dp[E];   // pre-diagonal entries e^{i theta}
  float2 dm[E];   // mid-diagonal entries
  float yv[E];    // measurements
  float2 dq[E];   // post-diagonal entries
  float2 xo[E];   // previous iterate (or x for POST_PHASE_CONJ_GT)
  float2 sv[E];   // saved intermediate
  float gt[E];    // phase-cotangent accumulator
  typename T::Twiddles w;
  const Rsrc r_in = rsrc(a.in - (IN_WIN ? m_cut : i_cut));
  const Rsrc r_out = rsrc(a.out - u_cut);
  const Rsrc r_pre = TAB ? rsrc(a.ep_pre) : rsrc(a.th_pre);
  const Rsrc r_mid = TAB ? rsrc(a.ep_mid) : rsrc(a.th_mid);
  const Rsrc r_post = TAB ? rsrc(a.ep_post) : rsrc(a.th_post);
  const Rsrc r_y = rsrc(a.y - m_cut);
  const Rsrc r_save = rsrc(a.save);
  const Rsrc r_gth = rsrc(a.gth);
  const Rsrc r_xin = rsrc(a.xin - u_cut);
  constexpr unsigned PB = TAB ? 8 : 4;  // bytes of a phase entry
  const unsigned p_all = off(active, g_lane + o_th, PB);
  auto ld_phase = [&](Rsrc r, unsigned o, int j) -> float2 {
    if constexpr (TAB) return ld2(r, o, (unsigned)(j * g_step) * 8u);
    else return make_float2(ld1(r, o, (unsigned)(j * g_step) * 4u), 0.f);
  };
  if constexpr (IN_WIN) {
    const int lane = m_off - o_win + o_in;
#pragma unroll
    for (int j = 0; j < E; ++j) v[j] = ld2(r_in, off(m_in(j), lane, 8), (unsigned)(j * m_step) * 8u);
  } else if (in_full) {
    const unsigned o = off(active, i_lane + o_in, 8);
#pragma unroll
    for (int j = 0; j < E; ++j) v[j] = ld2(r_in, o, (unsigned)(j * i_step) * 8u);
  } else {
#pragma unroll
    for (int j = 0; j < E; ++j) v[j] = ld2(r_in, off(in_win(j), i_lane + o_in, 8), (unsigned)(j * i_step) * 8u);
  }
  // Twiddles after what the first butterflies wait for, since loads return in
  // order, and no arithmetic before the last load is issued (the barrier below):
  // GD on a 512 x 512 grid 19.2 -> 18.6 us an iteration, power iteration 21.0 ->
  // 20.6, a four-column store pass 0.17 us.
  if constexpr (!PRE_PH) T::load_twiddles(w, EV ? a.tw_n : a.tw, t);
#pragma unroll
  for (int j = 0; j < E; ++j) {
    if constexpr (PRE_PH) dp[j] = ld_phase(r_pre, in_win(j) ? p_all : kOob, j);
    if constexpr (MID_PH) dm[j] = ld_phase(r_mid, p_all, j);
    if constexpr (MID_Y) yv[j] = ld1(r_y, off(m_in(j), m_off, 4), (unsigned)(j * m_step) * 4u);
    if constexpr (MID_SAVED || MID == MID_STEP_BAR)
      sv[j] = ld2(r_save, off(active, g_lane + o_sv, 8), (unsigned)(j * g_step) * 8u);
    if constexpr (MID_SAVED)
      gt[j] = a.gth_set ? 0.f : ld1(r_gth, off(active, g_lane + o_gt, 4), (unsigned)(j * g_step) * 4u);
    if constexpr (MID == MID_STEP_BAR)
      gt[j] = a.gy != nullptr ? ld1(rsrc(a.gy - m_cut), off(m_in(j), m_off, 4), (unsigned)(j * m_step) * 4u) : 0.f;
    if constexpr (MID != MID_STORE && POST_PH) {
      const bool ow = out_win(j);
      dq[j] = ld_phase(r_post, ow ? p_all : kOob, j);
      if constexpr (POST_X) xo[j] = ld2(r_out, off(ow, u_lane + o_out, 8), (unsigned)(j * u_step) * 8u);
      if constexpr (POST == POST_PHASE_CONJ_GT || POST == POST_GTV) {
        xo[j] = ld2(r_xin, off(ow, u_lane + o_xin, 8), (unsigned)(j * u_step) * 8u);
        gt[j] = a.gth_set ? 0.f : ld1(r_gth, off(ow, g_lane + o_gt, 4), (unsigned)(j * g_step) * 4u);
      }
    }
  }
  if constexpr (PRE_PH) T::load_twiddles(w, EV ? a.tw_n : a.tw, t);
  __builtin_amdgcn_sched_barrier(0);  // no arithmetic, and so no wait, among the loads
  // phases -> diagonal entries where no table was given (the sixteen-
  // element shape forms the mid and post entries where they are used, so
  // that only the phases stay live across the first transform)
  constexpr bool LATE_PH = !TAB && E >= 16;
  // POLY: a diagonal's entries from its phases, or from its table where this
  // thread has one past the polynomials' range
  auto entries = [&](float2(&d)[E], const float2* tab, auto&& offset) {
    float top = 0.f;
#pragma unroll
    for (int j = 0; j < E; ++j) top = fmaxf(top, fabsf(d[j].x));
    if (top > a.th_poly_max) {
#pragma unroll
      for (int j = 0; j < E; ++j) d[j] = ld2(rsrc(tab), offset(j), (unsigned)(j * g_step) * 8u);
    } else {
#pragma unroll
      for (int j = 0; j < E; ++j) d[j] = phase_poly(d[j].x);
    }
  };
  const unsigned e_all = off(active, g_lane + o_th, 8);
  static_assert(!POLY || (!TAB && !LATE_PH), "POLY kernels form the entries from phases");
  if constexpr (POLY && PRE_PH) entries(dp, a.ep_pre, [&](int j) { return in_win(j) ? e_all : kOob; });
  if constexpr (!TAB && !POLY) {
#pragma unroll
    for (int j = 0; j < E; ++j) {
      if constexpr (PRE_PH) dp[j] = phase_turns(dp[j].x);
      if constexpr (MID_PH && !LATE_PH) dm[j] = phase_turns(dm[j].x);
      if constexpr (POST_PH && !LATE_PH) dq[j] = phase_turns(dq[j].x);
    }
  }
  // a weight of measurement j, zero outside the window (without WIN the lanes
  // outside hold zeros anyway: their loads returned none)
  auto in_weight = [&](int j, float wgt) -> float { return !WIN || m_in(j) ? wgt : 0.f; };
  auto Dm = [&](int j) -> float2 {
    if constexpr (LATE_PH) return phase_turns(dm[j].x);
    else return dm[j];
  };
  auto Dq = [&](int j) -> float2 {
    if constexpr (LATE_PH) return phase_turns(dq[j].x);
    else return dq[j];
  };

  float s_pre = a.scale_pre;
  float s_prev = 1.f;  // 1/||u_prev|| for the spectral update
  if constexpr (PRE == PRE_PHASE || POST_IS_SPEC) {  // the only shapes that take the previous norm
    if (part_in != nullptr) {
      // a stack keeps each problem's partials together (npart apiece), and
      // a pass that reads them has whole problems in each tile
      const float* pin = a.stack > 1 ? part_in + (tile * B / a.ntr_p) * npart : part_in;
      s_prev = inv_norm_from_partials<T::THREADS>(pin, npart);
      if (PRE == PRE_PHASE) s_pre *= s_prev;
    }
  }

  // the step of the lane's problem (the reverse GD step's factor -eta/m)
  float step = a.step;
  if constexpr (PRE == PRE_PHASE_STEP || POST == POST_GTV) {
    if (a.step_v != nullptr && active) step = a.step_v[sp];
  }
  if constexpr (PRE == PRE_PHASE_STEP) s_pre *= step;

  // ---- pre-diagonal, first transform
#pragma unroll
  for (int j = 0; j < E; ++j) {
    if constexpr (PRE_PH) v[j] = cmul(v[j], cscale(dp[j], s_pre));  // (only these passes have a scale_pre)
  }
  int ph = 0;
  T::template fft<INV1>(v, lds, ph, w, t, bl);

  // ---- mid operation.  A pass of two transforms along one axis scales by
  // 1/sqrt(N) twice; where a factor is applied between them, both go into it as
  // 1/N (FOLD), which the powers of two hold exactly: two multiplications an
  // element less, and none of the bias that the rounded 1/sqrt(N) leaves.
  constexpr bool FOLD = FFT2 && !mid_rev_phase(MID);
  static_assert(!FOLD || POST == POST_STORE, "a folded scale has no post operation to precede");
  constexpr float kInvN = 1.f / (float)N;
  const float s_mid = a.scale_mid, s_out = a.scale_out;
  float acc = 0.f;
  if constexpr (POLY && MID_PH) entries(dm, a.ep_mid, [&](int) { return e_all; });
  if constexpr (MID == MID_PHASE || MID == MID_PHASE_CONJ) {
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const float2 d = cscale(Dm(j), kInvN);
      v[j] = (MID == MID_PHASE_CONJ) ? cmulc(v[j], d) : cmul(v[j], d);
    }
  } else if constexpr (mid_rev_phase(MID)) {
    const unsigned o8 = off(active, g_lane + o_sv, 8), o4 = off(active, g_lane + o_gt, 4);
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const unsigned j8 = (unsigned)(j * g_step) * 8u, j4 = (unsigned)(j * g_step) * 4u;
      const float2 u = cscale(v[j], s_mid);
      if constexpr (MID == MID_PHASE_SAVE) {
        v[j] = cmul(u, Dm(j));
        st2(r_save, o8, j8, v[j]);
      } else if constexpr (MID == MID_PHASE_CONJ_SAVE) {
        v[j] = cmulc(u, Dm(j));
        st2(r_save, o8, j8, v[j]);
      } else if constexpr (MID == MID_PHASE_CONJ_GT) {
        // Im(u conj(s)) = u.y s.x - u.x s.y
        st1(r_gth, o4, j4, gt[j] + (u.y * sv[j].x - u.x * sv[j].y));
        v[j] = cmulc(u, Dm(j));
      } else {  // MID_PHASE_GT: Im(conj(u) s) = u.x s.y - u.y s.x
        st1(r_gth, o4, j4, gt[j] + (u.x * sv[j].y - u.y * sv[j].x));
        v[j] = cmul(u, Dm(j));
      }
    }
  } else if constexpr (MID == MID_STEP) {
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const float2 z = cscale(v[j], s_mid);
      st2(r_save, off(active, g_lane + o_sv, 8), (unsigned)(j * g_step) * 8u, z);
      v[j] = cscale(v[j], in_weight(j, cabs2(z) - yv[j]) * kInvN);
    }
  } else if constexpr (MID == MID_STEP_BAR) {
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const bool in = m_in(j);
      const float2 rb = cscale(v[j], s_mid), z = sv[j];
      const float w = 2.f * cabs2(z) - yv[j];
      const float2 z2 = cmul(z, z);
      if (a.gy != nullptr)
        st1(rsrc(a.gy - m_cut), off(in, m_off, 4), (unsigned)(j * m_step) * 4u, gt[j] - (rb.x * z.x + rb.y * z.y));
      v[j] = make_float2(in ? (w * rb.x + z2.x * rb.x + z2.y * rb.y) * s_out : 0.f,
                         in ? (w * rb.y + z2.y * rb.x - z2.x * rb.y) * s_out : 0.f);
    }
  } else if constexpr (MID == MID_INT_BAR) {
#pragma unroll
    for (int j = 0; j < E; ++j) v[j] = cscale(v[j], in_weight(j, 2.f * yv[j]) * kInvN);
  } else if constexpr (MID == MID_GD) {
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const float d = in_weight(j, cabs2(cscale(v[j], s_mid)) - yv[j]);  // zero residual outside the measurement window
      acc += d * d;
      v[j] = cscale(v[j], d * kInvN);
    }
  } else if constexpr (MID == MID_GD_POIS) {
    float z2[E];
#pragma unroll
    for (int j = 0; j < E; ++j) {
      z2[j] = cabs2(cscale(v[j], s_mid));
      v[j] = cscale(v[j], in_weight(j, poisson_weight(z2[j], yv[j], a.loss_eps)) * kInvN);
    }
    if (part_out != nullptr) {  // the logarithms only for a loss trace
#pragma unroll
      for (int j = 0; j < E; ++j) acc += m_in(j) ? poisson_term(z2[j], yv[j], a.loss_eps) : 0.f;
    }
  } else if constexpr (MID == MID_SPEC) {
    const float ybar = (float)(a.ysum[active ? sp : 0] * (double)a.inv_m);  // the problem's sum(y) (a stack: one each)
#pragma unroll
    for (int j = 0; j < E; ++j) {
      float wgt = a.lam;
      if (yv[j] > 0.f) wgt = fmaxf(1.f - ybar / yv[j], a.lam);
      v[j] = cscale(v[j], in_weight(j, wgt) * kInvN);
    }
  } else if constexpr (MID == MID_STORE) {
    const Rsrc r_z = rsrc(a.z_out - m_cut), r_yo = rsrc(a.y_out - m_cut);
#pragma unroll
    for (int j = 0; j < E; ++j) {
      float2 z = cscale(v[j], s_mid);
      const bool in = m_in(j);
      if (a.z_out) st2(r_z, off(in, m_off, 8), (unsigned)(j * m_step) * 8u, z);
      if (a.y_out) st1(r_yo, off(in, m_off, 4), (unsigned)(j * m_step) * 4u, cabs2(z));
    }
  }

  // ---- second transform, post-diagonal, update, store
  if constexpr (FFT2) T::template fft<INV2>(v, lds, ph, w, t, bl);
  if constexpr (MID != MID_STORE && POST == POST_STORE) {
    auto val = [&](int j) { return FOLD ? v[j] : cscale(v[j], s_out); };
    if (out_full) {
      const unsigned o = off(active, u_lane + o_out, 8);
#pragma unroll
      for (int j = 0; j < E; ++j) st2(r_out, o, (unsigned)(j * u_step) * 8u, val(j));
    } else {
#pragma unroll
      for (int j = 0; j < E; ++j) st2(r_out, off(out_win(j), u_lane + o_out, 8), (unsigned)(j * u_step) * 8u, val(j));
    }
  } else if constexpr (MID != MID_STORE) {
    if constexpr (POLY) entries(dq, a.ep_post, [&](int j) { return out_win(j) ? e_all : kOob; });
    constexpr bool CHECK = (POST == POST_GD || POST == POST_SPEC);  // the last update of a solve
    bool bad = false;
    if constexpr (POST_IS_GD) {
      if (a.step_v != nullptr && active) step = a.step_v[sp];
    }
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const bool ow = out_win(j);
      const unsigned ju = (unsigned)(j * u_step) * 8u, j4 = (unsigned)(j * g_step) * 4u;
      float2 val = cscale(v[j], s_out);
      const float2 qj = Dq(j);
      if constexpr (POST == POST_PHASE_CONJ_GT) {
        const float2 u1 = cmul(xo[j], qj);  // u_1 = D_1 U x at this position
        st1(r_gth, off(ow, g_lane + o_gt, 4), j4, gt[j] + (val.y * u1.x - val.x * u1.y));
      }
      val = cmulc(val, qj);
      if constexpr (POST == POST_GTV) {
        const float2 vb = cscale(xo[j], step);
        st1(r_gth, off(ow, g_lane + o_gt, 4), j4, gt[j] + (vb.x * val.y - vb.y * val.x));
        continue;
      }
      if constexpr (POST == POST_PHASE_CONJ_GT) {
        if (a.xadd != nullptr)
          val = cadd(ld2(rsrc(a.xadd - u_cut), off(ow, sp * a.s_xadd + u_lane, 8), ju), val);
      }
      if constexpr (POST_IS_GD) {
        val = make_float2(xo[j].x - step * val.x, xo[j].y - step * val.y);
      } else if constexpr (POST_IS_SPEC) {
        val = make_float2(s_prev * (a.step * val.x - a.two_lam * xo[j].x),
                          s_prev * (a.step * val.y - a.two_lam * xo[j].y));
        acc += ow ? cabs2(val) : 0.f;
      }
      st2(r_out, off(ow, u_lane + o_out, 8), ju, val);
      if constexpr (CHECK) bad |= ow && !finite2(val);
      if constexpr (POST_FWD) v[j] = ow ? cmul(val, qj) : make_float2(0.f, 0.f);  // zero outside the support
    }
    if constexpr (CHECK) flag_nonfinite(a.nf, bad);
  }

  if constexpr (POST_FWD) {
    // the next iteration's [U, D_1, F_0] into the compact buffer (full columns)
    T::template fft<false>(v, lds, ph, w, t, bl);
    const Rsrc r_o2 = rsrc(a.out2);
    const int o2ld = (int)a.out2_ld;
    const unsigned o = off(active, o_out2 + t * o2ld + b, 8);
#pragma unroll
    for (int j = 0; j < E; ++j) st2(r_o2, o, (unsigned)(j * ACT * o2ld) * 8u, cscale(v[j], s_out));
  }

  if constexpr (MID == MID_GD || MID == MID_GD_POIS || POST_IS_SPEC) {
    if (part_out != nullptr) {
      float sum = block_sum<T::THREADS>(acc, red);
      if (threadIdx.x == 0) part_out[tile] = sum;
    }
  }
}

// Whether a pass shape reads any phase diagonal.
template <int PRE, int MID, int POST>
constexpr bool pass_has_phase() {
  return PRE != PRE_NONE || MID == MID_PHASE || MID == MID_PHASE_CONJ || mid_rev_phase(MID) || POST != POST_STORE;
}

// pass_tile with the phase source picked at run time (the tables are set
// for every diagonal of a pass or for none), window-aware so that it serves
// every geometry.
template <int N, int B, bool COL, int PRE, int MID, bool FFT2, bool INV1, bool INV2, int POST, int EV = 0>
__device__ __forceinline__ void pass_tile_rt(const PassArgs& a, int tile, float2* lds, float* red, const float* part_in,
                                             int npart, float* part_out) {
  if constexpr (pass_has_phase<PRE, MID, POST>()) {
    if (a.ep_pre != nullptr || a.ep_mid != nullptr || a.ep_post != nullptr) {
      pass_tile<N, B, COL, PRE, MID, FFT2, INV1, INV2, POST, true, EV, true, true>(a, tile, lds, red, part_in, npart,
                                                                                  part_out);
      return;
    }
  }
  pass_tile<N, B, COL, PRE, MID, FFT2, INV1, INV2, POST, true, EV, false, true>(a, tile, lds, red, part_in, npart,
                                                                               part_out);
}

template <int N, int B, bool COL, int PRE, int MID, bool FFT2, bool INV1, bool INV2, int POST, bool DB = true,
          int EV = 0, bool TAB = false, bool WIN = false>
__global__ void __launch_bounds__((TileV<N, B, COL, DB, EV>::THREADS)) pass_kernel(const PassArgs a) {
  extern __shared__ float2 lds[];
  __shared__ float red[TileV<N, B, COL, DB, EV>::THREADS];
  pass_tile<N, B, COL, PRE, MID, FFT2, INV1, INV2, POST, DB, EV, TAB, WIN>(a, xcd_tile(blockIdx.x, gridDim.x), lds,
                                                                            red, a.part_in, a.npart, a.part_out);
}

}  // namespace sr
