// The line operator of an alternating pass (see qhd_kernels_axis.hip): F^{-1} E F along one
// mesh line, E the kinetic factor of one axis, and what a line does in a sub-step.
#pragma once

#include "line_fft.h"
#include "pass_common.h"
#include "qhd_internal.h"

namespace qhd {

// entries of one kinetic-factor table of an axis of N points
template <int N, int MODEL>
__host__ __device__ constexpr int etab_len() {
  return MODEL == kModelQAA ? ilog2_c(N) + 1 : N / 2 + 1;
}

// Tables E(a0) then E(a1) of one instance, by the whole block (the caller synchronises around
// it).  The two entries of |frequency| N / 2 come last: a block of N threads or half as many has
// whole rounds before them.  (As fourth powers of the entries of N / 4 they cost no round, but
// carried four times those entries' error: 3.6e-7 rad a step, 1.1e-7 by their own angle.)
template <int N, int MODEL>
__device__ __forceinline__ void fill_etab_pair(double2* __restrict__ tab, const InstDev& I, int axis, double a0, double a1) {
  constexpr int H = etab_len<N, MODEL>();
  constexpr int R = MODEL == kModelQAA ? H : N / 2;  // entries per table before the last ones
  constexpr double inv_n = 1.0 / N;
  const double unit = MODEL == kModelQAA ? I.dt * kInv2Pi : I.kin_turns[axis];
  for (int e = threadIdx.x; e < 2 * H; e += blockDim.x) {
    const bool last = e >= 2 * R;
    const int cur = last ? e - 2 * R : (e >= R ? 1 : 0), k = last ? R : e - cur * R;
    const double c = (cur ? a1 : a0) * unit;
    const double turns = c * (double)(MODEL == kModelQAA ? 2 * k - ilog2_c(N) : k * k);
    // 128-point axes by the exact angle (state error of 8 x 128^2 after 600 steps 3.5e-6 -> 1.8e-6,
    // with a constant schedule 5.8e-6 -> 1.5e-6; 262 x 128^2 32.9 -> 33.2 us per step); at other
    // lengths the errors stand below those of separate axis passes without it, and it costs
    // registers (512-point columns 78 -> 104) or latency (one 64^2 instance +0.9 us)
    double2 v;
    if constexpr (N == 128) v = phase_turns_exact(turns);
    else v = phase_turns_d(turns);
    tab[cur * H + k] = make_double2(v.x * inv_n, v.y * inv_n);
  }
}

// Tables of instances i0 .. i0 + count - 1: per instance E(a_{j-1}) then E(a_j), j = the
// stage of sub-step s
template <int N, int MODEL, bool Y4>
__device__ __forceinline__ void fill_etab(double2* __restrict__ tab, const InstDev* __restrict__ inst, int i0, int count,
                                          int axis, long long s) {
  for (int d = 0; d < count; ++d, tab += 2 * etab_len<N, MODEL>()) {
    const InstDev& I = inst[i0 + d];
    const long long j = I.steps_done + s;
    double a0, a1, b;
    sched_ab<Y4>(I, j - 1, a0, b);
    sched_ab<Y4>(I, j, a1, b);
    fill_etab_pair<N, MODEL>(tab, I, axis, a0, a1);
  }
}

// multiply the transformed line's slots t + q TPL by their factors
template <int N, int P, typename W>
__device__ __forceinline__ void mul_kinetic(W (&reg)[P], int t, const double2* __restrict__ tab) {
  constexpr int TPL = N / P;
  const double2* __restrict__ up = tab + t;        // |freq| = t + q TPL below N / 2
  const double2* __restrict__ down = tab + N - t;  // and N - (t + q TPL) from there
#pragma unroll
  for (int q = 0; q < P; ++q) reg[q] = cmul_fd(reg[q], q < P / 2 ? up[q * TPL] : down[-q * TPL]);
}
template <int N, int P>
__device__ __forceinline__ void mul_field(double2 (&reg)[P], int t, const double2* __restrict__ tab) {
  // popcount(t + q TPL) = popcount(t) + popcount(q)
  const double2* __restrict__ b = tab + __builtin_popcount(t);
#pragma unroll
  for (int q = 0; q < P; ++q) reg[q] = cmul_fd(reg[q], b[__builtin_popcount(q)]);
}

// Where a line works in FP64 beside its twiddle and factor products.  K, the frequency-space ends
// of the line operators (the last forward and the first inverse stage and the kinetic factor):
// always.  V, the position-space ends (the last inverse and the first forward stage and the
// potential factor): lines of 128 and 256 points.  XI, the stages and exchanges between on the
// way back to position space: 128 points.
// Early in a run every line of a near-uniform state concentrates into one coefficient and is
// rounded alike, late the state is localised; FP32 rounding of such values moves the norm, and
// alike-rounded values move it all one way.  Where all four ends are FP64 the two exchanges are
// what is left: a value that comes back through both is rounded twice and walks by a unit in the
// last place per pass, through one it comes back to itself.
// Largest norm drift of the 768-instance batch per 1e4 steps, and state error of 8 x 128^2 after
// 600 steps (4 x 256^2 after 400): separate axis passes (K for columns, all four ends for
// 128-point rows) 128^2 5.5e-6, 4.3e-6; 256^2 5.2e-6, 3.4e-6.  128^2 with K alone 1.3e-5; V
// alone 6.9e-6, 3.4e-6; both ends 1.5e-5, 2.1e-6; and XI 4.9e-6, 1.9e-6 (the exchange towards
// frequency space instead 4.0e-6, 1.4e-6 but 8 % longer; both 3.7e-6, 1.1e-6 and 11 %).  256^2
// with K 8.9e-6, 3.2e-6, with both ends 4.0e-6, 2.7e-6 (3 % longer).  512^2 with K 4.1e-6 (5.4e-6
// separate; both ends 2.6e-6, 3 % longer).  (With the factors of N / 2 by their own angle the
// chosen ones are 4.1e-6, 3.0e-6 and 4.3e-6 at 128^2, 256^2 and 512^2.)
template <int N>
struct LinePrec {
  using V = typename std::conditional<N == 128 || N == 256, double2, float2>::type;
  using K = double2;
  using XI = typename std::conditional<N == 128, double2, float2>::type;
};

// Twiddles of a line.  128 points with 16 per lane: radices 8 and 16 in this order: the first
// stage's scatter then puts neighbouring lanes on other banks where a line is a column of an
// array of odd stride (512 resident 128^2, us per step, radices 16 and 8: 56, so 46; rows and
// streamed columns 1 % longer).
template <int N, int P>
using LineTwiddles = typename std::conditional<N == 128 && P == 16, TwiddlesLds<N, P, TwPow<N, P>::value, 8>,
                                               TwiddlesFor<N, P>>::type;
template <int N, int P>
struct LineTwSize {
  static constexpr int value = TwLdsSize<N, P>::value;
};
template <>
struct LineTwSize<128, 16> {
  static constexpr int value = LineTwiddles<128, 16>::kEntries;
};

// F^{-1} E F of one line, from `in` to `out` (float2 or double2: the type of the first and
// of the last stage; they may be the same array)
template <int N, int P, bool BLOCK_SYNC, typename IX, typename TIN, typename TOUT, typename TW>
__device__ __forceinline__ void line_kinetic(TIN (&in)[P], TOUT (&out)[P], int t, const TW& tw,
                                             float2* __restrict__ lds, const double2* __restrict__ tab) {
  typename LinePrec<N>::K k[P];
  line_fft_io<N, P, -1, BLOCK_SYNC, IX>(in, k, t, tw, lds);
  mul_kinetic<N, P>(k, t, tab);
  line_fft_io<N, P, +1, BLOCK_SYNC, IX, typename LinePrec<N>::XI>(k, out, t, tw, lds);
}

// A line's whole pass: the owed operator, the potential factor (fget(q): f of slot q) and
// this step's operator; kPassFixUp: the owed operator alone.  (It is set only in general launches,
// but tested in all: the branch keeps the loads of f behind the owed operator.  Without it 128-point
// rows take 180 registers instead of 148, and 1024 x 128^2 run 107 us a step instead of 95.)
template <int N, int P, bool BLOCK_SYNC, typename IX, typename TW, typename F>
__device__ __forceinline__ void line_pass(float2 (&reg)[P], int t, const TW& tw, float2* __restrict__ lds,
                                          const double2* __restrict__ tab, bool prev, double cpot, int kind, F&& fget) {
  constexpr int H = etab_len<N, kModelQHD>();
  typename LinePrec<N>::V x[P];
  if (prev) {
    line_kinetic<N, P, BLOCK_SYNC, IX>(reg, x, t, tw, lds, tab);
  } else {
#pragma unroll
    for (int q = 0; q < P; ++q) assign(x[q], reg[q]);
  }
  if (kind != kPassFixUp) {
#pragma unroll
    for (int q = 0; q < P; ++q) x[q] = cmul_fd(x[q], phase_turns_d(cpot * fget(q)));
    line_kinetic<N, P, BLOCK_SYNC, IX>(x, x, t, tw, lds, tab + H);
  }
#pragma unroll
  for (int q = 0; q < P; ++q) assign(reg[q], x[q]);
}

template <int N, int P, int LS = 1>
__device__ __forceinline__ void line_field(double2 (&reg)[P], int t, const double2* __restrict__ tab) {
  line_wht<N, P, double2, LS>(reg, t);
  mul_field<N, P>(reg, t, tab);
  line_wht<N, P, double2, LS>(reg, t);
}

// What a line does in sub-step s in a launch of axis `axis`.  GEN, the general form of a pass: the
// stages of the fourth-order scheme, mixed launches (members on either axis: those whose turn it
// is take their whole pass, the others theirs in a launch of the other axis) and fix-up launches
// (only the owed operator, of the members that owe it).  In a plain launch every member takes its
// axis: the test of the member's own one cost 0.5 to 1 % (one 64^2 instance, 128^2 x 1024).
struct LineTask {
  bool active, prev, entry;
  double cpot;  // turns per unit f of the merged potential factor
};
template <bool GEN>
__device__ __forceinline__ bool line_active(const InstDev& I, long long s, long long max_steps, int axis, int kind) {
  if (GEN && kind == kPassFixUp) return pays_owed(I, axis == 0 ? kModeOweX : kModeOweY);
  if (GEN && kind == kPassMixed && ((I.axis + s) & 1) != axis) return false;
  return s < step_limit(I, max_steps);
}
template <bool GEN>
__device__ __forceinline__ LineTask line_task(const InstDev& I, long long s, long long max_steps, int axis, int kind) {
  LineTask k;
  k.prev = s > 0 || I.mode == (axis == 0 ? kModeOweX : kModeOweY);
  k.entry = s == 0 && I.mode == kModeClean;
  k.active = line_active<GEN>(I, s, max_steps, axis, kind);
  k.cpot = potential_turns<GEN>(I, I.steps_done + s, k.entry);
  return k;
}

}  // namespace qhd
