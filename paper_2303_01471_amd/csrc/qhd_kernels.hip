// HIP kernels of the QHD split-operator engine (gfx950 / CDNA4) beside the 2-D step passes
// (qhd_kernels_axis.hip): the leapfrog stages of the QAA model, the 1-D steps, the row
// form of the readouts, uploads, and the per-chunk bookkeeping.
#include <climits>

#include "launch_util.h"
#include "line_fft.h"
#include "pass_common.h"
#include "qhd_internal.h"

namespace qhd {

// ------------------------------------------------------------------------------------
// Leapfrog stages of the QAA model (the paper's integrator for its baseline QAA).  The
// state stays in position space, R = psi.x, I = psi.y.  A stage applies
//     H v = a W^{-1} D0 W v + b f v,   D0 = d_x(u) + d_y(v), d(u) = 2 popcount(u) - bits,
// to its source component v and adds c H v to its target component, in two passes that
// use the separability of D0: the row pass stores u = a W_x^{-1} d_x W_x v + b f v into
// the class scratch buffer (same tiled layout as psi); the column pass adds
// a W_y^{-1} d_y W_y v and updates the target.  Lines in FP64.

template <int NX, int P>
__global__ void __launch_bounds__(256) k_lf_row_2d(const InstDev* __restrict__ inst, const int* __restrict__ nact_p, int ny_log2,
                                                   const float2* __restrict__ psi, const double* __restrict__ f,
                                                   float* __restrict__ scratch, int s, long long max_steps) {
  const int ninst = *nact_p;  // members active in this sub-step (device, set per chunk)
  constexpr int TPL = NX / P;
  constexpr int LPW = 256 / TPL;
  constexpr int BITS = ilog2_c(NX);
  const int ll = threadIdx.x / TPL, t = threadIdx.x % TPL;
  const long long total = (long long)ninst << ny_log2;
  long long begin, end;
  block_share(total, LPW, begin, end);
  for (long long l0 = begin; l0 < end; l0 += LPW) {
    const long long L = l0 + ll;
    const bool valid = L < end;
    const long long Lc = valid ? L : end - 1;
    int i = (int)(Lc >> ny_log2);
    const int y = (int)(Lc & ((1 << ny_log2) - 1));
    if constexpr (64 * P <= 8 * NX) i = __builtin_amdgcn_readfirstlane(i);  // as in the row pass
    const InstDev& I = inst[i];
    const bool active = valid && s < step_limit(I, max_steps);
    double a, b, c;
    bool kick;
    leapfrog_stage(I, I.steps_done + s, a, b, c, kick);
    const float2* __restrict__ pl = psi + I.psi_off;
    double v[P], h[P];
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const float2 z = pl[row_slot<NX, TPL>(t, q, y)];
      v[q] = kick ? z.x : z.y;
      h[q] = v[q];
    }
    line_wht<NX, P>(h, t);
#pragma unroll
    for (int q = 0; q < P; ++q) h[q] *= (double)(2 * __builtin_popcount(t + q * TPL) - BITS);
    line_wht<NX, P>(h, t);
    if (active) {
      const double* __restrict__ fl = f + I.psi_off;
      float* __restrict__ ul = scratch + I.psi_off;
      constexpr double kInvN = 1.0 / NX;
#pragma unroll
      for (int q = 0; q < P; ++q) {
        const long long o = row_slot<NX, TPL>(t, q, y);
        ul[o] = (float)fma(a * kInvN, h[q], b * fl[o] * v[q]);
      }
    }
  }
}

template <int NY, int P>
__global__ void __launch_bounds__(256) k_lf_col_2d(const InstDev* __restrict__ inst, const int* __restrict__ nact_p, int nx_log2,
                                                   float2* __restrict__ psi, const float* __restrict__ scratch, int s,
                                                   long long max_steps) {
  const int ninst = *nact_p;  // members active in this sub-step (device, set per chunk)
  using C = ColCfg<NY, P>;
  constexpr int TPL = C::TPL, ITEMS = C::ITEMS, NT = C::NT, STRIDE = C::STRIDE, SUBS = C::SUBS;
  constexpr int TILES = NY / 8;
  constexpr int BITS = ilog2_c(NY);
  __shared__ float2 lds[C::LINES * STRIDE];
  __shared__ float ulds[C::LINES * STRIDE];
  const int tid = threadIdx.x;
  const int line0 = tid / TPL, t = tid % TPL;
  const int nx = 1 << nx_log2, tc_log2 = nx_log2 - 3, tcols = nx >> 3;
  const long long total = (long long)ninst << tc_log2;
  long long begin, end;
  block_share(total, ITEMS, begin, end);
  for (long long g0 = begin; g0 < end; g0 += ITEMS) {
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      const long long g = g0 + it;
      if (g < end) {
        const int i = (int)(g >> tc_log2), tc = (int)(g & (tcols - 1));
        const InstDev& I = inst[i];
        if (s < step_limit(I, max_steps)) {
          const float4* __restrict__ src = reinterpret_cast<const float4*>(psi + I.psi_off) + tc * 32;
          const float4* __restrict__ srcu = reinterpret_cast<const float4*>(scratch + I.psi_off) + tc * 16;
          float2* __restrict__ dst = lds + it * 8 * STRIDE;
          float* __restrict__ dstu = ulds + it * 8 * STRIDE;
#pragma unroll
          for (int e = tid; e < TILES * 32; e += NT) {
            const int ty = e >> 5, w = e & 31;
            const float4 v = src[(long long)ty * tcols * 32 + w];
            const int y = ty * 8 + (w >> 2), xx = (w & 3) << 1;
            dst[xx * STRIDE + lds_slot(y)] = make_float2(v.x, v.y);
            dst[(xx + 1) * STRIDE + lds_slot(y)] = make_float2(v.z, v.w);
          }
#pragma unroll
          for (int e = tid; e < TILES * 16; e += NT) {
            const int ty = e >> 4, w = e & 15;
            const float4 v = srcu[(long long)ty * tcols * 16 + w];
            const int y = ty * 8 + (w >> 1), xx = (w & 1) << 2;
            dstu[xx * STRIDE + lds_slot(y)] = v.x;
            dstu[(xx + 1) * STRIDE + lds_slot(y)] = v.y;
            dstu[(xx + 2) * STRIDE + lds_slot(y)] = v.z;
            dstu[(xx + 3) * STRIDE + lds_slot(y)] = v.w;
          }
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int sub = 0; sub < SUBS; ++sub) {
      const int line = line0 + sub * (NT / TPL);
      float2* my = lds + line * STRIDE;
      const float* myu = ulds + line * STRIDE;
      // wave-uniform with at least 8 lanes per line, as in the staged column pass
      const long long g = g0 + (TPL >= 8 ? __builtin_amdgcn_readfirstlane(line / 8) : line / 8);
      const long long gc = g < end ? g : end - 1;
      const InstDev& I = inst[(int)(gc >> tc_log2)];
      double a, b, c;
      bool kick;
      leapfrog_stage(I, I.steps_done + s, a, b, c, kick);
      const bool twice = lf_joins_next(I, s, max_steps);
      double h[P];
#pragma unroll
      for (int q = 0; q < P; ++q) {
        const float2 z = my[lds_slot(t + q * TPL)];
        h[q] = kick ? z.x : z.y;
      }
      line_wht<NY, P>(h, t);
#pragma unroll
      for (int q = 0; q < P; ++q) h[q] *= (double)(2 * __builtin_popcount(t + q * TPL) - BITS);
      line_wht<NY, P>(h, t);
      constexpr double kInvN = 1.0 / NY;
#pragma unroll
      for (int q = 0; q < P; ++q) {
        const int slot = lds_slot(t + q * TPL);
        const double w = fma(a * kInvN, h[q], (double)myu[slot]);
        float2 z = my[slot];
        if (kick) z.y = (float)fma(c, w, (double)z.y);
        else z.x = (float)fma(c, w, (double)z.x);
        if (twice) z.y = (float)fma(c, w, (double)z.y);
        my[slot] = z;
      }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      const long long g = g0 + it;
      if (g < end) {
        const int i = (int)(g >> tc_log2), tc = (int)(g & (tcols - 1));
        const InstDev& I = inst[i];
        if (s < step_limit(I, max_steps)) {
          float4* __restrict__ dstg = reinterpret_cast<float4*>(psi + I.psi_off) + tc * 32;
          const float2* __restrict__ srcl = lds + it * 8 * STRIDE;
#pragma unroll
          for (int e = tid; e < TILES * 32; e += NT) {
            const int ty = e >> 5, w = e & 31;
            const int y = ty * 8 + (w >> 2), xx = (w & 3) << 1;
            const float2 p0 = srcl[xx * STRIDE + lds_slot(y)];
            const float2 p1 = srcl[(xx + 1) * STRIDE + lds_slot(y)];
            dstg[(long long)ty * tcols * 32 + w] = make_float4(p0.x, p0.y, p1.x, p1.y);
          }
        }
      }
    }
    __syncthreads();
  }
}

// The same for 64- and 128-point columns with a tile column per wavefront, lanes (t, column),
// straight to and from registers: the transforms cross lanes only inside the wavefront, so
// there is no LDS and no barrier, the whole tile column is in flight at once, and the values
// are those of the staged form bit by bit.  256 instances, us per stage, staged and
// this: 128^2 21.1 and 17.1, 64^2 9.6 and 7.4.
template <int NY>
__global__ void __launch_bounds__(256) k_lf_col_tw(const InstDev* __restrict__ inst, const int* __restrict__ nact_p, int nx_log2,
                                                   float2* __restrict__ psi, const float* __restrict__ scratch, int s,
                                                   long long max_steps) {
  const int ninst = *nact_p;  // members active in this sub-step (device, set per chunk)
  constexpr int P = NY / 8, BITS = ilog2_c(NY);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t = lane >> 3;
  const int tc_log2 = nx_log2 - 3, tcols = 1 << tc_log2;
  const long long total = (long long)ninst << tc_log2;
  long long begin, end;
  block_share(total, 4, begin, end);
  for (long long g = begin + wave; g < end; g += 4) {
    const int i = (int)(g >> tc_log2), tc = (int)(g & (tcols - 1));
    const InstDev& I = inst[i];
    if (!(s < step_limit(I, max_steps))) continue;
    double a, b, c;
    bool kick;
    leapfrog_stage(I, I.steps_done + s, a, b, c, kick);
    const bool twice = lf_joins_next(I, s, max_steps);
    const long long off = I.psi_off + ((long long)tc << 6);
    const LaneView<float2> pv(psi + off, lane);
    const float* __restrict__ uv = scratch + off;
    float2 z[P];
    float u[P];
#pragma unroll
    for (int q = 0; q < P; ++q) {
      z[q] = pv.load(q * tcols * 64);
      u[q] = uv[q * tcols * 64 + lane];
    }
    double h[P];
#pragma unroll
    for (int q = 0; q < P; ++q) h[q] = kick ? z[q].x : z[q].y;
    line_wht<NY, P, double, 8>(h, t);
#pragma unroll
    for (int q = 0; q < P; ++q) h[q] *= (double)(2 * __builtin_popcount(t + 8 * q) - BITS);
    line_wht<NY, P, double, 8>(h, t);
    constexpr double kInvN = 1.0 / NY;
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const double w = fma(a * kInvN, h[q], (double)u[q]);
      if (kick) z[q].y = (float)fma(c, w, (double)z[q].y);
      else z[q].x = (float)fma(c, w, (double)z[q].x);
      if (twice) z[q].y = (float)fma(c, w, (double)z[q].y);
      pv.store(q * tcols * 64, z[q]);
    }
  }
}

// ------------------------------------------------------------------------------------
// 1-D steps: V (merged halves) . F . K . F^{-1}, the state in position space with the
// trailing half step of the last step pending.  A line (TPL lanes of one wavefront) needs
// nothing from another, so one launch runs every sub-step of the chunk with psi and f in
// registers: a serial chain per line, bound by its latency (two transforms, their LDS
// exchanges and the phases), so blocks of one wavefront spread the lines over the CUs and a
// lane holds few points.  Us per step, one launch per step -> this kernel: one 8-point line
// 3.4 -> 1.2, 256 points 5.3 -> 1.7, 1024 points 10.4 -> 4.7; 200 lines of 256 5.8 -> 1.7.

// Points per lane: 4 while a line then fits one wavefront (256 points: 1.7 us a step, 2.6
// with 8; 5000 lines of 256, where the chip is full: 6.0 and 5.7), 8 and 16 above.
constexpr int line_step_points(int n) { return n <= 256 ? 4 : n / 64; }

template <int N, int P>
__global__ void __launch_bounds__(64) k_line_steps_1d(const InstDev* __restrict__ inst, const int* __restrict__ nact_p,
                                                      float2* __restrict__ psi,
                                                      const double* __restrict__ f,
                                                      const double2* __restrict__ twtab, long long max_steps) {
  const int ninst = *nact_p;  // members active in the chunk (device, set per chunk)
  constexpr int TPL = N / P;
  constexpr int LPW = 64 / TPL;
  constexpr int SLOTS = LineLds<N>::kSlots;
  __shared__ float2 lds[LPW * SLOTS];
  const int ll = threadIdx.x / TPL, t = threadIdx.x % TPL;
  float2* my = lds + ll * SLOTS;
  Twiddles<N, P> tw;
  tw.load(twtab, t);
  constexpr double inv_n = 1.0 / (double)N;
  for (long long l0 = (long long)blockIdx.x * LPW; l0 < ninst; l0 += (long long)gridDim.x * LPW) {
    const long long L = l0 + ll;
    if (L >= ninst) continue;  // (the lanes of a line leave together; no block barrier below)
    const InstDev& I = inst[(int)L];
    const long long lim = step_limit(I, max_steps), base = I.psi_off;
    float2 reg[P];
    double fv[P];
#pragma unroll
    for (int q = 0; q < P; ++q) {
      reg[q] = psi[base + t + q * TPL];
      fv[q] = f[base + t + q * TPL];
    }
    // b of the stage before, carried along (potential_turns evaluates the schedule twice)
    double a, b, b_prev = 0.0;
    if (I.steps_done > 0 && lim > 0) sched_ab(I, I.steps_done - 1, a, b_prev);
    for (long long s = 0; s < lim; ++s) {
      const long long j = I.steps_done + s;
      sched_ab(I, j, a, b);
      const double cpot = merged_turns(I, j, s == 0 && I.mode == kModeClean, b, b_prev);
      b_prev = b;
      const double ck = a * I.kin_turns[0];
#pragma unroll
      for (int q = 0; q < P; ++q) reg[q] = cmul_fd(reg[q], phase_turns_d(cpot * fv[q]));
      double2 kd[P];
      line_fft_io<N, P, -1>(reg, kd, t, tw, my);
#pragma unroll
      for (int q = 0; q < P; ++q) {
        const int nf = freq(t + q * TPL, N);
        const double2 w = phase_turns_d(ck * (double)(nf * nf));
        kd[q] = cmul_fd(kd[q], make_double2(w.x * inv_n, w.y * inv_n));
      }
      line_fft_io<N, P, +1>(kd, reg, t, tw, my);
    }
#pragma unroll
    for (int q = 0; q < P; ++q) psi[base + t + q * TPL] = reg[q];
  }
}

__global__ void k_chunk_plan(const InstDev* __restrict__ inst, int ninst, long long max_steps, int S,
                             int* __restrict__ nact) {
  for (int s = blockIdx.x * blockDim.x + threadIdx.x; s < S; s += gridDim.x * blockDim.x) {
    int n = 0;
    for (int k = ninst - 1; k >= 0; --k) {
      if (s < step_limit(inst[k], max_steps)) {
        n = k + 1;
        break;
      }
    }
    nact[s] = n;
  }
}

__global__ void k_reset_inst(InstDev* __restrict__ inst, int ninst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ninst) return;
  inst[i].steps_done = 0;
  inst[i].mode = kModeClean;
  inst[i].axis = 0;
}

__global__ void k_commit(InstDev* __restrict__ inst, int ninst, long long max_steps, bool alt) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ninst) return;
  const long long lim = step_limit(inst[i], max_steps);
  if (lim > 0) advance(inst[i], lim, alt);
}

// ------------------------------------------------------------------------------------
// Observe (readouts of App. B / Algorithm 1 / main-text fig. 2)

// deterministic sum over the TPL lanes of one line (lanes are contiguous)
template <int TPL>
__device__ __forceinline__ double line_sum(double v) {
#pragma unroll
  for (int o = TPL / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

template <int NX, int P, int MODEL = kModelQHD>
__global__ void __launch_bounds__(256) k_observe_2d(const InstDev* __restrict__ inst, int ninst,
                                                    int ny_log2, int slab_log2,
                                                    const float2* __restrict__ psi,
                                                    const double* __restrict__ f,
                                                    const double2* __restrict__ twtab,
                                                    float2* __restrict__ out_psi,
                                                    float* __restrict__ out_rho,
                                                    double* __restrict__ partials, int stride) {
  constexpr int TPL = NX / P;
  constexpr int LPW = 256 / TPL;
  constexpr int SLOTS = LineLds<NX>::kSlots;
  __shared__ float2 lds[LPW * SLOTS];
  const int ll = threadIdx.x / TPL, t = threadIdx.x % TPL;
  float2* my = lds + ll * SLOTS;
  Twiddles<NX, P> tw;
  tw.load(twtab, t);
  const long long total = (long long)ninst << ny_log2;
  for (long long l0 = (long long)blockIdx.x * LPW; l0 < total; l0 += (long long)gridDim.x * LPW) {
    const long long L = l0 + ll;
    const bool valid = L < total;
    const long long Lc = valid ? L : total - 1;
    const int i = (int)(Lc >> ny_log2), y = (int)(Lc & ((1 << ny_log2) - 1));
    const InstDev& I = inst[i];
    if (I.mode == kModeOweY) continue;  // the column form's
    // leapfrog keeps the state in position space, in step with the clock
    const bool pending = I.mode != kModeClean && I.scheme != kSchemeLeapfrog;
    const long long base = I.psi_off;
    float2 reg[P];
#pragma unroll
    for (int q = 0; q < P; ++q) reg[q] = psi[base + tile_index(t + q * TPL, y, NX)];
    double fv[P];
#pragma unroll
    for (int q = 0; q < P; ++q) fv[q] = f[base + tile_index(t + q * TPL, y, NX)];
    if (pending) {
      // the line operator along x of the last stage where it is owed (matrix-core classes:
      // back to position space); the symmetric scheme also owes the trailing half step
      double2 in[P];
#pragma unroll
      for (int q = 0; q < P; ++q) assign(in[q], reg[q]);
      if (I.mode == kModeOweX) {
        double a, b;
        sched_ab(I, I.steps_done - 1, a, b);
        if constexpr (MODEL == kModelQAA) line_wht<NX, P>(in, t);
        else line_fft_io<NX, P, -1>(reg, in, t, tw, my);
#pragma unroll
        for (int q = 0; q < P; ++q) {
          const double2 e = phase_turns_d(a * axis_turns<MODEL>(I, 0, t + q * TPL, NX));
          in[q] = cmul_fd(in[q], make_double2(e.x * (1.0 / NX), e.y * (1.0 / NX)));
        }
      }
      if (I.mode == kModeOweX || I.mode == kModePending) {
        if constexpr (MODEL == kModelQAA) {
          line_wht<NX, P>(in, t);
#pragma unroll
          for (int q = 0; q < P; ++q) assign(reg[q], in[q]);
        } else {
          line_fft_io<NX, P, +1>(in, reg, t, tw, my);
        }
      }
      if (I.scheme != kSchemeLie) {
        const double cpot = closing_turns(I);
#pragma unroll
        for (int q = 0; q < P; ++q) reg[q] = cmul_fd(reg[q], phase_turns_d(cpot * fv[q]));
      }
    }
    const long long rs = I.argmin / NX;
    const int xs = (int)(I.argmin % NX);
    const int ys = (int)(rs & ((1 << slab_log2) - 1)), zs = (int)(rs >> slab_log2);
    const int yy = y & ((1 << slab_log2) - 1), zz = y >> slab_log2;
    double sr = 0.0, sf = 0.0, sm = 0.0;
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const int x = t + q * TPL;
      const float2 v = reg[q];
      const double rho = (double)v.x * v.x + (double)v.y * v.y;
      sr += rho;
      sf += fv[q] * rho;
      if (in_ball(x - xs, yy - ys, zz - zs, I)) sm += rho;
      if (valid) {
        const long long o = I.out_off + (long long)y * NX + x;
        if (out_psi) out_psi[o] = v;
        if (out_rho) out_rho[o] = (float)rho;
      }
    }
    sr = line_sum<TPL>(sr);
    sf = line_sum<TPL>(sf);
    sm = line_sum<TPL>(sm);
    if (valid && t == 0) {
      double* pt = partials + 3 * ((long long)i * stride + y);
      pt[0] = sr;
      pt[1] = sf;
      pt[2] = sm;
    }
  }
}

template <int N, int P>
__global__ void __launch_bounds__(256) k_observe_1d(const InstDev* __restrict__ inst, int ninst,
                                                    const float2* __restrict__ psi,
                                                    const double* __restrict__ f,
                                                    float2* __restrict__ out_psi,
                                                    float* __restrict__ out_rho,
                                                    double* __restrict__ partials) {
  constexpr int TPL = N / P;
  constexpr int LPW = (256 / TPL) > 0 ? 256 / TPL : 1;
  const int ll = threadIdx.x / TPL, t = threadIdx.x % TPL;
  for (long long l0 = (long long)blockIdx.x * LPW; l0 < ninst; l0 += (long long)gridDim.x * LPW) {
    const long long L = l0 + ll;
    const bool valid = L < ninst;
    const int i = (int)(valid ? L : ninst - 1);
    const InstDev& I = inst[i];
    // the symmetric scheme leaves its trailing half step pending; the first-order
    // product leaves nothing
    const bool close = I.mode == kModePending && I.scheme != kSchemeLie;
    const double cpot = close ? closing_turns(I) : 0.0;
    const int xs = (int)I.argmin;
    double sr = 0.0, sf = 0.0, sm = 0.0;
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const int x = t + q * TPL;
      const long long p = I.psi_off + x;
      const double fv = f[p];
      float2 v = psi[p];
      if (close) v = cmul_fd(v, phase_turns_d(cpot * fv));
      const double rho = (double)v.x * v.x + (double)v.y * v.y;
      sr += rho;
      sf += fv * rho;
      const double dx = __dmul_rn((double)(x - xs), I.h[0]);
      if (__dmul_rn(dx, dx) < I.r2) sm += rho;
      if (valid) {
        const long long o = I.out_off + x;
        if (out_psi) out_psi[o] = v;
        if (out_rho) out_rho[o] = (float)rho;
      }
    }
    sr = line_sum<TPL>(sr);
    sf = line_sum<TPL>(sf);
    sm = line_sum<TPL>(sm);
    if (valid && t == 0) {
      partials[3 * L + 0] = sr;
      partials[3 * L + 1] = sf;
      partials[3 * L + 2] = sm;
    }
  }
}

// Fixed-order compensated sum of each instance's line partials, one block per instance:
// every thread sums a contiguous run of lines (Neumaier), then the 256 runs are combined
// pairwise in a fixed tree (sums and compensations separately), so the result does not
// depend on timing.
__device__ __forceinline__ void neumaier_add(double& s, double& comp, double v) {
  const double t = s + v;
  comp += (fabs(s) >= fabs(v)) ? ((s - t) + v) : ((v - t) + s);
  s = t;
}

__global__ void __launch_bounds__(256) k_finalize(const InstDev* __restrict__ inst, const double* __restrict__ partials,
                                                  int lines_x, int lines_y, int stride, double* __restrict__ results) {
  __shared__ double ss[3][256], sc[3][256];
  const int i = blockIdx.x;
  const int lines = inst[i].mode == kModeOweY ? lines_y : lines_x;
  const int per = (lines + 255) / 256;
  const int l0 = threadIdx.x * per, l1 = l0 + per < lines ? l0 + per : lines;
  double s[3] = {0.0, 0.0, 0.0}, comp[3] = {0.0, 0.0, 0.0};
  for (int l = l0; l < l1; ++l) {
    const double* pl = partials + 3 * ((long long)i * stride + l);
#pragma unroll
    for (int c = 0; c < 3; ++c) neumaier_add(s[c], comp[c], pl[c]);
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    ss[c][threadIdx.x] = s[c];
    sc[c][threadIdx.x] = comp[c];
  }
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        double a = ss[c][threadIdx.x], ca = sc[c][threadIdx.x] + sc[c][threadIdx.x + o];
        neumaier_add(a, ca, ss[c][threadIdx.x + o]);
        ss[c][threadIdx.x] = a;
        sc[c][threadIdx.x] = ca;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < 3) results[3 * i + threadIdx.x] = ss[threadIdx.x][0] + sc[threadIdx.x][0];
}

// ------------------------------------------------------------------------------------
// uploads

__global__ void k_import_f_2d(const double* __restrict__ user, double* __restrict__ dst, int nx,
                              int ny) {
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= (long long)nx * ny) return;
  const int x = (int)(p % nx), y = (int)(p / nx);
  dst[tile_index(x, y, nx)] = user[p];
}

__global__ void k_import_psi_2d(const float2* __restrict__ user, float2* __restrict__ dst, int nx,
                                int ny) {
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= (long long)nx * ny) return;
  const int x = (int)(p % nx), y = (int)(p / nx);
  dst[tile_index(x, y, nx)] = user[p];
}

__global__ void k_copy_f(const double* __restrict__ src, double* __restrict__ dst, long long n) {
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p < n) dst[p] = src[p];
}

__global__ void k_copy_psi(const float2* __restrict__ src, float2* __restrict__ dst, long long n) {
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p < n) dst[p] = src[p];
}

__global__ void k_fill(float2* __restrict__ dst, long long n, float v) {
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p < n) dst[p] = make_float2(v, 0.0f);
}

// lowest-index minimiser; also counts non-finite entries.  Stage 1: every block reduces a
// contiguous share of f to (value, index, non-finite count); stage 2: one block reduces
// the blocks' partials.  Ties go to the lower index in both stages, so the result is the
// lowest-index minimiser whatever the block count.
__device__ __forceinline__ void argmin_merge(double& v, long long& i, double v2, long long i2) {
  if (v2 < v || (v2 == v && i2 < i)) {
    v = v2;
    i = i2;
  }
}

template <int NT>
__device__ __forceinline__ void argmin_block(double bv, long long bi, long long bad, double* sv, long long* si,
                                             long long* sbad) {
  sv[threadIdx.x] = bv;
  si[threadIdx.x] = bi;
  sbad[threadIdx.x] = bad;
  __syncthreads();
  for (int o = NT / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      double v = sv[threadIdx.x];
      long long id = si[threadIdx.x];
      argmin_merge(v, id, sv[threadIdx.x + o], si[threadIdx.x + o]);
      sv[threadIdx.x] = v;
      si[threadIdx.x] = id;
      sbad[threadIdx.x] += sbad[threadIdx.x + o];
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(256) k_argmin_partial(const double* __restrict__ f, long long n,
                                                        double* __restrict__ part_val,
                                                        long long* __restrict__ part_idx,
                                                        long long* __restrict__ part_bad) {
  __shared__ double sv[256];
  __shared__ long long si[256], sbad[256];
  const long long per = (n + gridDim.x - 1) / gridDim.x;
  const long long b0 = (long long)blockIdx.x * per, b1 = b0 + per < n ? b0 + per : n;
  double bv = INFINITY;
  long long bi = LLONG_MAX, bad = 0;
  for (long long p = b0 + threadIdx.x; p < b1; p += 256) {
    const double v = f[p];
    if (!isfinite(v)) {
      ++bad;
      continue;
    }
    argmin_merge(bv, bi, v, p);
  }
  argmin_block<256>(bv, bi, bad, sv, si, sbad);
  if (threadIdx.x == 0) {
    part_val[blockIdx.x] = sv[0];
    part_idx[blockIdx.x] = si[0];
    part_bad[blockIdx.x] = sbad[0];
  }
}

__global__ void __launch_bounds__(kArgminBlocks) k_argmin_final(const double* __restrict__ part_val,
                                                                const long long* __restrict__ part_idx,
                                                                const long long* __restrict__ part_bad,
                                                                double* __restrict__ out_val,
                                                                long long* __restrict__ out_idx) {
  __shared__ double sv[kArgminBlocks];
  __shared__ long long si[kArgminBlocks], sbad[kArgminBlocks];
  argmin_block<kArgminBlocks>(part_val[threadIdx.x], part_idx[threadIdx.x], part_bad[threadIdx.x], sv, si, sbad);
  if (threadIdx.x == 0) {
    out_val[0] = sv[0];
    out_idx[0] = si[0];
    out_idx[1] = sbad[0];
  }
}

// ------------------------------------------------------------------------------------
// launchers

hipError_t launch_lf_row_2d(int nx, int ny, const InstDev* inst, int ninst, const int* nact, const float2* psi, const double* f,
                            float* scratch, int s, long long max_steps, int grid_cap, hipStream_t stream) {
  const int blocks = pass_blocks_row_2d(nx, ny, ninst, grid_cap, 8);
  QHD_SWITCH_N(nx, {
    constexpr int P_ = pts_per_lane<N_>();
    QHD_LAUNCH((k_lf_row_2d<N_, P_>), dim3(blocks), dim3(256), 0, stream, inst, nact, ilog2(ny), psi, f,
                       scratch, s, max_steps);
    return hipGetLastError();
  });
}

hipError_t launch_lf_col_2d(int nx, int ny, const InstDev* inst, int ninst, const int* nact, float2* psi, const float* scratch, int s,
                            long long max_steps, int grid_cap, hipStream_t stream) {
  QHD_SWITCH_N(ny, {
    if constexpr (N_ == 64 || N_ == 128) {
      const int blocks = blocks_for((long long)ninst * (nx / 8), 4, grid_cap);
      QHD_LAUNCH((k_lf_col_tw<N_>), dim3(blocks), dim3(256), 0, stream, inst, nact, ilog2(nx), psi, scratch, s,
                 max_steps);
    } else {
      constexpr int P_ = pts_per_lane<N_>();
      const int blocks = pass_blocks_col_2d(nx, ny, ninst, grid_cap, kColStaged);
      QHD_LAUNCH((k_lf_col_2d<N_, P_>), dim3(blocks), dim3(ColCfg<N_, P_>::NT), 0, stream, inst, nact,
                 ilog2(nx), psi, scratch, s, max_steps);
    }
    return hipGetLastError();
  });
}

hipError_t launch_line_steps_1d(int n, const InstDev* inst, int ninst, const int* nact, float2* psi, const double* f,
                                const double2* tw, long long max_steps, int grid_cap, hipStream_t stream) {
  QHD_SWITCH_N(n, {
    constexpr int P_ = line_step_points(N_);
    const int blocks = blocks_for(ninst, 64 / (N_ / P_), grid_cap);
    QHD_LAUNCH((k_line_steps_1d<N_, P_>), dim3(blocks), dim3(64), 0, stream, inst, nact, psi, f, tw, max_steps);
    return hipGetLastError();
  });
}

hipError_t launch_commit(InstDev* inst, int ninst, long long max_steps, bool alt, hipStream_t stream) {
  QHD_LAUNCH(k_commit, dim3((ninst + 255) / 256), dim3(256), 0, stream, inst, ninst,
                     max_steps, alt);
  return hipGetLastError();
}

hipError_t launch_chunk_plan(const InstDev* inst, int ninst, long long max_steps, int S, int* nact,
                             hipStream_t stream) {
  if (S <= 0) return hipSuccess;
  QHD_LAUNCH(k_chunk_plan, dim3((S + 255) / 256), dim3(256), 0, stream, inst, ninst, max_steps, S, nact);
  return hipGetLastError();
}

hipError_t launch_reset_inst(InstDev* inst, int ninst, hipStream_t stream) {
  QHD_LAUNCH(k_reset_inst, dim3((ninst + 255) / 256), dim3(256), 0, stream, inst, ninst);
  return hipGetLastError();
}

hipError_t launch_observe_2d(int nx, int rows, int ny, const InstDev* inst, int ninst,
                             const float2* psi, const double* f, const double2* tw,
                             float2* out_psi, float* out_rho, double* partials, int stride,
                             hipStream_t stream, int model) {
  QHD_SWITCH_N(nx, {
    constexpr int P_ = pts_per_lane<N_>();
    constexpr int LPW_ = 256 / (N_ / P_);
    const int blocks = blocks_for((long long)ninst * rows, LPW_, 4096);
    if (model == kModelQAA)
      QHD_LAUNCH((k_observe_2d<N_, P_, kModelQAA>), dim3(blocks), dim3(256), 0, stream, inst, ninst,
                         ilog2(rows), ilog2(ny), psi, f, tw, out_psi, out_rho, partials, stride);
    else
      QHD_LAUNCH((k_observe_2d<N_, P_>), dim3(blocks), dim3(256), 0, stream, inst, ninst,
                         ilog2(rows), ilog2(ny), psi, f, tw, out_psi, out_rho, partials, stride);
    return hipGetLastError();
  });
}

hipError_t launch_observe_1d(int n, const InstDev* inst, int ninst, const float2* psi,
                             const double* f, float2* out_psi, float* out_rho, double* partials,
                             hipStream_t stream) {
  QHD_SWITCH_N(n, {
    constexpr int P_ = pts_per_lane<N_>();
    constexpr int TPL_ = N_ / P_;
    constexpr int LPW_ = (256 / TPL_) > 0 ? 256 / TPL_ : 1;
    const int blocks = blocks_for(ninst, LPW_, 4096);
    QHD_LAUNCH((k_observe_1d<N_, P_>), dim3(blocks), dim3(256), 0, stream, inst, ninst,
                       psi, f, out_psi, out_rho, partials);
    return hipGetLastError();
  });
}

hipError_t launch_finalize(const InstDev* inst, const double* partials, int lines, int lines_y, int stride, int ninst,
                           double* results, hipStream_t stream) {
  QHD_LAUNCH(k_finalize, dim3(ninst), dim3(256), 0, stream, inst, partials, lines, lines_y, stride, results);
  return hipGetLastError();
}

hipError_t launch_import_f(int ndim, int nx, int ny, const double* user, double* dst,
                           hipStream_t stream) {
  const long long n = (long long)nx * ny;
  const int blocks = (int)((n + 255) / 256);
  if (ndim == 2)
    QHD_LAUNCH(k_import_f_2d, dim3(blocks), dim3(256), 0, stream, user, dst, nx, ny);
  else
    QHD_LAUNCH(k_copy_f, dim3(blocks), dim3(256), 0, stream, user, dst, n);
  return hipGetLastError();
}

hipError_t launch_import_psi(int ndim, int nx, int ny, const float2* user, float2* dst,
                             hipStream_t stream) {
  const long long n = (long long)nx * ny;
  const int blocks = (int)((n + 255) / 256);
  if (ndim == 2)
    QHD_LAUNCH(k_import_psi_2d, dim3(blocks), dim3(256), 0, stream, user, dst, nx, ny);
  else
    QHD_LAUNCH(k_copy_psi, dim3(blocks), dim3(256), 0, stream, user, dst, n);
  return hipGetLastError();
}

hipError_t launch_fill_psi(float2* dst, long long count, float value, hipStream_t stream) {
  const int blocks = (int)((count + 255) / 256);
  QHD_LAUNCH(k_fill, dim3(blocks), dim3(256), 0, stream, dst, count, value);
  return hipGetLastError();
}

hipError_t launch_argmin(const double* f, long long count, double* out_val, long long* out_idx, double* part_val,
                         long long* part_idx, long long* part_bad, hipStream_t stream) {
  QHD_LAUNCH(k_argmin_partial, dim3(kArgminBlocks), dim3(256), 0, stream, f, count, part_val, part_idx,
                     part_bad);
  QHD_LAUNCH(k_argmin_final, dim3(1), dim3(kArgminBlocks), 0, stream, part_val, part_idx, part_bad, out_val,
                     out_idx);
  return hipGetLastError();
}

}  // namespace qhd
