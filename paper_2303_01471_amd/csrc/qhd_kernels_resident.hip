// Resident 2-D QHD steps (gfx950): one workgroup owns an instance of at most 128 x 128
// points for a whole evolve call.
//
// The steps are those of the alternating passes (qhd_kernels_axis.hip; App. C.2.1, eq.
// prod_qhd_fft; App. E.1, Algorithm 1 in its symmetric form with midpoint coefficients): a
// step takes one axis, the line operator owed from the step before, the merged potential
// half steps and its own operator.  Here the state stays in LDS across all the steps of the
// call: it is read from HBM once at the start (8x8-tiled layout), every step runs out of
// LDS with one block barrier, and it is written back once at the end, so a step moves no
// HBM bytes for psi (f, FP64, is re-read every step and stays in L2 / the last-level cache).
// Small instances, whose streaming passes are bound by launch latency, run at the speed of
// one CU.
//
// LDS layout: row-major, point (x, y) at y * RS + slot(x), slot(x) = x + x / 8 (one pad
// entry per 8, as the line transforms' exchange buffers use), RS odd, so both a row
// (contiguous, padded) and a column (stride RS) are exchanged in place: a line loads
// its points into registers, and its own storage then serves as the exchange buffer
// of its transforms.  The QAA model (App. E.2's baseline) runs the same steps with FP64
// Walsh-Hadamard lines, which need no LDS exchange.  Every line gives the values of the
// streaming passes bit for bit (of the forms with 16 points per lane where it has 128).
#include "axis_line.h"
#include "line_fft.h"
#include "pass_common.h"
#include "qhd_internal.h"

namespace qhd {

// MANY (128 x 32 and 32 x 128, more members than CUs): 256 threads, so that two instances fit a
// CU beside each other (us per step, 512 and 256 threads: 2000 x 128 x 32 53 and 42, 2000 x 32 x
// 128 47 and 38; one instance 6.6 and 7.6, 5.9 and 6.4)
template <int NX, int NY, int MODEL, bool MANY>
struct ResCfg {
  // 128-point lines take 16 points per lane (radices 8 and 16: one exchange per transform)
  static constexpr int PX = NX >= 128 ? 16 : 8, PY = NY >= 128 ? 16 : 8;
  static constexpr int TX = NX / PX, TY = NY / PY;             // lanes per row / column line
  static constexpr int LANES = NX * NY / PX > NX * NY / PY ? NX * NY / PX : NX * NY / PY;
  // 16 points need more than the 128 registers of a 1024-thread block (1024 and 512 threads, us
  // per step: 1000 x 128 x 64 64 and 42, 1000 x 64 x 128 62 and 42, 512 x 128^2 57 and 46)
  static constexpr int MAXT = MANY ? 256 : PX == 16 || PY == 16 ? 512 : 1024;
  static constexpr int NT = LANES < MAXT ? LANES : MAXT;
  static constexpr int RS = ((NX + NX / 8) | 1);               // row stride in slots (odd)
  static constexpr int ROWS_PER_IT = NT / TX, COLS_PER_IT = NT / TY;
  static_assert(NX >= 32 && NY >= 32 && NX <= 128 && NY <= 128, "resident sizes: 32..128 per axis");
};

template <int NX, int NY, int MODEL, bool Y4, bool MANY>
__global__ void __launch_bounds__((ResCfg<NX, NY, MODEL, MANY>::NT)) k_resident_2d(const InstDev* __restrict__ inst, const int* __restrict__ nact_p,
                                                                     float2* __restrict__ psi,
                                                                     const double* __restrict__ f,
                                                                     const double2* __restrict__ twx,
                                                                     const double2* __restrict__ twy,
                                                                     long long max_steps) {
  const int ninst = *nact_p;  // members active in this sub-step (device, set per chunk)
  using C = ResCfg<NX, NY, MODEL, MANY>;
  constexpr int PX = C::PX, PY = C::PY, TX = C::TX, TY = C::TY, NT = C::NT, RS = C::RS;
  constexpr int HX = etab_len<NX, MODEL>(), HY = etab_len<NY, MODEL>();
  constexpr bool SHARE_TW = NX == NY;
  __shared__ float2 st[NY * RS];
  __shared__ double2 twlx[MODEL == kModelQAA ? 1 : LineTwSize<NX, PX>::value];
  __shared__ double2 twly[MODEL == kModelQAA || SHARE_TW ? 1 : LineTwSize<NY, PY>::value];
  // E(a_{j-1}) and E(a_j) of the axis of the current step; the other axis's are filled for
  // the next step meanwhile
  __shared__ double2 ex[2 * HX], ey[2 * HY];
  const int tid = threadIdx.x;
  const int rl = tid / TX, rt = tid % TX;  // row step: line of this lane group, lane in the line
  const int cl = tid / TY, ct = tid % TY;  // column step
  LineTwiddles<NX, PX> tx;
  LineTwiddles<NY, PY> ty;
  if constexpr (MODEL != kModelQAA) {
    load_twiddles(tx, twx, twlx, rt);
    load_twiddles(ty, twy, SHARE_TW ? twlx : twly, ct);  // equal sizes share one table
  }
  for (int i = blockIdx.x; i < ninst; i += gridDim.x) {
    const InstDev& I = inst[i];
    const long long lim = step_limit(I, max_steps);
    if (lim <= 0) continue;  // block-uniform
    const int start_axis = I.axis;
    float2* __restrict__ pg = psi + I.psi_off;
    const double* __restrict__ fg = f + I.psi_off;
    // tiled HBM -> row-major LDS: element 2e and 2e+1 are (x, y) and (x + 1, y), x even
    for (int e = tid; e < NX * NY / 2; e += NT) {
      const float4 v = reinterpret_cast<const float4*>(pg)[e];
      const int idx = 2 * e, tile = idx >> 6, w = idx & 63;
      const int y = ((tile / (NX / 8)) << 3) + (w >> 3), x = ((tile % (NX / 8)) << 3) + (w & 7);
      st[y * RS + lds_slot(x)] = make_float2(v.x, v.y);
      st[y * RS + lds_slot(x) + 1] = make_float2(v.z, v.w);
    }
    // a, b of the step before, this one and the next, carried along: one evaluation of the
    // schedule per step (line_task and fill_etab take four: 39 x 32^2 and 44 fourth-order steps, 572 -> 551 us)
    double ap, bp, ac, bc;
    sched_ab<Y4>(I, I.steps_done - 1, ap, bp);
    sched_ab<Y4>(I, I.steps_done, ac, bc);
    if (start_axis == 0) fill_etab_pair<NX, MODEL>(ex, I, 0, ap, ac);
    else fill_etab_pair<NY, MODEL>(ey, I, 1, ap, ac);
    __syncthreads();
    for (long long s = 0; s < lim; ++s) {
      double an, bn;
      sched_ab<Y4>(I, I.steps_done + s + 1, an, bn);
      const bool row = ((start_axis + s) & 1) == 0;
      struct { bool prev; double cpot; } k;
      k.prev = s > 0 || I.mode == (row ? kModeOweX : kModeOweY);
      k.cpot = merged_turns(I, I.steps_done + s, s == 0 && I.mode == kModeClean, bc, bp);
      if (row) {
        fill_etab_pair<NY, MODEL>(ey, I, 1, ac, an);  // read after the barrier
#pragma unroll 1
        for (int y = rl; y < NY; y += C::ROWS_PER_IT) {
          float2* my = st + y * RS;
          if constexpr (MODEL == kModelQAA) {
            double2 reg[PX];
#pragma unroll
            for (int q = 0; q < PX; ++q) assign(reg[q], my[lds_slot(rt + q * TX)]);
            if (k.prev) line_field<NX, PX>(reg, rt, ex);
#pragma unroll
            for (int q = 0; q < PX; ++q)
              reg[q] = cmul_fd(reg[q], phase_turns_d(k.cpot * fg[tile_index(rt + q * TX, y, NX)]));
            line_field<NX, PX>(reg, rt, ex + HX);
#pragma unroll
            for (int q = 0; q < PX; ++q) assign(my[lds_slot(rt + q * TX)], reg[q]);
          } else {
            float2 reg[PX];
#pragma unroll
            for (int q = 0; q < PX; ++q) reg[q] = my[lds_slot(rt + q * TX)];
            wave_lds_sync();
            line_pass<NX, PX, false, SlotIx>(reg, rt, tx, my, ex, k.prev, k.cpot, 0,
                                             [&](int q) { return fg[tile_index(rt + q * TX, y, NX)]; });
#pragma unroll
            for (int q = 0; q < PX; ++q) my[lds_slot(rt + q * TX)] = reg[q];
          }
        }
      } else {
        fill_etab_pair<NX, MODEL>(ex, I, 0, ac, an);
#pragma unroll 1
        for (int x = cl; x < NX; x += C::COLS_PER_IT) {
          float2* my = st + lds_slot(x);
          if constexpr (MODEL == kModelQAA) {
            double2 reg[PY];
#pragma unroll
            for (int q = 0; q < PY; ++q) assign(reg[q], my[(ct + q * TY) * RS]);
            if (k.prev) line_field<NY, PY>(reg, ct, ey);
#pragma unroll
            for (int q = 0; q < PY; ++q)
              reg[q] = cmul_fd(reg[q], phase_turns_d(k.cpot * fg[tile_index(x, ct + q * TY, NX)]));
            line_field<NY, PY>(reg, ct, ey + HY);
#pragma unroll
            for (int q = 0; q < PY; ++q) assign(my[(ct + q * TY) * RS], reg[q]);
          } else {
            float2 reg[PY];
#pragma unroll
            for (int q = 0; q < PY; ++q) reg[q] = my[(ct + q * TY) * RS];
            wave_lds_sync();
            line_pass<NY, PY, false, StrideIx<RS>>(reg, ct, ty, my, ey, k.prev, k.cpot, 0,
                                                   [&](int q) { return fg[tile_index(x, ct + q * TY, NX)]; });
#pragma unroll
            for (int q = 0; q < PY; ++q) my[(ct + q * TY) * RS] = reg[q];
          }
        }
      }
      ac = an;
      bp = bc;
      bc = bn;
      __syncthreads();
    }
    // row-major LDS -> tiled HBM
    for (int e = tid; e < NX * NY / 2; e += NT) {
      const int idx = 2 * e, tile = idx >> 6, w = idx & 63;
      const int y = ((tile / (NX / 8)) << 3) + (w >> 3), x = ((tile % (NX / 8)) << 3) + (w & 7);
      const float2 p0 = st[y * RS + lds_slot(x)], p1 = st[y * RS + lds_slot(x) + 1];
      reinterpret_cast<float4*>(pg)[e] = make_float4(p0.x, p0.y, p1.x, p1.y);
    }
    __syncthreads();  // the next instance's load reuses the LDS
  }
}

bool resident_supported(int nx, int ny) {
  auto ok = [](int n) { return n == 32 || n == 64 || n == 128; };
  return ok(nx) && ok(ny);
}

hipError_t launch_resident_2d(int nx, int ny, const InstDev* inst, int ninst, const int* nact, float2* psi,
                              const double* f,
                              const double2* tw_nx, const double2* tw_ny, long long max_steps, int model,
                              bool y4, hipStream_t stream) {
  if (ninst <= 0) return hipSuccess;
  if (!resident_supported(nx, ny)) return hipErrorInvalidValue;
  auto go = [&](auto kernel, int threads) {
    QHD_LAUNCH(kernel, dim3(ninst), dim3(threads), 0, stream, inst, nact, psi, f, tw_nx, tw_ny, max_steps);
    return hipGetLastError();
  };
#define QHD_RES_LAUNCH(NX_, NY_, MANY_)                                                              \
  if (nx == NX_ && ny == NY_ && (!MANY_ || ninst > 256)) {                                           \
    if (model == kModelQAA)                                                                          \
      return go(k_resident_2d<NX_, NY_, kModelQAA, false, MANY_>, ResCfg<NX_, NY_, kModelQAA, MANY_>::NT); \
    if (y4) return go(k_resident_2d<NX_, NY_, kModelQHD, true, MANY_>, ResCfg<NX_, NY_, kModelQHD, MANY_>::NT); \
    return go(k_resident_2d<NX_, NY_, kModelQHD, false, MANY_>, ResCfg<NX_, NY_, kModelQHD, MANY_>::NT); \
  }
  QHD_RES_LAUNCH(32, 128, true)
  QHD_RES_LAUNCH(128, 32, true)
  QHD_RES_LAUNCH(32, 32, false)
  QHD_RES_LAUNCH(32, 64, false)
  QHD_RES_LAUNCH(32, 128, false)
  QHD_RES_LAUNCH(64, 32, false)
  QHD_RES_LAUNCH(64, 64, false)
  QHD_RES_LAUNCH(64, 128, false)
  QHD_RES_LAUNCH(128, 32, false)
  QHD_RES_LAUNCH(128, 64, false)
  QHD_RES_LAUNCH(128, 128, false)
#undef QHD_RES_LAUNCH
  return hipErrorInvalidValue;
}

}  // namespace qhd
