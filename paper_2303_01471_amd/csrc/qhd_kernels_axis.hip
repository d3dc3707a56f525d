// HIP kernels of the 2-D split-operator steps (gfx950 / CDNA4): one HBM pass per step,
// alternating between the two axes.
//
// One symmetric step of the product formula (App. C.2.1, eqs. prod_qhd and
// prod_qhd_fft; App. E.1, Algorithm 1, taken in its symmetric form with midpoint
// coefficients) is
//
//     psi <- V_j^{1/2} K_j V_j^{1/2} psi,
//     V_j^{1/2} = exp(-i (dt/2) b_j f(x)),   K_j = F^{-1} exp(-i dt a_j |k|^2 / 2) F,
//
// with a_j = a(t_{j+1/2}), b_j = b(t_{j+1/2}).  |k|^2 is a sum over the axes, so the kinetic
// factor is a product of two commuting line operators, K_j = X_j Y_j with
// X_j = F_x^{-1} E_x(a_j) F_x along the mesh rows and Y_j likewise along the columns.  Only
// V_j couples the axes, and it is diagonal where both are done, so consecutive steps may
// take the two line operators in turn:
//
//     V_0^{1/2} X_0 | Y_0 . V_0^{1/2} V_1^{1/2} . Y_1 | X_1 . V_1^{1/2} V_2^{1/2} . X_2 | ...
//
// Each bar is an HBM pass and every pass does a whole step's work along one axis: the line
// operator owed by the step before, the merged potential half steps, and its own step's
// operator along the same axis.  A step reads and writes psi once and reads f once (24
// bytes per grid point); taking both axes of one step in turn, each in a pass of its own,
// moved 40 and took two launches for the same four line transforms.  The state between
// passes is in position space and owes the line operator of its last stage along the axis
// that the last pass did not take (InstDev::mode), and its trailing half step.  A new state
// starts on x; the axis that each member takes next is part of its record (InstDev::axis), and
// where members of a class differ a sub-step launches both axes in the general form of the passes.
//
// Lie (V_j, then K_j) and the stages of the fourth-order composition take the same form.
// QAA (App. C.2): the transverse field is diagonal after a Walsh-Hadamard transform of each
// axis and a sum over the axes, so the same passes run with those lines in FP64.
//
// Memory layout in HBM (2-D): 8x8 tiles of 64 consecutive complex64 values, tile rows of the
// mesh stored one after another, so that a tile row (8 mesh rows) and a tile column (8 mesh
// columns) are both made of 512-byte contiguous chunks.  f is stored as FP64 in the same
// layout: carrying f at FP64 precision matters because the potential phase accumulates
// f * integral(b dt) (up to ~8e4 f at T = 20), far beyond FP32's 2^-24 relative precision.
//
// Phases: every phase argument is formed in FP64 and reduced to [-1/2, 1/2] turns, evaluated
// in FP32 and given one Newton magnitude correction in FP64; each factor multiplies in FP64
// and the product is rounded once.  The kinetic factors E(a_{j-1}) and E(a_j) of an
// instance, with the 1/n of the inverse transform folded in exactly, sit in an LDS table
// per block, indexed by |frequency| (QHD: n/2 + 1 entries) or by popcount (QAA).
//
// Rounding: the whole mesh never concentrates into one coefficient here (a near-uniform
// state does after both transforms), only each line into its own, and the rounding errors
// of the lines are independent.
#include "axis_line.h"
#include "launch_util.h"
#include "line_fft.h"
#include "pass_common.h"
#include "qhd_internal.h"

namespace qhd {

// ------------------------------------------------------------------------------------
// Row pass: lines along x, one line per TPL lanes.

// 512-point QHD rows with 16 points per lane (PAD16): one pad slot per 16 line entries (the
// radix-16 scatter of the first stage then puts a group of 16 lanes on 16 distinct bank
// pairs) and a table of first twiddle powers.
template <int NX, int P, int MODEL>
struct RowCfg {
  static constexpr bool PAD16 = MODEL == kModelQHD && NX == 512 && P == 16;
  static constexpr int SLOTS = PAD16 ? NX + NX / 16 : LineLds<NX>::kSlots;
  static constexpr int WAVES = P == 16 && NX == 512 ? 3 : 1;
  static constexpr int TPL = NX / P;
  static constexpr int NT = 256;
  static constexpr int LPW = NT / TPL;  // lines per block
};
struct Slot16Ix {
  __device__ static constexpr int at(int i) { return i + (i >> 4); }
};
template <>
struct IxShift<Slot16Ix> {
  static constexpr int value = 4;
};

template <int NX, int P, int MODEL = kModelQHD, bool GEN = true>
__global__ void __launch_bounds__((RowCfg<NX, P, MODEL>::NT)) __attribute__((amdgpu_waves_per_eu(RowCfg<NX, P, MODEL>::WAVES)))
k_row_axis_2d(const InstDev* __restrict__ inst, const int* __restrict__ nact_p, int ny_log2,
              float2* __restrict__ psi, const double* __restrict__ f, const double2* __restrict__ twtab, int s,
              long long max_steps, int kind) {
  const int ninst = *nact_p;  // members active in this sub-step (device, set per chunk)
  using RC = RowCfg<NX, P, MODEL>;
  constexpr int TPL = RC::TPL, LPW = RC::LPW, SLOTS = RC::SLOTS, H = etab_len<NX, MODEL>();
  __shared__ float2 lds[MODEL == kModelQAA ? 1 : LPW * SLOTS];
  extern __shared__ double2 etab[];  // tables of the block's instances, sized at launch
  const int ll = threadIdx.x / TPL, t = threadIdx.x % TPL;
  float2* my = lds + (MODEL == kModelQAA ? 0 : ll * SLOTS);
  using TW = typename std::conditional<RC::PAD16, TwiddlesLds<NX, P, true>, LineTwiddles<NX, P>>::type;
  __shared__ double2 twl[MODEL == kModelQAA ? 1 : (RC::PAD16 ? TwiddlesLds<NX, P, true>::kEntries : LineTwSize<NX, P>::value)];
  TW tw;
  if constexpr (MODEL != kModelQAA) load_twiddles(tw, twtab, twl, t);
  // instances of the block's lines: one, or LPW / ny whole ones
  constexpr int LPW_LOG2 = ilog2_c(LPW);
  const int per_block = LPW_LOG2 > ny_log2 ? 1 << (LPW_LOG2 - ny_log2) : 1;
  const long long total = (long long)ninst << ny_log2;
  long long begin, end;
  block_share(total, LPW, begin, end);
  int cached = -1;
  for (long long l0 = begin; l0 < end; l0 += LPW) {
    const int i0 = (int)(l0 >> ny_log2);
    const long long L = l0 + ll;
    const bool valid = L < end;
    const long long Lc = valid ? L : end - 1;
    int i = (int)(Lc >> ny_log2);
    const int y = (int)(Lc & ((1 << ny_log2) - 1));
    // a wavefront's rows (64 P / NX of them, aligned) lie in one instance when they are
    // at most 8, the smallest mesh size: the index is then wave-uniform and the instance
    // record is read with scalar loads instead of a chain of waited vector loads
    if constexpr (64 * P <= 8 * NX) i = __builtin_amdgcn_readfirstlane(i);
    const InstDev& I = inst[i];
    float2* __restrict__ pl = psi + I.psi_off;
    const double* __restrict__ fl = f + I.psi_off;
    // wave-uniform instance, whole-tile slot stride: buffer views (scalar base)
    constexpr bool VIEW = 64 * P <= 8 * NX && TPL % 8 == 0;
    const int off = VIEW ? (int)row_slot<NX, TPL>(t, 0, y) : 0;
    const LaneView<float2> ps(pl, off);
    const LaneView<double> fs(fl, off);
    float2 reg[P];  // in flight while the tables are filled
#pragma unroll
    for (int q = 0; q < P; ++q) {
      if constexpr (VIEW) reg[q] = ps.load(q * TPL * 8);
      else reg[q] = pl[row_slot<NX, TPL>(t, q, y)];
    }
    auto fget = [&](int q) -> double {
      if constexpr (VIEW) return fs.load(q * TPL * 8);
      else return fl[row_slot<NX, TPL>(t, q, y)];
    };
    if (i0 != cached) {  // block-uniform
      if (cached >= 0) __syncthreads();  // the previous instance's readers
      fill_etab<NX, MODEL, GEN>(etab, inst, i0, per_block < ninst - i0 ? per_block : ninst - i0, 0, s);
      __syncthreads();
      cached = i0;
    }
    const LineTask k = line_task<GEN>(I, s, max_steps, 0, kind);
    const double2* tab = etab + (i - i0) * 2 * H;
    if constexpr (MODEL == kModelQAA) {
      double2 x[P];
#pragma unroll
      for (int q = 0; q < P; ++q) assign(x[q], reg[q]);
      if (k.prev) line_field<NX, P>(x, t, tab);
      if (kind != kPassFixUp) {
#pragma unroll
        for (int q = 0; q < P; ++q) x[q] = cmul_fd(x[q], phase_turns_d(k.cpot * fget(q)));
        line_field<NX, P>(x, t, tab + H);
      }
#pragma unroll
      for (int q = 0; q < P; ++q) assign(reg[q], x[q]);
    } else {
      using IX = typename std::conditional<RC::PAD16, Slot16Ix, SlotIx>::type;
      line_pass<NX, P, false, IX>(reg, t, tw, my, tab, k.prev, k.cpot, kind, fget);
    }
    if (valid && k.active) {
#pragma unroll
      for (int q = 0; q < P; ++q) {
        if constexpr (VIEW) ps.store(q * TPL * 8, reg[q]);
        else pl[row_slot<NX, TPL>(t, q, y)] = reg[q];
      }
    }
  }
}

// ------------------------------------------------------------------------------------
// Column pass, staged form: a tile column (8 mesh columns) is copied through LDS with
// 512-byte tile loads; each column is then one line of TPL lanes.  f is read in the line
// layout (64-byte pieces).  The general form: short columns, QAA, and a choice of the
// tuning cache at the other lengths.

template <int NY, int P, int MODEL = kModelQHD, bool GEN = true>
__global__ void __launch_bounds__((ColCfg<NY, P>::NT)) __attribute__((amdgpu_waves_per_eu(ColCfg<NY, P>::MIN_WAVES)))
k_col_axis_2d(const InstDev* __restrict__ inst, const int* __restrict__ nact_p, int nx_log2,
              float2* __restrict__ psi, const double* __restrict__ f, const double2* __restrict__ twtab, int s,
              long long max_steps, int kind) {
  const int ninst = *nact_p;  // members active in this sub-step (device, set per chunk)
  using C = ColCfg<NY, P>;
  constexpr int TPL = C::TPL, ITEMS = C::ITEMS, NT = C::NT, STRIDE = C::STRIDE, SUBS = C::SUBS;
  constexpr int TILES = NY / 8, H = etab_len<NY, MODEL>();
  __shared__ float2 lds[C::LINES * STRIDE];
  __shared__ double2 etab[ITEMS * 2 * H];
  const int tid = threadIdx.x;
  const int line0 = tid / TPL, t = tid % TPL;  // first column of this lane group
  __shared__ double2 twl[MODEL == kModelQAA ? 1 : LineTwSize<NY, P>::value];
  LineTwiddles<NY, P> tw;
  if constexpr (MODEL != kModelQAA) load_twiddles(tw, twtab, twl, t);
  const int tc_log2 = nx_log2 - 3, tcols = 1 << tc_log2, nx = 1 << nx_log2;
  const long long total = (long long)ninst << tc_log2;
  long long begin, end;
  block_share(total, ITEMS, begin, end);
  int cached = -1, cached_n = 0;
  auto live = [&](const InstDev& I) { return line_active<GEN>(I, s, max_steps, 1, kind); };
  for (long long g0 = begin; g0 < end; g0 += ITEMS) {
    const long long glast = g0 + ITEMS <= end ? g0 + ITEMS - 1 : end - 1;
    const int i0 = (int)(g0 >> tc_log2), count = (int)(glast >> tc_log2) - i0 + 1;
    if (i0 != cached || count > cached_n) {
      // the previous items' readers passed the barrier that ends their store
      fill_etab<NY, MODEL, GEN>(etab, inst, i0, count, 1, s);
      cached = i0;
      cached_n = count;
    }
    // stage the tile columns: each thread moves float4 = two complex values; the item
    // decode is wave-uniform
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      const long long g = g0 + it;
      if (g < end) {
        const int i = (int)(g >> tc_log2), tc = (int)(g & (tcols - 1));
        const InstDev& I = inst[i];
        if (live(I)) {
          const float4* __restrict__ src = reinterpret_cast<const float4*>(psi + I.psi_off) + tc * 32;
          float2* __restrict__ dst = lds + it * 8 * STRIDE;
#pragma unroll
          for (int e = tid; e < TILES * 32; e += NT) {
            const int ty = e >> 5, w = e & 31;
            const float4 v = src[(long long)ty * tcols * 32 + w];
            const int y = ty * 8 + (w >> 2), xx = (w & 3) << 1;
            dst[xx * STRIDE + lds_slot(y)] = make_float2(v.x, v.y);
            dst[(xx + 1) * STRIDE + lds_slot(y)] = make_float2(v.z, v.w);
          }
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int sub = 0; sub < SUBS; ++sub) {
      const int line = line0 + sub * (NT / TPL);
      float2* my = lds + line * STRIDE;
      // with at least 8 lanes per line a wavefront's lines (aligned) lie in one 8-line item
      const int item_of_line = TPL >= 8 ? __builtin_amdgcn_readfirstlane(line / 8) : line / 8;
      const long long g = g0 + item_of_line;
      const long long gc = g < end ? g : end - 1;
      const int i = (int)(gc >> tc_log2), tc = (int)(gc & (tcols - 1));
      const InstDev& I = inst[i];
      const int x = tc * 8 + (line & 7);
      const LineTask k = line_task<GEN>(I, s, max_steps, 1, kind);
      const double2* tab = etab + (i - i0) * 2 * H;
      const double* __restrict__ fl = f + I.psi_off;
      float2 reg[P];
#pragma unroll
      for (int q = 0; q < P; ++q) reg[q] = my[lds_slot(t + q * TPL)];
      wave_lds_sync();
      if constexpr (MODEL == kModelQAA) {
        double2 kd[P];
#pragma unroll
        for (int q = 0; q < P; ++q) assign(kd[q], reg[q]);
        if (k.prev) line_field<NY, P>(kd, t, tab);
        if (kind != kPassFixUp) {
#pragma unroll
          for (int q = 0; q < P; ++q) kd[q] = cmul_fd(kd[q], phase_turns_d(k.cpot * fl[tile_index(x, t + q * TPL, nx)]));
          line_field<NY, P>(kd, t, tab + H);
        }
#pragma unroll
        for (int q = 0; q < P; ++q) assign(reg[q], kd[q]);
      } else {
        line_pass<NY, P, false, SlotIx>(reg, t, tw, my, tab, k.prev, k.cpot, kind,
                                        [&](int q) { return fl[tile_index(x, t + q * TPL, nx)]; });
      }
#pragma unroll
      for (int q = 0; q < P; ++q) my[lds_slot(t + q * TPL)] = reg[q];
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      const long long g = g0 + it;
      if (g < end) {
        const int i = (int)(g >> tc_log2), tc = (int)(g & (tcols - 1));
        const InstDev& I = inst[i];
        if (live(I)) {
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

// ------------------------------------------------------------------------------------
// Column pass, split form (512-point columns, QHD).  A block of 8 wavefronts takes
// one tile column (8 columns x 512 rows) per item, in two lane layouts:
//   tile view   lane l of wavefront w holds column l & 7, rows t + 64 q with
//               t = (l >> 3) + 8 w: slot q of a wavefront is one whole 8x8 tile, loaded
//               from (and stored to) HBM straight into registers, psi and f alike;
//   line view   wavefront w holds column w as one line, lane t = l with rows t + 64 q.
// Of each line operator the tile view runs the first forward and the last inverse stage,
// the line view the stages between and the kinetic factor with wavefront-local
// exchanges; the views meet in the columns' LDS lines behind block barriers.  The
// potential factor applies in the tile view.

template <int NY>
struct ColSplitCfg {
  static constexpr int P = 8, TPL = NY / P, NT = 512;
  static constexpr int STRIDE = ColCfg<NY, P>::STRIDE;  // line stride in LDS slots
};

template <int NY, bool GEN>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(6)))
k_col_axis_split(const InstDev* __restrict__ inst, const int* __restrict__ nact_p, int nx_log2,
                 float2* __restrict__ psi, const double* __restrict__ f, const double2* __restrict__ twtab, int s,
                 long long max_steps, int kind) {
  const int ninst = *nact_p;  // members active in this sub-step (device, set per chunk)
  using C = ColSplitCfg<NY>;
  constexpr int P = C::P, TPL = C::TPL, STRIDE = C::STRIDE, H = NY / 2 + 1;
  static_assert(TPL == 64 && StagePlan<NY, P>::count() == 3, "split form: 512-point lines, radices 8, 8, 8");
  __shared__ float2 lds[8 * STRIDE];
  __shared__ double2 etab[2 * H];
  __shared__ double2 twl[LineTwSize<NY, P>::value];
  // the wavefront index is uniform: tile offsets are then scalar and not held per lane
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c_tv = lane & 7, t_tv = (lane >> 3) + 8 * wave;  // tile view: column, line position
  float2* my = lds + wave * STRIDE;                           // line view: this wavefront's column
  float2* mc = lds + c_tv * STRIDE;                           // tile view: this lane's column
  LineTwiddles<NY, P> tw;
  load_twiddles(tw, twtab, twl, lane);
  LineTwiddles<NY, P> twt = tw;  // the same table seen from the tile view's line positions
  twt.tab = twl + t_tv;
  const int tc_log2 = nx_log2 - 3, tcols = 1 << tc_log2;
  const long long total = (long long)ninst << tc_log2;
  long long begin, end;
  block_share(total, 1, begin, end);
  int cached = -1;
  // the line operator on the tile view's values, from `in` to `out` (float2 or double2)
  auto kinetic = [&](auto& in, auto& out, const double2* __restrict__ tab) {
    using TIN = typename std::remove_reference<decltype(in[0])>::type;
    using TOUT = typename std::remove_reference<decltype(out[0])>::type;
    using K = typename LinePrec<NY>::K;
    stage_outputs_to_lds<NY, P, -1, 0, TIN, SlotIx>(in, t_tv, twt, mc);
    __syncthreads();
    {
      float2 reg[P];
      K k[P];
      stage_inputs<NY, P, SlotIx>(reg, lane, my);
      wave_lds_sync();
      fft_stage_io<NY, P, -1, 1, false, float2, SlotIx>(reg, reg, lane, tw, my);
      fft_stage_io<NY, P, -1, 2, false, K, SlotIx>(reg, k, lane, tw, my);
      mul_kinetic<NY, P>(k, lane, tab);
      fft_stage_io<NY, P, +1, 0, false, K, SlotIx>(k, reg, lane, tw, my);
      stage_outputs_to_lds<NY, P, +1, 1, float2, SlotIx>(reg, lane, tw, my);
    }
    __syncthreads();
    float2 mid[P];
    stage_inputs<NY, P, SlotIx>(mid, t_tv, mc);
    fft_stage_io<NY, P, +1, 2, false, TOUT, SlotIx>(mid, out, t_tv, twt, mc);
    __syncthreads();  // the next first stage rewrites the lines
  };
  for (long long g0 = begin; g0 < end; ++g0) {
    const int i = (int)(g0 >> tc_log2), tc = (int)(g0 & (tcols - 1));
    const InstDev& I = inst[i];
    const LineTask k = line_task<GEN>(I, s, max_steps, 1, kind);
    if (!k.active) continue;  // block-uniform
    const LaneView<float2> pv(psi + I.psi_off + tc * 64, lane);
    const LaneView<double> fv(f + I.psi_off + tc * 64, lane);
    float2 x[P];
#pragma unroll
    for (int q = 0; q < P; ++q) x[q] = pv.load((wave + 8 * q) * tcols * 64);
    if (i != cached) {
      // the previous item's readers passed its last barrier; this item's readers wait for
      // the barrier after the first stage
      fill_etab<NY, kModelQHD, GEN>(etab, inst, i, 1, 1, s);
      cached = i;
    }
    typename LinePrec<NY>::V v[P];
    if (k.prev) {
      kinetic(x, v, etab);
    } else {
#pragma unroll
      for (int q = 0; q < P; ++q) assign(v[q], x[q]);
    }
    if (kind != kPassFixUp) {
#pragma unroll
      for (int q = 0; q < P; ++q)
        v[q] = cmul_fd(v[q], phase_turns_d(k.cpot * fv.load((wave + 8 * q) * tcols * 64)));
      kinetic(v, v, etab + H);
    }
#pragma unroll
    for (int q = 0; q < P; ++q) {
      assign(x[q], v[q]);
      pv.store((wave + 8 * q) * tcols * 64, x[q]);
    }
  }
}

// ------------------------------------------------------------------------------------
// Column pass, tile-wave form (NY >= 64).  Lane l of wavefront w of an item
// owns column c = l & 7 of a tile column and row group t = (l >> 3) + 8 w, and
// holds the rows t + q*TPL (q = 0..P-1).  Slot q of a wavefront is then exactly
// one 8x8 tile (64 consecutive complex values, 512 bytes): loads and stores are
// fully coalesced and go straight to registers.  A column spans W = TPL/8
// wavefronts; with W > 1 the FFT exchanges use workgroup barriers and a block takes one
// item, so that every branch around them is block-uniform.

template <int NY, int P>
struct ColTwCfg {
  static constexpr int TPL = NY / P;
  static constexpr int W = TPL / 8;                       // wavefronts per tile column
  static constexpr int ITEMS = W > 1 ? 1 : 4;             // tile columns per block
  static constexpr int NT = ITEMS * W * 64;
  static constexpr int STRIDE = ((LineLds<NY>::kSlots + 13) / 16) * 16 + 2;
  // 16 points per lane: three waves per SIMD (168 VGPRs)
  static constexpr int MIN_WAVES = (NT == 512) ? 2 : (P >= 16 ? 3 : 1);
  static_assert(TPL % 8 == 0, "tile-wave column pass needs TPL multiple of 8");
};

template <int NY, int P, int MODEL, bool GEN>
__global__ void __launch_bounds__((ColTwCfg<NY, P>::NT)) __attribute__((amdgpu_waves_per_eu(ColTwCfg<NY, P>::MIN_WAVES)))
k_col_axis_tw(const InstDev* __restrict__ inst, const int* __restrict__ nact_p, int nx_log2,
              float2* __restrict__ psi, const double* __restrict__ f, const double2* __restrict__ twtab, int s,
              long long max_steps, int kind) {
  const int ninst = *nact_p;  // members active in this sub-step (device, set per chunk)
  using C = ColTwCfg<NY, P>;
  constexpr int W = C::W, ITEMS = C::ITEMS, STRIDE = C::STRIDE, H = etab_len<NY, MODEL>();
  static_assert(MODEL != kModelQAA || W == 1, "Walsh-Hadamard columns stay in one wavefront");
  __shared__ float2 lds[MODEL == kModelQAA ? 1 : ITEMS * 8 * STRIDE];
  __shared__ double2 etab[ITEMS * 2 * H];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // item within the block and wave within the item; wave-uniform, so the instance
  // record is read with scalar loads
  const int item = __builtin_amdgcn_readfirstlane(wave / W), wv = __builtin_amdgcn_readfirstlane(wave - item * W);
  const int c = lane & 7;
  const int t = (lane >> 3) + 8 * wv;
  float2* my = lds + (MODEL == kModelQAA ? 0 : (item * 8 + c) * STRIDE);
  __shared__ double2 twl[MODEL == kModelQAA ? 1 : LineTwSize<NY, P>::value];
  LineTwiddles<NY, P> tw;
  if constexpr (MODEL != kModelQAA) load_twiddles(tw, twtab, twl, t);
  const int tc_log2 = nx_log2 - 3, tcols = 1 << tc_log2;
  const long long total = (long long)ninst << tc_log2;
  long long begin, end;
  block_share(total, ITEMS, begin, end);
  int cached = -1, cached_n = 0;
  for (long long g0 = begin; g0 < end; g0 += ITEMS) {
    const long long glast = g0 + ITEMS <= end ? g0 + ITEMS - 1 : end - 1;
    const int i0 = (int)(g0 >> tc_log2), count = (int)(glast >> tc_log2) - i0 + 1;
    const long long g = g0 + item;
    const bool valid = g < end;
    const long long gc = valid ? g : end - 1;
    const int i = (int)(gc >> tc_log2), tc = (int)(gc & (tcols - 1));
    const InstDev& I = inst[i];
    // the item's tile column: scalar base, the lane's offset in one register, slot
    // offsets scalar (tile rows t + q TPL, W tile rows apart)
    const long long off = I.psi_off + ((long long)tc << 6);
    const LaneView<float2> pv(psi + off, lane + wv * tcols * 64);
    const LaneView<double> fv(f + off, lane + wv * tcols * 64);
    float2 in[P];  // in flight while the tables are filled
#pragma unroll
    for (int q = 0; q < P; ++q) in[q] = pv.load(q * W * tcols * 64);
    if (i0 != cached || count > cached_n) {  // block-uniform
      if (cached >= 0) __syncthreads();  // the previous items' readers are done
      fill_etab<NY, MODEL, GEN>(etab, inst, i0, count, 1, s);
      __syncthreads();
      cached = i0;
      cached_n = count;
    }
    const LineTask k = line_task<GEN>(I, s, max_steps, 1, kind);
    const bool active = valid && k.active;
    const double2* tab = etab + (i - i0) * 2 * H;
    if constexpr (MODEL == kModelQAA) {
      double2 reg[P];
#pragma unroll
      for (int q = 0; q < P; ++q) assign(reg[q], in[q]);
      if (k.prev) line_field<NY, P, 8>(reg, t, tab);
      if (kind != kPassFixUp) {
#pragma unroll
        for (int q = 0; q < P; ++q) reg[q] = cmul_fd(reg[q], phase_turns_d(k.cpot * fv.load(q * W * tcols * 64)));
        line_field<NY, P, 8>(reg, t, tab + H);
      }
      if (active) {
#pragma unroll
        for (int q = 0; q < P; ++q) {
          float2 z;
          assign(z, reg[q]);
          pv.store(q * W * tcols * 64, z);
        }
      }
    } else {
      line_pass<NY, P, (W > 1), SlotIx>(in, t, tw, my, tab, k.prev, k.cpot, kind,
                                        [&](int q) { return fv.load(q * W * tcols * 64); });
      if (active) {
#pragma unroll
        for (int q = 0; q < P; ++q) pv.store(q * W * tcols * 64, in[q]);
      }
    }
  }
}

// ------------------------------------------------------------------------------------
// Column form of the readouts, for instances that owe the line operator along y (the row
// form is k_observe_2d): the operator on a copy in LDS, then, in the tile layout, the
// trailing potential half step, the sums and the outputs.  One triple of partial sums per
// tile column.
template <int NY, int P, int MODEL>
__global__ void __launch_bounds__(256) k_observe_col_2d(const InstDev* __restrict__ inst, int ninst, int nx_log2,
                                                        const float2* __restrict__ psi, const double* __restrict__ f,
                                                        const double2* __restrict__ twtab, float2* __restrict__ out_psi,
                                                        float* __restrict__ out_rho, double* __restrict__ partials,
                                                        int stride) {
  constexpr int TPL = NY / P, NT = 256, LPR = NT / TPL;  // lines per round
  constexpr int STRIDE = ColCfg<NY, P>::STRIDE, TILES = NY / 8, H = etab_len<NY, MODEL>();
  __shared__ float2 lds[8 * STRIDE];
  __shared__ double2 etab[2 * H];
  __shared__ double2 twl[MODEL == kModelQAA ? 1 : LineTwSize<NY, P>::value];
  __shared__ double red[3][NT];
  const int tid = threadIdx.x, line0 = tid / TPL, t = tid % TPL;
  LineTwiddles<NY, P> tw;
  if constexpr (MODEL != kModelQAA) load_twiddles(tw, twtab, twl, t);
  const int tc_log2 = nx_log2 - 3, tcols = 1 << tc_log2, nx = 1 << nx_log2;
  const long long total = (long long)ninst << tc_log2;
  for (long long g = blockIdx.x; g < total; g += gridDim.x) {
    const int i = (int)(g >> tc_log2), tc = (int)(g & (tcols - 1));
    const InstDev& I = inst[i];
    if (I.mode != kModeOweY) continue;  // block-uniform
    fill_etab<NY, MODEL, true>(etab, inst, i, 1, 1, 0);  // E(a) of stage steps_done - 1 first
    const float4* __restrict__ src = reinterpret_cast<const float4*>(psi + I.psi_off) + tc * 32;
    for (int e = tid; e < TILES * 32; e += NT) {
      const int ty = e >> 5, w = e & 31;
      const float4 v = src[(long long)ty * tcols * 32 + w];
      const int y = ty * 8 + (w >> 2), xx = (w & 3) << 1;
      lds[xx * STRIDE + lds_slot(y)] = make_float2(v.x, v.y);
      lds[(xx + 1) * STRIDE + lds_slot(y)] = make_float2(v.z, v.w);
    }
    __syncthreads();
    for (int line = line0; line < 8; line += LPR) {
      float2* my = lds + line * STRIDE;
      float2 reg[P];
#pragma unroll
      for (int q = 0; q < P; ++q) reg[q] = my[lds_slot(t + q * TPL)];
      wave_lds_sync();
      if constexpr (MODEL == kModelQAA) {
        double2 kd[P];
#pragma unroll
        for (int q = 0; q < P; ++q) assign(kd[q], reg[q]);
        line_field<NY, P>(kd, t, etab);
#pragma unroll
        for (int q = 0; q < P; ++q) assign(reg[q], kd[q]);
      } else {
        line_kinetic<NY, P, false, SlotIx>(reg, reg, t, tw, my, etab);
      }
#pragma unroll
      for (int q = 0; q < P; ++q) my[lds_slot(t + q * TPL)] = reg[q];
    }
    __syncthreads();
    const double cpot = closing_turns(I);
    const bool half = I.scheme != kSchemeLie;
    const int xs = (int)(I.argmin & (nx - 1)), ys = (int)(I.argmin >> nx_log2);
    double sr = 0.0, sf = 0.0, sm = 0.0;
    for (int e = tid; e < NY * 8; e += NT) {
      const int y = e >> 3, xx = e & 7, x = tc * 8 + xx;
      const double fv = f[I.psi_off + tile_index(x, y, nx)];
      float2 v = lds[xx * STRIDE + lds_slot(y)];
      if (half) v = cmul_fd(v, phase_turns_d(cpot * fv));
      const double rho = (double)v.x * v.x + (double)v.y * v.y;
      sr += rho;
      sf += fv * rho;
      if (in_ball(x - xs, y - ys, 0, I)) sm += rho;
      const long long o = I.out_off + (long long)y * nx + x;
      if (out_psi) out_psi[o] = v;
      if (out_rho) out_rho[o] = (float)rho;
    }
    red[0][tid] = sr;
    red[1][tid] = sf;
    red[2][tid] = sm;
    __syncthreads();
    for (int o = NT / 2; o > 0; o >>= 1) {
      if (tid < o) {
#pragma unroll
        for (int q = 0; q < 3; ++q) red[q][tid] += red[q][tid + o];
      }
      __syncthreads();
    }
    if (tid < 3) partials[3 * ((long long)i * stride + tc) + tid] = red[tid][0];
    __syncthreads();  // the next item reuses the LDS
  }
}

__global__ void __launch_bounds__(256) k_count_owing(const InstDev* __restrict__ inst, int ninst, int owe,
                                                     int* __restrict__ owing) {
  __shared__ int last[256];
  int n = 0;
  for (int i = threadIdx.x; i < ninst; i += 256)
    if (pays_owed(inst[i], owe)) n = i + 1;
  last[threadIdx.x] = n;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) last[threadIdx.x] = max(last[threadIdx.x], last[threadIdx.x + o]);
    __syncthreads();
  }
  if (threadIdx.x == 0) *owing = last[0];
}

// the members that go on take `axis` next; those that a fix-up launch paid for the other axis
// owe only the potential half step
__global__ void k_set_axis(InstDev* __restrict__ inst, int ninst, int axis) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ninst || inst[i].steps_done >= inst[i].nsteps) return;
  if (pays_owed(inst[i], axis == 0 ? kModeOweY : kModeOweX)) inst[i].mode = kModeKDone;
  inst[i].axis = axis;
}

// ------------------------------------------------------------------------------------
// launchers

int row_points_resolve(int nx, int points_per_lane) {
  if (nx >= 1024) return 16;
  if (points_per_lane == 16 && nx >= 128) return 16;
  return 8;
}

int pass_blocks_row_2d(int nx, int ny, int ninst, int grid_cap, int points_per_lane) {
  const int P = row_points_resolve(nx, points_per_lane);
  const int lpw = 256 / (nx / P);
  return blocks_for((long long)ninst * ny, lpw, grid_cap);
}

// points per lane of the tile-wave columns
template <int N>
constexpr int col_tw_p() { return N >= 128 && N != 512 ? 16 : 8; }
int col_tw_points(int ny) { return ny >= 128 && ny != 512 ? 16 : 8; }

int col_variant_resolve(int ny, int variant) {
  const bool tw_ok = ny >= 64 && ny <= 1024;
  if (variant == kColTileWave && tw_ok) return kColTileWave;
  if (variant == kColStaged16 && (ny == 256 || ny == 512)) return kColStaged16;
  if (variant == kColSplit && ny == 512) return kColSplit;
  if (variant == kColStaged) return kColStaged;
  // 512 points: by whole steps the split form is the better one but for mid-sized batches (us per
  // step, split and tile-wave: 1 member 10.2 and 10.6, 4: 14.7 and 14.9, 16: 33.9 and 32.1, 64: 112
  // and 113, 263: 464 and 470), although a tile-wave pass launched alone over and over may time
  // faster
  return (ny >= 64 && ny <= 256) || ny == 1024 ? kColTileWave : (ny == 512 ? kColSplit : kColStaged);
}

int pass_blocks_col_2d(int nx, int ny, int ninst, int grid_cap, int variant) {
  int items;
  const int v = col_variant_resolve(ny, variant);
  if (v == kColTileWave) {
    items = ny / col_tw_points(ny) / 8 > 1 ? 1 : 4;
  } else if (v == kColSplit) {
    items = 1;
  } else {
    const int tpl = ny / (v == kColStaged16 || ny >= 1024 ? 16 : 8);
    items = (8 * tpl >= 256) ? 1 : 256 / (8 * tpl);
  }
  return blocks_for((long long)ninst * (nx / 8), items, grid_cap);
}

namespace {

struct PassArgs {
  const InstDev* inst;
  const int* nact;
  float2* psi;
  const double* f;
  const double2* tw;
  int s;
  long long max_steps;
  int kind;
  hipStream_t stream;
};

template <int N, int P, int MODEL, bool GEN>
hipError_t go_row(int blocks, int ny, const PassArgs& a) {
  const int lpw = RowCfg<N, P, MODEL>::LPW;
  const int per_block = lpw > ny ? lpw / ny : 1;
  const size_t dyn = (size_t)per_block * 2 * etab_len<N, MODEL>() * sizeof(double2);
  QHD_LAUNCH((k_row_axis_2d<N, P, MODEL, GEN>), dim3(blocks), dim3(RowCfg<N, P, MODEL>::NT), dyn, a.stream, a.inst, a.nact, ilog2(ny), a.psi,
             a.f, a.tw, a.s, a.max_steps, a.kind);
  return hipGetLastError();
}

template <bool GEN>
hipError_t row_pass_qhd(int nx, int ny, int blocks, int points, const PassArgs& a) {
  if (points == 16 && nx == 128) return go_row<128, 16, kModelQHD, GEN>(blocks, ny, a);
  if (points == 16 && nx == 256) return go_row<256, 16, kModelQHD, GEN>(blocks, ny, a);
  if (points == 16 && nx == 512) return go_row<512, 16, kModelQHD, GEN>(blocks, ny, a);
  QHD_SWITCH_N(nx, { return (go_row<N_, pts_per_lane<N_>(), kModelQHD, GEN>)(blocks, ny, a); });
}

template <int N, int P, int MODEL, bool GEN>
hipError_t go_col_staged(int blocks, int nx, const PassArgs& a) {
  QHD_LAUNCH((k_col_axis_2d<N, P, MODEL, GEN>), dim3(blocks), dim3(ColCfg<N, P>::NT), 0, a.stream, a.inst, a.nact,
             ilog2(nx), a.psi, a.f, a.tw, a.s, a.max_steps, a.kind);
  return hipGetLastError();
}

template <int N, int MODEL, bool GEN>
hipError_t go_col_tw(int blocks, int nx, const PassArgs& a) {
  if constexpr (N >= 64 && (MODEL == kModelQHD || N <= 128)) {
    constexpr int P_ = col_tw_p<N>();
    QHD_LAUNCH((k_col_axis_tw<N, P_, MODEL, GEN>), dim3(blocks), dim3(ColTwCfg<N, P_>::NT), 0, a.stream, a.inst, a.nact,
               ilog2(nx), a.psi, a.f, a.tw, a.s, a.max_steps, a.kind);
    return hipGetLastError();
  } else {
    return hipErrorInvalidValue;
  }
}

template <bool GEN>
hipError_t col_pass_qhd(int nx, int ny, int blocks, int v, const PassArgs& a) {
  if (v == kColTileWave) QHD_SWITCH_N(ny, { return (go_col_tw<N_, kModelQHD, GEN>)(blocks, nx, a); });
  if (v == kColSplit) {
    QHD_LAUNCH((k_col_axis_split<512, GEN>), dim3(blocks), dim3(ColSplitCfg<512>::NT), 0, a.stream, a.inst, a.nact,
               ilog2(nx), a.psi, a.f, a.tw, a.s, a.max_steps, a.kind);
    return hipGetLastError();
  }
  if (v == kColStaged16)
    return ny == 256 ? go_col_staged<256, 16, kModelQHD, GEN>(blocks, nx, a)
                     : go_col_staged<512, 16, kModelQHD, GEN>(blocks, nx, a);
  QHD_SWITCH_N(ny, { return (go_col_staged<N_, pts_per_lane<N_>(), kModelQHD, GEN>)(blocks, nx, a); });
}

template <bool GEN>
hipError_t col_pass_qaa(int nx, int ny, int blocks, const PassArgs& a) {
  QHD_SWITCH_N(ny, {
    if constexpr (N_ == 64 || N_ == 128) return (go_col_tw<N_, kModelQAA, GEN>)(blocks, nx, a);
    else return (go_col_staged<N_, pts_per_lane<N_>(), kModelQAA, GEN>)(blocks, nx, a);
  });
}

}  // namespace

hipError_t launch_row_pass_2d(int nx, int ny, const InstDev* inst, int ninst, const int* nact, float2* psi,
                              const double* f, const double2* tw, int s, long long max_steps, int grid_cap,
                              int points_per_lane, hipStream_t stream, int model, bool y4, int kind) {
  const PassArgs a{inst, nact, psi, f, tw, s, max_steps, kind, stream};
  const bool general = y4 || kind != kPassPlain;
  if (model == kModelQAA) {  // the QAA model runs the symmetric scheme or leapfrog
    const int blocks = pass_blocks_row_2d(nx, ny, ninst, grid_cap, 8);
    if (general) QHD_SWITCH_N(nx, { return (go_row<N_, pts_per_lane<N_>(), kModelQAA, true>)(blocks, ny, a); });
    QHD_SWITCH_N(nx, { return (go_row<N_, pts_per_lane<N_>(), kModelQAA, false>)(blocks, ny, a); });
  }
  const int blocks = pass_blocks_row_2d(nx, ny, ninst, grid_cap, points_per_lane);
  const int points = row_points_resolve(nx, points_per_lane);
  return general ? row_pass_qhd<true>(nx, ny, blocks, points, a) : row_pass_qhd<false>(nx, ny, blocks, points, a);
}

hipError_t launch_col_pass_2d(int nx, int ny, const InstDev* inst, int ninst, const int* nact, float2* psi,
                              const double* f, const double2* tw, int s, long long max_steps, int grid_cap,
                              int variant, hipStream_t stream, int model, bool y4, int kind) {
  const PassArgs a{inst, nact, psi, f, tw, s, max_steps, kind, stream};
  const bool general = y4 || kind != kPassPlain;
  if (model == kModelQAA) {
    // 64- and 128-point Walsh-Hadamard columns lie in one wavefront of the tile-wave form;
    // the others are staged (in-wave shuffles along a line)
    const int v = ny == 64 || ny == 128 ? kColTileWave : kColStaged;
    const int blocks = pass_blocks_col_2d(nx, ny, ninst, grid_cap, v);
    return general ? col_pass_qaa<true>(nx, ny, blocks, a) : col_pass_qaa<false>(nx, ny, blocks, a);
  }
  const int blocks = pass_blocks_col_2d(nx, ny, ninst, grid_cap, variant);
  const int v = col_variant_resolve(ny, variant);
  return general ? col_pass_qhd<true>(nx, ny, blocks, v, a) : col_pass_qhd<false>(nx, ny, blocks, v, a);
}

hipError_t launch_observe_col_2d(int nx, int ny, const InstDev* inst, int ninst, const float2* psi, const double* f,
                                 const double2* tw_ny, float2* out_psi, float* out_rho, double* partials, int stride,
                                 hipStream_t stream, int model) {
  QHD_SWITCH_N(ny, {
    constexpr int P_ = pts_per_lane<N_>();
    const int blocks = blocks_for((long long)ninst * (nx / 8), 1, 4096);
    if (model == kModelQAA)
      QHD_LAUNCH((k_observe_col_2d<N_, P_, kModelQAA>), dim3(blocks), dim3(256), 0, stream, inst, ninst, ilog2(nx), psi,
                 f, tw_ny, out_psi, out_rho, partials, stride);
    else
      QHD_LAUNCH((k_observe_col_2d<N_, P_, kModelQHD>), dim3(blocks), dim3(256), 0, stream, inst, ninst, ilog2(nx), psi,
                 f, tw_ny, out_psi, out_rho, partials, stride);
    return hipGetLastError();
  });
}

hipError_t launch_count_owing(const InstDev* inst, int ninst, int owe, int* owing, hipStream_t stream) {
  QHD_LAUNCH(k_count_owing, dim3(1), dim3(256), 0, stream, inst, ninst, owe, owing);
  return hipGetLastError();
}

hipError_t launch_set_axis(InstDev* inst, int ninst, int axis, hipStream_t stream) {
  QHD_LAUNCH(k_set_axis, dim3((ninst + 255) / 256), dim3(256), 0, stream, inst, ninst, axis);
  return hipGetLastError();
}

}  // namespace qhd
