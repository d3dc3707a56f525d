// Kernels of the relaxed QHD for box-constrained QP (App. F.2, eq.
// relaxed-qhd-discrete; Algorithm 2): the state lives on the (r+1)^d lattice
// (NP = r + 1 points per axis, axis 1 fastest), one FP32 complex value per point.
//
// The kinetic factor of one step is one NP x NP complex matrix
//     M = e^{i theta A'} = U diag(e^{i theta lambda_m}) U^T,   theta = dt a r^2 / 2,
// along every axis (A' = U diag(lambda) U^T); the factors of different axes commute.  The
// axes are split into sets whose lattice fits one block's LDS, and the sets are swept up
// and down in turn: the last set of a step is the first of the next one, so both steps'
// matrices and the potential factor exp(-i beta f) between them are one pass over memory
// ("K V K").  Two sets: one pass of 24 B per point and step.
//
// A' couples neighbours only (M[m][n] is real for even m - n and imaginary for odd) and is
// symmetric under m -> r - m, so for even r a line splits into its even and odd parts, each
// with a real-times-complex matrix of half the size: 82 FP64 multiply-adds per line of 9
// points instead of 324; for odd r the first property alone halves them.  The matrices are
// formed in FP64 for a run of steps by one small kernel; the passes read them with
// wave-uniform (scalar) loads.  Lines accumulate in FP64 and round to FP32 once per axis.
#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>

#include "line_fft.h"
#include "rqp_internal.h"

namespace qhd {

namespace {

constexpr int kThreads = 256;

template <int NP>
struct AxisMat {
  static constexpr bool SPLIT = (NP & 1) != 0;      // r even: even and odd parts of a line
  static constexpr int H = NP / 2, HE = H + 1;      // sizes of the odd and the even part
  static constexpr int SIZE = SPLIT ? HE * HE + H * H : NP * NP;
  static_assert(SIZE < kRqpMatStride, "the step's potential coefficient follows the matrix");
};

// the entries of M that line_apply uses (real or imaginary part by the parity of m - n), and
// after them the potential coefficient in turns; block = step
template <int NP>
__global__ void __launch_bounds__(kThreads) k_rqp_matrix(const double* __restrict__ U, const double* __restrict__ lam,
                                                        RqpSteps steps, double* __restrict__ tab) {
  using A = AxisMat<NP>;
  __shared__ double2 ph[NP];
  const int s = blockIdx.x;
  double* __restrict__ M = tab + s * kRqpMatStride;
  if (threadIdx.x < NP) {
    double sn, c;
    sincos(steps.theta[s] * lam[threadIdx.x], &sn, &c);
    ph[threadIdx.x] = make_double2(c, sn);
  }
  __syncthreads();
  auto entry = [&](int m, int n) {
    double acc = 0.0;
    const bool im = ((m - n) & 1) != 0;
#pragma unroll
    for (int k = 0; k < NP; ++k) acc = fma(U[m * NP + k] * U[n * NP + k], im ? ph[k].y : ph[k].x, acc);
    return acc;
  };
  for (int e = threadIdx.x; e < A::SIZE; e += blockDim.x) {
    double v;
    if constexpr (!A::SPLIT) {
      v = entry(e / NP, e % NP);
    } else {
      const bool even = e < A::HE * A::HE;
      const int q = even ? e : e - A::HE * A::HE, w = even ? A::HE : A::H;
      const int m = q / w, n = q % w;
      v = entry(m, n);
      if (n < A::H) v = 0.5 * (even ? v + entry(m, NP - 1 - n) : v - entry(m, NP - 1 - n));
    }
    M[e] = v;
  }
  if (threadIdx.x == 0) M[A::SIZE] = steps.beta_turns[s];
}

// A wave-uniform zero the compiler cannot see through (no memory access).  Offsetting
// the matrix by it once per line keeps the matrix reads (scalar loads, the same entry for
// every lane) inside the line loops instead of in vector registers.
__device__ __forceinline__ int opaque_zero() {
  int z;
  asm volatile("s_mov_b32 %0, 0" : "=s"(z));
  return z;
}

// acc += (IM ? i w : w) x
template <bool IM>
__device__ __forceinline__ void axpy(double2& acc, double w, double2 x) {
  if constexpr (IM) {
    acc.x = fma(-w, x.y, acc.x);
    acc.y = fma(w, x.x, acc.y);
  } else {
    acc.x = fma(w, x.x, acc.x);
    acc.y = fma(w, x.y, acc.y);
  }
}

template <int ROW, int N>
__device__ __forceinline__ double2 row_dot(const double* __restrict__ w, const double2* x) {
  double2 acc = make_double2(0.0, 0.0);
#pragma unroll
  for (int n = 0; n < N; ++n) {
    if ((ROW - n) & 1)
      axpy<true>(acc, w[n], x[n]);
    else
      axpy<false>(acc, w[n], x[n]);
  }
  return acc;
}

template <int NP, int M, typename STORE>
__device__ __forceinline__ void apply_rows(const double* __restrict__ W, const double2* x, const double2* u,
                                           const double2* v, STORE store) {
  using A = AxisMat<NP>;
  if constexpr (!A::SPLIT) {
    if constexpr (M < NP) {
      store(M, row_dot<M, NP>(W + M * NP, x));
      apply_rows<NP, M + 1>(W, x, u, v, store);
    }
  } else if constexpr (M < A::HE) {
    const double2 e = row_dot<M, A::HE>(W + M * A::HE, u);
    if constexpr (M == A::H) {
      store(M, e);
    } else {
      const double2 o = row_dot<M, A::H>(W + A::HE * A::HE + M * A::H, v);
      store(M, make_double2(e.x + o.x, e.y + o.y));
      store(NP - 1 - M, make_double2(e.x - o.x, e.y - o.y));
    }
    apply_rows<NP, M + 1>(W, x, u, v, store);
  }
}

// one line of the LDS tile (points `s` apart) times the axis matrix
template <int NP>
__device__ __forceinline__ void line_apply(const double* __restrict__ Mg, float2* __restrict__ line, int s) {
  using A = AxisMat<NP>;
  const double* __restrict__ W = Mg + opaque_zero();
  double2 x[NP];
#pragma unroll
  for (int m = 0; m < NP; ++m) assign(x[m], line[m * s]);
  auto store = [&](int m, double2 y) { assign(line[m * s], y); };
  if constexpr (!A::SPLIT) {
    apply_rows<NP, 0>(W, x, x, x, store);
  } else {
    double2 u[A::HE], v[A::H];
#pragma unroll
    for (int m = 0; m < A::H; ++m) {
      const double2 a = x[m], b = x[NP - 1 - m];
      u[m] = make_double2(a.x + b.x, a.y + b.y);
      v[m] = make_double2(a.x - b.x, a.y - b.y);
    }
    u[A::H] = x[A::H];
    apply_rows<NP, 0>(W, x, u, v, store);
  }
}

// One pass of a set of axes.  A tile is a block's LDS: for the leading set (axes 1..count) a
// run of whole chunks of NP^count contiguous points; for a trailing set the n = NP^count
// rows that share the indices of all other axes, times `span` consecutive inner points.
//   mat0 given: the matrix mat0 along the set's axes (the step before's)
//   rounds:     then, per round, the potential factor and the matrix of the next entry of
//               mat1 (one round per step: more than one only if the set holds every axis)
// Each axis rounds to FP32 on its LDS store.  Each thread owns at most NP points of the
// tile (loads, potential, stores) and one line of each axis.
//
// 256 instances of 9^5 points, us per step: 91 (axes 1-3, both steps') and 82 (axes 4-5) in
// turn, bound about equally by memory (24 B per point: 61) and by FP64 issue; one pass for
// axes 1-4, one for axis 5 and a matrix launch took 179.  f is loaded with the state, ahead of
// the matrices that come before its use.  Four waves per SIMD where 128 VGPRs hold a line (82
// against 87 us a step with three; with five the line spills: 193); for NP = 16 the bound
// spills (16^3: 14.8 against 12.8).
template <int NP, int NT, bool LEAD>
__global__ void __launch_bounds__(NT, NT == 256 && NP <= 9 ? 4 : 1) k_rqp_pass(float2* __restrict__ psi,
                                                const double* __restrict__ f, RqpSet S, long long total_points,
                                                long long tiles, const double* __restrict__ mat0, const double* __restrict__ mat1,
                                                int rounds) {
  constexpr int PTS = NP < kRqpTilePoints / NT ? NP : kRqpTilePoints / NT;
  extern __shared__ float2 seg[];
  const int tid = threadIdx.x;
  // tiles in eight contiguous runs, one per XCD: neighbouring tiles share cache lines
  const long long per = (tiles + 7) >> 3;
  for (long long q = blockIdx.x >> 3; q < per; q += gridDim.x >> 3) {
    const long long tile = (long long)(blockIdx.x & 7) * per + q;
    if (tile >= tiles) break;
    long long base;
    int npts, width = 0;
    if constexpr (LEAD) {
      base = tile * S.span;
      npts = (int)(total_points - base < (long long)S.span ? total_points - base : (long long)S.span);
    } else {
      const long long outer = tile / S.inner_tiles;
      const int inner = (int)(tile - outer * S.inner_tiles) * S.span;
      base = outer * S.s0 * S.n + inner;
      npts = S.n * S.span;
      width = S.s0 - inner < S.span ? S.s0 - inner : S.span;  // the last tile of a row may be narrower
    }
    float2 v[PTS];
    double fv[PTS];
    // Offset of element e of the tile from its base (false: none there).  The base is the
    // same for the whole block and a byte offset fits 32 bits, so an address is one register.
    float2* __restrict__ zt = psi + base;
    const double* __restrict__ ft = f + base;
    auto at = [](auto* p, unsigned off) {
      using B = typename std::conditional<std::is_const<typename std::remove_pointer<decltype(p)>::type>::value, const char, char>::type;
      return reinterpret_cast<decltype(p)>(reinterpret_cast<B*>(p) + off * (unsigned)sizeof(*p));
    };
    auto point = [&](int e, unsigned& off) {
      if constexpr (LEAD) {
        off = (unsigned)e;
        return e < npts;
      } else {
        const int row = S.span == 1 ? e : (int)__umulhi((unsigned)e, S.magic_span);
        const int w = e - row * S.span;
        off = (unsigned)row * (unsigned)S.s0 + (unsigned)w;
        return e < npts && w < width;
      }
    };
#pragma unroll
    for (int i = 0; i < PTS; ++i) {
      unsigned off;
      const bool in = point(tid + i * NT, off);
      v[i] = in ? *at(zt, off) : make_float2(0.0f, 0.0f);
      fv[i] = rounds > 0 && in ? *at(ft, off) : 0.0;
    }
    auto axes = [&](const double* __restrict__ M) {
      int s = LEAD ? 1 : S.span;
      for (int k = 0; k < S.count; ++k) {
        if (tid * NP < npts) {
          const int outer = s == 1 ? tid : (int)__umulhi((unsigned)tid, S.magic[k]);
          line_apply<NP>(M, seg + (tid - outer * s) + outer * s * NP, s);
        }
        __syncthreads();
        s *= NP;
      }
    };
    auto potential = [&](double beta) {
#pragma unroll
      for (int i = 0; i < PTS; ++i) v[i] = cmul_fd(v[i], phase_turns_d(beta * fv[i]));
    };
    auto put = [&]() {
#pragma unroll
      for (int i = 0; i < PTS; ++i)
        if (tid + i * NT < npts) seg[tid + i * NT] = v[i];
    };
    auto get = [&]() {
#pragma unroll
      for (int i = 0; i < PTS; ++i)
        if (tid + i * NT < npts) v[i] = seg[tid + i * NT];
    };
    if (mat0) {
      put();
      __syncthreads();
      axes(mat0);
      get();
    }
    for (int rd = 0; rd < rounds; ++rd) {
      const double* __restrict__ M = mat1 + (long long)rd * kRqpMatStride;
      potential(M[AxisMat<NP>::SIZE]);
      put();  // (each thread's own points: nobody else reads them before the barrier)
      __syncthreads();
      axes(M);
      get();
    }
    int again = tid;  // the offsets are formed anew: kept, they cost a wave per SIMD
    asm volatile("" : "+v"(again));
#pragma unroll
    for (int i = 0; i < PTS; ++i) {
      unsigned off;
      if (point(again + i * NT, off)) *at(zt, off) = v[i];
    }
    __syncthreads();  // the next tile reuses the LDS
  }
}

// f on the lattice: f = 1/2 x^T Q x + b^T x, x_k = j_k / r (FP64); Qb = [Q (d x d), b (d)]
// per instance
__global__ void k_rqp_objective(double* __restrict__ f, const double* __restrict__ Qb, int d, int NP,
                                long long N, long long total) {
  const long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= total) return;
  const long long inst = g / N;
  long long p = g - inst * N;
  const double* Q = Qb + inst * (long long)(d * d + d);
  const double* b = Q + d * d;
  const double inv_r = 1.0 / (double)(NP - 1);
  double x[kRqpMaxDim];
  for (int k = 0; k < d; ++k) {
    x[k] = (double)(p % NP) * inv_r;
    p /= NP;
  }
  double v = 0.0;
  for (int k = 0; k < d; ++k) {
    double qx = 0.0;
    for (int l = 0; l < d; ++l) qx = fma(Q[k * d + l], x[l], qx);
    v = fma(x[k], fma(0.5, qx, b[k]), v);
  }
  f[g] = v;
}

// one block per instance: lowest-index minimiser of f
__global__ void __launch_bounds__(kThreads) k_rqp_argmin(const double* __restrict__ f, long long N,
                                                        double* __restrict__ fmin, long long* __restrict__ amin) {
  __shared__ double sv[kThreads];
  __shared__ long long si[kThreads];
  const double* fi = f + (long long)blockIdx.x * N;
  double bv = INFINITY;
  long long bi = LLONG_MAX;
  for (long long p = threadIdx.x; p < N; p += kThreads) {
    const double v = fi[p];
    if (v < bv) {
      bv = v;
      bi = p;
    }
  }
  sv[threadIdx.x] = bv;
  si[threadIdx.x] = bi;
  __syncthreads();
  for (int o = kThreads / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      const double v = sv[threadIdx.x + o];
      const long long id = si[threadIdx.x + o];
      if (v < sv[threadIdx.x] || (v == sv[threadIdx.x] && id < si[threadIdx.x])) {
        sv[threadIdx.x] = v;
        si[threadIdx.x] = id;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    fmin[blockIdx.x] = sv[0];
    amin[blockIdx.x] = si[0];
  }
}

// psi <- discrete Gaussian prod_k amp[j_k]; grid (points, instances)
template <int NP>
__global__ void __launch_bounds__(kThreads) k_rqp_init(float2* __restrict__ psi, const double* __restrict__ amp, int d,
                                                      unsigned N, int batch) {
  __shared__ double a[NP];
  if (threadIdx.x < NP) a[threadIdx.x] = amp[threadIdx.x];
  __syncthreads();
  const unsigned p0 = blockIdx.x * kThreads + threadIdx.x;
  if (p0 >= N) return;
  double v = 1.0;
  for (unsigned k = 0, p = p0; k < (unsigned)d; ++k, p /= NP) v *= a[p % NP];
  const float2 z = make_float2((float)v, 0.0f);
  for (long long i = blockIdx.y; i < batch; i += gridDim.y) psi[i * N + p0] = z;
}

// Sums of rho, f rho, rho over the minimisers, in FP64 and in a fixed order (per-thread
// strided sums, a tree, then the blocks of an instance in turn by k_rqp_reduce); optional
// rho and state output.  Grid (blocks of an instance, instances): with one block per
// instance 256 instances of 9^5 points took 250 us, the chip idle.
__global__ void __launch_bounds__(kThreads) k_rqp_observe(const float2* __restrict__ psi, const double* __restrict__ f,
                                                         long long N, const double* __restrict__ fmin, double tol,
                                                         double* __restrict__ part, double* __restrict__ out,
                                                         float* __restrict__ prob, float2* __restrict__ psi_out,
                                                         double close_turns, int batch) {
  __shared__ double s0[kThreads], s1[kThreads], s2[kThreads];
  for (int inst = blockIdx.y; inst < batch; inst += gridDim.y) {
    const long long off = (long long)inst * N;
    const double thr = fmin[inst] + tol;
    double a = 0.0, b = 0.0, c = 0.0;
    for (long long p = (long long)blockIdx.x * kThreads + threadIdx.x; p < N; p += (long long)gridDim.x * kThreads) {
      const float2 v = psi[off + p];
      const double rho = (double)v.x * v.x + (double)v.y * v.y;
      const double fv = f[off + p];
      a += rho;
      b = fma(fv, rho, b);
      if (fv <= thr) c += rho;
      if (prob) prob[off + p] = (float)rho;
      if (psi_out) psi_out[off + p] = close_turns != 0.0 ? cmul_fd(v, phase_turns_d(close_turns * fv)) : v;
    }
    s0[threadIdx.x] = a;
    s1[threadIdx.x] = b;
    s2[threadIdx.x] = c;
    __syncthreads();
    for (int o = kThreads / 2; o > 0; o >>= 1) {
      if ((int)threadIdx.x < o) {
        s0[threadIdx.x] += s0[threadIdx.x + o];
        s1[threadIdx.x] += s1[threadIdx.x + o];
        s2[threadIdx.x] += s2[threadIdx.x + o];
      }
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      double* o = gridDim.x == 1 ? out + 3ll * inst : part + 3 * ((long long)inst * gridDim.x + blockIdx.x);
      o[0] = s0[0];
      o[1] = s1[0];
      o[2] = s2[0];
    }
    __syncthreads();
  }
}

// out[g][c] = sum over the `blocks` partial rows of group g; thread = (group, column)
template <typename T>
__global__ void k_rqp_reduce(const double* __restrict__ part, int blocks, int cols, long long groups,
                             T* __restrict__ out) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= groups * cols) return;
  const long long g = e / cols;
  const double* p = part + g * blocks * cols + (e - g * cols);
  double s = 0.0;
  for (int b = 0; b < blocks; ++b) s += p[(long long)b * cols];
  out[e] = (T)s;
}

// Marginal distributions over j_k; grid (blocks of an instance, axes, instances).  A thread
// takes whole lines of its axis, so its NP bins stay in registers.
template <int NP>
__global__ void __launch_bounds__(kThreads) k_rqp_marginals(const float2* __restrict__ psi, long long N, int d,
                                                           double* __restrict__ part, float* __restrict__ marg,
                                                           int batch) {
  __shared__ double red[kThreads / 64][NP];
  const int k = blockIdx.y;
  unsigned stride = 1;
  for (int q = 0; q < k; ++q) stride *= NP;
  const unsigned lines = (unsigned)(N / NP);
  for (int inst = blockIdx.z; inst < batch; inst += gridDim.z) {
    const float2* __restrict__ z = psi + (long long)inst * N;
    double bin[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) bin[j] = 0.0;
    for (unsigned L = blockIdx.x * kThreads + threadIdx.x; L < lines; L += gridDim.x * kThreads) {
      const unsigned outer = L / stride;
      const unsigned p = outer * stride * NP + (L - outer * stride);
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        const float2 v = z[p + j * stride];
        bin[j] += (double)v.x * v.x + (double)v.y * v.y;
      }
    }
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      for (int o = 32; o > 0; o >>= 1) bin[j] += __shfl_xor(bin[j], o, 64);
      if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][j] = bin[j];
    }
    __syncthreads();
    if ((int)threadIdx.x < NP) {
      double s = 0.0;
      for (int w = 0; w < kThreads / 64; ++w) s += red[w][threadIdx.x];
      const long long row = (long long)inst * d + k;
      if (gridDim.x == 1)
        marg[row * NP + threadIdx.x] = (float)s;
      else
        part[(row * gridDim.x + blockIdx.x) * NP + threadIdx.x] = s;
    }
    __syncthreads();
  }
}

template <int NP>
hipError_t matrices_np(const double* U, const double* lam, const RqpSteps& steps, int count, double* tab,
                       hipStream_t st) {
  hipLaunchKernelGGL((k_rqp_matrix<NP>), dim3((unsigned)count), dim3(kThreads), 0, st, U, lam, steps, tab);
  return hipGetLastError();
}

template <int NP, int NT, bool LEAD>
hipError_t pass_np(float2* psi, const double* f, const RqpSet& S, long long total_points,
                   const double* mat0, const double* mat1, int rounds, hipStream_t st) {
  const int points = LEAD ? S.span : S.n * S.span;
  if (points < NP || points > NT * NP || points % NP != 0 || points > kRqpTilePoints ||
      S.count < 1 || S.count > kRqpMaxDim) return hipErrorInvalidValue;
  const long long tiles = LEAD ? (total_points + S.span - 1) / S.span
                               : total_points / ((long long)S.s0 * S.n) * S.inner_tiles;
  long long blocks = (tiles + 7) / 8;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL((k_rqp_pass<NP, NT, LEAD>), dim3((unsigned)(8 * blocks)), dim3(NT), sizeof(float2) * points, st,
                     psi, f, S, total_points, tiles, mat0, mat1, rounds);
  return hipGetLastError();
}

template <int NP>
hipError_t pass_any(float2* psi, const double* f, const RqpSet& S, long long total_points,
                    const double* mat0, const double* mat1, int rounds, hipStream_t st) {
  if (S.threads == kThreads)
    return S.first == 0 ? pass_np<NP, kThreads, true>(psi, f, S, total_points, mat0, mat1, rounds, st)
                        : pass_np<NP, kThreads, false>(psi, f, S, total_points, mat0, mat1, rounds, st);
  return S.first == 0 ? pass_np<NP, 1024, true>(psi, f, S, total_points, mat0, mat1, rounds, st)
                      : pass_np<NP, 1024, false>(psi, f, S, total_points, mat0, mat1, rounds, st);
}

template <int NP>
hipError_t marginals_np(const float2* psi, long long N, int d, int batch, double* part, int blocks, float* marg,
                        hipStream_t st) {
  hipLaunchKernelGGL((k_rqp_marginals<NP>), dim3((unsigned)blocks, (unsigned)d, (unsigned)(batch < 65535 ? batch : 65535)),
                     dim3(kThreads), 0, st, psi, N, d, part, marg, batch);
  if (blocks == 1) return hipGetLastError();
  const long long groups = (long long)batch * d;
  hipLaunchKernelGGL((k_rqp_reduce<float>), dim3((unsigned)((groups * NP + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                     st, part, blocks, NP, groups, marg);
  return hipGetLastError();
}

template <int NP>
hipError_t init_np(float2* psi, const double* amp, int d, long long N, int batch, hipStream_t st) {
  const int rows = batch < 16384 ? batch : 16384;
  hipLaunchKernelGGL((k_rqp_init<NP>), dim3((unsigned)((N + kThreads - 1) / kThreads), (unsigned)rows), dim3(kThreads),
                     0, st, psi, amp, d, (unsigned)N, batch);
  return hipGetLastError();
}

}  // namespace

// run the call with NP_ = NP as a constant
#define QHD_RQP_CASE(n, ...) \
  case n: {                  \
    constexpr int NP_ = n;   \
    return __VA_ARGS__;      \
  }
#define QHD_RQP_SWITCH(NP, ...)                                                                              \
  switch (NP) {                                                                                              \
    QHD_RQP_CASE(2, __VA_ARGS__) QHD_RQP_CASE(3, __VA_ARGS__) QHD_RQP_CASE(4, __VA_ARGS__)                   \
    QHD_RQP_CASE(5, __VA_ARGS__) QHD_RQP_CASE(6, __VA_ARGS__) QHD_RQP_CASE(7, __VA_ARGS__)                   \
    QHD_RQP_CASE(8, __VA_ARGS__) QHD_RQP_CASE(9, __VA_ARGS__) QHD_RQP_CASE(10, __VA_ARGS__)                  \
    QHD_RQP_CASE(11, __VA_ARGS__) QHD_RQP_CASE(12, __VA_ARGS__) QHD_RQP_CASE(13, __VA_ARGS__)                \
    QHD_RQP_CASE(14, __VA_ARGS__) QHD_RQP_CASE(15, __VA_ARGS__) QHD_RQP_CASE(16, __VA_ARGS__)                \
    default:                                                                                                 \
      return hipErrorInvalidValue;                                                                           \
  }

hipError_t rqp_matrices(int NP, const double* U, const double* lam, const RqpSteps& steps, int count, double* tab,
                        hipStream_t st) {
  if (count < 1 || count > kRqpStepRun) return hipErrorInvalidValue;
  QHD_RQP_SWITCH(NP, matrices_np<NP_>(U, lam, steps, count, tab, st))
}

hipError_t rqp_pass(int NP, float2* psi, const double* f, const RqpSet& S, long long total_points,
                    const double* mat0, const double* mat1, int rounds, hipStream_t st) {
  QHD_RQP_SWITCH(NP, pass_any<NP_>(psi, f, S, total_points, mat0, mat1, rounds, st))
}

hipError_t rqp_marginals(int NP, const float2* psi, long long N, int d, int batch, double* part, float* marg,
                         hipStream_t st) {
  const int blocks = rqp_observe_blocks(N);
  QHD_RQP_SWITCH(NP, marginals_np<NP_>(psi, N, d, batch, part, blocks, marg, st))
}

hipError_t rqp_objective(double* f, const double* Qb, int d, int NP, long long N, int batch, hipStream_t st) {
  const long long total = N * batch;
  hipLaunchKernelGGL(k_rqp_objective, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, f, Qb, d, NP, N, total);
  return hipGetLastError();
}

hipError_t rqp_argmin(const double* f, long long N, int batch, double* fmin, long long* amin, hipStream_t st) {
  hipLaunchKernelGGL(k_rqp_argmin, dim3((unsigned)batch), dim3(kThreads), 0, st, f, N, fmin, amin);
  return hipGetLastError();
}

hipError_t rqp_init(float2* psi, const double* amp, int d, int NP, long long N, int batch, hipStream_t st) {
  QHD_RQP_SWITCH(NP, init_np<NP_>(psi, amp, d, N, batch, st))
}

hipError_t rqp_observe(const float2* psi, const double* f, long long N, int batch, const double* fmin, double tol,
                       double* part, double* out, float* prob, float2* psi_out, double close_turns, hipStream_t st) {
  const int blocks = rqp_observe_blocks(N);
  hipLaunchKernelGGL(k_rqp_observe, dim3((unsigned)blocks, (unsigned)(batch < 65535 ? batch : 65535)), dim3(kThreads), 0,
                     st, psi, f, N, fmin, tol, part, out, prob, psi_out, close_turns, batch);
  if (blocks == 1) return hipGetLastError();
  hipLaunchKernelGGL((k_rqp_reduce<double>), dim3((unsigned)((3ll * batch + kThreads - 1) / kThreads)), dim3(kThreads),
                     0, st, part, blocks, 3, (long long)batch, out);
  return hipGetLastError();
}

}  // namespace qhd
