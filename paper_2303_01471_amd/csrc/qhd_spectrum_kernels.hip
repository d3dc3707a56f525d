// Kernels of the spectrum entry point: the matrix-vector product
//     H(t) v = a(t) F^{-1} diag(|k|^2/2) F v + b(t) f v
// (the Fourier-diagonal kinetic operator of the split-operator scheme, App. C.2.1
// eq. prod_qhd_fft) on a plain row-major (x fastest) complex64 vector of one 2-D
// instance, and the Krylov vector operations of the Lanczos iteration.
#include <hip/hip_runtime.h>

#include "line_fft.h"
#include "pass_common.h"
#include "qhd_internal.h"

namespace qhd {

namespace {

template <int N>
constexpr int spec_p() { return N >= 1024 ? 16 : (N >= 8 ? 8 : N); }
// Blocks of the line kernels: one wavefront, so that the lines spread over the CUs and their
// exchanges take no block barrier (128 columns: 11.4 us in blocks of 256)
constexpr int kSpecLineThreads = 64;

// The matrix-vector product takes three launches, each with the values the separate
// operations round to: F_x from `in` to scratch; F_y, the kinetic diagonal and F_y^{-1} of
// the columns in one kernel; F_x^{-1} and the potential term.  A 128^2 vector is 128 KB, so
// every launch is latency (about 4 us); seven of them (copy, four transforms, diagonal,
// potential) and three more for the coefficients and scales made an iteration 78 us, now
// 47 (400 vectors).

// lines along x: line y is [y*N .. y*N+N); one line per TPL lanes.  With `f` the result w
// becomes w + b f v, f read from the plan's 8x8-tiled FP64 copy.
template <int N, int S, bool FINISH>
__global__ void __launch_bounds__(kSpecLineThreads) k_spec_rows(const float2* __restrict__ in, float2* __restrict__ out, int nlines,
                                                   const double2* __restrict__ twtab, const float2* __restrict__ v,
                                                   const double* __restrict__ f, double b) {
  constexpr int P = spec_p<N>(), TPL = N / P;
  constexpr int LPW = kSpecLineThreads / TPL;
  constexpr int SLOTS = LineLds<N>::kSlots;
  __shared__ float2 lds[LPW * SLOTS];
  const int ll = threadIdx.x / TPL, t = threadIdx.x % TPL;
  float2* my = lds + ll * SLOTS;
  Twiddles<N, P> tw;
  tw.load(twtab, t);
  for (long long l0 = (long long)blockIdx.x * LPW; l0 < nlines; l0 += (long long)gridDim.x * LPW) {
    const long long L = l0 + ll;
    const bool valid = L < nlines;
    const long long base = (valid ? L : 0) * N;
    float2 reg[P];
#pragma unroll
    for (int q = 0; q < P; ++q) reg[q] = in[base + t + q * TPL];
    line_fft<N, P, S>(reg, t, tw, my);
    if (valid) {
#pragma unroll
      for (int q = 0; q < P; ++q) {
        const int x = t + q * TPL;
        if constexpr (FINISH) {
          const double bf = b * f[tile_index(x, (int)L, N)];
          const float2 a = reg[q], c = v[base + x];
          reg[q] = make_float2((float)(a.x + bf * c.x), (float)(a.y + bf * c.y));
        }
        out[base + x] = reg[q];
      }
    }
  }
}

// Lines along y (stride nx): F_y, times s |k|^2 / 2 a with |k|^2 = (2 pi n_x / L_x)^2 +
// (2 pi n_y / L_y)^2 (cx, cy: its factors times a / 2), F_y^{-1}.  LPW adjacent columns per
// block, lane order (t, column) so that a slot access of consecutive threads touches
// consecutive columns.
template <int N>
__global__ void __launch_bounds__(kSpecLineThreads) k_spec_cols(float2* __restrict__ v, int nx, const double2* __restrict__ twtab,
                                                   double cx, double cy, double s) {
  constexpr int P = spec_p<N>(), TPL = N / P;
  constexpr int LPW = kSpecLineThreads / TPL;
  constexpr int SLOTS = LineLds<N>::kSlots;
  __shared__ float2 lds[LPW * SLOTS];
  const int ll = threadIdx.x % LPW, t = threadIdx.x / LPW;
  float2* my = lds + ll * SLOTS;
  Twiddles<N, P> tw;
  tw.load(twtab, t);
  for (long long c0 = (long long)blockIdx.x * LPW; c0 < nx; c0 += (long long)gridDim.x * LPW) {
    const long long x = c0 + ll;
    const bool valid = x < nx;
    float2* __restrict__ col = v + (valid ? x : 0);
    float2 reg[P];
#pragma unroll
    for (int q = 0; q < P; ++q) reg[q] = col[(long long)(t + q * TPL) * nx];
    line_fft<N, P, -1>(reg, t, tw, my);
    const int fx = freq((int)x, nx);
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const int fy = freq(t + q * TPL, N);
      const double m = s * fma(cx, (double)fx * fx, cy * (double)fy * fy);
      reg[q] = make_float2((float)(m * reg[q].x), (float)(m * reg[q].y));
    }
    wave_lds_sync();  // the transforms share the LDS
    line_fft<N, P, +1>(reg, t, tw, my);
    if (valid) {
#pragma unroll
      for (int q = 0; q < P; ++q) col[(long long)(t + q * TPL) * nx] = reg[q];
    }
    wave_lds_sync();
  }
}

// partials[(i * nblk + block) * 2 + {0,1}] = block's share of <V_i, w> (conj on V_i), FP64
__global__ void __launch_bounds__(256) k_spec_multidot(const float2* __restrict__ V, long long n, int count,
                                                       const float2* __restrict__ w, double* __restrict__ partials) {
  __shared__ double sr[256], si[256];
  const int i = blockIdx.y;
  const float2* __restrict__ vi = V + (long long)i * n;
  double ar = 0.0, ai = 0.0;
#pragma unroll 4
  for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < n; e += (long long)gridDim.x * 256) {
    const float2 a = vi[e], c = w[e];
    ar += (double)a.x * c.x + (double)a.y * c.y;
    ai += (double)a.x * c.y - (double)a.y * c.x;
  }
  sr[threadIdx.x] = ar;
  si[threadIdx.x] = ai;
  __syncthreads();
  if (threadIdx.x >= 64) return;
  // the tree t += t + 128, 64, .., 1: the upper levels from LDS, the rest inside the wavefront
  const int t = threadIdx.x;
  ar = (sr[t] + sr[t + 128]) + (sr[t + 64] + sr[t + 192]);
  ai = (si[t] + si[t + 128]) + (si[t + 64] + si[t + 192]);
  for (int o = 32; o > 0; o >>= 1) {
    ar += __shfl_down(ar, o, 64);
    ai += __shfl_down(ai, o, 64);
  }
  if (t == 0) {
    partials[((long long)i * gridDim.x + blockIdx.x) * 2 + 0] = ar;
    partials[((long long)i * gridDim.x + blockIdx.x) * 2 + 1] = ai;
  }
}

// Coefficient c of vector i (k = 2 i + c): the sum of its block partials in block order
// (FP64, the additions a host-side sum would make)
__device__ __forceinline__ double block_sum(const double* __restrict__ partials, int k) {
  double p[kSpecDotBlocks], acc = 0.0;
#pragma unroll
  for (int b = 0; b < kSpecDotBlocks; ++b) p[b] = partials[((long long)(k >> 1) * kSpecDotBlocks + b) * 2 + (k & 1)];
#pragma unroll
  for (int b = 0; b < kSpecDotBlocks; ++b) acc += p[b];
  return acc;
}

// coefficients [k0, k1) (pairs) into LDS, from device memory or from the dots' partials
__device__ __forceinline__ void load_coef(double* __restrict__ cl, const double* __restrict__ c, bool partials, int k0, int k1) {
  for (int k = 2 * k0 + (int)threadIdx.x; k < 2 * k1; k += blockDim.x) cl[k - 2 * k0] = partials ? block_sum(c, k) : c[k];
  __syncthreads();
}

// y <- y / |y| from its <y, y> partials; keep[0] = |y|
__global__ void k_spec_normalise(float2* __restrict__ w, long long n, const double* __restrict__ partials,
                                 double* __restrict__ keep) {
  const double acc = block_sum(partials, 0);
  const double nrm = sqrt(acc > 0.0 ? acc : 0.0);
  const double scale = 1.0 / nrm;
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e == 0) keep[0] = nrm;
  if (e >= n) return;
  const float2 z = w[e];
  w[e] = make_float2((float)(scale * (double)z.x), (float)(scale * (double)z.y));
}

// w <- scale (w - sum_i c_i V_i), c_i complex (FP64): in device memory, or with `partials`
// as the block partials of the dots; keep[0], when set, gets the real part of the newest one
// (the Lanczos diagonal entry).
__global__ void k_spec_multiaxpy(float2* __restrict__ w, const float2* __restrict__ V, long long n, int count,
                                 const double* __restrict__ c, bool partials, double scale, double* __restrict__ keep) {
  extern __shared__ double cl[];
  load_coef(cl, c, partials, 0, count);
  if (keep && blockIdx.x == 0 && threadIdx.x == 0) keep[0] = cl[2 * (count - 1)];
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  double xr = w[e].x, xi = w[e].y;
  for (int i = 0; i < count; ++i) {
    const float2 a = V[(long long)i * n + e];
    const double cr = cl[2 * i], ci = cl[2 * i + 1];
    xr -= cr * a.x - ci * a.y;
    xi -= cr * a.y + ci * a.x;
  }
  w[e] = make_float2((float)(scale * xr), (float)(scale * xi));
}

// Grouped form of the same update for long bases: group g of the grid's y dimension
// sums c_i V_i over its share of i into part[g] (FP64), then k_spec_axpy_fin subtracts
// the groups' sums in group order.  One thread per element and group instead of one per
// element gives the loads of a 16 K-point vector enough waves to be in flight.
__global__ void k_spec_axpy_part(const float2* __restrict__ V, long long n, int count, const double* __restrict__ c,
                                 bool partials, double2* __restrict__ part, double* __restrict__ keep) {
  extern __shared__ double cl[];
  const int g = blockIdx.y, groups = gridDim.y;
  const int per = (count + groups - 1) / groups;
  const int i0 = min(count, g * per), i1 = min(count, i0 + per);
  load_coef(cl, c, partials, i0, i1);
  if (keep && blockIdx.x == 0 && threadIdx.x == 0 && i0 < i1 && i1 == count) keep[0] = cl[2 * (count - 1 - i0)];
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  double xr = 0.0, xi = 0.0;
#pragma unroll 16
  for (int i = i0; i < i1; ++i) {  // (loads of 16 vectors in flight)
    const float2 a = V[(long long)i * n + e];
    const double cr = cl[2 * (i - i0)], ci = cl[2 * (i - i0) + 1];
    xr += cr * a.x - ci * a.y;
    xi += cr * a.y + ci * a.x;
  }
  part[(long long)g * n + e] = make_double2(xr, xi);
}

__global__ void k_spec_axpy_fin(float2* __restrict__ w, long long n, const double2* __restrict__ part, int groups,
                                double scale) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  double xr = w[e].x, xi = w[e].y;
  for (int g = 0; g < groups; ++g) {
    const double2 p = part[(long long)g * n + e];
    xr -= p.x;
    xi -= p.y;
  }
  w[e] = make_float2((float)(scale * xr), (float)(scale * xi));
}

// deterministic start vector from a counter-based hash (splitmix64 of the index)
__global__ void k_spec_random(float2* __restrict__ v, long long n, unsigned long long seed) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  unsigned long long z = seed + 0x9E3779B97F4A7C15ull * (unsigned long long)(e + 1);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  const float r = (float)((z >> 40) * (1.0 / 16777216.0)) - 0.5f;
  const float i = (float)((z & 0xFFFFFF) * (1.0 / 16777216.0)) - 0.5f;
  v[e] = make_float2(r, i);
}

inline unsigned grid1(long long n) { return (unsigned)((n + 255) / 256); }

}  // namespace

hipError_t spec_matvec(const float2* in, float2* scratch, float2* out, int nx, int ny, const double2* tw_x,
                       const double2* tw_y, double cx, double cy, const double* f, double b, hipStream_t st) {
  const double s = 1.0 / ((double)nx * (double)ny);
#define QHD_SPEC_SIZES(n, ...)                                                                    \
  switch (n) {                                                                                    \
    QHD_SPEC(8, __VA_ARGS__) QHD_SPEC(16, __VA_ARGS__) QHD_SPEC(32, __VA_ARGS__)                  \
    QHD_SPEC(64, __VA_ARGS__) QHD_SPEC(128, __VA_ARGS__) QHD_SPEC(256, __VA_ARGS__)               \
    QHD_SPEC(512, __VA_ARGS__) QHD_SPEC(1024, __VA_ARGS__)                                        \
    default:                                                                                      \
      return hipErrorInvalidValue;                                                                \
  }
#define QHD_SPEC(N, ...)                                         \
  case N: {                                                      \
    constexpr int N_ = N, LPW = kSpecLineThreads / (N_ / spec_p<N_>());       \
    __VA_ARGS__;                                                 \
    break;                                                       \
  }
  QHD_SPEC_SIZES(nx, hipLaunchKernelGGL((k_spec_rows<N_, -1, false>), dim3((unsigned)((ny + LPW - 1) / LPW)), dim3(kSpecLineThreads),
                                        0, st, in, scratch, ny, tw_x, nullptr, nullptr, 0.0))
  QHD_SPEC_SIZES(ny, hipLaunchKernelGGL((k_spec_cols<N_>), dim3((unsigned)((nx + LPW - 1) / LPW)), dim3(kSpecLineThreads), 0, st,
                                        scratch, nx, tw_y, cx, cy, s))
  QHD_SPEC_SIZES(nx, hipLaunchKernelGGL((k_spec_rows<N_, +1, true>), dim3((unsigned)((ny + LPW - 1) / LPW)), dim3(kSpecLineThreads),
                                        0, st, scratch, out, ny, tw_x, in, f, b))
#undef QHD_SPEC
#undef QHD_SPEC_SIZES
  return hipGetLastError();
}

hipError_t spec_multidot(const float2* V, long long n, int count, const float2* w, double* partials,
                         hipStream_t st) {
  hipLaunchKernelGGL(k_spec_multidot, dim3(kSpecDotBlocks, count), dim3(256), 0, st, V, n, count, w, partials);
  return hipGetLastError();
}

hipError_t spec_multiaxpy(float2* w, const float2* V, long long n, int count, const double* c, bool partials, double scale,
                          hipStream_t st, double2* part, int groups, double* keep) {
  if (groups > 1 && count >= 2 * groups) {
    const int per = (count + groups - 1) / groups;
    hipLaunchKernelGGL(k_spec_axpy_part, dim3(grid1(n), groups), dim3(256), sizeof(double) * 2 * per, st, V, n, count, c,
                       partials, part, keep);
    hipLaunchKernelGGL(k_spec_axpy_fin, dim3(grid1(n)), dim3(256), 0, st, w, n, part, groups, scale);
  } else {
    hipLaunchKernelGGL(k_spec_multiaxpy, dim3(grid1(n)), dim3(256), sizeof(double) * 2 * (count > 0 ? count : 1), st, w,
                       V, n, count, c, partials, scale, keep);
  }
  return hipGetLastError();
}

hipError_t spec_normalise(float2* w, long long n, const double* partials, double* keep, hipStream_t st) {
  hipLaunchKernelGGL(k_spec_normalise, dim3(grid1(n)), dim3(256), 0, st, w, n, partials, keep);
  return hipGetLastError();
}

hipError_t spec_random(float2* v, long long n, unsigned long long seed, hipStream_t st) {
  hipLaunchKernelGGL(k_spec_random, dim3(grid1(n)), dim3(256), 0, st, v, n, seed);
  return hipGetLastError();
}

}  // namespace qhd
