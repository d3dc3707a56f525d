// Declarations shared by the relaxed-QP host code (rqp.cpp) and its kernels
// (rqp_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace qhd {

constexpr int kRqpMaxDim = 8;
constexpr int kRqpMaxPoints = 16;    // r + 1 <= 16
constexpr int kRqpTilePoints = 8192; // points of a pass's LDS tile (64 KB of FP32 complex)
constexpr int kRqpMatStride = 264;   // doubles per step: the axis matrix, then the potential coefficient
constexpr int kRqpStepRun = 65;      // steps whose matrices one launch forms (64 and the one before them)

// theta (kinetic) and potential coefficient (turns) of a run of steps
struct RqpSteps {
  double theta[kRqpStepRun], beta_turns[kRqpStepRun];
};

// A set of consecutive axes that one pass applies in LDS, and the tiles of that pass.
struct RqpSet {
  int first, count;         // axes first + 1 .. first + count
  int threads;              // block size: 256 or 1024, each thread at most r + 1 points
  int n, s0;                // NP^count points of the set's lattice, NP^first points inside it
  int span;                 // first == 0: points of a tile (whole chunks of n); else inner points
  int inner_tiles;          // tiles over the s0 inner points (first > 0)
  unsigned magic_span;      // ceil(2^32 / span)
  unsigned magic[kRqpMaxDim];  // ceil(2^32 / stride) of each axis' LDS stride
};

// matrices and potential coefficients of `count` steps into tab[count][kRqpMatStride]
hipError_t rqp_matrices(int NP, const double* U, const double* lam, const RqpSteps& steps, int count, double* tab,
                        hipStream_t st);
// One pass over whole instances: mat0 (or NULL) along the set's axes, then
// `rounds` times the potential factor and the matrix of the next entry of mat1.
hipError_t rqp_pass(int NP, float2* psi, const double* f, const RqpSet& S, long long total_points,
                    const double* mat0, const double* mat1, int rounds, hipStream_t st);
// Blocks per instance of the readouts, by the lattice alone: the order of an instance's sums does
// not depend on the batch.  4096 points each, at most 256 blocks: enough for one large instance
// (all readouts of one 16^6 507 us; 9^5: one 61, 256 of them 320), small ones need no second pass.
inline int rqp_observe_blocks(long long N) {
  const long long most = N / 4096 + 1;
  return (int)(most < 256 ? most : 256);
}
// part: batch * d * rqp_observe_blocks() * NP doubles, unused with one block per instance
hipError_t rqp_marginals(int NP, const float2* psi, long long N, int d, int batch, double* part, float* marg,
                         hipStream_t st);
hipError_t rqp_objective(double* f, const double* Qb, int d, int NP, long long N, int batch, hipStream_t st);
hipError_t rqp_argmin(const double* f, long long N, int batch, double* fmin, long long* amin, hipStream_t st);
hipError_t rqp_init(float2* psi, const double* amp, int d, int NP, long long N, int batch, hipStream_t st);
// Sums per instance (rho, f rho, rho over the minimisers), optional rho output and, with
// psi_out, the state times exp(-2 pi i close_turns f) (the owed potential half step);
// part: 3 * batch * rqp_observe_blocks() doubles, unused with one block per instance
hipError_t rqp_observe(const float2* psi, const double* f, long long N, int batch, const double* fmin, double tol,
                       double* part, double* out, float* prob, float2* psi_out, double close_turns, hipStream_t st);

}  // namespace qhd
