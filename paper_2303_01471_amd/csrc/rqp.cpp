// Relaxed QHD for box-constrained QP: the C ABI of include/qhd_rqp.h.
//
// Host side: validation, the eigen-decomposition of the relaxed chain adjacency A'
// (FP64 cyclic Jacobi, once per handle), the split of the axes into sets, the schedule per
// step, and the launch sequence of the symmetric steps.  Kernels in rqp_kernels.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../../include/qhd_rqp.h"
#include "rqp_internal.h"

namespace qhd {
void set_error_message(const char* msg);
}

using namespace qhd;

struct qhd_rqp_s {
  qhd_rqp_desc desc{};
  std::vector<double> table;  // TABLE schedule (host copy)
  int batch = 0, NP = 0, device = 0;
  long long N = 0;
  float2* psi = nullptr;
  double* f = nullptr;
  double* Qb = nullptr;     // per instance [Q (d x d), b (d)]
  double* U = nullptr;      // eigenvectors of A' (columns), row-major NP x NP
  double* lam = nullptr;    // eigenvalues of A'
  double* tab = nullptr;    // per step of a run: axis matrix and potential coefficient
  double* part = nullptr;   // readouts: per-block sums and marginals
  double* amp = nullptr;    // discrete Gaussian amplitudes of one axis
  double* fmin = nullptr;
  long long* amin = nullptr;
  double* sums = nullptr;   // [batch][3]
  double* host_sums = nullptr;  // pinned
  std::vector<double> fmin_h;
  std::vector<long long> amin_h;
  std::vector<char> has_obj;
  long long steps_done = 0;
  bool pending = false;     // the trailing potential half step of the last step is owed
  // The axes in sets, swept up and down in turn: inside a call the last set of a step is one pass
  // with the first of the next.  A call ends with its last set applied: what the device holds
  // is then the same whether calls are eager, captured, replayed or reset in between.
  std::vector<RqpSet> sets;
  int next = 0;             // the set that the next step begins with
  RqpSteps steps{};         // host copy of the run being formed
  bool unfused = false;     // each axis of a set in passes of its own, the same values
};

namespace {

qhd_status rfail(qhd_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  set_error_message(buf);
  return st;
}

#define RQP_TRY(expr)                                                                                 \
  do {                                                                                                \
    hipError_t e_ = (expr);                                                                           \
    if (e_ != hipSuccess)                                                                             \
      return rfail(e_ == hipErrorOutOfMemory ? QHD_ENOMEM : QHD_EDEVICE, "%s: %s", #expr,             \
                   hipGetErrorString(e_));                                                            \
  } while (0)

// symmetric tridiagonal A' of one axis: off-diagonal sqrt((j+1)(r-j)/r), j = 0..r-1
std::vector<double> relaxed_adjacency(int r) {
  const int n = r + 1;
  std::vector<double> A((size_t)n * n, 0.0);
  for (int j = 0; j < r; ++j) {
    const double v = std::sqrt((double)(j + 1) * (double)(r - j) / (double)r);
    A[(size_t)(j + 1) * n + j] = A[(size_t)j * n + j + 1] = v;
  }
  return A;
}

// cyclic Jacobi: A = Z diag(w) Z^T for a real symmetric n x n matrix (row-major)
void jacobi(std::vector<double> A, int n, std::vector<double>& w, std::vector<double>& Z) {
  Z.assign((size_t)n * n, 0.0);
  for (int k = 0; k < n; ++k) Z[(size_t)k * n + k] = 1.0;
  for (int sweep = 0; sweep < 100; ++sweep) {
    double off = 0.0;
    for (int p = 0; p < n; ++p)
      for (int q = p + 1; q < n; ++q) off += A[(size_t)p * n + q] * A[(size_t)p * n + q];
    if (off < 1e-32) break;
    for (int p = 0; p < n - 1; ++p)
      for (int q = p + 1; q < n; ++q) {
        const double apq = A[(size_t)p * n + q];
        if (std::fabs(apq) < 1e-300) continue;
        const double app = A[(size_t)p * n + p], aqq = A[(size_t)q * n + q];
        const double th = 0.5 * (aqq - app) / apq;
        const double t = (th >= 0 ? 1.0 : -1.0) / (std::fabs(th) + std::sqrt(th * th + 1.0));
        const double c = 1.0 / std::sqrt(t * t + 1.0), s = t * c;
        for (int k = 0; k < n; ++k) {  // A <- A J
          const double akp = A[(size_t)k * n + p], akq = A[(size_t)k * n + q];
          A[(size_t)k * n + p] = c * akp - s * akq;
          A[(size_t)k * n + q] = s * akp + c * akq;
        }
        for (int k = 0; k < n; ++k) {  // A <- J^T A
          const double apk = A[(size_t)p * n + k], aqk = A[(size_t)q * n + k];
          A[(size_t)p * n + k] = c * apk - s * aqk;
          A[(size_t)q * n + k] = s * apk + c * aqk;
        }
        for (int k = 0; k < n; ++k) {  // Z <- Z J
          const double zkp = Z[(size_t)k * n + p], zkq = Z[(size_t)k * n + q];
          Z[(size_t)k * n + p] = c * zkp - s * zkq;
          Z[(size_t)k * n + q] = s * zkp + c * zkq;
        }
      }
  }
  w.resize(n);
  for (int k = 0; k < n; ++k) w[k] = A[(size_t)k * n + k];
}

// a, b of step j at the step midpoint (TABLE: the j-th pair)
void schedule(const qhd_rqp_s* h, long long j, double& a, double& b) {
  const qhd_rqp_desc& d = h->desc;
  if (d.sched_kind == QHD_SCHED_TABLE) {
    a = h->table[2 * j];
    b = h->table[2 * j + 1];
    return;
  }
  if (d.sched_kind == QHD_SCHED_CONST) {
    a = d.sched_p[0];
    b = d.sched_p[1];
    return;
  }
  const double t = ((double)j + 0.5) * d.dt;
  if (d.sched_kind == QHD_SCHED_LINEAR) {
    const double g = t / d.sched_p[0];
    a = 1.0 - g;
    b = g;
  } else {
    const double t3 = t * t * t;
    a = 2.0 / (d.sched_p[0] + t3);
    b = 2.0 * t3;
  }
}

// theta and potential coefficient of steps j0 .. j0 + count - 1 (the first entry is only the
// step before; with `before` false step j0 + 1 has no half step to merge with)
void step_table(qhd_rqp h, long long j0, int count, bool before) {
  const qhd_rqp_desc& d = h->desc;
  const double r2 = (double)d.r * (double)d.r;
  double prev = 0.0;
  for (int q = 0; q < count; ++q) {
    double a = 0.0, b = 0.0;
    if (q > 0 || before) schedule(h, j0 + q, a, b);
    // merged potential half steps: the trailing half of the step before and the leading half
    const double beta = 0.5 * d.dt * b + (q > 1 || before ? 0.5 * d.dt * prev : 0.0);
    h->steps.theta[q] = 0.5 * d.dt * a * r2;
    h->steps.beta_turns[q] = beta * 0.15915494309189533577;
    prev = b;
  }
}

void release(qhd_rqp h) {
  if (!h) return;
  (void)hipSetDevice(h->device);
  for (void* p : {(void*)h->psi, (void*)h->f, (void*)h->Qb, (void*)h->U, (void*)h->lam, (void*)h->tab, (void*)h->amp,
                  (void*)h->fmin, (void*)h->amin, (void*)h->sums, (void*)h->part})
    if (p) (void)hipFree(p);
  if (h->host_sums) (void)hipHostFree(h->host_sums);
  delete h;
}

constexpr int kNarrow = 8;                       // inner points of a trailing tile at least (64 B)

long long ipow(int b, int e) {
  long long v = 1;
  for (int k = 0; k < e; ++k) v *= b;
  return v;
}

// Tiles of axes first + 1 .. first + count.  256 threads and their 256 lines where the set's
// lattice fits (9^5: 729 leading points, 81 trailing rows by 27), else 1024.  Fewer whole
// chunks or inner points per tile while that leaves the chip short of blocks.
RqpSet make_set(int NP, int first, int count, long long total) {
  RqpSet S{};
  S.first = first;
  S.count = count;
  S.n = (int)ipow(NP, count);
  S.s0 = (int)ipow(NP, first);
  const int narrow = first == 0 ? 1 : std::min(kNarrow, S.s0);
  S.threads = (long long)S.n * narrow <= 256 * NP ? 256 : 1024;
  const int most = std::min(S.threads * NP, kRqpTilePoints) / S.n;  // chunks or inner points
  const long long chunks = total / S.n;
  int span = (int)std::max<long long>(std::min<long long>(most, chunks / 1024), std::min(narrow, most));
  if (first == 0) {
    S.span = span * S.n;
  } else {
    span = std::min(span, S.s0);
    S.inner_tiles = (S.s0 + span - 1) / span;
    S.span = (S.s0 + S.inner_tiles - 1) / S.inner_tiles;
  }
  auto magic = [](long long s) { return (unsigned)((((1ull << 32) + s - 1) / s) & 0xffffffffull); };
  S.magic_span = magic(S.span);
  long long s = first == 0 ? 1 : S.span;
  for (int k = 0; k < count; ++k, s *= NP) S.magic[k] = magic(s);
  return S;
}

// The fewest sets whose tiles fit, and among those the most even split: the passes then
// share the matrix work (9^5 as 3 + 2 axes).
std::vector<RqpSet> make_sets(int NP, int d, long long total) {
  const long long most = std::min(1024ll * NP, (long long)kRqpTilePoints);
  int lead = 1, trail = 0;
  while (lead < d && ipow(NP, lead + 1) <= most) ++lead;
  while (trail < d && ipow(NP, trail + 1) * kNarrow <= most) ++trail;
  const int ntrail = (d - lead + trail - 1) / trail;
  int first = std::min(lead, (d + ntrail) / (ntrail + 1));
  while (d - first > ntrail * trail) ++first;
  std::vector<RqpSet> sets{make_set(NP, 0, ntrail ? first : d, total)};
  for (int k = 0, at = first; k < ntrail; ++k) {
    const int c = (d - at + ntrail - k - 1) / (ntrail - k);
    sets.push_back(make_set(NP, at, c, total));
    at += c;
  }
  return sets;
}

// One pass of set i: mat0 (or NULL), then `rounds` steps from mat1 on.
hipError_t set_pass(qhd_rqp h, int i, long long total, const double* mat0, const double* mat1, int rounds,
                    hipStream_t st) {
  const RqpSet& S = h->sets[i];  // (total: whole instances)
  if (!h->unfused) return rqp_pass(h->NP, h->psi, h->f, S, total, mat0, mat1, rounds, st);
  // the reference form of the same arithmetic: one pass per axis and matrix
  hipError_t e = hipSuccess;
  for (int rd = mat0 ? -1 : 0; rd < rounds; ++rd)
    for (int k = 0; k < S.count && e == hipSuccess; ++k) {
      const double* m = rd < 0 ? mat0 : mat1 + (long long)rd * kRqpMatStride;
      const RqpSet axis = make_set(h->NP, S.first + k, 1, total);
      const bool pot = rd >= 0 && k == 0;  // the potential factor comes before the first axis
      e = rqp_pass(h->NP, h->psi, h->f, axis, total, pot ? nullptr : m, m, pot ? 1 : 0, st);
    }
  return e;
}

qhd_status validate(const qhd_rqp_desc* d, int batch) {
  if (!d) return rfail(QHD_EINVAL, "desc is NULL");
  if (batch < 1) return rfail(QHD_EINVAL, "batch must be >= 1");
  if (d->dim < 1 || d->dim > kRqpMaxDim) return rfail(QHD_EINVAL, "dim must be in [1, %d]", kRqpMaxDim);
  if (d->r < 1 || d->r + 1 > kRqpMaxPoints) return rfail(QHD_EINVAL, "r must be in [1, %d]", kRqpMaxPoints - 1);
  if (!std::isfinite(d->dt) || !(d->dt > 0.0)) return rfail(QHD_EINVAL, "dt must be finite and > 0");
  if (d->nsteps < 0) return rfail(QHD_EINVAL, "nsteps must be >= 0");
  if (!std::isfinite(d->min_tol) || d->min_tol < 0.0) return rfail(QHD_EINVAL, "min_tol must be finite and >= 0");
  switch (d->sched_kind) {
    case QHD_SCHED_NESTEROV:
    case QHD_SCHED_LINEAR:
      if (!std::isfinite(d->sched_p[0]) || !(d->sched_p[0] > 0.0))
        return rfail(QHD_EINVAL, "schedule parameter sched_p[0] must be > 0");
      break;
    case QHD_SCHED_CONST:
      if (!std::isfinite(d->sched_p[0]) || !std::isfinite(d->sched_p[1]))
        return rfail(QHD_EINVAL, "CONST schedule needs finite a0, b0");
      break;
    case QHD_SCHED_TABLE:
      if (d->nsteps > 0 && !d->sched_table) return rfail(QHD_EINVAL, "TABLE schedule needs sched_table");
      for (long long j = 0; j < 2 * d->nsteps; ++j)
        if (!std::isfinite(d->sched_table[j])) return rfail(QHD_EINVAL, "sched_table[%lld] is not finite", j);
      break;
    default:
      return rfail(QHD_EINVAL, "unknown sched_kind %d", d->sched_kind);
  }
  double pts = 1.0;
  for (int k = 0; k < d->dim; ++k) pts *= (double)(d->r + 1);
  if (pts > (double)(1 << 24)) return rfail(QHD_EUNSUPPORTED, "(r + 1)^d = %.0f lattice points exceeds 2^24", pts);
  if (pts * batch > 4.0e9) return rfail(QHD_EUNSUPPORTED, "batch x (r + 1)^d exceeds 4e9 points");
  return QHD_OK;
}

}  // namespace

extern "C" {

qhd_status qhd_rqp_create(const qhd_rqp_desc* desc, int32_t batch, qhd_rqp* out) {
  set_error_message("");
  if (!out) return rfail(QHD_EINVAL, "out is NULL");
  *out = nullptr;
  qhd_status st = validate(desc, batch);
  if (st != QHD_OK) return st;
  qhd_rqp h = new qhd_rqp_s;
  h->desc = *desc;
  if (desc->sched_kind == QHD_SCHED_TABLE)
    h->table.assign(desc->sched_table, desc->sched_table + 2 * desc->nsteps);
  h->desc.sched_table = nullptr;
  h->batch = batch;
  h->NP = desc->r + 1;
  h->N = 1;
  for (int k = 0; k < desc->dim; ++k) h->N *= h->NP;
  const char* unfused = std::getenv("QHD_RQP_UNFUSED");  // 1: one pass per axis and matrix
  h->unfused = unfused && std::strcmp(unfused, "1") == 0;
  h->sets = make_sets(h->NP, desc->dim, h->N * batch);
  h->fmin_h.assign(batch, 0.0);
  h->amin_h.assign(batch, 0);
  h->has_obj.assign(batch, 0);
  hipError_t e = hipGetDevice(&h->device);
  const size_t pts = (size_t)h->N * batch;
  const int d = desc->dim, NP = h->NP;
  if (e == hipSuccess) e = hipMalloc(&h->psi, sizeof(float2) * pts);
  if (e == hipSuccess) e = hipMalloc(&h->f, sizeof(double) * pts);
  if (e == hipSuccess) e = hipMalloc(&h->Qb, sizeof(double) * (size_t)batch * (d * d + d));
  if (e == hipSuccess) e = hipMalloc(&h->U, sizeof(double) * NP * NP);
  if (e == hipSuccess) e = hipMalloc(&h->lam, sizeof(double) * NP);
  if (e == hipSuccess) e = hipMalloc(&h->tab, sizeof(double) * kRqpStepRun * kRqpMatStride);
  const int blocks = rqp_observe_blocks(h->N);
  if (e == hipSuccess && blocks > 1)
    e = hipMalloc(&h->part, sizeof(double) * batch * (size_t)blocks * std::max(3, d * NP));
  if (e == hipSuccess) e = hipMalloc(&h->amp, sizeof(double) * NP);
  if (e == hipSuccess) e = hipMalloc(&h->fmin, sizeof(double) * batch);
  if (e == hipSuccess) e = hipMalloc(&h->amin, sizeof(long long) * batch);
  if (e == hipSuccess) e = hipMalloc(&h->sums, sizeof(double) * 3 * batch);
  if (e == hipSuccess) e = hipHostMalloc((void**)&h->host_sums, sizeof(double) * 3 * batch);
  if (e == hipSuccess) {
    std::vector<double> w, Z, amp(NP);
    jacobi(relaxed_adjacency(desc->r), NP, w, Z);
    double c = std::ldexp(1.0, -desc->r);  // C(r, j) / 2^r, built up multiplicatively
    for (int j = 0; j <= desc->r; ++j) {
      amp[j] = std::sqrt(c);
      c = c * (double)(desc->r - j) / (double)(j + 1);
    }
    e = hipMemcpy(h->U, Z.data(), sizeof(double) * NP * NP, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(h->lam, w.data(), sizeof(double) * NP, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(h->amp, amp.data(), sizeof(double) * NP, hipMemcpyHostToDevice);
  }
  if (e == hipSuccess) e = hipMemset(h->f, 0, sizeof(double) * pts);
  if (e == hipSuccess) e = rqp_init(h->psi, h->amp, d, NP, h->N, batch, nullptr);
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) {
    st = rfail(e == hipErrorOutOfMemory ? QHD_ENOMEM : QHD_EDEVICE, "relaxed-QP allocation: %s", hipGetErrorString(e));
    release(h);
    return st;
  }
  *out = h;
  return QHD_OK;
}

qhd_status qhd_rqp_set_objective(qhd_rqp h, int32_t i, const double* Q, const double* b) {
  set_error_message("");
  if (!h || !Q || !b) return rfail(QHD_EINVAL, "NULL argument");
  if (i < 0 || i >= h->batch) return rfail(QHD_EINVAL, "instance index %d out of range", i);
  const int d = h->desc.dim;
  std::vector<double> qb((size_t)d * d + d);
  for (int k = 0; k < d; ++k)
    for (int l = 0; l < d; ++l) {
      const double v = 0.5 * (Q[k * d + l] + Q[l * d + k]);
      if (!std::isfinite(v)) return rfail(QHD_EINVAL, "Q[%d][%d] is not finite", k, l);
      qb[(size_t)k * d + l] = v;
    }
  for (int k = 0; k < d; ++k) {
    if (!std::isfinite(b[k])) return rfail(QHD_EINVAL, "b[%d] is not finite", k);
    qb[(size_t)d * d + k] = b[k];
  }
  RQP_TRY(hipSetDevice(h->device));
  double* dst = h->Qb + (size_t)i * qb.size();
  RQP_TRY(hipMemcpy(dst, qb.data(), sizeof(double) * qb.size(), hipMemcpyHostToDevice));
  RQP_TRY(rqp_objective(h->f + (size_t)i * h->N, dst, d, h->NP, h->N, 1, nullptr));
  RQP_TRY(rqp_argmin(h->f + (size_t)i * h->N, h->N, 1, h->fmin + i, h->amin + i, nullptr));
  RQP_TRY(hipMemcpy(&h->fmin_h[i], h->fmin + i, sizeof(double), hipMemcpyDeviceToHost));
  RQP_TRY(hipMemcpy(&h->amin_h[i], h->amin + i, sizeof(long long), hipMemcpyDeviceToHost));
  h->has_obj[i] = 1;
  return QHD_OK;
}

qhd_status qhd_rqp_evolve(qhd_rqp h, int64_t max_steps, void* stream_v) {
  set_error_message("");
  if (!h) return rfail(QHD_EINVAL, "handle is NULL");
  for (int i = 0; i < h->batch; ++i)
    if (!h->has_obj[i]) return rfail(QHD_ESTATE, "instance %d: qhd_rqp_set_objective was not called", i);
  hipStream_t st = (hipStream_t)stream_v;
  RQP_TRY(hipSetDevice(h->device));
  const qhd_rqp_desc& d = h->desc;
  const long long rem = d.nsteps - h->steps_done;
  const long long n = (max_steps < 0 || max_steps > rem) ? rem : max_steps;
  const long long total = h->N * h->batch;
  const int last = (int)h->sets.size() - 1;
  for (long long s0 = 0; s0 < n; s0 += kRqpStepRun - 1) {
    const int run = (int)std::min<long long>(n - s0, kRqpStepRun - 1);
    // entry q of the table: step j0 - 1 + q
    const long long j0 = h->steps_done + s0;
    const bool before = h->pending || s0 > 0;
    step_table(h, j0 - 1, run + 1, before);
    RQP_TRY(rqp_matrices(h->NP, h->U, h->lam, h->steps, run + 1, h->tab, st));
    if (last == 0) {
      // one set holds every axis: the run's steps in one pass
      RQP_TRY(set_pass(h, 0, total, nullptr, h->tab + kRqpMatStride, run, st));
      continue;
    }
    for (int s = 0; s < run; ++s) {
      const double* now = h->tab + (long long)(s + 1) * kRqpMatStride;
      const int from = h->next;
      RQP_TRY(set_pass(h, from, total, s0 + s > 0 ? now - kRqpMatStride : nullptr, now, 1, st));
      const int dir = from == 0 ? 1 : -1;
      for (int k = from + dir; k > 0 && k < last; k += dir) RQP_TRY(set_pass(h, k, total, now, nullptr, 0, st));
      h->next = last - from;
    }
    if (s0 + run == n) RQP_TRY(set_pass(h, h->next, total, h->tab + (long long)run * kRqpMatStride, nullptr, 0, st));
  }
  if (n > 0) {
    h->steps_done += n;
    h->pending = true;
  }
  return QHD_OK;
}

qhd_status qhd_rqp_observe(qhd_rqp h, void* stream_v, qhd_rqp_obs* out, float* marginals_dev, float* prob_dev,
                           float* psi_dev) {
  set_error_message("");
  if (!h || !out) return rfail(QHD_EINVAL, "NULL argument");
  hipStream_t st = (hipStream_t)stream_v;
  RQP_TRY(hipSetDevice(h->device));
  // the owed potential half step is a phase: |phi|^2, and every readout, is unchanged; the
  // state output gets it (exp(-i (dt/2) b_{j-1} f) of the last step j-1, in turns)
  double close_turns = 0.0;
  if (psi_dev && h->pending && h->steps_done > 0) {
    double a, b;
    schedule(h, h->steps_done - 1, a, b);
    close_turns = 0.5 * h->desc.dt * b * 0.15915494309189533577;
  }
  const int d = h->desc.dim, NP = h->NP;
  RQP_TRY(rqp_observe(h->psi, h->f, h->N, h->batch, h->fmin, h->desc.min_tol, h->part, h->sums, prob_dev,
                      reinterpret_cast<float2*>(psi_dev), close_turns, st));
  if (marginals_dev) RQP_TRY(rqp_marginals(NP, h->psi, h->N, d, h->batch, h->part, marginals_dev, st));
  RQP_TRY(hipMemcpyAsync(h->host_sums, h->sums, sizeof(double) * 3 * h->batch, hipMemcpyDeviceToHost, st));
  RQP_TRY(hipStreamSynchronize(st));
  qhd_status status = QHD_OK;
  for (int i = 0; i < h->batch; ++i) {
    const double* s = h->host_sums + 3 * i;
    qhd_rqp_obs& o = out[i];
    o.norm = s[0];
    o.e_f = s[1] / s[0];
    o.p_min = s[2] / s[0];
    o.f_min = h->fmin_h[i];
    o.argmin_index = h->amin_h[i];
    o.steps_done = h->steps_done;
    o.t = (double)h->steps_done * h->desc.dt;
    if (!std::isfinite(o.norm) || !std::isfinite(o.e_f) || !std::isfinite(o.p_min))
      if (status == QHD_OK) status = rfail(QHD_ENUMERIC, "instance %d: non-finite readout", i);
  }
  return status;
}

qhd_status qhd_rqp_reset(qhd_rqp h, void* stream_v) {
  set_error_message("");
  if (!h) return rfail(QHD_EINVAL, "handle is NULL");
  RQP_TRY(hipSetDevice(h->device));
  RQP_TRY(rqp_init(h->psi, h->amp, h->desc.dim, h->NP, h->N, h->batch, (hipStream_t)stream_v));
  h->steps_done = 0;
  h->pending = false;
  h->next = 0;
  return QHD_OK;
}

qhd_status qhd_rqp_points(qhd_rqp h, int64_t* points) {
  set_error_message("");
  if (!h || !points) return rfail(QHD_EINVAL, "NULL argument");
  *points = h->N;
  return QHD_OK;
}

qhd_status qhd_rqp_destroy(qhd_rqp h) {
  set_error_message("");
  if (!h) return QHD_OK;
  (void)hipDeviceSynchronize();
  release(h);
  return QHD_OK;
}

}  // extern "C"
