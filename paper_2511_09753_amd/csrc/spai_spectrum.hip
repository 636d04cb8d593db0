// spai_spectrum.hip — extreme eigenvalues of a symmetric sparse matrix (the lambda_min /
// lambda_max columns the paper reports for its approximate inverses, Tables 4-6, and
// whether an iterate is positive definite, Section 7.1).
//
// Lanczos process with full reorthogonalisation (Lanczos 1950; Paige 1972; Golub and
// Van Loan, Matrix Computations, Section 10.1): v_0 = v0 / ||v0||, and per step
//   w = S v_j;  h = V_j^T w, w -= V_j h;  h' = V_j^T w, w -= V_j h'  (Gram-Schmidt twice)
//   alpha_j = h_j + h'_j,  beta_j = ||w||,  v_{j+1} = w / beta_j,
// stopping early once beta_j <= 1e-12 max_{i<=j} (|alpha_i| + beta_i) (an invariant
// subspace).  The Ritz values are the eigenvalues of the tridiagonal T_k =
// tridiag(beta, alpha, beta); its extreme ones are found by bisection on Sturm counts,
// and beta_k |y_k| (y the unit eigenvector of T_k, by inverse iteration) bounds the
// distance from each to an eigenvalue of S.  Ritz values are Rayleigh quotients, so
// lambda_min(S) <= theta_min and theta_max <= lambda_max(S).
//
// Device work: a workgroup owns a block of rows and takes it 256 rows at a time; each
// launch forms w for its rows (S v, or w - V h) and, from the same w in LDS, the partial
// products with every basis vector.  Partials are summed in a fixed order (deterministic).
// alpha, beta and the stopping test stay on the device; the host looks after 1, 4, 16 and 64 steps
// and then every 64.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "spai.h"
#include "spai_host.hpp"

namespace spai {

namespace {

constexpr int kThreads = 256;
constexpr int kLzThreads = 1024;
constexpr int kLzRows = 256;        // rows of w in LDS at a time
constexpr int kLzBlocks = 256;      // at most: one workgroup per compute unit
constexpr int kMaxSteps = 2048;

struct LzState {
  double scale;                     // max_i (|alpha_i| + beta_i)
  int steps, stop;                  // steps taken; 1: invariant subspace or a non-finite step
};

// One pass over the rows of a workgroup.  kLzMult: w = S v_{k-1}; kLzSub, kLzNorm: w -= V h
// (k basis vectors).  Then part[t * gridDim.x + block] = sum over its rows of V[i, t] w[i]
// (kLzNorm: part[block] = sum of w[i]^2).
// Bound by reading the basis (8 n k bytes) and, where that is small, by latency: a row's sum
// takes four threads (entries, or basis vectors, in strides of four), so that a tile of 256
// rows keeps 1024 threads loading; a wave then owns every sixteenth group of four basis
// vectors and reads their 256 rows as 16 coalesced loads against w in registers.  Forming w
// and the products in one launch saves a pass over w.  At n = 262,144 (14 entries per row,
// 100 steps, 50 vectors on average) kLzMult takes 46 us where a thread per row (its entries
// read 14 apart, one dependent load after another) and a launch for the products took 146;
// kLzSub 33 against 38, kLzNorm 22 against 25, and the serial sums of the partials 4.6
// against 15: 115 us a step against 330.  One workgroup of 16 waves per compute unit: capping
// the registers at 64 for two spilled and took 1.5 times as long.
enum { kLzMult = 0, kLzSub = 1, kLzNorm = 2 };
template <int MODE>
__global__ __launch_bounds__(kLzThreads) void k_lz_pass(PcgMat S, const double* __restrict__ V,
                                                        int64_t ldv, int k, int64_t n,
                                                        int64_t per,
                                                        const double* __restrict__ h,
                                                        double* __restrict__ w,
                                                        double* __restrict__ part,
                                                        const LzState* st) {
  if (st->stop) return;
  __shared__ double s_w[kLzRows];
  __shared__ double s_red[kLzThreads];
  __shared__ double s_acc[MODE == kLzNorm ? 1 : kMaxSteps + 1];
  constexpr int kWaves = kLzThreads / 64;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int64_t lo = (int64_t)blockIdx.x * per, hi = lo + per < n ? lo + per : n;
  double nrm = 0.0;
  if constexpr (MODE != kLzNorm)
    for (int t = tid; t < k; t += kLzThreads) s_acc[t] = 0.0;
  for (int64_t base = lo; base < hi; base += kLzRows) {
    if constexpr (MODE == kLzMult) {
      const int64_t i = base + (tid >> 2);
      const int l = tid & 3;
      const double* __restrict__ x = V + (int64_t)(k - 1) * ldv;
      double acc = 0.0;
      if (i < hi) {
        const int64_t e = S.row_end(i);
        for (int64_t q0 = S.row_begin(i) + l; q0 < e; q0 += 16) {
          int c[4];
          double v[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int64_t q = q0 + 4 * u;
            c[u] = -1;
            v[u] = 0.0;
            if (q < e) {
              c[u] = S.col[q];
              v[u] = S.v(q);
            }
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (c[u] >= 0) acc += v[u] * x[c[u]];
        }
      }
      acc += __shfl_xor(acc, 1, 64);
      acc += __shfl_xor(acc, 2, 64);
      if (l == 0) {
        s_w[tid >> 2] = acc;                       // 0 past the last row
        if (i < hi) w[i] = acc;
      }
    } else {
      const int r = tid & (kLzRows - 1), g = tid / kLzRows;
      const int64_t i = base + r;
      const int64_t ic = i < hi ? i : hi - 1;
      const double* __restrict__ v = V + ic;
      double acc = 0.0;
      int t = g;
      for (; t + 28 < k; t += 32) {                // eight loads in flight
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = v[(int64_t)(t + 4 * u) * ldv];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += x[u] * h[t + 4 * u];
      }
      for (; t < k; t += 4) acc += v[(int64_t)t * ldv] * h[t];
      s_red[tid] = acc;
      __syncthreads();
      if (g == 0) {
        const double sub = (s_red[r] + s_red[kLzRows + r]) +
                           (s_red[2 * kLzRows + r] + s_red[3 * kLzRows + r]);
        const double x = i < hi ? w[i] - sub : 0.0;
        if (i < hi) w[i] = x;
        if constexpr (MODE == kLzNorm) nrm += x * x;
        else s_w[r] = x;
      }
    }
    __syncthreads();
    if constexpr (MODE != kLzNorm) {
      // four basis vectors per wave at a time, 16 loads in flight; their four sums over
      // the wave in one transposed tree (7 exchanges instead of 24), vector t in lane 16 t
      double x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = s_w[lane + 64 * u];
      const double* __restrict__ vb = V + base + lane;
      for (int t0 = 4 * wv; t0 < k; t0 += 4 * kWaves) {
        double a[4];
        if (base + kLzRows <= hi && t0 + 4 <= k) {
          double v[4][4];
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int u = 0; u < 4; ++u) v[t][u] = vb[(int64_t)(t0 + t) * ldv + 64 * u];
#pragma unroll
          for (int t = 0; t < 4; ++t)
            a[t] = (v[t][0] * x[0] + v[t][1] * x[1]) + (v[t][2] * x[2] + v[t][3] * x[3]);
        } else {                                   // the last rows, the last vectors
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            double v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
              v[u] = t0 + t < k && base + lane + 64 * u < hi ? vb[(int64_t)(t0 + t) * ldv + 64 * u]
                                                             : 0.0;
            a[t] = (v[0] * x[0] + v[1] * x[1]) + (v[2] * x[2] + v[3] * x[3]);
          }
        }
        const bool up = lane >= 32, up16 = (lane & 16) != 0;
        const double b0 = (up ? a[2] : a[0]) + __shfl_xor(up ? a[0] : a[2], 32, 64);
        const double b1 = (up ? a[3] : a[1]) + __shfl_xor(up ? a[1] : a[3], 32, 64);
        double c = (up16 ? b1 : b0) + __shfl_xor(up16 ? b0 : b1, 16, 64);
#pragma unroll
        for (int d = 8; d >= 1; d >>= 1) c += __shfl_xor(c, d, 64);
        const int t = t0 + (lane >> 4);
        if ((lane & 15) == 0 && t < k) s_acc[t] += c;   // a basis vector belongs to one wave
      }
      __syncthreads();
    }
  }
  if constexpr (MODE == kLzNorm) {
    s_red[tid] = nrm;
    __syncthreads();
    for (int d = kLzThreads / 2; d >= 1; d >>= 1) {
      if (tid < d) s_red[tid] += s_red[tid + d];
      __syncthreads();
    }
    if (tid == 0) part[blockIdx.x] = s_red[0];
  } else {
    __syncthreads();
    for (int t = tid; t < k; t += kLzThreads) part[(int64_t)t * gridDim.x + blockIdx.x] = s_acc[t];
  }
}

// sum of p[0 .. m) over one wave in a fixed order, on every lane
__device__ __forceinline__ double lz_sum(const double* __restrict__ p, int m) {
  double a = 0.0;
#pragma unroll 4
  for (int c = threadIdx.x & 63; c < m; c += 64) a += p[c];
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) a += __shfl_xor(a, d, 64);
  return a;
}

// h[t] = sum_c part[t * m + c], one wave per basis vector
__global__ __launch_bounds__(kThreads) void k_lz_sum(const double* __restrict__ part, int k, int m,
                                                     double* __restrict__ h) {
  const int t = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  if (t >= k) return;
  const double a = lz_sum(part + (int64_t)t * m, m);
  if ((threadIdx.x & 63) == 0) h[t] = a;
}

// the end of step j: beta_j from the partials of ||w||^2 (every workgroup sums them, in one
// order), v_{j+1} = w / beta_j where a step follows (next), and on workgroup 0 alpha_j and
// the stopping test
__global__ __launch_bounds__(kThreads) void k_lz_next(const double* __restrict__ w, int64_t n,
                                                      const double* __restrict__ part, int m,
                                                      const double* __restrict__ h1,
                                                      const double* __restrict__ h2, int j,
                                                      double* __restrict__ next,
                                                      double* __restrict__ alpha,
                                                      double* __restrict__ beta, LzState* st) {
  if (st->stop) return;                            // a workgroup that sees this step's own
                                                   // stop leaves v_{j+1}, which nobody reads
  const double nb = lz_sum(part, m);
  const double b = sqrt(nb > 0.0 ? nb : nb == nb ? 0.0 : nb);
  if (next)
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads)
      next[i] = w[i] / b;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    const double a = h1[j] + h2[j];
    alpha[j] = a;
    beta[j] = b;
    const double sc = fmax(st->scale, fabs(a) + b);
    st->scale = sc;
    st->steps = j + 1;
    if (!isfinite(a) || !isfinite(b) || b <= 1e-12 * sc) st->stop = 1;
  }
}

__global__ void k_lz_div(const double* __restrict__ w, double b, int64_t n,
                         double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = w[i] / b;
}

__global__ void k_lz_start(LzState* st) {
  st->scale = 0.0;
  st->steps = 0;
  st->stop = 0;
}

// ---- host: the tridiagonal T_k

// number of eigenvalues of T below x (signs of the LDL^T pivots of T - x I)
int sturm_below(const std::vector<double>& a, const std::vector<double>& b, double x) {
  int cnt = 0;
  double d = 1.0;
  const double tiny = 1e-300;
  for (size_t i = 0; i < a.size(); ++i) {
    d = (a[i] - x) - (i ? (b[i - 1] * b[i - 1]) / d : 0.0);
    if (d == 0.0) d = -tiny;
    if (d < 0.0) ++cnt;
  }
  return cnt;
}

// the r-th smallest eigenvalue of T (r = 1..k) by bisection inside the Gershgorin interval
double tri_eig(const std::vector<double>& a, const std::vector<double>& b, int r) {
  const size_t k = a.size();
  double lo = a[0], hi = a[0];
  for (size_t i = 0; i < k; ++i) {
    const double rad = (i ? std::fabs(b[i - 1]) : 0.0) + (i + 1 < k ? std::fabs(b[i]) : 0.0);
    lo = std::min(lo, a[i] - rad);
    hi = std::max(hi, a[i] + rad);
  }
  for (int it = 0; it < 400; ++it) {
    const double mid = 0.5 * (lo + hi);
    if (mid <= lo || mid >= hi) break;
    if (sturm_below(a, b, mid) >= r) hi = mid; else lo = mid;
  }
  return 0.5 * (lo + hi);
}

// last component of the unit eigenvector of T for the eigenvalue theta (inverse iteration
// with a tridiagonal LU with partial pivoting)
double tri_last_component(const std::vector<double>& a, const std::vector<double>& b,
                          double theta, double scale) {
  const size_t k = a.size();
  if (k == 1) return 1.0;
  const double shift = theta + 1e-14 * scale;
  std::vector<double> y(k, 1.0), dl(k), d(k), du(k), du2(k), rhs(k);
  std::vector<char> swapped(k, 0);
  for (int pass = 0; pass < 3; ++pass) {
    for (size_t i = 0; i < k; ++i) {
      d[i] = a[i] - shift;
      du[i] = i + 1 < k ? b[i] : 0.0;
      dl[i] = i + 1 < k ? b[i] : 0.0;   // subdiagonal entry below row i
      du2[i] = 0.0;
      swapped[i] = 0;
      rhs[i] = y[i];
    }
    // elimination down the rows
    for (size_t i = 0; i + 1 < k; ++i) {
      if (std::fabs(d[i]) >= std::fabs(dl[i])) {
        const double piv = d[i] != 0.0 ? d[i] : 1e-300;
        const double m = dl[i] / piv;
        d[i] = piv;
        d[i + 1] -= m * du[i];
        rhs[i + 1] -= m * rhs[i];
        dl[i] = m;
      } else {                          // swap rows i and i + 1
        const double m = d[i] / dl[i];
        d[i] = dl[i];
        const double t = d[i + 1];
        d[i + 1] = du[i] - m * t;
        du2[i] = i + 2 < k ? du[i + 1] : 0.0;
        if (i + 2 < k) du[i + 1] = -m * du2[i];
        du[i] = t;
        std::swap(rhs[i], rhs[i + 1]);
        rhs[i + 1] -= m * rhs[i];
        dl[i] = m;
        swapped[i] = 1;
      }
    }
    if (d[k - 1] == 0.0) d[k - 1] = 1e-300;
    // back substitution
    y[k - 1] = rhs[k - 1] / d[k - 1];
    if (k >= 2) y[k - 2] = (rhs[k - 2] - du[k - 2] * y[k - 1]) / d[k - 2];
    for (size_t ii = k - 2; ii-- > 0;) y[ii] = (rhs[ii] - du[ii] * y[ii + 1] - du2[ii] * y[ii + 2]) / d[ii];
    double nrm = 0.0;
    for (double v : y) nrm = std::max(nrm, std::fabs(v));
    if (!(nrm > 0.0) || !std::isfinite(nrm)) return 1.0;
    for (double& v : y) v /= nrm;
  }
  double s2 = 0.0;
  for (double v : y) s2 += v * v;
  return y[k - 1] / std::sqrt(s2);
}

}  // namespace

int lanczos_run(const PcgMat& S, int steps, const double* dv0, double* out, int* steps_done,
                int64_t pool_limit, hipStream_t s) {
  const int64_t n = S.n;
  if (steps < 1 || steps > kMaxSteps) return fail(SPAI_ERR_ARG, "spectrum: steps outside 1..2048");
  if (!out) return fail(SPAI_ERR_ARG, "spectrum: null output");
  const int K = (int)std::min<int64_t>(steps, n);
  const int64_t ldv = n;
  DevPool pool;
  pool.limit = pool_limit;
  int rc;
  // rows per workgroup and workgroups
  const int64_t per = std::max<int64_t>(kLzRows, ((n + kLzBlocks - 1) / kLzBlocks + 63) / 64 * 64);
  const int nb = (int)((n + per - 1) / per);
  double *V, *w, *part, *h1, *h2, *ab;
  LzState* st;
  if ((rc = pool.alloc(&V, n * (int64_t)(K + 1))) || (rc = pool.alloc(&w, n)) ||
      (rc = pool.alloc(&part, (int64_t)nb * (K + 1))) || (rc = pool.alloc(&h1, K + 1)) ||
      (rc = pool.alloc(&h2, K + 1)))
    return rc;
  // alpha, beta and the state: in the basis's last column, which no step writes
  static_assert(sizeof(LzState) == 2 * sizeof(double), "the state takes two doubles");
  ab = V + n * (int64_t)K;
  if (n < 2 * (int64_t)K + 2 && (rc = pool.alloc(&ab, 2 * (int64_t)K + 2))) return rc;
  st = (LzState*)ab;
  double *d_alpha = ab + 2, *d_beta = d_alpha + K;
  const dim3 rows((unsigned)((n + kThreads - 1) / kThreads)), bs(kThreads), lb(kLzThreads);
  auto sum = [&](int k, double* h) {
    hipLaunchKernelGGL(k_lz_sum, dim3((k + kThreads / 64 - 1) / (kThreads / 64)), bs, 0, s, part, k,
                       nb, h);
  };
  hipLaunchKernelGGL(k_lz_start, dim3(1), dim3(1), 0, s, st);
  // v_0 = v0 / ||v0||
  double nrm2 = 0.0;
  HIPCHK(hipMemcpyAsync(w, dv0, sizeof(double) * n, hipMemcpyDeviceToDevice, s));
  hipLaunchKernelGGL(k_lz_pass<kLzNorm>, dim3(nb), lb, 0, s, S, V, ldv, 0, n, per, h1, w, part, st);
  sum(1, h1);
  HIPCHK(hipMemcpyAsync(&nrm2, h1, sizeof(double), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  if (!(nrm2 > 0.0) || !std::isfinite(nrm2))
    return fail(SPAI_ERR_ARG, "spectrum: start vector zero or not finite");
  hipLaunchKernelGGL(k_lz_div, rows, bs, 0, s, w, std::sqrt(nrm2), n, V);
  LzState hst{};
  for (int j = 0; j < K; ++j) {
    const int k = j + 1;
    hipLaunchKernelGGL(k_lz_pass<kLzMult>, dim3(nb), lb, 0, s, S, V, ldv, k, n, per, h1, w, part, st);
    sum(k, h1);
    hipLaunchKernelGGL(k_lz_pass<kLzSub>, dim3(nb), lb, 0, s, S, V, ldv, k, n, per, h1, w, part, st);
    sum(k, h2);
    hipLaunchKernelGGL(k_lz_pass<kLzNorm>, dim3(nb), lb, 0, s, S, V, ldv, k, n, per, h2, w, part, st);
    hipLaunchKernelGGL(k_lz_next, dim3(std::min<unsigned>(rows.x, 1024)), bs, 0, s, w, n, part, nb,
                       h1, h2, j, k < K ? V + (int64_t)k * ldv : nullptr, d_alpha, d_beta, st);
    HIPCHK(hipGetLastError());
    // an invariant subspace ends the process early: the host looks after 1, 4, 16 and 64 steps
    // and every 64, so that at most three times the steps taken run masked (15 us each, where
    // a look every step took 85 us a step at n = 600).  Looking every 64 alone, a process of one
    // step took 1.2 ms and one of three 1.2, 0.22 and 0.30 so; a look leaves the device idle for
    // some 25 us of the 11.4 ms that 100 steps take at n = 262,144
    if (k == K || k % 64 == 0 || k == 1 || k == 4 || k == 16) {
      HIPCHK(hipMemcpyAsync(&hst, st, sizeof(LzState), hipMemcpyDeviceToHost, s));
      HIPCHK(hipStreamSynchronize(s));
      if (hst.stop) break;
    }
  }
  std::vector<double> alpha((size_t)hst.steps), beta((size_t)hst.steps);
  HIPCHK(hipMemcpyAsync(alpha.data(), d_alpha, sizeof(double) * hst.steps, hipMemcpyDeviceToHost, s));
  HIPCHK(hipMemcpyAsync(beta.data(), d_beta, sizeof(double) * hst.steps, hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  const double scale = hst.scale;
  const int done = hst.steps;
  for (int j = 0; j < done; ++j)
    if (!std::isfinite(alpha[j]) || !std::isfinite(beta[j]))
      return fail(SPAI_ERR_NONFINITE, "spectrum: non-finite step");
  const int k = done;
  std::vector<double> a(alpha.begin(), alpha.begin() + k), b(beta.begin(), beta.begin() + k);
  const double bl = b[k - 1];
  b.resize(k - 1 > 0 ? k - 1 : 0);
  const double tmin = tri_eig(a, b, 1), tmax = tri_eig(a, b, k);
  out[0] = tmin;
  out[1] = tmax;
  out[2] = bl * std::fabs(tri_last_component(a, b, tmin, scale));
  out[3] = bl * std::fabs(tri_last_component(a, b, tmax, scale));
  if (steps_done) *steps_done = k;
  return SPAI_OK;
}

}  // namespace spai

using namespace spai;

extern "C" int spai_csr_spectrum(const spai_csr_t* S, int steps, const double* v0, double* out,
                                 int* steps_done, const spai_opts_t* opts) {
  try {
    if (!S || !v0 || !out) return fail(SPAI_ERR_ARG, "spai_csr_spectrum: null argument");
    int rc;
    HostCsr h;
    if ((rc = fetch_csr(S, h))) return rc;
    for (int64_t i = 0; i < h.n; ++i)
      for (int64_t q = h.rowptr[i]; q < h.rowptr[i + 1]; ++q) {
        const int64_t t = find_entry(h, h.col[q], (int32_t)i);
        if (t < 0 || h.val[t] != h.val[q])
          return fail(SPAI_ERR_NOT_SYMMETRIC, "spai_csr_spectrum: matrix not symmetric");
      }
    spai_opts_t o;
    spai_default_opts(&o);
    if (opts) o = *opts;
    hipStream_t s = (hipStream_t)o.stream;
    DevPool pool;
    pool.limit = o.device_pool_limit;
    int64_t* rp;
    int32_t* ci;
    double* va;
    double* dv0;
    if ((rc = pool.alloc(&rp, h.n + 1)) || (rc = pool.alloc(&ci, h.nnz)) ||
        (rc = pool.alloc(&va, h.nnz)) || (rc = pool.alloc(&dv0, h.n)))
      return rc;
    HIPCHK(hipMemcpyAsync(rp, h.rowptr.data(), sizeof(int64_t) * (h.n + 1), hipMemcpyHostToDevice, s));
    if (h.nnz) {
      HIPCHK(hipMemcpyAsync(ci, h.col.data(), sizeof(int32_t) * h.nnz, hipMemcpyHostToDevice, s));
      HIPCHK(hipMemcpyAsync(va, h.val.data(), sizeof(double) * h.nnz, hipMemcpyHostToDevice, s));
    }
    HIPCHK(hipMemcpyAsync(dv0, v0, sizeof(double) * h.n,
                          S->on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, s));
    PcgMat m;
    m.n = h.n;
    m.rowptr = rp;
    m.col = ci;
    m.val = va;
    const int64_t rest = o.device_pool_limit > 0
                             ? std::max<int64_t>(1, o.device_pool_limit - (int64_t)pool.used)
                             : 0;
    return lanczos_run(m, steps, dv0, out, steps_done, rest, s);
  } catch (const std::bad_alloc&) {
    return fail(SPAI_ERR_NOMEM, "host allocation failed");
  } catch (...) {
    return fail(SPAI_ERR_HIP, "unexpected exception");
  }
}
