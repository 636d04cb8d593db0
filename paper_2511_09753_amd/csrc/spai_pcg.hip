// spai_pcg.hip — preconditioned CG with the SPAI as preconditioner (z = M r), many
// right-hand sides at once (the vector solves of Section 7, Experiments 04 and 06).
//
// Every right-hand side runs its own textbook recurrence in float64; the block of
// vectors is row-major (n x nrhs, the nrhs values of a row contiguous), so one
// wavefront reads the 64 values of a row of X as one coalesced 512-byte line and the
// SpMM gathers whole rows (with at most 32 right-hand sides, pow2(nrhs) lanes share a
// row instead).  Frobenius-free per-RHS dots are reduced per workgroup in
// a fixed order and then across workgroups in a fixed order (deterministic).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "spai.h"
#include "spai_dev.hpp"
#include "spai_host.hpp"

namespace spai {
namespace {

constexpr int kThreads = 256;
constexpr int kGrid = 2048;

using Mat = PcgMat;
typedef double d2v __attribute__((ext_vector_type(2)));   // for nontemporal 16-byte stores

__device__ __forceinline__ double readlane_f64(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// a wave-uniform 64-bit value moved to scalar registers
__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const int lo = __builtin_amdgcn_readfirstlane((int)(v & 0xffffffffll));
  const int hi = __builtin_amdgcn_readfirstlane((int)(v >> 32));
  return ((int64_t)hi << 32) | (int64_t)(unsigned)lo;
}

enum { kLayEll = 0, kLayPad = 1, kLayCsr = 2 };

template <int LAY>
__device__ __forceinline__ int64_t row_lo(const Mat& A, int64_t i) {
  if (LAY == kLayEll) return i << A.eshift;
  if (LAY == kLayPad) return A.beg[i];
  return A.rowptr[i];
}
template <int LAY>
__device__ __forceinline__ int64_t row_hi(const Mat& A, int64_t i) {
  if (LAY == kLayEll) return (i + 1) << A.eshift;
  if (LAY == kLayPad) return A.beg[i] + A.len[i];
  return A.rowptr[i + 1];
}
template <typename VT>
__device__ __forceinline__ VT entry_val(const Mat& A, int64_t q) {
  if constexpr (sizeof(VT) == 4) return A.val32[q];
  else return A.val[q];
}
__device__ __forceinline__ float readlane_val(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double readlane_val(double v, int l) { return readlane_f64(v, l); }

// G gathers of one row, all issued before any is used: entry e0 + k of the row (held
// one per lane in cc) selects row col of X, whose 64-value piece starting at column c0
// is one 512-byte line; lane k's value sits at byte offset loff.  Entries past cnt
// repeat the last one, so every load is in bounds and there is no branch between them.
template <int G>
__device__ __forceinline__ void gather_row(const double* X, int nrhs, int c0, unsigned loff,
                                           int cc, int e0, int cnt, double (&xs)[G]) {
#pragma unroll
  for (int k = 0; k < G; ++k) {
    const int e = min(e0 + k, cnt - 1);
    const int col = __builtin_amdgcn_readlane(cc, e);
    const char* xrow = (const char*)(X + ((int64_t)col * nrhs + c0));   // uniform base
    xs[k] = *(const double*)(xrow + loff);
  }
}

// y += v_e x_e over the entries e0 .. min(e0 + G, cnt) in order (v_e widened to float64);
// the gathered value of the entry in column `diag` (the row's own index) is kept in xd
template <int G, typename VT>
__device__ __forceinline__ void accumulate_row(double& y, VT cv, int cc, int e0, int cnt,
                                               const double (&xs)[G], int diag, double& xd,
                                               bool& found) {
#pragma unroll
  for (int k = 0; k < G; ++k)
    if (e0 + k < cnt) {
      y += (double)readlane_val(cv, e0 + k) * xs[k];
      if (__builtin_amdgcn_readlane(cc, e0 + k) == diag) {
        xd = xs[k];
        found = true;
      }
    }
}

// Y[:, c0:c0+64) = K X[:, c0:c0+64) and, when dot is set, per-block partials of
// sum_i X[i, r] Y[i, r] (X[i, :] taken from the row's own diagonal gather), stored
// transposed: part[r * gridDim.x + block].
// One wave per row at a time, lane r owning right-hand side c0 + r, so every gather is
// one 512-byte line of X.  The row's entries are loaded by the lanes together (one per
// lane) and broadcast with readlane, so the row's gathers (up to 16 in flight) wait on
// a single entry load; the next row's entries and the descriptor of the row after it
// are loaded while the current row's gathers are in flight.  Row i's sum runs over its
// entries in stored (ascending column) order.  The rows are split into eight
// contiguous ranges, one per XCD (workgroups are dealt round-robin over the XCDs), and
// each wave takes kRowsPerWave consecutive positions of its range.  The launch is not
// persistent: workgroups are dispatched in order as others finish, so the positions in
// flight stay within a few thousand of each other and the rows of X they gather stay in
// the XCD's L2 (a persistent grid whose waves walk the range with a fixed stride drifts
// apart and gathers rows again from beyond L2).
constexpr int kRowsPerWave = 16;

template <typename VT, int LAY>
__global__ __launch_bounds__(kThreads) void k_spmm_wave(Mat A, const double* X, double* Y,
                                                        int dot, int nrhs, int c0,
                                                        const int32_t* order, double* part) {
  if (A.gate && *A.gate == 0) return;                     // every right-hand side stopped
  if (A.ran && c0 == 0 && blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(A.ran, 1);
  __shared__ double sh[kThreads];
  constexpr int WPB = kThreads / 64;
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int64_t xcd = blockIdx.x & 7, kb = blockIdx.x >> 3, nb = gridDim.x >> 3;
  const int64_t per = (A.n + 7) / 8;
  const int64_t r0 = xcd * per;
  const int64_t r1 = r0 + per < A.n ? r0 + per : A.n;
  (void)nb;
  const int64_t stride = 1;
  const bool on = c0 + lane < nrhs;
  const int64_t cofs = c0 + lane;
  const unsigned loff = on ? (unsigned)lane * 8u : 0u;   // idle lanes re-read column c0
  auto rowof = [&](int64_t k) -> int64_t { return order ? (int64_t)order[k] : k; };
  double acc = 0.0;
  int64_t k = r0 + (kb * WPB + wv) * kRowsPerWave;
  const int64_t kend = k + kRowsPerWave < r1 ? k + kRowsPerWave : r1;
  // position k: row i, its descriptor (a, b) and first 64 entries (ec, ev), one per lane;
  // position k + stride: row ni and descriptor (na, nbe); position k + 2 stride: row mi
  int64_t i = 0, ni = 0, mi = 0, a = 0, b = 0, na = 0, nbe = 0;
  int ec = -1;
  VT ev = 0;
  if (k < kend) {
    i = rowof(k);
    a = row_lo<LAY>(A, i);
    b = row_hi<LAY>(A, i);
    if (a + lane < b) {
      ec = A.col[a + lane];
      ev = entry_val<VT>(A, a + lane);
    }
  }
  if (k + stride < kend) {
    ni = rowof(k + stride);
    na = row_lo<LAY>(A, ni);
    nbe = row_hi<LAY>(A, ni);
  }
  if (k + 2 * stride < kend) mi = rowof(k + 2 * stride);
  for (; k < kend; k += stride) {
    const int64_t kn = k + stride;
    const int cnt = __popcll(__ballot(ec >= 0));   // ELL padding (column -1) sits last
    int nc = -1;
    VT nv = 0;
    int64_t ma = 0, mb = 0, li = 0;
    auto prefetch = [&]() {
      if (kn < kend && na + lane < nbe) {
        nc = A.col[na + lane];
        nv = entry_val<VT>(A, na + lane);
      }
      if (kn + stride < kend) {
        ma = row_lo<LAY>(A, mi);
        mb = row_hi<LAY>(A, mi);
      }
      if (kn + 2 * stride < kend) li = rowof(kn + 2 * stride);
    };
    // X[i, :] for the dot: the row's own (diagonal) gather
    const int diag = dot ? (int)i : -1;
    double xd = 0.0;
    bool found = false;
    double y = 0.0;
    if (cnt == 0) {
      prefetch();
    } else if (cnt <= 8) {
      double xs[8];
      gather_row<8>(X, nrhs, c0, loff, ec, 0, cnt, xs);
      prefetch();
      accumulate_row<8>(y, ev, ec, 0, cnt, xs, diag, xd, found);
    } else {
      double xs[16];
      gather_row<16>(X, nrhs, c0, loff, ec, 0, cnt, xs);
      prefetch();
      accumulate_row<16>(y, ev, ec, 0, cnt, xs, diag, xd, found);
      for (int e0 = 16; e0 < cnt; e0 += 16) {
        gather_row<16>(X, nrhs, c0, loff, ec, e0, cnt, xs);
        accumulate_row<16>(y, ev, ec, e0, cnt, xs, diag, xd, found);
      }
      for (int64_t q = a + 64; q < b; q += 64) {   // rows longer than 64 entries
        int cc = -1;
        VT cv = 0;
        if (q + lane < b) {
          cc = A.col[q + lane];
          cv = entry_val<VT>(A, q + lane);
        }
        const int cn = __popcll(__ballot(cc >= 0));
        if (cn == 0) break;
        for (int e0 = 0; e0 < cn; e0 += 16) {
          gather_row<16>(X, nrhs, c0, loff, cc, e0, cn, xs);
          accumulate_row<16>(y, cv, cc, e0, cn, xs, diag, xd, found);
        }
      }
    }
    if (on) {
      Y[i * nrhs + cofs] = y;
      if (dot) {
        // a row without a diagonal entry loads X[i, :] after all
        const double wv = found ? xd : X[i * nrhs + cofs];
        acc += wv * y;
      }
    }
    ec = nc;
    ev = nv;
    a = na;
    b = nbe;
    na = ma;
    nbe = mb;
    i = ni;
    ni = mi;
    mi = li;
  }
  if (!part) return;
  sh[threadIdx.x] = acc;
  __syncthreads();
  if (threadIdx.x < 64 && c0 + (int)threadIdx.x < nrhs) {
    double sum = 0.0;
    for (int w = 0; w < WPB; ++w) sum += sh[w * 64 + threadIdx.x];
    part[(int64_t)(c0 + threadIdx.x) * gridDim.x + blockIdx.x] = sum;
  }
}

// The product for an even number of right-hand sides: two rows per wave at a time,
// lanes 0-31 the row at one position and lanes 32-63 the row at the next, lane l of a
// half owning right-hand sides c0 + 2 (l mod 32) and the one after, so every gather is
// one 16-byte load per lane and one load instruction serves two rows (half the
// address-unit work of k_spmm_wave per row).  A half's row entries are loaded 32 at a
// time (one per lane of the half) and broadcast with readlane; the gathers of both
// rows are issued in groups of four before any is used (groups of eight hold 100
// registers, five waves per SIMD, and the 64-right-hand-side solve at 96^3 took 6%
// longer than with four at six waves) -- of two for A in ELL, whose short rows do best
// with more, smaller groups (350 against 353 ms per solve) --, entries past a row's count
// repeating its last one so every load is in bounds.  Each row's sum runs over its
// entries in stored order, and the dot terms are added in position order, so the rows
// of Y and the dot partials are those of k_spmm_wave bit for bit.  Positions are
// dealt as in k_spmm_wave (eight XCD ranges, kRowsPerWave consecutive positions per
// wave, a non-persistent launch).
template <typename VT, int LAY>
__global__ __launch_bounds__(kThreads) void k_spmm_pair(Mat A, const double* X, double* Y,
                                                        int dot, int nrhs, int c0,
                                                        const int32_t* order, double* part) {
  if (A.gate && *A.gate == 0) return;                     // every right-hand side stopped
  if (A.ran && c0 == 0 && blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(A.ran, 1);
  constexpr int G = LAY == kLayEll ? 2 : 4;
  __shared__ double sh[kThreads];
  constexpr int WPB = kThreads / 64;
  const int lane = threadIdx.x & 63;
  const int half = lane >> 5;
  const int hl = lane & 31;
  const int wv = threadIdx.x >> 6;
  const int64_t xcd = blockIdx.x & 7, kb = blockIdx.x >> 3;
  const int64_t per = (A.n + 7) / 8;
  const int64_t r0 = xcd * per;
  const int64_t r1 = r0 + per < A.n ? r0 + per : A.n;
  const bool on = c0 + 2 * hl < nrhs;
  const unsigned loff = on ? (unsigned)hl * 16u : 0u;   // idle lanes re-read column c0
  auto rowof = [&](int64_t k) -> int64_t { return order ? (int64_t)order[k] : k; };
  double acc0 = 0.0, acc1 = 0.0;
  const int64_t kbeg = r0 + (kb * WPB + wv) * kRowsPerWave;
  const int64_t kend = kbeg + kRowsPerWave < r1 ? kbeg + kRowsPerWave : r1;
  // this half's position k + half: row i, descriptor [a, b), first 32 entries (ec, ev)
  auto load_pos = [&](int64_t p, int64_t& i, int64_t& a, int64_t& b) {
    i = -1;
    a = 0;
    b = 0;
    if (p < kend) {
      i = rowof(p);
      a = row_lo<LAY>(A, i);
      b = row_hi<LAY>(A, i);
    }
  };
  auto load_ent = [&](int64_t a, int64_t b, int& cc, VT& cv) {
    cc = -1;
    cv = 0;
    if (a + hl < b) {
      cc = A.col[a + hl];
      cv = entry_val<VT>(A, a + hl);
    }
  };
  int64_t i, a, b, ni, na, nb;
  int ec, nec = -1;
  VT ev, nev = 0;
  load_pos(kbeg + half, i, a, b);
  load_ent(a, b, ec, ev);
  load_pos(kbeg + 2 + half, ni, na, nb);
  for (int64_t k = kbeg; k < kend; k += 2) {
    const bool has = i >= 0;
    double y0 = 0.0, y1 = 0.0;
    double2 xd = make_double2(0.0, 0.0);
    bool found = false;
    int64_t q0 = 0;                     // entries a + q0 .. a + q0 + 31 are in (ec, ev)
    bool first = true;
    for (;;) {
      const unsigned long long bal = __ballot(ec >= 0);   // ELL padding (column -1) last
      const int cA = __popcll(bal & 0xffffffffull), cB = __popcll(bal >> 32);
      const int cmax = cA > cB ? cA : cB;
      if (first) {                      // the next pair's entries while these are gathered
        load_ent(na, nb, nec, nev);
        first = false;
      }
      if (cmax == 0) break;
      const int cmine = half ? cB : cA;
      for (int e0 = 0; e0 < cmax; e0 += G) {
        double2 xs[G];
        int cs[G];
#pragma unroll
        for (int t = 0; t < G; ++t) {
          const int e = e0 + t;
          const int eA = cA ? min(e, cA - 1) : 0, eB = cB ? min(e, cB - 1) : 0;
          const int colA = __builtin_amdgcn_readlane(ec, eA);
          const int colB = __builtin_amdgcn_readlane(ec, 32 + eB);
          int col = half ? colB : colA;
          cs[t] = col;
          col = col < 0 ? 0 : col;
          const char* xrow = (const char*)(X + ((int64_t)col * nrhs + c0));
          xs[t] = *(const double2*)(xrow + loff);
        }
#pragma unroll
        for (int t = 0; t < G; ++t) {
          const int e = e0 + t;
          const VT vA = readlane_val(ev, e < 32 ? e : 31);
          const VT vB = readlane_val(ev, 32 + (e < 32 ? e : 31));
          if (e < cmine) {
            const double v = (double)(half ? vB : vA);
            y0 += v * xs[t].x;
            y1 += v * xs[t].y;
            if (cs[t] == (int)i) {
              xd = xs[t];
              found = true;
            }
          }
        }
      }
      // rows longer than 32 entries: the next 32 of each half's row
      q0 += 32;
      if (__ballot(a + q0 < b) == 0ull) break;   // every lane takes part in the ballot
      load_ent(a + q0, b, ec, ev);
    }
    double t0 = 0.0, t1 = 0.0;          // this row's terms of the dot
    if (has && on) {
      // stored nontemporally: the next kernel reads Y once
      d2v* yr = (d2v*)(Y + (i * nrhs + c0 + 2 * hl));
      d2v yv;
      yv.x = y0;
      yv.y = y1;
      __builtin_nontemporal_store(yv, yr);
      if (dot) {
        // a row without a diagonal entry loads X[i, :] after all
        const double2 w = found ? xd : *(const double2*)(X + (i * nrhs + c0 + 2 * hl));
        t0 = w.x * y0;
        t1 = w.y * y1;
      }
    }
    if (dot) {
      // both halves add the pair's terms in position order, as k_spmm_wave adds its
      // rows one after the other, so the partials equal that kernel's bit for bit
      const double o0 = __shfl_xor(t0, 32, SPAI_WAVE), o1 = __shfl_xor(t1, 32, SPAI_WAVE);
      const bool hasA = __shfl_xor((int)has, half ? 32 : 0, SPAI_WAVE) != 0;
      const bool hasB = __shfl_xor((int)has, half ? 0 : 32, SPAI_WAVE) != 0;
      if (on && hasA) {
        acc0 += half ? o0 : t0;
        acc1 += half ? o1 : t1;
      }
      if (on && hasB) {
        acc0 += half ? t0 : o0;
        acc1 += half ? t1 : o1;
      }
    }
    i = ni;
    a = na;
    b = nb;
    ec = nec;
    ev = nev;
    load_pos(k + 4 + half, ni, na, nb);
  }
  if (!part) return;
  // per right-hand side r = 2 (l mod 32) + s, wave w's sum (the same in both halves) at
  // sh[w 64 + r], reduced over the waves in order as in k_spmm_wave
  if (half == 0) {
    sh[wv * 64 + 2 * hl] = acc0;
    sh[wv * 64 + 2 * hl + 1] = acc1;
  }
  __syncthreads();
  if (threadIdx.x < 64 && c0 + (int)threadIdx.x < nrhs) {
    double sum = 0.0;
    for (int w = 0; w < WPB; ++w) sum += sh[w * 64 + threadIdx.x];
    part[(int64_t)(c0 + threadIdx.x) * gridDim.x + blockIdx.x] = sum;
  }
}

// The sum of sh[k], k = t, t + R, ... below kThreads, from 0 in that order: 16 loads in
// flight, the additions one after the other (the order is the result's).
__device__ __forceinline__ double column_sum(const double* sh, int t, int R) {
  double s = 0.0;
  int k = t;
  for (; k + 15 * R < kThreads; k += 16 * R) {
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = sh[k + u * R];
#pragma unroll
    for (int u = 0; u < 16; ++u) s += v[u];
  }
  for (; k < kThreads; k += R) s += sh[k];
  return s;
}

struct RhsState {
  double bnorm, rz, pq, rr, alpha, beta;
  double alpha_prev;                // the previous iteration's alpha (its x term may be pending)
  int active, iters, status, pad;   // status 0 running, 1 converged, 2 maxiter, 4 indefinite
};
__device__ void rhs_alpha(RhsState& g, double pq, int* nactive);
__device__ void rhs_conv(RhsState& g, double rr, double rtol, int* nactive);
__device__ void rhs_beta(RhsState& g, double rz_new);

// What the last workgroup of a product or of the r update does with the partials: the
// right-hand sides' sums (part[r * rstep + b * bstep], nrhs of them, nblocks partials each)
// and the scalar step that consumes them (0: alpha, 1: beta, 2: convergence).  ticket counts
// the workgroups that have written theirs (null: a launch of its own sums them); the last
// one leaves it at 0 for the next launch.  One launch less per reduction: where partials and
// workgroups are few the sums take less time than a launch, 2 to 4 us each of the three in an
// iteration; beyond that one workgroup per right-hand side sums them faster.  20^3, 4
// right-hand sides: a solve 1.57 ms fused, 1.71 not.  Products, 256 x 256 grid, 8 right-hand
// sides (512 workgroups): 11.3 and 10.7; 28^3, 16 of them (344): 2.95 and 2.99.  The r update:
// 52^3, 4 right-hand sides (4396 partials, as many waves) 8.35 and 7.85, 256 x 256, 4 (4096)
// 9.8 and 9.4, 46^3, 2 (1522) 4.6 both.
struct Finish {
  int* ticket = nullptr;
  RhsState* S = nullptr;
  int* nactive = nullptr;
  int step = 0, nrhs = 0;
  int64_t rstep = 0, bstep = 0;
  double rtol = 0.0;
};
constexpr int kFusedParts = 8192;
constexpr int kFusedGrid = 400;     // and the workgroups that draw a ticket
constexpr int kFusedRows = 2048;    // partials of the r update

__device__ __forceinline__ void finish_blocks(const Finish& f, const double* part, int nblocks) {
  __shared__ int last;
  // this workgroup's partials (agent_store) have arrived before its ticket is drawn
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0)
    last = __hip_atomic_fetch_add(f.ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
           (int)gridDim.x - 1;
  __syncthreads();
  if (!last) return;
  for (int r = threadIdx.x >> 6; r < f.nrhs; r += blockDim.x >> 6) {
    const double v = blocks_sum_wave(part + r * f.rstep, f.bstep, nblocks);
    if ((threadIdx.x & 63) == 0) {
      if (f.step == 0) rhs_alpha(f.S[r], v, f.nactive);
      else if (f.step == 1) rhs_beta(f.S[r], v);
      else rhs_conv(f.S[r], v, f.rtol, f.nactive);
    }
  }
  if (threadIdx.x == 0) *f.ticket = 0;
}

// a launch that returns at once takes its scalar step all the same (every right-hand side has
// stopped, so no sum is read): the step carries a pending x term on
__device__ __forceinline__ void finish_stopped(const Finish& f) {
  if (!f.ticket || blockIdx.x != 0 || (int)threadIdx.x >= f.nrhs) return;
  if (f.step == 0) rhs_alpha(f.S[threadIdx.x], 0.0, f.nactive);
  else if (f.step == 1) rhs_beta(f.S[threadIdx.x], 0.0);
}

// The product for at most 32 right-hand sides.  A wave of k_spmm_wave would leave
// 64 - nrhs lanes idle; here R = pow2(nrhs) lanes share a row (lane r owns right-hand
// side r), and each lane sums its row's entries in stored order, eight entries and their
// gathers issued together (the order of k_spmm_wave: the rows of Y are the same bit for
// bit).  Positions are dealt as in k_spmm_wave: eight contiguous XCD ranges, each workgroup
// a contiguous chunk of narrow_chunk(R) positions.  With dot set, per-block partials of
// sum_i X[i, r] Y[i, r], stored transposed as there: thread (g, r) of 256 adds its rows g,
// g + G, ..., then g runs over the G groups.
// W = 4: 1024 threads take those rows side by side instead of 256 one after the other and
// leave the terms in LDS for the same sums.  Where a launch has few workgroups (wide_grid) the
// product is bound by the latency of a thread's rows (descriptor, entries, gathers, one row
// after the other): 256 x 256 grid, 4 right-hand sides (256 workgroups) 12.4 us with its
// reduction, against 13.3 and a reduction of 4.1; with more workgroups 256 threads keep more
// waves resident (registers).  Those take no reduction's end: the code alone, never run there,
// cost 5% (64^3, float32 M, 8 right-hand sides: z = M r 65 us against 70).
template <int R>
constexpr int narrow_rpt() { return R / 4 > 4 ? R / 4 : 4; }   // rows per thread of 256
template <int R>
constexpr int narrow_chunk() { return (kThreads / R) * narrow_rpt<R>(); }

template <typename VT, int LAY, int R, int W>
__global__ __launch_bounds__(kThreads* W) void k_spmm_narrow(Mat A, const double* X, double* Y,
                                                             int dot, int nrhs,
                                                             const int32_t* order, double* part,
                                                             Finish fin) {
  static_assert(narrow_chunk<R>() >= (kThreads / 64) * kRowsPerWave,
                "no more workgroups than the partial buffer holds");
  if (A.gate && *A.gate == 0) {                            // every right-hand side stopped
    if constexpr (W > 1) finish_stopped(fin);
    return;
  }
  if (A.ran && blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(A.ran, 1);
  constexpr int G = kThreads / R;
  constexpr int RPT = narrow_rpt<R>();
  __shared__ double sh[W == 1 ? kThreads : RPT * kThreads];
  const int t = threadIdx.x % kThreads;
  const int r = t % R, g = t / R;
  const int64_t xcd = blockIdx.x & 7, kb = blockIdx.x >> 3;
  const int64_t per = (A.n + 7) / 8;
  const int64_t r0 = xcd * per;
  const int64_t r1 = r0 + per < A.n ? r0 + per : A.n;
  const int64_t base = r0 + kb * (int64_t)narrow_chunk<R>();
  double acc = 0.0;
  if (W > 1 || r < nrhs) {
    for (int j = W > 1 ? threadIdx.x / kThreads : 0; j < RPT; j += W) {
      const int64_t k = base + (int64_t)j * G + g;
      if (W == 1 && k >= r1) break;
      double term = 0.0;
      if (W == 1 || (r < nrhs && k < r1)) {
        const int64_t i = order ? (int64_t)order[k] : k;
        const int64_t a = row_lo<LAY>(A, i), b = row_hi<LAY>(A, i);
        double y = 0.0, xd = 0.0;
        bool found = false;
        for (int64_t q0 = a; q0 < b; q0 += 8) {
          int cc[8];
          VT vv[8];
          double xx[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            cc[u] = -1;
            vv[u] = 0;
            if (q0 + u < b) {
              cc[u] = A.col[q0 + u];
              vv[u] = entry_val<VT>(A, q0 + u);
            }
          }
#pragma unroll
          for (int u = 0; u < 8; ++u) xx[u] = cc[u] >= 0 ? X[(int64_t)cc[u] * nrhs + r] : 0.0;
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (cc[u] >= 0) {               // ELL padding (column -1) sits last
              y += (double)vv[u] * xx[u];
              if (cc[u] == (int)i) {
                xd = xx[u];
                found = true;
              }
            }
          if (cc[7] < 0) break;
        }
        Y[i * nrhs + r] = y;
        if (dot) {
          // a row without a diagonal entry loads X[i, r] after all
          const double wx = found ? xd : X[i * nrhs + r];
          if (W == 1) acc += wx * y;
          else term = wx * y;
        }
      }
      if (W > 1) sh[j * kThreads + t] = term;
    }
  }
  if (!part) return;
  if (W > 1) {
    __syncthreads();
    if (threadIdx.x < kThreads)
#pragma unroll
      for (int j = 0; j < RPT; ++j) acc += sh[j * kThreads + t];
    __syncthreads();
  }
  if (threadIdx.x < kThreads) sh[t] = acc;
  __syncthreads();
  if (threadIdx.x < R && t < nrhs)
    agent_store(&part[(int64_t)t * gridDim.x + blockIdx.x], column_sum(sh, t, R));
  if constexpr (W > 1)
    if (fin.ticket) finish_blocks(fin, part, (int)gridDim.x);
}

// The product for at most two right-hand sides: four lanes per row and right-hand side, lane
// l of them holding entries 2 l and 2 l + 1 of each eight, so that a row's entries are read
// side by side and a wave's load touches 16 rows' pieces instead of 64 (a thread per row reads
// its entries 8 or more words from its neighbour's: the address unit, at one cache line per
// lane and load, was what the product waited for).  A row's sum still runs over its entries in
// stored order, from 0: lane 0 adds its two, hands the sum to lane 1, and so on; lane 3 ends
// with it.  1024 threads take the G = 256 / R rows of a pass of k_spmm_narrow at a time, four
// passes with their loads in flight together, and the partials are that kernel's: the same
// bit for bit.  256 x 256 grid, one right-hand side (64 workgroups): z = M r 19.4 us against
// 31.7, q = A p 12.9 against 17.1 (each with its reduction).  Solves with one and two: 64^3
// 9.6 ms against 14.1 and 12.0 against 13.7, 96^3 47 against 88 and 55 against 77.  From three right-hand sides on a
// thread per value is faster (four of them, 44.3 us an iteration against 47.1): its lanes
// share their rows' loads already.
constexpr int kQuadRhs = 2;         // padded right-hand sides
template <int R>
__device__ __forceinline__ double quad_shift(double v) {       // lane l's value to lane l + 1
  const long long b = __double_as_longlong(v);
  const int lo = lane_dpp<0x110 + R>((int)(b & 0xffffffffll));  // row_shr R
  const int hi = lane_dpp<0x110 + R>((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
template <int R>
__device__ __forceinline__ double quad_return(double v) {      // lane 3's value to lane 0
  const long long b = __double_as_longlong(v);
  const int lo = lane_dpp<0x100 + 3 * R>((int)(b & 0xffffffffll));  // row_shl 3 R
  const int hi = lane_dpp<0x100 + 3 * R>((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
// y (in lane 0) plus the eight terms in order; the sum is lane 3's.  Every lane takes part.
template <int R>
__device__ __forceinline__ double quad_sum(int l, double y, double p0, double p1) {
  double s = (y + p0) + p1;
#pragma unroll
  for (int k = 1; k < 4; ++k) {
    const double t = (quad_shift<R>(s) + p0) + p1;
    s = l == k ? t : s;
  }
  return s;
}

template <typename VT, int LAY, int R>
__global__ __launch_bounds__(4 * kThreads) void k_spmm_quad(Mat A, const double* X, double* Y,
                                                            int dot, int nrhs,
                                                            const int32_t* order, double* part,
                                                            Finish fin) {
  if (A.gate && *A.gate == 0) return finish_stopped(fin);  // every right-hand side stopped
  if (A.ran && blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(A.ran, 1);
  constexpr int G = kThreads / R;
  constexpr int RPT = narrow_rpt<R>();
  static_assert(R <= 4 && RPT == 4, "four lanes per value within 16");
  __shared__ double sh[kThreads];
  const int r = threadIdx.x % R, l = (threadIdx.x / R) & 3, g = threadIdx.x / (4 * R);
  const int64_t xcd = blockIdx.x & 7, kb = blockIdx.x >> 3;
  const int64_t per = (A.n + 7) / 8;
  const int64_t r0 = xcd * per;
  const int64_t r1 = r0 + per < A.n ? r0 + per : A.n;
  const int64_t base = r0 + kb * (int64_t)narrow_chunk<R>();
  const int rc = r < nrhs ? r : 0;
  int64_t row[RPT], a[RPT], b[RPT];
#pragma unroll
  for (int j = 0; j < RPT; ++j) {
    const int64_t k = base + (int64_t)j * G + g;
    row[j] = -1;
    if (k < r1) row[j] = order ? (int64_t)order[k] : k;
  }
#pragma unroll
  for (int j = 0; j < RPT; ++j) {
    a[j] = b[j] = 0;
    if (row[j] >= 0) {
      a[j] = row_lo<LAY>(A, row[j]);
      b[j] = row_hi<LAY>(A, row[j]);
    }
  }
  // entries q, q + 1 of a row that ends at e (column -1: none)
  auto two = [&](int64_t q, int64_t e, int (&c)[2], VT (&v)[2]) {
    typedef int i2 __attribute__((ext_vector_type(2), aligned(4)));
    typedef VT v2 __attribute__((ext_vector_type(2), aligned(sizeof(VT))));
    c[0] = c[1] = -1;
    v[0] = v[1] = 0;
    if (q + 1 < e) {
      const i2 cc = *(const i2*)(A.col + q);
      c[0] = cc.x;
      c[1] = cc.y;
      v2 vv;
      if constexpr (sizeof(VT) == 4) vv = *(const v2*)(A.val32 + q);
      else vv = *(const v2*)(A.val + q);
      v[0] = vv.x;
      v[1] = vv.y;
    } else if (q < e) {
      c[0] = A.col[q];
      v[0] = entry_val<VT>(A, q);
    }
  };
  int c[RPT][2];
  VT v[RPT][2];
  double xd[RPT], x[RPT][2];
#pragma unroll
  for (int j = 0; j < RPT; ++j) two(a[j] + 2 * l, b[j], c[j], v[j]);
#pragma unroll
  for (int j = 0; j < RPT; ++j) {
    xd[j] = dot && row[j] >= 0 ? X[row[j] * nrhs + rc] : 0.0;
    x[j][0] = c[j][0] >= 0 ? X[(int64_t)c[j][0] * nrhs + rc] : 0.0;
    x[j][1] = c[j][1] >= 0 ? X[(int64_t)c[j][1] * nrhs + rc] : 0.0;
  }
  double acc = 0.0;
#pragma unroll
  for (int j = 0; j < RPT; ++j) {
    double p0 = c[j][0] >= 0 ? (double)v[j][0] * x[j][0] : 0.0;
    double p1 = c[j][1] >= 0 ? (double)v[j][1] * x[j][1] : 0.0;
    double y = quad_sum<R>(l, 0.0, p0, p1);
    // rows longer than eight entries (the wave goes on together: lanes without one add 0)
    for (int64_t q = 8; __ballot(a[j] + q < b[j]) != 0ull; q += 8) {
      int cc[2];
      VT vv[2];
      two(a[j] + q + 2 * l, b[j], cc, vv);
      p0 = cc[0] >= 0 ? (double)vv[0] * X[(int64_t)cc[0] * nrhs + rc] : 0.0;
      p1 = cc[1] >= 0 ? (double)vv[1] * X[(int64_t)cc[1] * nrhs + rc] : 0.0;
      y = quad_sum<R>(l, quad_return<R>(y), p0, p1);
    }
    if (l == 3 && r < nrhs && row[j] >= 0) {
      Y[row[j] * nrhs + r] = y;
      acc += xd[j] * y;
    }
  }
  if (!part) return;
  if (l == 3) sh[g * R + r] = acc;
  __syncthreads();
  if ((int)threadIdx.x < nrhs)
    agent_store(&part[(int64_t)threadIdx.x * gridDim.x + blockIdx.x], column_sum(sh, threadIdx.x, R));
  if (fin.ticket) finish_blocks(fin, part, (int)gridDim.x);
}

// per-block partials of sum_i A[i, r] B[i, r] (B may be A), optionally of (B - C)
__global__ __launch_bounds__(kThreads) void k_dot_rows(const double* Xa, const double* Xb,
                                                       const double* Xc, int64_t n, int nrhs,
                                                       int c0, int cw, int R, double* part) {
  __shared__ double sh[kThreads];
  const int t = threadIdx.x;
  const int r = t % R;
  const int rows_per = kThreads / R;
  const int roff = t / R;
  double acc = 0.0;
  for (int64_t base = (int64_t)blockIdx.x * rows_per; base < n; base += (int64_t)gridDim.x * rows_per) {
    const int64_t i = base + roff;
    if (i < n && r < cw) {
      const int64_t o = i * nrhs + c0 + r;
      double a = Xa[o];
      double b = Xb[o];
      if (Xc) {
        a = a - Xc[o];
        b = a;
      }
      acc += a * b;
    }
  }
  sh[t] = acc;
  __syncthreads();
  if (t < cw) part[(int64_t)blockIdx.x * nrhs + c0 + t] = column_sum(sh, t, R);
}

// one workgroup per right-hand side: fixed strided partial sums, then a fixed tree
// sum_b p[b] over the workgroup in a fixed order (on thread 0)
__device__ double rows_sum(const double* p, int nblocks, double* sh) {
  // eight loads in flight per thread, added in the order of the plain loop
  double s = 0.0;
  int b = threadIdx.x;
  for (; b + 7 * kThreads < nblocks; b += 8 * kThreads) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[b + u * kThreads];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  for (; b < nblocks; b += kThreads) s += p[b];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int w = kThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  return sh[0];
}

// sum_b part[b * nrhs + r] in a fixed order (on thread 0)
__device__ double parts_sum(const double* part, int nblocks, int nrhs, int r, double* sh) {
  double s = 0.0;
  int b = threadIdx.x;
  for (; b + 7 * kThreads < nblocks; b += 8 * kThreads) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)(b + u * kThreads) * nrhs + r];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  for (; b < nblocks; b += kThreads) s += part[(int64_t)b * nrhs + r];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int w = kThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  return sh[0];
}

// out[r] = sum_b part[r * nblocks + b] in a fixed order (the products' transposed partials)
__global__ __launch_bounds__(kThreads) void k_reduce_rows(const double* part, int nblocks,
                                                          double* out) {
  __shared__ double sh[kThreads];
  const int r = blockIdx.x;
  const double v = rows_sum(part + (int64_t)r * nblocks, nblocks, sh);
  if (threadIdx.x == 0) out[r] = v;
}

__global__ __launch_bounds__(kThreads) void k_reduce_parts(const double* part, int nblocks,
                                                           int nrhs, double* out) {
  __shared__ double sh[kThreads];
  const int r = blockIdx.x;
  const double v = parts_sum(part, nblocks, nrhs, r, sh);
  if (threadIdx.x == 0) out[r] = v;
}

__global__ void k_init_rhs(RhsState* S, const double* bb, int nrhs, int* nactive) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nrhs) return;
  S[r].bnorm = sqrt(bb[r]);
  S[r].iters = 0;
  S[r].alpha = S[r].beta = 0.0;
  if (S[r].bnorm == 0.0) {
    S[r].active = 0;
    S[r].status = 1;
  } else {
    S[r].active = 1;
    S[r].status = 0;
    atomicAdd(nactive, 1);
  }
}

__global__ void k_set_rz(RhsState* S, const double* rz, int nrhs) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < nrhs) S[r].rz = rz[r];
}

// alpha = (r, z) / (p, A p), with the indefiniteness checks of the recurrence
// alpha = (r, z) / (p, q) of one right-hand side; a non-positive (r, z) or (p, q) stops it
// as indefinite
__device__ void rhs_alpha(RhsState& g, double pq, int* nactive) {
  g.alpha_prev = g.alpha;
  g.alpha = 0.0;
  if (!g.active) return;
  g.pq = pq;
  if (!(g.rz > 0.0) || !(g.pq > 0.0)) {
    g.active = 0;
    g.status = 4;
    atomicSub(nactive, 1);
    return;
  }
  g.alpha = g.rz / g.pq;
  g.iters += 1;
}

// r -= alpha q (inactive right-hand sides have alpha = 0), fused with the per-block
// partials of ||r||^2 for every right-hand side; x is updated later, with p.  Blocks read
// for the last time before they are written again (q here, z and x in the p updates)
// are loaded nontemporally, and x and the new p are stored so, as are the products'
// outputs: they do not push out of the caches what a product gathers (the 64-right-hand-
// side solve at 96^3 339 -> 330 ms; r, which the next product gathers, gained nothing).
// A block of partials belongs to kThreads threads; W of them share a workgroup (W = 4 where
// its last workgroup finishes the reduction: one draws a ticket where four did, and tickets
// of one address come one after the other, about 10 ns each).
template <int W>
__global__ __launch_bounds__(kThreads* W) void k_axpy(double* __restrict__ rv,
                                                      const double* __restrict__ q,
                                                      const RhsState* S, int64_t n, int nrhs,
                                                      int R, int nblocks, double* part,
                                                      const int* gate, Finish fin) {
  if (*gate == 0) return;                                  // every right-hand side stopped
  __shared__ double sh[kThreads * W];
  const int t = threadIdx.x % kThreads, wb = threadIdx.x / kThreads;
  const int block = blockIdx.x * W + wb;
  const int r = t % R;
  const int rows_per = kThreads / R;
  const int roff = t / R;
  double acc = 0.0;
  if (r < nrhs && block < nblocks) {
    const double a = S[r].alpha;
    for (int64_t base = (int64_t)block * rows_per; base < n; base += (int64_t)nblocks * rows_per) {
      const int64_t i = base + roff;
      if (i < n) {
        const int64_t o = i * nrhs + r;
        double rr = rv[o];
        if (a != 0.0) {
          rr = rr - a * __builtin_nontemporal_load(&q[o]);
          rv[o] = rr;
        }
        acc += rr * rr;
      }
    }
  }
  sh[threadIdx.x] = acc;
  __syncthreads();
  if (t < nrhs && block < nblocks)
    agent_store(&part[(int64_t)block * nrhs + t], column_sum(sh + wb * kThreads, t, R));
  if (fin.ticket) finish_blocks(fin, part, nblocks);
}

// convergence of one right-hand side on the recursive residual: ||r|| <= rtol ||b||
__device__ void rhs_conv(RhsState& g, double rr, double rtol, int* nactive) {
  if (!g.active) return;
  g.rr = rr;
  if (sqrt(g.rr) <= rtol * g.bnorm) {
    g.active = 0;
    g.status = 1;
    atomicSub(nactive, 1);
  }
}

__global__ void k_conv(RhsState* S, const double* rr, double rtol, int nrhs, int* nactive) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nrhs) return;
  rhs_conv(S[r], rr[r], rtol, nactive);
}

// beta = (r, z)_new / (r, z)_old of one right-hand side
__device__ void rhs_beta(RhsState& g, double rz_new) {
  g.beta = 0.0;
  if (!g.active) return;
  g.beta = rz_new / g.rz;
  g.rz = rz_new;
}

// The reductions of an iteration with the scalar step that consumes them (one launch
// instead of two; the same sums and the same step): step 0 alpha from (p, q), 1 beta from
// (r, z) -- both from the products' partials -- and convergence from ||r||^2 partials.
__global__ __launch_bounds__(kThreads) void k_reduce_rows_step(const double* part, int nblocks,
                                                               double* out, RhsState* S, int step,
                                                               int* nactive) {
  __shared__ double sh[kThreads];
  const int r = blockIdx.x;
  const double v = rows_sum(part + (int64_t)r * nblocks, nblocks, sh);
  if (threadIdx.x == 0) {
    out[r] = v;
    if (step == 0) rhs_alpha(S[r], v, nactive);
    else rhs_beta(S[r], v);
  }
}

__global__ __launch_bounds__(kThreads) void k_reduce_parts_conv(const double* part, int nblocks,
                                                                int nrhs, double* out,
                                                                RhsState* S, double rtol,
                                                                int* nactive) {
  __shared__ double sh[kThreads];
  const int r = blockIdx.x;
  const double v = parts_sum(part, nblocks, nrhs, r, sh);
  if (threadIdx.x == 0) {
    out[r] = v;
    rhs_conv(S[r], v, rtol, nactive);
  }
}

// The x update taken two iterations at a time (up to 64 right-hand sides): p alternates
// between two buffers, an even iteration only forms the next p, and the odd one after it
// adds both iterations' terms to x, first alpha_prev p_prev, then alpha p (the additions
// and their order are those of one update per iteration, so x is the same bit for bit).
// Reading x once per two iterations saves half a block pass per iteration.
//
// even iteration: pn = z + beta p for the running right-hand sides
__global__ __launch_bounds__(kThreads) void k_pupd_p(double* __restrict__ pn,
                                                     const double* __restrict__ p,
                                                     const double* __restrict__ z,
                                                     const RhsState* __restrict__ S, int64_t n,
                                                     int nrhs, int R) {
  const int t = threadIdx.x;
  const int r = t % R;
  const int rows_per = kThreads / R;
  const int roff = t / R;
  if (r >= nrhs || S[r].active == 0) return;
  const double b = S[r].beta;
  for (int64_t base = (int64_t)blockIdx.x * rows_per; base < n; base += (int64_t)gridDim.x * rows_per) {
    const int64_t i = base + roff;
    if (i < n) {
      const int64_t o = i * nrhs + r;
      __builtin_nontemporal_store(__builtin_nontemporal_load(&z[o]) + b * p[o], &pn[o]);
    }
  }
}

// odd iteration: x += alpha_prev pp, x += alpha p; then pp = z + beta p (pp holds the even
// iteration's p, read before it is overwritten)
__global__ __launch_bounds__(kThreads) void k_pupd_x2(double* __restrict__ pp,
                                                      const double* __restrict__ p,
                                                      double* __restrict__ x,
                                                      const double* __restrict__ z,
                                                      const RhsState* __restrict__ S, int64_t n,
                                                      int nrhs, int R) {
  const int t = threadIdx.x;
  const int r = t % R;
  const int rows_per = kThreads / R;
  const int roff = t / R;
  if (r >= nrhs) return;
  const double a0 = S[r].alpha_prev, a1 = S[r].alpha;
  const bool act = S[r].active != 0;
  const bool upx = a0 != 0.0 || a1 != 0.0;
  if (!upx && !act) return;
  const double b = S[r].beta;
  for (int64_t base = (int64_t)blockIdx.x * rows_per; base < n; base += (int64_t)gridDim.x * rows_per) {
    const int64_t i = base + roff;
    if (i < n) {
      const int64_t o = i * nrhs + r;
      const double po = p[o];
      if (upx) {
        double xv = __builtin_nontemporal_load(&x[o]);
        if (a0 != 0.0) xv = xv + a0 * pp[o];
        if (a1 != 0.0) xv = xv + a1 * po;
        __builtin_nontemporal_store(xv, &x[o]);
      }
      if (act) __builtin_nontemporal_store(__builtin_nontemporal_load(&z[o]) + b * po, &pp[o]);
    }
  }
}

// the pending x term of a solve that stopped after an even iteration: x += alpha p
__global__ __launch_bounds__(kThreads) void k_x_flush(double* __restrict__ x,
                                                      const double* __restrict__ p,
                                                      const RhsState* __restrict__ S, int64_t n,
                                                      int nrhs, int R) {
  const int t = threadIdx.x;
  const int r = t % R;
  const int rows_per = kThreads / R;
  const int roff = t / R;
  if (r >= nrhs) return;
  const double a = S[r].alpha;
  if (a == 0.0) return;
  for (int64_t base = (int64_t)blockIdx.x * rows_per; base < n; base += (int64_t)gridDim.x * rows_per) {
    const int64_t i = base + roff;
    if (i < n) {
      const int64_t o = i * nrhs + r;
      x[o] = x[o] + a * p[o];
    }
  }
}

// the same updates for more than 64 right-hand sides (flat indexing)
__global__ __launch_bounds__(kThreads) void k_axpy_wide(double* rv, const double* q,
                                                        const RhsState* S, int64_t n, int nrhs) {
  const int64_t tot = n * nrhs;
  for (int64_t o = (int64_t)blockIdx.x * kThreads + threadIdx.x; o < tot; o += (int64_t)gridDim.x * kThreads) {
    const double a = S[o % nrhs].alpha;
    if (a != 0.0) rv[o] = rv[o] - a * q[o];
  }
}

__global__ __launch_bounds__(kThreads) void k_pupd_wide(double* p, double* x, const double* z,
                                                        const RhsState* S, int64_t n, int nrhs) {
  const int64_t tot = n * nrhs;
  for (int64_t o = (int64_t)blockIdx.x * kThreads + threadIdx.x; o < tot; o += (int64_t)gridDim.x * kThreads) {
    const int r = (int)(o % nrhs);
    const double a = S[r].alpha;
    const double po = p[o];
    if (a != 0.0) x[o] = x[o] + a * po;
    if (S[r].active) p[o] = z[o] + S[r].beta * po;
  }
}

__global__ __launch_bounds__(kThreads) void k_copy(double* dst, const double* src, int64_t tot) {
  for (int64_t o = (int64_t)blockIdx.x * kThreads + threadIdx.x; o < tot; o += (int64_t)gridDim.x * kThreads)
    dst[o] = src[o];
}

__global__ __launch_bounds__(kThreads) void k_fill(double* dst, double v, int64_t tot) {
  for (int64_t o = (int64_t)blockIdx.x * kThreads + threadIdx.x; o < tot; o += (int64_t)gridDim.x * kThreads)
    dst[o] = v;
}

// ---- the whole solve in one workgroup -------------------------------------------------
// A small solve is a chain of launches, seven an iteration at 2.5 to 7 us each with a few
// rows of work in every one.  With at most kTinyElems values per block of vectors one
// workgroup of 1024 threads runs all of it: the vectors that are gathered (p, r) and the
// terms of the dots in LDS, x, z and q in registers of the thread that owns a position and a
// right-hand side, barriers instead of launches (where A and M have few enough entries,
// tiny_limit: the kernel itself counts them and declines).  Up to 1024 values (U = 1) the first eight
// entries of a thread's rows of A and M stay in registers too.  Bound by the ordered sums
// (chains of up to 256 dependent additions) and, with U = 4, the rows' entries from L2.
// 17 x 17 and 32 x 32 grids, one right-hand side: 7 us an iteration against 63 and 50 launched
// (32 with fused reductions).
// Every sum is that of the launched kernels: the products' terms by XCD range and thread of
// the 256 (one workgroup per range here), the rows' by blocks of kThreads / R rows, each
// from 0 in order, and the partials by halves (an unlaunched workgroup's is 0).  The results
// are the same bit for bit.
constexpr int kTinyElems = 4096;
constexpr int kTinyRows = 1024;     // beyond, one compute unit reads the rows too slowly: 4096
                                    // rows and one right-hand side 58 us an iteration, launched 60
constexpr int kTinyThreads = 1024;
constexpr int kTinyRhs = 32;
constexpr int kTinyDeclined = -1;   // TinyOut.status of a solve that one workgroup is not to take
// Stored entries of A and M, times right-hand sides, that one workgroup reads (row after row,
// eight entries a load) no slower than the launched products: beyond, they are faster.  The
// lanes of four right-hand sides share a row's loads, which other numbers split over the waves'
// ends; up to 1024 values the rows' first entries stay in registers, and rows are shared the
// more, the more right-hand sides there are.  us an iteration, one workgroup | launched, some
// 30 to 60 us a solve more where it declines: one right-hand side 31 | 41 at 40,000, 60 | 47 at
// 72,000; three, 900 values 39 | 54 at 74,000, 108 | 83 at 206,000; three, 2200 values and more
// 43 | 48 at 70,000, 66 | 48 at 119,000; six 36 | 42 at 83,000, 43 | 40 at 98,000; four 42 | 45
// at 128,000, 49 | 46 at 176,000; sixteen 43 | 44 at 172,000.
__host__ __device__ inline int tiny_limit(int n, int nrhs) {
  if (nrhs % 4 == 0) return 160000;
  if (n * nrhs <= 1024) return nrhs < 3 ? 32000 * (nrhs + 1) : 128000;
  return nrhs > 4 ? 84000 : 64000;
}
// Iterations of one launch: a kernel cannot be interrupted, and a solve that stagnates runs to
// its max_iter (any int).  1024 take 7 to 50 ms, 0.02 ms of it the launch and the host's look;
// what goes on is kept in TinyKeep.
constexpr int kTinyIters = 1024;

struct TinyOut {
  int iters, status;
  int active, pad;                  // right-hand sides still running (rr is then not set)
  double bnorm, rr;                 // ||b||, sum of (b - A x)^2
};

// a solve between two launches
struct TinyKeep {
  TinyOut out[kTinyRhs];
  RhsState S[kTinyRhs];
  double x[kTinyElems], r[kTinyElems], p[kTinyElems];
};

// eight entries of a row from q0 (column -1: none)
template <typename VT, int LAY>
__device__ __forceinline__ void tiny_chunk(const Mat& A, int64_t q0, int64_t b, int (&cc)[8],
                                           VT (&vv)[8]) {
  if constexpr (LAY == kLayEll) {                 // aligned pieces of the padded row
    const int4 c0 = *(const int4*)(A.col + q0), c1 = *(const int4*)(A.col + q0 + 4);
    cc[0] = c0.x; cc[1] = c0.y; cc[2] = c0.z; cc[3] = c0.w;
    cc[4] = c1.x; cc[5] = c1.y; cc[6] = c1.z; cc[7] = c1.w;
    if constexpr (sizeof(VT) == 8) {
#pragma unroll
      for (int u = 0; u < 8; u += 2) {
        const double2 v = *(const double2*)(A.val + q0 + u);
        vv[u] = v.x;
        vv[u + 1] = v.y;
      }
    } else {
#pragma unroll
      for (int u = 0; u < 8; ++u) vv[u] = entry_val<VT>(A, q0 + u);
    }
  } else {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      cc[u] = -1;
      vv[u] = 0;
      if (q0 + u < b) {
        cc[u] = A.col[q0 + u];
        vv[u] = entry_val<VT>(A, q0 + u);
      }
    }
  }
}

// a row of the product: its first eight entries are in (cc, vv)
template <typename VT, int LAY>
__device__ __forceinline__ double tiny_row(const Mat& A, int64_t i, const int (&c0)[8],
                                           const VT (&v0)[8], const double* x, int nrhs, int r) {
  double y = 0.0;
#pragma unroll
  for (int u = 0; u < 8; ++u)
    if (c0[u] >= 0) y += (double)v0[u] * x[c0[u] * nrhs + r];
  if (c0[7] >= 0) {
    const int64_t b = row_hi<LAY>(A, i);
    for (int64_t q0 = row_lo<LAY>(A, i) + 8; q0 < b; q0 += 8) {
      int cc[8];
      VT vv[8];
      tiny_chunk<VT, LAY>(A, q0, b, cc, vv);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (cc[u] >= 0) y += (double)vv[u] * x[cc[u] * nrhs + r];
      if (cc[7] < 0) break;
    }
  }
  return y;
}

// s = 0; s += ((t[g] + t[G + g]) + t[2 G + g]) + ... (J terms) for g < cnt in order, cnt a
// multiple of eight, the next K g's loads ahead of the additions
template <int J>
__device__ __forceinline__ double tiny_chain(const double* t, int G, int cnt) {
  constexpr int K = J == 1 ? 8 : J == 2 ? 4 : 2;
  double s = 0.0;
  double v[J][K];
#pragma unroll
  for (int j = 0; j < J; ++j)
#pragma unroll
    for (int c = 0; c < K; ++c) v[j][c] = t[j * G + c];
#pragma unroll 1
  for (int g = K; g <= cnt; g += K) {
    double w[J][K];
    const int gn = g < cnt ? g : 0;               // (the last round's loads are not used)
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
      for (int c = 0; c < K; ++c) w[j][c] = t[j * G + gn + c];
#pragma unroll
    for (int c = 0; c < K; ++c) {
      double a = v[0][c];
#pragma unroll
      for (int j = 1; j < J; ++j) a += v[j][c];
      s += a;
    }
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
      for (int c = 0; c < K; ++c) v[j][c] = w[j][c];
  }
  return s;
}

// Where the terms of the sums sit in LDS: each chain of additions contiguous (an odd number
// of doubles from one chain to the next: different banks), zeros behind its last term.
// By position: a chain per XCD range and right-hand side, J rows of G terms (thread g of the
// 256 adds its J rows first) or, with a row per thread, one of `cnt`; by row: a chain per
// block of G rows and right-hand side.
struct TinyLay {
  int G, J, cnt, lp, blocks;        // lp: doubles per chain by position (G + 1 by row)
  int by_pos, by_row;               // doubles in all
};
__host__ __device__ inline TinyLay tiny_lay(int n, int nrhs, int R) {
  TinyLay l;
  const int per = (n + 7) / 8;
  l.G = kThreads / R;
  l.J = (per + l.G - 1) / l.G;
  l.cnt = l.J > 1 ? l.G : (per + 7) / 8 * 8;
  l.lp = l.J * l.cnt + 1;
  l.blocks = (n + l.G - 1) / l.G;
  l.by_pos = 8 * nrhs * l.lp;
  l.by_row = l.blocks * nrhs * (l.G + 1);
  return l;
}
constexpr int kTinyTerms = 5248;    // of each kind

template <typename MT, int LAYA, int LAYM, int U>
__global__ __launch_bounds__(kTinyThreads) void k_pcg_tiny(Mat A, Mat M, const double* __restrict__ B,
                                                           double* __restrict__ X, int nrhs, int R,
                                                           double rtol, int it0, int it1, int max_iter,
                                                           const int32_t* order, TinyKeep* keep) {
  __shared__ double s_p[kTinyThreads * U], s_r[kTinyThreads * U];
  __shared__ double s_t[kTinyTerms], s_n[kTinyTerms];       // terms by position, by row
  __shared__ RhsState S[kTinyRhs];
  __shared__ int s_active, s_entries;
  const int tid = threadIdx.x;
  const int n = (int)A.n, tot = n * nrhs;
  if (it0 == 0) {                   // n <= kTinyThreads: a thread a row
    if (tid == 0) s_entries = 0;
    __syncthreads();
    int64_t len = 0;
    if (tid < n)
      len = row_hi<LAYA>(A, tid) - row_lo<LAYA>(A, tid) + row_hi<LAYM>(M, tid) - row_lo<LAYM>(M, tid);
    const int sum = wave_sum_int((int)len);        // (a row has at most n entries, or 64 in ELL)
    if ((tid & 63) == 0) atomicAdd(&s_entries, sum);
    __syncthreads();
    if (s_entries > tiny_limit(n, nrhs) / nrhs) {
      if (tid == 0) keep->out[0] = TinyOut{0, kTinyDeclined, 0, 0, 0.0, 0.0};
      return;
    }
  }
  const int per = (n + 7) / 8;
  const TinyLay lay = tiny_lay(n, nrhs, R);
  const int G = lay.G;              // rows of a pass of 256 threads
  for (int k = tid; k < lay.by_pos; k += kTinyThreads) s_t[k] = 0.0;
  for (int k = tid; k < lay.by_row; k += kTinyThreads) s_n[k] = 0.0;
  __syncthreads();
  // element e = tid + u kTinyThreads is position e / nrhs and right-hand side e mod nrhs: its
  // row and right-hand side (-1: none), its x, and q or z
  int place[U], tat[U], nat[U];     // and the places of its terms
  double x[U], w[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int e = tid + u * kTinyThreads;
    place[u] = -1;
    tat[u] = nat[u] = 0;
    if (e < tot) {
      const int k = e / nrhs, r = e - k * nrhs;
      const int i = order ? order[k] : k;
      place[u] = i * kTinyRhs + r;
      tat[u] = (r * 8 + k / per) * lay.lp + k % per;
      nat[u] = (r * lay.blocks + i / G) * (G + 1) + i % G;
    }
    x[u] = w[u] = 0.0;
  }
  int ca[8], cm[8];                 // U = 1: the rows' first entries
  double va[8];
  MT vm[8];
  if constexpr (U == 1) {
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      ca[c] = cm[c] = -1;
      va[c] = 0.0;
      vm[c] = 0;
    }
    if (place[0] >= 0) {
      const int64_t i = place[0] / kTinyRhs;
      const int64_t a = row_lo<LAYA>(A, i), m = row_lo<LAYM>(M, i);
      if (a < row_hi<LAYA>(A, i)) tiny_chunk<double, LAYA>(A, a, row_hi<LAYA>(A, i), ca, va);
      if (m < row_hi<LAYM>(M, i)) tiny_chunk<MT, LAYM>(M, m, row_hi<LAYM>(M, i), cm, vm);
    }
  }
  // f(u, row, r, own): own the element by row.  (U > 1: the place is
  // opaque each time, as left to itself the compiler keeps the addresses and entries of all
  // the rows across the iterations, and spills them.)
  auto each = [&](auto f) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (place[u] >= 0) {
        int pl = place[u];
        if constexpr (U > 1) asm volatile("" : "+v"(pl));
        const int i = pl / kTinyRhs, r = pl % kTinyRhs;
        f(u, i, r, i * nrhs + r);
      }
  };
  auto row_a = [&](int i, const double* v, int r) {
    if constexpr (U > 1) {
      const int64_t a = row_lo<LAYA>(A, i), b = row_hi<LAYA>(A, i);
#pragma unroll
      for (int c = 0; c < 8; ++c) ca[c] = -1;
      if (a < b) tiny_chunk<double, LAYA>(A, a, b, ca, va);
    }
    return tiny_row<double, LAYA>(A, i, ca, va, v, nrhs, r);
  };
  auto row_m = [&](int i, const double* v, int r) {
    if constexpr (U > 1) {
      const int64_t a = row_lo<LAYM>(M, i), b = row_hi<LAYM>(M, i);
#pragma unroll
      for (int c = 0; c < 8; ++c) cm[c] = -1;
      if (a < b) tiny_chunk<MT, LAYM>(M, a, b, cm, vm);
    }
    return tiny_row<MT, LAYM>(M, i, cm, vm, v, nrhs, r);
  };
  // the sums of s_t in the products' order (by position), step(r, sum) on one thread each ...
  auto product_sums = [&](auto step) {
    if (tid < 8 * nrhs) {
      const int xcd = tid & 7, r = tid >> 3;
      const double* t = s_t + tid * lay.lp;
      double s = lay.J == 1   ? tiny_chain<1>(t, 0, lay.cnt)
                 : lay.J == 2 ? tiny_chain<2>(t, G, G)
                 : lay.J == 3 ? tiny_chain<3>(t, G, G)
                              : tiny_chain<4>(t, G, G);
      // lanes 8 r .. 8 r + 7 hold the eight workgroups' partials
      s = lane_xor_add<4>(s);
      s = lane_xor_add<2>(s);
      s = lane_xor_add<1>(s);
      if (xcd == 0) step(r, s);
    }
  };
  // ... and of s_n in the order of a pass over the rows, from the last threads on
  auto row_sums = [&](auto step) {
    const int at = kTinyThreads - 1 - tid;
    if (at < 32 * nrhs) {
      const int blk = at & 31, r = at >> 5;
      double s = 0.0;
      if (blk < lay.blocks) s = tiny_chain<1>(s_n + (r * lay.blocks + blk) * (G + 1), 0, G);
      s = lane_xor_add<16>(s);
      s = lane_xor_add<8>(s);
      s = lane_xor_add<4>(s);
      s = lane_xor_add<2>(s);
      s = lane_xor_add<1>(s);
      if (blk == 0) step(r, s);
    }
  };
  if (tid == 0) s_active = 0;
  if (it0 > 0) {                    // where the launch before this one stopped
    each([&](int u, int i, int r, int own) {
      x[u] = keep->x[own];
      s_r[own] = keep->r[own];
      s_p[own] = keep->p[own];
    });
    __syncthreads();
    if (tid < nrhs) {
      S[tid] = keep->S[tid];
      if (S[tid].active) atomicAdd(&s_active, 1);
    }
  } else {                          // x_0 = 0, r = b, z = M r, p = z
    each([&](int u, int i, int r, int own) {
      const double b = B[own];
      s_r[own] = b;
      s_n[nat[u]] = b * b;
    });
    __syncthreads();
    each([&](int u, int i, int r, int own) {
      w[u] = row_m(i, s_r, r);
      s_p[own] = w[u];
      s_t[tat[u]] = s_r[own] * w[u];
    });
    row_sums([&](int r, double bb) {
      RhsState& g = S[r];
      g = RhsState{};
      g.bnorm = sqrt(bb);
      if (g.bnorm == 0.0) {
        g.status = 1;
      } else {
        g.active = 1;
        atomicAdd(&s_active, 1);
      }
    });
    __syncthreads();
    product_sums([&](int r, double v) { S[r].rz = v; });
  }
  __syncthreads();
  for (int it = it0; it < it1 && s_active > 0; ++it) {
    each([&](int u, int i, int r, int own) {      // q = A p, (p, q), alpha
      w[u] = row_a(i, s_p, r);
      s_t[tat[u]] = s_p[own] * w[u];
    });
    __syncthreads();
    product_sums([&](int r, double v) { rhs_alpha(S[r], v, &s_active); });
    __syncthreads();
    each([&](int u, int i, int r, int own) {      // r -= alpha q, x += alpha p
      const double a = S[r].alpha;
      double rr = s_r[own];
      if (a != 0.0) {
        rr = rr - a * w[u];
        s_r[own] = rr;
        x[u] = x[u] + a * s_p[own];
      }
      s_n[nat[u]] = rr * rr;
    });
    __syncthreads();
    each([&](int u, int i, int r, int own) {      // z = M r
      w[u] = row_m(i, s_r, r);
      s_t[tat[u]] = s_r[own] * w[u];
    });
    // ||r||^2 and the convergence test, while the first threads wait for z; then (r, z)
    row_sums([&](int r, double v) { rhs_conv(S[r], v, rtol, &s_active); });
    __syncthreads();
    product_sums([&](int r, double v) { rhs_beta(S[r], v); });
    __syncthreads();
    each([&](int u, int i, int r, int own) {      // p = z + beta p
      if (S[r].active) s_p[own] = w[u] + S[r].beta * s_p[own];
    });
    __syncthreads();
  }
  if (s_active > 0 && it1 < max_iter) {
    each([&](int u, int i, int r, int own) {
      keep->x[own] = x[u];
      keep->r[own] = s_r[own];
      keep->p[own] = s_p[own];
    });
    if (tid < nrhs) {
      keep->S[tid] = S[tid];
      keep->out[tid].active = s_active;
    }
    return;
  }
  // x, and the true residual: p's place takes x for the product
  each([&](int u, int i, int r, int own) {
    X[own] = x[u];
    s_p[own] = x[u];
  });
  __syncthreads();
  each([&](int u, int i, int r, int own) {
    const double d = B[own] - row_a(i, s_p, r);
    s_n[nat[u]] = d * d;
  });
  __syncthreads();
  row_sums([&](int r, double v) {
    keep->out[r] = TinyOut{S[r].iters, S[r].status, 0, 0, S[r].bnorm, v};
  });
}

// which solves: the vectors fit, and each XCD range is one workgroup of the narrow product
// and the rows at most 32 blocks (so the partials above are all there are)
static bool tiny_fits(int64_t n, int nrhs) {
  if (nrhs > kTinyRhs || n > kTinyRows || n * nrhs > kTinyElems) return false;
  int R = 1;
  while (R < nrhs) R <<= 1;
  const int rpt = R / 4 > 4 ? R / 4 : 4;
  const TinyLay l = tiny_lay((int)n, nrhs, R);
  return (n + 7) / 8 <= (int64_t)l.G * rpt && l.J <= 4 && l.blocks <= 32 &&
         l.by_pos <= kTinyTerms && l.by_row <= kTinyTerms;
}

template <typename MT, int LAYA>
static void launch_tiny(const Mat& A, const Mat& M, const double* B, double* X, int nrhs, int R,
                        double rtol, int it0, int it1, int max_iter, const int32_t* order,
                        TinyKeep* keep, hipStream_t s) {
  auto go = [&](auto one, auto four) {
    if (A.n * nrhs <= kTinyThreads)
      hipLaunchKernelGGL(one, dim3(1), dim3(kTinyThreads), 0, s, A, M, B, X, nrhs, R, rtol, it0,
                         it1, max_iter, order, keep);
    else
      hipLaunchKernelGGL(four, dim3(1), dim3(kTinyThreads), 0, s, A, M, B, X, nrhs, R, rtol, it0,
                         it1, max_iter, order, keep);
  };
  constexpr int kFour = kTinyElems / kTinyThreads;
  if (M.beg) go(k_pcg_tiny<MT, LAYA, kLayPad, 1>, k_pcg_tiny<MT, LAYA, kLayPad, kFour>);
  else go(k_pcg_tiny<MT, LAYA, kLayCsr, 1>, k_pcg_tiny<MT, LAYA, kLayCsr, kFour>);
}

// (*declined: nothing has been solved)
static int pcg_tiny(const Mat& A, const Mat& M, int nrhs, const double* B, double* X, double rtol,
                    int max_iter, int* iters, double* relres, const int32_t* order, hipStream_t s,
                    PcgWork* work, bool* declined) {
  DevPool local;
  TinyKeep* keep = nullptr;
  int rc;
  if (work && work->tiny) {
    keep = (TinyKeep*)work->tiny;
  } else {
    DevPool& pool = work ? work->tiny_pool : local;
    if ((rc = pool.alloc(&keep, 1))) return rc;
    if (work) work->tiny = keep;
  }
  int R = 1;
  while (R < nrhs) R <<= 1;
  TinyOut h[kTinyRhs];
  int it0 = 0;
  do {
    const int it1 = max_iter - it0 > kTinyIters ? it0 + kTinyIters : max_iter;
    auto by_a = [&](auto mt) {
      using MT = decltype(mt);
      if (A.eshift >= 0)
        launch_tiny<MT, kLayEll>(A, M, B, X, nrhs, R, rtol, it0, it1, max_iter, order, keep, s);
      else
        launch_tiny<MT, kLayCsr>(A, M, B, X, nrhs, R, rtol, it0, it1, max_iter, order, keep, s);
    };
    if (M.val32) by_a(float{});
    else by_a(double{});
    HIPCHK(hipGetLastError());
    HIPCHK(hipMemcpyAsync(h, keep->out, sizeof(TinyOut) * nrhs, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    it0 = it1;
  } while (h[0].active > 0);
  *declined = h[0].status == kTinyDeclined;
  if (*declined) return SPAI_OK;
  bool indef = false, unconv = false;
  for (int r = 0; r < nrhs; ++r) {
    if (iters) iters[r] = h[r].iters;
    if (relres) relres[r] = h[r].bnorm > 0.0 ? std::sqrt(h[r].rr) / h[r].bnorm : 0.0;
    if (h[r].status == 4) indef = true;
    if (h[r].status == 0) unconv = true;
  }
  return indef ? PCG_INDEFINITE : unconv ? SPAI_MAXITER : SPAI_OK;
}

struct Solver {
  Mat A, M;
  Mat Ag, Mg;                        // A and M as the iterations use them (gated, counted)
  int* runs = nullptr;               // products that did their work, per kind: nactive + 1
  int runs_seen[2] = {0, 0};
  int ctr_host[3] = {0, 0, 0};       // the last host copy of nactive and runs
  int64_t n;
  int nrhs;
  hipStream_t s;
  double *x, *r, *z, *p, *q, *part, *tmp;
  double* p1 = nullptr;              // the second p buffer (up to 64 right-hand sides)
  const double* b;
  RhsState* S;
  int* nactive;
  const int32_t* order = nullptr;   // row visiting order of the products (null: natural)
  // workgroups of the x, p update: 5 per compute unit (20 waves; the 64-right-hand-side solve
  // at 96^3 took 352 ms, against 361 ms with the full 2048 and 363 ms with 3 per unit)
  int pupd_grid = kGrid;
  // products with at most as many workgroups take 1024 threads: with 8 and 16 right-hand sides
  // up to four a compute unit (a solve, 40^3, 16 of them and 1000 workgroups: 6.0 ms against 6.2
  // with 256 threads; 46^3, 8: 5.8 and 6.3), else two (40^3, 32 and 1000: 10.7 and 9.8, a
  // thread's two rows not side by side; 52^3, 4, float32 M and 552: 8.1 and 7.7)
  static constexpr int wide_grid(int R) { return R == 8 || R == 16 ? 1024 : 512; }
  static_assert(kFusedGrid <= 512, "a product of 256 threads takes no reduction's end");
  int* ticket = nullptr;             // of the fused reductions
  // optional timing of the products inside the iterations: HIP events recorded on the
  // solver's stream around each A p (kind 0) and M r (kind 1), read back per chunk
  PcgTiming* timing = nullptr;
  std::vector<hipEvent_t> ev;
  std::vector<int> ev_kind;
  int ev_used = 0;

  // the last workgroup of a launch of nb workgroups finishes its reduction (step as in
  // Finish; part[r * rstep + b * bstep]), where the partials are few
  Finish finish(int step, int64_t nb, int64_t grid, int64_t rstep, int64_t bstep,
                double rtol = 0.0) const {
    Finish f;
    if (step == 2 ? nb * nrhs > kFusedRows : nb * nrhs > kFusedParts || grid > kFusedGrid) return f;
    f.ticket = ticket;
    f.S = S;
    f.nactive = nactive;
    f.step = step;
    f.nrhs = nrhs;
    f.rstep = rstep;
    f.bstep = bstep;
    f.rtol = rtol;
    return f;
  }
  int prod_step = -1;                // the scalar step of the product being launched (-1: none)
  bool prod_done = false;            // its last workgroup takes that step

  // Y = K X with the per-RHS dots (X, Y) reduced into out and the scalar step `step` applied
  // to them in the same launch (0: alpha, 1: beta)
  void timed_spmm(int kind, const Mat& K, const double* X, double* Y, double* out, int step) {
    const bool rec = timing && ev_used + 2 <= (int)ev.size();
    if (rec) (void)hipEventRecord(ev[ev_used], s);
    prod_step = step;
    if (K.val32) spmm_v<float>(K, X, Y, part);
    else spmm_v<double>(K, X, Y, part);
    prod_step = -1;
    if (rec) {
      (void)hipEventRecord(ev[ev_used + 1], s);
      ev_kind[ev_used / 2] = kind;
      ev_used += 2;
    }
    if (!prod_done)
      hipLaunchKernelGGL(k_reduce_rows_step, dim3(nrhs), dim3(kThreads), 0, s, part, spmm_grid, out,
                         S, step, nactive);
    prod_done = false;
  }
  // after a synchronisation: add the recorded product times to the totals
  // (calls: the products that did their work; a product of a solve whose right-hand sides
  // have all stopped returns at once, and its few microseconds stay in the time)
  void collect_timing() {
    for (int i = 0; i + 1 < ev_used; i += 2) {
      float ms = 0.f;
      if (hipEventElapsedTime(&ms, ev[i], ev[i + 1]) == hipSuccess) {
        timing->ms[ev_kind[i / 2]] += ms;
      } else {
        (void)hipGetLastError();
      }
    }
    ev_used = 0;
    for (int k = 0; k < 2; ++k) {
      timing->calls[k] += ctr_host[1 + k] - runs_seen[k];
      runs_seen[k] = ctr_host[1 + k];
    }
  }

  static int pow2(int w) {
    int R = 1;
    while (R < w) R <<= 1;
    return R;
  }

  // workgroups of a product: 8 XCD ranges of ceil(n / 8) positions, kRowsPerWave
  // positions per wave, kThreads / 64 waves per workgroup (blocks of its partials)
  static int spmm_blocks(int64_t n) {
    const int64_t per = (n + 7) / 8, rows = (int64_t)(kThreads / 64) * kRowsPerWave;
    return (int)(8 * ((per + rows - 1) / rows));
  }
  int spmm_grid = 8;

  template <typename VT, int LAY, int R>
  void spmm_narrow(const Mat& K, const double* X, double* Y, double* pt) {
    const int64_t per = (n + 7) / 8;
    spmm_grid = (int)(8 * ((per + narrow_chunk<R>() - 1) / narrow_chunk<R>()));
    Finish f;
    if (prod_step >= 0) f = finish(prod_step, spmm_grid, spmm_grid, spmm_grid, 1);
    prod_done = f.ticket != nullptr;
    if constexpr (R <= kQuadRhs) {
      hipLaunchKernelGGL((k_spmm_quad<VT, LAY, R>), dim3(spmm_grid), dim3(4 * kThreads), 0, s, K, X, Y,
                         pt ? 1 : 0, nrhs, order, pt, f);
    } else if (spmm_grid <= wide_grid(R))
      hipLaunchKernelGGL((k_spmm_narrow<VT, LAY, R, 4>), dim3(spmm_grid), dim3(4 * kThreads), 0, s, K,
                         X, Y, pt ? 1 : 0, nrhs, order, pt, f);
    else
      hipLaunchKernelGGL((k_spmm_narrow<VT, LAY, R, 1>), dim3(spmm_grid), dim3(kThreads), 0, s, K, X,
                         Y, pt ? 1 : 0, nrhs, order, pt, f);
  }
  template <typename VT, int LAY>
  void spmm_as(const Mat& K, const double* X, double* Y, double* pt) {
    switch (nrhs <= 32 ? pow2(nrhs) : 0) {   // few right-hand sides: rows share a wave
      case 1: return spmm_narrow<VT, LAY, 1>(K, X, Y, pt);
      case 2: return spmm_narrow<VT, LAY, 2>(K, X, Y, pt);
      case 4: return spmm_narrow<VT, LAY, 4>(K, X, Y, pt);
      case 8: return spmm_narrow<VT, LAY, 8>(K, X, Y, pt);
      case 16: return spmm_narrow<VT, LAY, 16>(K, X, Y, pt);
      case 32: return spmm_narrow<VT, LAY, 32>(K, X, Y, pt);
      default: break;
    }
    spmm_grid = spmm_blocks(n);
    for (int c0 = 0; c0 < nrhs; c0 += 64) {
      if (nrhs % 2 == 0)   // 16-byte gathers, two rows per wave
        hipLaunchKernelGGL((k_spmm_pair<VT, LAY>), dim3(spmm_grid), dim3(kThreads), 0, s, K, X,
                           Y, pt ? 1 : 0, nrhs, c0, order, pt);
      else
        hipLaunchKernelGGL((k_spmm_wave<VT, LAY>), dim3(spmm_grid), dim3(kThreads), 0, s, K, X,
                           Y, pt ? 1 : 0, nrhs, c0, order, pt);
    }
  }
  template <typename VT>
  void spmm_v(const Mat& K, const double* X, double* Y, double* pt) {
    if (K.eshift >= 0) spmm_as<VT, kLayEll>(K, X, Y, pt);
    else if (K.beg) spmm_as<VT, kLayPad>(K, X, Y, pt);
    else spmm_as<VT, kLayCsr>(K, X, Y, pt);
  }
  // Y = Mat X, and with out set the per-RHS dots (X, Y) reduced into out
  void spmm(const Mat& K, const double* X, double* Y, double* out) {
    if (K.val32) spmm_v<float>(K, X, Y, out ? part : nullptr);
    else spmm_v<double>(K, X, Y, out ? part : nullptr);
    if (out)
      hipLaunchKernelGGL(k_reduce_rows, dim3(nrhs), dim3(kThreads), 0, s, part, spmm_grid, out);
  }

  // workgroups of a pass over the rows, kThreads / R of them at a time: at most kGrid, and
  // none without rows (their partials would be zeros at the end of every sum)
  int row_blocks(int R) const {
    return (int)std::min<int64_t>(kGrid, (n * R + kThreads - 1) / kThreads);
  }

  void dot(const double* Xa, const double* Xb, const double* Xc, double* out) {
    const int nb = row_blocks(pow2(std::min(64, nrhs)));   // of the widest group of columns
    for (int c0 = 0; c0 < nrhs; c0 += 64) {
      const int cw = std::min(64, nrhs - c0);
      const int R = pow2(cw);
      hipLaunchKernelGGL(k_dot_rows, dim3(nb), dim3(kThreads), 0, s, Xa, Xb, Xc, n, nrhs, c0, cw, R,
                         part);
    }
    hipLaunchKernelGGL(k_reduce_parts, dim3(nrhs), dim3(kThreads), 0, s, part, nb, nrhs, out);
  }

  // one PCG iteration; each reduction applies the scalar step that consumes it.  odd:
  // the parity of the iteration's index (p in p1, and x updated for this and the previous)
  void iteration(double rtol, int odd) {
    const dim3 gs((nrhs + 63) / 64), bs(64);
    const bool two = nrhs <= 64;
    double* pc = two && odd ? p1 : p;                          // this iteration's p
    timed_spmm(0, Ag, pc, q, tmp, 0);                         // q = A p, (p, q), alpha
    if (nrhs <= 64) {                                            // r update fused with ||r||^2
      const int nb = row_blocks(pow2(nrhs));
      const int g4 = (nb + 3) / 4;
      const Finish f = finish(2, nb, g4, 1, nrhs, rtol);
      if (f.ticket)
        hipLaunchKernelGGL(k_axpy<4>, dim3(g4), dim3(4 * kThreads), 0, s, r, q, S, n, nrhs, pow2(nrhs),
                           nb, part, nactive, f);
      else
        hipLaunchKernelGGL(k_axpy<1>, dim3(nb), dim3(kThreads), 0, s, r, q, S, n, nrhs, pow2(nrhs), nb,
                           part, nactive, f);
      if (!f.ticket)
        hipLaunchKernelGGL(k_reduce_parts_conv, dim3(nrhs), dim3(kThreads), 0, s, part, nb, nrhs, tmp,
                           S, rtol, nactive);                  // convergence test
    } else {
      hipLaunchKernelGGL(k_axpy_wide, dim3(kGrid), dim3(kThreads), 0, s, r, q, S, n, nrhs);
      dot(r, r, nullptr, tmp);
      hipLaunchKernelGGL(k_conv, gs, bs, 0, s, S, tmp, rtol, nrhs, nactive);
    }
    timed_spmm(1, Mg, r, z, tmp, 1);                          // z = M r, (r, z), beta
    const int ug = std::min(pupd_grid, row_blocks(pow2(std::min(64, nrhs))));
    if (two && !odd)                                             // p1 = z + beta p
      hipLaunchKernelGGL(k_pupd_p, dim3(ug), dim3(kThreads), 0, s, p1, p, z, S, n, nrhs,
                         pow2(nrhs));
    else if (two)                                                // x += both terms, p = z + beta p1
      hipLaunchKernelGGL(k_pupd_x2, dim3(ug), dim3(kThreads), 0, s, p, p1, x, z, S, n,
                         nrhs, pow2(nrhs));
    else
      hipLaunchKernelGGL(k_pupd_wide, dim3(kGrid), dim3(kThreads), 0, s, p, x, z, S, n, nrhs);
  }
};

int upload_csr(DevPool& pool, const HostCsr& h, bool f32, Mat& m, hipStream_t s) {
  int rc;
  int64_t* rp;
  int32_t* c;
  if ((rc = pool.alloc(&rp, h.n + 1)) || (rc = pool.alloc(&c, h.nnz))) return rc;
  HIPCHK(hipMemcpyAsync(rp, h.rowptr.data(), sizeof(int64_t) * (h.n + 1), hipMemcpyHostToDevice, s));
  HIPCHK(hipMemcpyAsync(c, h.col.data(), sizeof(int32_t) * h.nnz, hipMemcpyHostToDevice, s));
  m = Mat{};
  m.n = h.n;
  m.rowptr = rp;
  m.col = c;
  if (f32) {
    std::vector<float> v(h.nnz);
    for (int64_t q = 0; q < h.nnz; ++q) v[q] = (float)h.val[q];
    float* d;
    if ((rc = pool.alloc(&d, h.nnz))) return rc;
    HIPCHK(hipMemcpyAsync(d, v.data(), sizeof(float) * h.nnz, hipMemcpyHostToDevice, s));
    HIPCHK(hipStreamSynchronize(s));
    m.val32 = d;
  } else {
    double* d;
    if ((rc = pool.alloc(&d, h.nnz))) return rc;
    HIPCHK(hipMemcpyAsync(d, h.val.data(), sizeof(double) * h.nnz, hipMemcpyHostToDevice, s));
    m.val = d;
  }
  return SPAI_OK;
}

}  // namespace
}  // namespace spai

using namespace spai;

namespace spai {

int pcg_run(const PcgMat& A, const PcgMat& M, int nrhs, const double* dB, double* dX, double rtol,
            int max_iter, int* iters, double* relres, const int32_t* order, hipStream_t s,
            PcgTiming* timing, PcgWork* work) {
  // (A is ELL or CSR, M padded columns or CSR; the per-product timing wants the launches)
  int rc;
  if (tiny_fits(A.n, nrhs) && !timing && !A.beg && !A.val32 && M.eshift < 0) {
    bool declined = false;
    rc = pcg_tiny(A, M, nrhs, dB, dX, rtol, max_iter, iters, relres, order, s, work, &declined);
    if (rc < 0 || !declined) return rc;
  }
  DevPool local;
  DevPool& pool = work ? work->pool : local;
  Solver S{};
  struct EvGuard {
    std::vector<hipEvent_t>* v;
    ~EvGuard() {
      for (hipEvent_t e : *v) (void)hipEventDestroy(e);
    }
  } evg{&S.ev};
  S.A = A;
  S.M = M;
  S.n = A.n;
  S.nrhs = nrhs;
  S.s = s;
  S.order = order;
  const int64_t tot = S.n * nrhs;
  // every block is initialised or written before it is read in each solve, so kept
  // blocks need no clearing beyond the state reset below
  if (work && work->n == S.n && work->nrhs == nrhs) {
    S.r = (double*)work->blk[0];
    S.z = (double*)work->blk[1];
    S.p = (double*)work->blk[2];
    S.p1 = (double*)work->blk[3];
    S.q = (double*)work->blk[4];
    S.part = (double*)work->blk[5];
    S.tmp = (double*)work->blk[6];
    S.S = (RhsState*)work->blk[7];
    S.nactive = (int*)work->blk[8];
  } else {
    if (work) {
      work->pool.release();
      work->n = -1;
    }
    if ((rc = pool.alloc(&S.r, tot)) || (rc = pool.alloc(&S.z, tot)) || (rc = pool.alloc(&S.p, tot)) ||
        (nrhs <= 64 && (rc = pool.alloc(&S.p1, tot))) ||
        (rc = pool.alloc(&S.q, tot)) ||
        (rc = pool.alloc(&S.part, (int64_t)std::max<int64_t>(kGrid, Solver::spmm_blocks(S.n)) * nrhs)) ||
        (rc = pool.alloc(&S.tmp, nrhs)) || (rc = pool.alloc(&S.S, nrhs)) || (rc = pool.alloc(&S.nactive, 4)))
      return rc;
    if (work) {
      void* const b[9] = {S.r, S.z, S.p, S.p1, S.q, S.part, S.tmp, S.S, S.nactive};
      for (int i = 0; i < 9; ++i) work->blk[i] = b[i];
      work->n = S.n;
      work->nrhs = nrhs;
    }
  }
  S.b = dB;
  S.x = dX;
  {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
        cus > 0)
      S.pupd_grid = 5 * cus;
    else
      (void)hipGetLastError();
  }
  if (timing) {                         // two products per iteration, 8 iterations per chunk
    S.timing = timing;
    S.ev.resize(32, nullptr);
    S.ev_kind.resize(16, 0);
    for (auto& e : S.ev)
      if (hipEventCreate(&e) != hipSuccess) {
        (void)hipGetLastError();
        e = nullptr;
        S.timing = nullptr;
      }
  }
  if (S.timing) S.runs = S.nactive + 1;   // read with the active count in one copy
  S.Ag = S.A;
  S.Mg = S.M;
  S.Ag.gate = S.Mg.gate = S.nactive;
  S.Ag.ran = S.runs;
  S.Mg.ran = S.runs ? S.runs + 1 : nullptr;
  S.ticket = S.nactive + 3;
  HIPCHK(hipMemsetAsync(S.nactive, 0, 4 * sizeof(int), s));
  HIPCHK(hipMemsetAsync(S.S, 0, sizeof(RhsState) * nrhs, s));
  const dim3 gs((nrhs + 63) / 64), bs(64);
  // x_0 = 0, r = b, z = M r, p = z
  hipLaunchKernelGGL(k_fill, dim3(kGrid), dim3(kThreads), 0, s, S.x, 0.0, tot);
  hipLaunchKernelGGL(k_copy, dim3(kGrid), dim3(kThreads), 0, s, S.r, dB, tot);
  S.dot(dB, dB, nullptr, S.tmp);
  hipLaunchKernelGGL(k_init_rhs, gs, bs, 0, s, S.S, S.tmp, nrhs, S.nactive);
  S.spmm(S.M, S.r, S.z, S.tmp);
  hipLaunchKernelGGL(k_set_rz, gs, bs, 0, s, S.S, S.tmp, nrhs);
  hipLaunchKernelGGL(k_copy, dim3(kGrid), dim3(kThreads), 0, s, S.p, S.z, tot);
  HIPCHK(hipGetLastError());
  // iterate in chunks, checking the running count between chunks.  On a stream of
  // its own (not the null stream) and without the per-product timing, a full chunk is
  // captured once as a HIP graph and replayed: every launch of an iteration has fixed
  // arguments, and converged right-hand sides are masked on the device.
  int it = 0;
  const int chunk = 8;
  hipGraph_t graph = nullptr;
  hipGraphExec_t gexec = nullptr;
  struct GraphGuard {
    hipGraph_t* g;
    hipGraphExec_t* e;
    ~GraphGuard() {
      if (*e) (void)hipGraphExecDestroy(*e);
      if (*g) (void)hipGraphDestroy(*g);
    }
  } gguard{&graph, &gexec};
  bool use_graph = s != nullptr && !S.timing;
  while (it < max_iter) {
    HIPCHK(hipMemcpyAsync(S.ctr_host, S.nactive, (S.timing ? 3 : 1) * sizeof(int),
                          hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    if (S.timing) S.collect_timing();
    if (S.ctr_host[0] == 0) break;
    const int k = std::min(chunk, max_iter - it);
    if (use_graph && k == chunk && !gexec) {
      if (hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal) == hipSuccess) {
        for (int t = 0; t < k; ++t) S.iteration(rtol, (it + t) & 1);
        if (hipStreamEndCapture(s, &graph) != hipSuccess ||
            hipGraphInstantiate(&gexec, graph, nullptr, nullptr, 0) != hipSuccess) {
          (void)hipGetLastError();
          if (graph) (void)hipGraphDestroy(graph);
          graph = nullptr;
          gexec = nullptr;
          return fail(SPAI_ERR_HIP, "pcg: capturing the iteration graph failed");
        }
      } else {
        (void)hipGetLastError();
        use_graph = false;
      }
    }
    if (use_graph && k == chunk && gexec) {
      HIPCHK(hipGraphLaunch(gexec, s));
    } else {
      for (int t = 0; t < k; ++t) S.iteration(rtol, (it + t) & 1);
    }
    HIPCHK(hipGetLastError());
    it += k;
  }
  if (nrhs <= 64 && (it & 1))      // the last iteration was even: its x term is pending
    hipLaunchKernelGGL(k_x_flush, dim3(S.pupd_grid), dim3(kThreads), 0, s, S.x, S.p, S.S, S.n, nrhs,
                       Solver::pow2(nrhs));
  // true residual ||b - A x|| / ||b||
  S.spmm(S.A, S.x, S.q, nullptr);
  S.dot(dB, dB, S.q, S.tmp);     // sum (b - Ax)^2
  std::vector<double> rr(nrhs);
  HIPCHK(hipMemcpyAsync(rr.data(), S.tmp, sizeof(double) * nrhs, hipMemcpyDeviceToHost, s));
  std::vector<RhsState> hs(nrhs);
  HIPCHK(hipMemcpyAsync(hs.data(), S.S, sizeof(RhsState) * nrhs, hipMemcpyDeviceToHost, s));
  if (S.timing)
    HIPCHK(hipMemcpyAsync(S.ctr_host, S.nactive, 3 * sizeof(int), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  if (S.timing) S.collect_timing();
  bool indef = false, unconv = false;
  for (int r = 0; r < nrhs; ++r) {
    if (iters) iters[r] = hs[r].iters;
    if (relres) relres[r] = hs[r].bnorm > 0.0 ? std::sqrt(rr[r]) / hs[r].bnorm : 0.0;
    if (hs[r].status == 4) indef = true;
    if (hs[r].status == 0) unconv = true;
  }
  if (indef) return PCG_INDEFINITE;
  if (unconv) return SPAI_MAXITER;
  return SPAI_OK;
}

}  // namespace spai

extern "C" int pcg_solve(const spai_csr_t* A, const spai_csr_t* M, int nrhs, const double* B,
                         double* X, double rtol, int max_iter, int* iters, double* relres,
                         const spai_opts_t* opts) {
  try {
    if (!A || !M || nrhs < 1 || !B || !X || !(rtol >= 0.0) || max_iter < 0)
      return fail(SPAI_ERR_ARG, "pcg_solve: bad arguments");
    int rc;
    HostCsr hA, hM;
    if ((rc = fetch_csr(A, hA)) || (rc = fetch_csr(M, hM))) return rc;
    if (hM.n != hA.n) return fail(SPAI_ERR_ARG, "pcg_solve: A and M differ in size");
    spai_opts_t o;
    spai_default_opts(&o);
    if (opts) o = *opts;
    hipStream_t s = (hipStream_t)o.stream;
    DevPool pool;
    Mat dA, dM;
    if ((rc = upload_csr(pool, hA, false, dA, s))) return rc;
    if ((rc = upload_csr(pool, hM, o.precision == SPAI_PREC_MIXED, dM, s))) return rc;
    const int64_t tot = hA.n * nrhs;
    const double* dB = B;
    double* dX = X;
    if (!A->on_device) {
      double *b2, *x2;
      if ((rc = pool.alloc(&b2, tot)) || (rc = pool.alloc(&x2, tot))) return rc;
      HIPCHK(hipMemcpyAsync(b2, B, sizeof(double) * tot, hipMemcpyHostToDevice, s));
      dB = b2;
      dX = x2;
    }
    std::vector<int32_t> ord;
    locality_order(hA, kBallRows, ord);
    int32_t* d_order;
    if ((rc = pool.alloc(&d_order, hA.n))) return rc;
    HIPCHK(hipMemcpyAsync(d_order, ord.data(), sizeof(int32_t) * hA.n, hipMemcpyHostToDevice, s));
    HIPCHK(hipStreamSynchronize(s));
    rc = pcg_run(dA, dM, nrhs, dB, dX, rtol, max_iter, iters, relres, d_order, s, nullptr);
    if (rc < 0) return rc;
    if (!A->on_device) {
      HIPCHK(hipMemcpyAsync(X, dX, sizeof(double) * tot, hipMemcpyDeviceToHost, s));
      HIPCHK(hipStreamSynchronize(s));
    }
    return rc;
  } catch (const std::bad_alloc&) {
    return fail(SPAI_ERR_NOMEM, "host allocation failed");
  } catch (...) {
    return fail(SPAI_ERR_HIP, "unexpected exception");
  }
}
