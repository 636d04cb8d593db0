// spai_loss.hip — f(M) = ||I - A M||_F^2 (Section 2) on fixed patterns and its adjoint.
//
// With R = I - A M:  df = -2 (R, dA M + A dM)_F, so
//   d f / d A = -2 R M^T   restricted to supp(A),
//   d f / d M = -2 A^T R   restricted to supp(M)   (= -2 A R of Section 2 for symmetric A).
// Neither A M nor R is stored.  Row i of R is rebuilt from the rows of M selected by A's
// row i, which gives f and d f / d A; column j of R is row j of R^T = I - M^T A^T, so the
// same kernel on M^T and A^T (symmetric patterns, values gathered through the transpose
// map) gives d f / d M.  Rows and columns past its tile are left to k_loss_rows and
// k_loss_cols.  One row per 64-lane wavefront, every sum in a fixed order, so the results are
// deterministic.
#include <hip/hip_runtime.h>

#include <map>
#include <mutex>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "spai.h"
#include "spai_dev.hpp"
#include "spai_host.hpp"

namespace spai {
namespace {

// (offsets only, no integer round trip of the pointer, so the compiler still sees
// LDS addresses and emits ds_* instructions rather than flat ones)
struct Carve2 {
  char* base;
  unsigned off = 0;
  __device__ explicit Carve2(char* b) : base(b) {}
  template <typename U> __device__ U* take(int count) {
    off = (off + 7u) & ~7u;
    U* r = (U*)(base + off);
    off += (unsigned)(sizeof(U) * (unsigned)count);
    return r;
  }
};

struct Pat {                    // CSR pattern
  int64_t n;
  const int64_t* rowptr;
  const int32_t* col;
};

// position of (col[q], row(q)) for every stored entry q of a symmetric pattern, in tmap
// and / or the value there, in tval; an entry without its mirror maps to itself and raises
// err bit 2.  Sixteen lanes share a row, so that the binary searches of a row (four or five
// dependent loads) run side by side: 2.4M + 6.6M entries took 158 us a thread per row.
constexpr int kMapLanes = 16;
template <typename T>
__global__ __launch_bounds__(256) void k_transpose(Pat P, int64_t* tmap, const T* val, T* tval,
                                                   int* err) {
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kMapLanes;
  if (i >= P.n) return;
  const int64_t e = P.rowptr[i + 1];
  for (int64_t q = P.rowptr[i] + threadIdx.x % kMapLanes; q < e; q += kMapLanes) {
    const int32_t k = P.col[q];
    int64_t lo = P.rowptr[k];
    const int64_t end = P.rowptr[k + 1];
    int64_t hi = end;
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (P.col[mid] < (int32_t)i) lo = mid + 1; else hi = mid;
    }
    int64_t at = q;
    if (lo < end && P.col[lo] == (int32_t)i) at = lo;
    else atomicOr(err, 2);
    if (tmap) tmap[q] = at;
    if (tval) tval[q] = val[at];
  }
}

__global__ void k_to_f32(const double* a, float* b, int64_t nnz) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < nnz) b[q] = (float)a[q];
}

// Row i of I - X Y, with X and Y in CSR: rowpart[i] = ||row||^2 and, with gX set,
// gX[q] = -2 dL (row) . (row col(q) of Y) for the entries q of X's row i.  (A, M) gives f and
// d f / d A; (M^T, A^T) gives d f / d M, X's values read and gX written through xmap (MAP).
//
// One wave per row.  The rows of Y that X's row selects are taken G lanes each (G = 16, 32
// or 64, the first that holds the longest), 64 / G rows a round, at most kLossRounds rounds
// held in registers: every load of a row is in flight together.  Their columns are mapped to
// cells without clashes (no probing); the first entry of each cell, in the order of rounds and
// lanes, takes the next rank, so the ranks do not depend on the order of the writes.  The
// products are added into per-rank sums in LDS, one row of Y per lane group a round (distinct
// columns, so distinct ranks), each group with sums of its own that are added last.  The row
// of R then stays in LDS for the gradients, one group sum per entry of X.  Descriptors are
// loaded one and two rows ahead.
// Bound by instruction issue and LDS latency at 17 waves per compute unit (9 KB of LDS).
// 512 x 512 nine-point graph, M on pattern(A^2) (9 rows of 25 entries, and 25 of 9): 290 us
// for the value and with d f / d A, 469 us for d f / d M.  One instance per number of rounds
// (297 and 486, at four waves per SIMD), against 405 and 622 with every round tested for and
// 455 and 668 with sums over the wave through the LDS pipe as well; with the columns in an
// ordered hash set 463 and 678; with binary searches in a 19 KB tile (8 waves per compute
// unit) and an LDS sort 2600 and 2800.
// A row outside this (more than 64 entries in X's row or a row of Y, more rounds or more
// distinct columns than there is room for, a clash under every multiplier) is marked
// rowpart[i] = -1 and left to k_loss_rows, or to k_loss_cols (MAP).
constexpr int kLossRounds = 8;
constexpr int kLossSums = 512;      // per-rank sums of all groups
constexpr int kLossEntries = 509;   // entries of the selected rows together (the left tiers' limit)
constexpr double kLossLeft = -1.0;  // rowpart of a row left to the larger tiles

template <typename T, bool MAP>
__global__ __launch_bounds__(SPAI_WAVE) __attribute__((amdgpu_waves_per_eu(5))) void k_loss_lean(Pat X, const T* Xv, const int64_t* xmap,
                                                         Pat Y, const T* Yv, double* rowpart,
                                                         double* gX, double dL) {
  // a lane without an entry in a round works on a place of its own behind the tables, so the
  // rounds need no branches
  __shared__ int cell[kBtCells + SPAI_WAVE];      // column, then first entry, then rank
  __shared__ double sums[kLossSums + SPAI_WAVE];
  const int lane = lane_id();
  ColumnWalk w(X.n, blockIdx.x, gridDim.x);
  struct Row {
    int64_t qa = 0, yb = 0;
    int deg = 0, l = -1, len = 0;
    T a = (T)0;
  };
  auto ends = [&](int64_t i, Row& r) {            // the row's range in X
    r = Row{};
    if (i < w.end) {
      r.qa = X.rowptr[i];
      r.deg = (int)min<int64_t>(X.rowptr[i + 1] - r.qa, INT_MAX);
    }
  };
  auto entries = [&](Row& r) {                    // its entries, one per lane
    if (lane < r.deg) {
      r.l = X.col[r.qa + lane];
      r.a = MAP ? Xv[xmap[r.qa + lane]] : Xv[r.qa + lane];
    }
  };
  auto spans = [&](Row& r) {                      // where their rows of Y sit
    if (r.l >= 0) {
      r.yb = Y.rowptr[r.l];
      r.len = (int)min<int64_t>(Y.rowptr[r.l + 1] - r.yb, INT_MAX / SPAI_WAVE);
    }
  };
  Row cur, nxt;
  ends(w.begin, cur);
  entries(cur);
  spans(cur);
  ends(w.begin + w.step, nxt);
  for (int64_t i = w.begin; i < w.end; i += w.step) {
    entries(nxt);
    Row far;
    ends(i + 2 * w.step, far);
    // the rows of Y, G = 2^lg lanes each
    const int lg = __ballot(cur.len > 32) ? 6 : __ballot(cur.len > 16) ? 5 : 4;
    const int groups = SPAI_WAVE >> lg;
    int rounds = (cur.deg + groups - 1) >> (6 - lg);
    const int cap = kLossSums >> (6 - lg);                       // ranks a group has room for
    const int g = lane >> lg, e = lane & ((1 << lg) - 1);
    const double av = (double)cur.a;
    bool left = cur.deg > SPAI_WAVE || rounds > kLossRounds || __ballot(cur.len > SPAI_WAVE);
    if (!left && (cur.deg << lg) > kLossEntries) left = wave_sum_int(cur.len) > kLossEntries;
    if (left) rounds = 0;                         // marked below
    // one instance per number of rounds: no round is tested for
    auto work = [&](auto rc) {
      constexpr int RR = decltype(rc)::value;
      int c[RR];
      T v[RR];
#pragma unroll
      for (int r = 0; r < RR; ++r) {
        const int t = (r << (6 - lg)) + g;                       // at most 63
        const int64_t yb = __shfl(cur.yb, t, SPAI_WAVE);
        const int len = __shfl(cur.len, t, SPAI_WAVE);           // 0 past the row's entries
        c[r] = -1;
        v[r] = (T)0;
        if (e < len) {
          c[r] = Y.col[yb + e];
          v[r] = Yv[yb + e];
        }
      }
      spans(nxt);
      // an entry's cell, then the place of its sum
      int at[RR];
      int a = 0;
      for (; a < kBtMuls; ++a) {
        const unsigned m = bt_mul(a);
        const int own = (int)bt_cell((int)i, m);
#pragma unroll
        for (int r = 0; r < RR; ++r) {
          at[r] = c[r] >= 0 ? (int)bt_cell(c[r], m) : kBtCells + lane;
          cell[at[r]] = c[r];
        }
        cell[own] = (int)i;                       // the same word from every lane
        __syncthreads();
        bool clash = cell[own] != (int)i;
#pragma unroll
        for (int r = 0; r < RR; ++r) clash |= cell[at[r]] != c[r];
        __syncthreads();
        if (__ballot(clash) == 0ull) {
#pragma unroll
          for (int r = 0; r < RR; ++r) cell[at[r]] = INT_MAX;
          __syncthreads();
          cell[own] = 0;                          // rank 0: the row's own column i
          break;
        }
      }
      if (a == kBtMuls) return false;
      __syncthreads();
#pragma unroll
      for (int r = 0; r < RR; ++r) atomicMin(&cell[at[r]], 1 + r * SPAI_WAVE + lane);
      __syncthreads();
      int mine[RR], nk = 1;
#pragma unroll
      for (int r = 0; r < RR; ++r) {
        const bool first = c[r] >= 0 && cell[at[r]] == 1 + r * SPAI_WAVE + lane;
        const unsigned long long bal = __ballot(first);
        mine[r] = first ? nk + __popcll(bal & lanemask_lt()) : -1;
        nk += __popcll(bal);
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < RR; ++r) cell[mine[r] >= 0 ? at[r] : kBtCells + lane] = mine[r];
      __syncthreads();
#pragma unroll
      for (int r = 0; r < RR; ++r) {
        const int rk = cell[at[r]];
        at[r] = c[r] >= 0 ? g * cap + rk : kLossSums + lane;
      }
      if (nk > cap) return false;
      for (int q = 0; q < groups; ++q)
        for (int k = lane; k < nk; k += SPAI_WAVE) sums[q * cap + k] = 0.0;
      __syncthreads();
      double av_v[RR];
#pragma unroll
      for (int r = 0; r < RR; ++r)
        av_v[r] = __shfl(av, (r << (6 - lg)) + g, SPAI_WAVE) * (double)v[r];
#pragma unroll
      for (int r = 0; r < RR; ++r) {
        sums[at[r]] += av_v[r];
        wave_sync();                              // the next round may add to it from another lane
      }
      __syncthreads();
      double acc = 0.0;
      for (int k = lane; k < nk; k += SPAI_WAVE) {
        double s = sums[k];
        if (groups >= 2) s += sums[cap + k];
        if (groups == 4) s += sums[2 * cap + k] + sums[3 * cap + k];
        const double rho = (k == 0 ? 1.0 : 0.0) - s;
        sums[k] = rho;
        acc += rho * rho;
      }
      acc = wave_sum(acc);
      if (lane == 0) rowpart[i] = acc;
      __syncthreads();
      if (gX) {
        double p[RR];
#pragma unroll
        for (int r = 0; r < RR; ++r) {
          const double rho = sums[c[r] >= 0 ? at[r] - g * cap : 0];
          p[r] = c[r] >= 0 ? rho * (double)v[r] : 0.0;
        }
        if (lg == 6)
#pragma unroll
          for (int r = 0; r < RR; ++r) p[r] = lane_xor_add<32>(p[r]);
        if (lg >= 5)
#pragma unroll
          for (int r = 0; r < RR; ++r) p[r] = lane_xor_add<16>(p[r]);
#pragma unroll
        for (int r = 0; r < RR; ++r) p[r] = lane_xor_add<8>(p[r]);
#pragma unroll
        for (int r = 0; r < RR; ++r) p[r] = lane_xor_add<4>(p[r]);
#pragma unroll
        for (int r = 0; r < RR; ++r) p[r] = lane_xor_add<2>(p[r]);
#pragma unroll
        for (int r = 0; r < RR; ++r) p[r] = lane_xor_add<1>(p[r]);
#pragma unroll
        for (int r = 0; r < RR; ++r) {
          const int t = (r << (6 - lg)) + g;
          if (e == 0 && t < cur.deg) {
            const int64_t q = cur.qa + t;
            gX[MAP ? xmap[q] : q] = -2.0 * dL * p[r];
          }
        }
        __syncthreads();
      }
      return true;
    };
    bool done = false;
    switch (rounds) {
      case 1: done = work(std::integral_constant<int, 1>{}); break;
      case 2: done = work(std::integral_constant<int, 2>{}); break;
      case 3: done = work(std::integral_constant<int, 3>{}); break;
      case 4: done = work(std::integral_constant<int, 4>{}); break;
      case 5: done = work(std::integral_constant<int, 5>{}); break;
      case 6: done = work(std::integral_constant<int, 6>{}); break;
      case 7: done = work(std::integral_constant<int, 7>{}); break;
      case 8: done = work(std::integral_constant<int, 8>{}); break;
      default: spans(nxt);                        // no entries, or more than this kernel takes
    }
    if (!done && lane == 0) rowpart[i] = kLossLeft;
    cur = nxt;
    nxt = far;
  }
}

// body(i) for the rows that k_loss_lean left (rowpart[i] = kLossLeft), walked as it walks them:
// 64 of a workgroup's rows are looked at together
template <typename F>
__device__ __forceinline__ void left_rows(int64_t n, const double* rowpart, F body) {
  ColumnWalk w(n, blockIdx.x, gridDim.x);
  for (int64_t i0 = w.begin; i0 < w.end; i0 += SPAI_WAVE * w.step) {
    const int64_t i = i0 + lane_id() * w.step;
    const bool mine = i < w.end && rowpart[i] == kLossLeft;
    for (unsigned long long m = __ballot(mine); m; m &= m - 1)
      body(i0 + (int64_t)(__ffsll((long long)m) - 1) * w.step);
  }
}

// The rows of I - X Y that k_loss_lean left, in a larger LDS tile: sorted
// keys, and the sums pulled with binary searches.  Up to DG entries in X's row and
// L, H / 2 - 2 entries of Y; a row beyond that raises err bit 1.
template <typename T>
__global__ __launch_bounds__(SPAI_WAVE) void k_loss_rows(Pat X, const T* Xv, Pat Y, const T* Yv,
                                                         double* rowpart, double* gX, double dL,
                                                         int* err, int L, int H, int DG) {
  extern __shared__ char smem[];
  Carve2 cv(smem);
  int* s_li = cv.take<int>(L);
  int* s_keys = cv.take<int>(H);
  int* s_sorted = cv.take<int>(H);
  int* s_off = cv.take<int>(DG + 1);
  double* s_lv = cv.take<double>(L);
  double* s_a = cv.take<double>(DG);
  double* s_rho = cv.take<double>(H / 2);
  const int lane = lane_id();
  auto body = [&](int64_t i) {
    const int64_t qa = X.rowptr[i];
    const int deg = (int)(X.rowptr[i + 1] - qa);
    int ltot = 0;
    for (int t = lane; t < deg; t += SPAI_WAVE) {
      const int l = X.col[qa + t];
      ltot += (int)(Y.rowptr[l + 1] - Y.rowptr[l]);
    }
    ltot = wave_sum_int(ltot);
    if (deg > DG || ltot > L || ltot + 2 >= H / 2) {
      if (lane == 0) atomicOr(err, 1);
      return;
    }
    int run = 0;
    for (int base = 0; base < deg; base += SPAI_WAVE) {
      const int t = base + lane;
      int len = 0;
      if (t < deg) {
        const int l = X.col[qa + t];
        len = (int)(Y.rowptr[l + 1] - Y.rowptr[l]);
        s_a[t] = (double)Xv[qa + t];
      }
      const int inc = wave_incl_scan(len);
      if (t < deg) s_off[t] = run + inc - len;
      run += wave_last(inc);
    }
    if (lane == 0) s_off[deg] = run;
    __syncthreads();
    for (int t = 0; t < deg; ++t) {
      const int l = X.col[qa + t];
      const int64_t b = Y.rowptr[l];
      const int len = s_off[t + 1] - s_off[t];
      for (int e = lane; e < len; e += SPAI_WAVE) {
        s_li[s_off[t] + e] = Y.col[b + e];
        s_lv[s_off[t] + e] = (double)Yv[b + e];
      }
    }
    ks_clear(s_keys, H);
    __syncthreads();
    if (lane == 0) ks_insert(s_keys, H, (int)i);
    for (int e = lane; e < ltot; e += SPAI_WAVE) ks_insert(s_keys, H, s_li[e]);
    __syncthreads();
    const int nk = ks_sorted(s_keys, H, s_sorted);
    __syncthreads();
    double acc = 0.0;
    for (int t0 = lane; t0 < nk; t0 += SPAI_WAVE) {
      const int j = s_sorted[t0];
      double s = 0.0;
      for (int t = 0; t < deg; ++t) {
        const int o = s_off[t];
        const int e = bsearch_idx(s_li + o, s_off[t + 1] - o, j);
        if (e >= 0) s += s_a[t] * s_lv[o + e];
      }
      const double rho = ((j == (int)i) ? 1.0 : 0.0) - s;
      s_rho[t0] = rho;
      acc += rho * rho;
    }
    acc = wave_sum(acc);
    if (lane == 0) rowpart[i] = acc;
    __syncthreads();
    if (gX) {
      for (int t = 0; t < deg; ++t) {
        const int o = s_off[t];
        const int len = s_off[t + 1] - o;
        double g = 0.0;
        for (int e = lane; e < len; e += SPAI_WAVE) {
          const int pos = bsearch_idx(s_sorted, nk, s_li[o + e]);
          g += s_rho[pos] * s_lv[o + e];
        }
        g = wave_sum(g);
        if (lane == 0) gX[qa + t] = -2.0 * dL * g;
      }
    }
    __syncthreads();
  };
  left_rows(X.n, rowpart, body);
}

// The columns of the gradient in M that k_loss_lean left: column j of R = I - A M is pulled
// over the rows of A that its support selects, against the entries of m_j in LDS, and so is
// -2 (A^T R)(k, j) for the rows k of m_j -- a search in m_j or in the column's rows per entry
// of A, where k_loss_rows on M^T would search every row of A for each of the column's rows,
// and take a sum over the wave per entry of M.  Up to L entries in m_j that select at most
// H / 2 - 3 of A; beyond, err bit 1.  Seven-point 40^3, M on pattern(A^3) (63 entries a column):
// gradient in M 9.1 ms by k_loss_rows, 1.6 so; nine-point 256^2, pattern(A^3) (49), 7.2
// and 1.35.
template <typename T>
__global__ __launch_bounds__(SPAI_WAVE) void k_loss_cols(Pat A, const T* Av, const T* Atv, Pat M,
                                                         const T* Mv, const int64_t* tmap,
                                                         const double* rowpart, double* gM,
                                                         double dL, int* err, int L, int H) {
  extern __shared__ char smem[];
  Carve2 cv(smem);
  int* s_mi = cv.take<int>(L);
  int* s_pre = cv.take<int>(L);
  int* s_keys = cv.take<int>(H);
  int* s_sorted = cv.take<int>(H);
  double* s_mv = cv.take<double>(L);
  double* s_r = cv.take<double>(H / 2);
  const int lane = lane_id();
  left_rows(M.n, rowpart, [&](int64_t j) {
    const int64_t mb = M.rowptr[j];
    const int64_t lm64 = M.rowptr[j + 1] - mb;      // column j of M: row j, the pattern is symmetric
    if (lm64 > L) {
      if (lane == 0) atomicOr(err, 1);
      return;
    }
    const int lm = (int)lm64;
    for (int e = lane; e < lm; e += SPAI_WAVE) {
      s_mi[e] = M.col[mb + e];
      s_mv[e] = (double)Mv[tmap[mb + e]];           // M(l, j)
    }
    __syncthreads();
    // the entries of A in the rows l of m_j, numbered through their prefix
    int run = 0;
    for (int base = 0; base < lm; base += SPAI_WAVE) {
      const int e = base + lane;
      int d = 0;
      if (e < lm) d = (int)min<int64_t>(A.rowptr[s_mi[e] + 1] - A.rowptr[s_mi[e]], H);
      const int inc = wave_incl_scan(d);
      if (e < lm) s_pre[e] = run + inc;
      run += wave_last(inc);
    }
    if (run + 2 >= H / 2) {
      if (lane == 0) atomicOr(err, 1);
      __syncthreads();
      return;
    }
    ks_clear(s_keys, H);
    __syncthreads();
    if (lane == 0) ks_insert(s_keys, H, (int)j);
    for (int p = lane; p < run; p += SPAI_WAVE) {
      const int e = upper_bound_int(s_pre, lm, p);
      const int before = e ? s_pre[e - 1] : 0;
      ks_insert(s_keys, H, A.col[A.rowptr[s_mi[e]] + (p - before)]);
    }
    __syncthreads();
    const int nu = ks_sorted(s_keys, H, s_sorted);
    __syncthreads();
    for (int t = lane; t < nu; t += SPAI_WAVE) {
      const int u = s_sorted[t];
      double s = 0.0;
      for (int64_t q = A.rowptr[u]; q < A.rowptr[u + 1]; ++q) {
        const int e = bsearch_idx(s_mi, lm, A.col[q]);
        if (e >= 0) s += (double)Av[q] * s_mv[e];
      }
      s_r[t] = ((u == (int)j) ? 1.0 : 0.0) - s;
    }
    __syncthreads();
    for (int e = lane; e < lm; e += SPAI_WAVE) {
      const int k = s_mi[e];
      double g = 0.0;
      for (int64_t q = A.rowptr[k]; q < A.rowptr[k + 1]; ++q) {
        const int pos = bsearch_idx(s_sorted, nu, A.col[q]);
        if (pos >= 0) g += (double)Atv[q] * s_r[pos];   // A(u, k) R(u, j), u = col q
      }
      gM[tmap[mb + e]] = -2.0 * dL * g;
    }
    __syncthreads();
  });
}

__global__ void k_sum_parts(const double* part, int64_t n, double* out) {
  __shared__ double sh[256];
  double acc = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 256) acc += part[i];
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sh[0];
}

__global__ void k_sum_chunks(const double* part, int64_t n, int64_t chunk, double* out) {
  __shared__ double sh[256];
  const int64_t lo = (int64_t)blockIdx.x * chunk;
  const int64_t hi = lo + chunk < n ? lo + chunk : n;
  double acc = 0.0;
  for (int64_t i = lo + threadIdx.x; i < hi; i += 256) acc += part[i];
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = sh[0];
}

constexpr int kGridRows = 256 * 17;       // k_loss_lean: the one-wave workgroups that fit (LDS)
constexpr int kGridLeft = 2048;
constexpr int kLeftL = 512, kLeftH = 1024, kLeftDeg = 64;   // k_loss_rows
constexpr int kColsL = 256;                                 // k_loss_cols: entries in a column of M

// row sums of I - A M, with gA the gradient in A
template <typename T>
void launch_rows(const Pat& A, const T* Av, const Pat& M, const T* Mv, double* rowpart, double* gA,
                 double dL, int* err, hipStream_t s) {
  hipLaunchKernelGGL((k_loss_lean<T, false>), dim3(kGridRows), dim3(SPAI_WAVE), 0, s, A, Av,
                     (const int64_t*)nullptr, M, Mv, rowpart, gA, dL);
  const size_t lds = (size_t)kLeftL * 4 + (size_t)kLeftH * 8 + (size_t)(kLeftDeg + 1) * 4 +
                     (size_t)kLeftL * 8 + (size_t)kLeftDeg * 8 + (size_t)(kLeftH / 2) * 8 + 64;
  hipLaunchKernelGGL((k_loss_rows<T>), dim3(kGridLeft), dim3(SPAI_WAVE), lds, s, A, Av, M, Mv, rowpart,
                     gA, dL, err, kLeftL, kLeftH, kLeftDeg);
}
// the gradient in M: the rows of R^T = I - M^T A^T (tmap: M's transpose map, Atv: A^T's values)
template <typename T>
void launch_cols(const Pat& A, const T* Av, const T* Atv, const Pat& M, const T* Mv,
                 const int64_t* tmap, double* rowpart, double* gM, double dL, int* err,
                 hipStream_t s) {
  hipLaunchKernelGGL((k_loss_lean<T, true>), dim3(kGridRows), dim3(SPAI_WAVE), 0, s, M, Mv, tmap, A, Atv,
                     rowpart, gM, dL);
  const size_t lds = (size_t)kColsL * 8 + (size_t)kLeftH * 8 + (size_t)kColsL * 8 +
                     (size_t)(kLeftH / 2) * 8 + 64;
  hipLaunchKernelGGL((k_loss_cols<T>), dim3(kGridLeft), dim3(SPAI_WAVE), lds, s, A, Av, Atv, M, Mv, tmap,
                     rowpart, gM, dL, err, kColsL, kLeftH);
}

struct LossCall {
  DevPool pool;
  Pat pA{}, pM{};
  const double* Av64 = nullptr;
  const double* Mv64 = nullptr;
  hipStream_t s = nullptr;
  int64_t nnzA = 0, nnzM = 0;
  int* err = nullptr;

  int load(const spai_csr_t* A, const spai_csr_t* M, const spai_opts_t* opts, bool check_pat) {
    int rc;
    if (!A || !M || A->n != M->n || A->n < 1) return fail(SPAI_ERR_ARG, "loss: bad shapes");
    spai_opts_t o;
    spai_default_opts(&o);
    if (opts) o = *opts;
    s = (hipStream_t)o.stream;
    nnzA = A->nnz;
    nnzM = M->nnz;
    if (check_pat || !A->on_device) {
      HostCsr hA, hM;
      if ((rc = fetch_csr(A, hA)) || (rc = fetch_csr(M, hM))) return rc;
      if (check_pat && ((rc = check_symmetric_pattern(hA)) || (rc = check_symmetric_pattern(hM))))
        return rc;
      if (!A->on_device) return upload(hA, hM);
    }
    pA = Pat{A->n, A->rowptr, A->colind};
    pM = Pat{M->n, M->rowptr, M->colind};
    Av64 = A->val;
    Mv64 = M->val;
    return SPAI_OK;
  }

  // the call's scratch, one block with the error flag in front (an allocation and its release
  // cost 30 to 400 us): `bytes` behind 256
  int scratch(char** p, size_t bytes) {
    int rc = pool.alloc(p, (int64_t)(256 + bytes));
    if (rc) return rc;
    err = (int*)*p;
    *p += 256;
    HIPCHK(hipMemsetAsync(err, 0, sizeof(int), s));
    return SPAI_OK;
  }

  int upload(const HostCsr& hA, const HostCsr& hM) {
    int rc;
    int64_t *ra, *rm;
    int32_t *ca, *cm;
    double *va, *vm;
    if ((rc = pool.alloc(&ra, hA.n + 1)) || (rc = pool.alloc(&ca, hA.nnz)) || (rc = pool.alloc(&va, hA.nnz)) ||
        (rc = pool.alloc(&rm, hM.n + 1)) || (rc = pool.alloc(&cm, hM.nnz)) || (rc = pool.alloc(&vm, hM.nnz)))
      return rc;
    HIPCHK(hipMemcpyAsync(ra, hA.rowptr.data(), 8 * (hA.n + 1), hipMemcpyHostToDevice, s));
    HIPCHK(hipMemcpyAsync(ca, hA.col.data(), 4 * hA.nnz, hipMemcpyHostToDevice, s));
    HIPCHK(hipMemcpyAsync(va, hA.val.data(), 8 * hA.nnz, hipMemcpyHostToDevice, s));
    HIPCHK(hipMemcpyAsync(rm, hM.rowptr.data(), 8 * (hM.n + 1), hipMemcpyHostToDevice, s));
    HIPCHK(hipMemcpyAsync(cm, hM.col.data(), 4 * hM.nnz, hipMemcpyHostToDevice, s));
    HIPCHK(hipMemcpyAsync(vm, hM.val.data(), 8 * hM.nnz, hipMemcpyHostToDevice, s));
    pA = Pat{hA.n, ra, ca};
    pM = Pat{hM.n, rm, cm};
    Av64 = va;
    Mv64 = vm;
    return SPAI_OK;
  }
};

// the float32 copies of the values (at `at`, value_bytes of the call's scratch), or the values
template <typename T>
size_t value_bytes(const LossCall& c) {
  return sizeof(T) == 8 ? 0 : sizeof(T) * (size_t)(c.nnzA + c.nnzM);
}
template <typename T>
void values(LossCall& c, char* at, const T** Av, const T** Mv) {
  if constexpr (sizeof(T) == 8) {
    *Av = (const T*)c.Av64;
    *Mv = (const T*)c.Mv64;
  } else {
    T *a = (T*)at, *m = a + c.nnzA;
    if (c.nnzA)
      hipLaunchKernelGGL(k_to_f32, dim3((unsigned)((c.nnzA + 255) / 256)), dim3(256), 0, c.s, c.Av64, a, c.nnzA);
    if (c.nnzM)
      hipLaunchKernelGGL(k_to_f32, dim3((unsigned)((c.nnzM + 255) / 256)), dim3(256), 0, c.s, c.Mv64, m, c.nnzM);
    *Av = a;
    *Mv = m;
  }
}

template <typename T>
int loss_fwd_t(LossCall& c, double* Lout) {
  int rc;
  const T *Av, *Mv;
  char* blk;
  const int nch = 512;
  const size_t n8 = sizeof(double) * (size_t)(c.pA.n + nch + 1);
  if ((rc = c.scratch(&blk, n8 + value_bytes<T>(c)))) return rc;
  double *rowpart = (double*)blk, *chunks = rowpart + c.pA.n, *out = chunks + nch;
  values<T>(c, blk + n8, &Av, &Mv);
  launch_rows<T>(c.pA, Av, c.pM, Mv, rowpart, nullptr, 1.0, c.err, c.s);
  HIPCHK(hipGetLastError());
  const int64_t chunk = (c.pA.n + nch - 1) / nch;
  const int nb = (int)((c.pA.n + chunk - 1) / chunk);
  hipLaunchKernelGGL(k_sum_chunks, dim3(nb), dim3(256), 0, c.s, rowpart, c.pA.n, chunk, chunks);
  hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(256), 0, c.s, chunks, (int64_t)nb, out);
  int herr = 0;
  HIPCHK(hipMemcpyAsync(Lout, out, sizeof(double), hipMemcpyDeviceToHost, c.s));
  HIPCHK(hipMemcpyAsync(&herr, c.err, sizeof(int), hipMemcpyDeviceToHost, c.s));
  HIPCHK(hipStreamSynchronize(c.s));
  if (herr) return fail(SPAI_ERR_CAPACITY, "loss: a row or column exceeded the per-column tile");
  return SPAI_OK;
}

template <typename T>
int loss_bwd_t(LossCall& c, double dL, double* gA, double* gM, bool host_out) {
  int rc;
  const T *Av, *Mv;
  double *dgA = gA, *dgM = gM;
  char* blk;                            // row sums, and for gM the transpose map of M and A^T's values
  const size_t n8 = sizeof(double) * (size_t)c.pA.n;
  const size_t m8 = gM ? sizeof(int64_t) * (size_t)c.nnzM : 0, a8 = gM ? sizeof(T) * (size_t)c.nnzA : 0;
  if ((rc = c.scratch(&blk, n8 + m8 + a8 + value_bytes<T>(c)))) return rc;
  double* rowpart = (double*)blk;
  int64_t* tM = (int64_t*)(blk + n8);
  T* Atv = (T*)(blk + n8 + m8);
  values<T>(c, blk + n8 + m8 + a8, &Av, &Mv);
  if (host_out) {
    if (gA && (rc = c.pool.alloc(&dgA, c.nnzA))) return rc;
    if (gM && (rc = c.pool.alloc(&dgM, c.nnzM))) return rc;
  }
  if (gA) launch_rows<T>(c.pA, Av, c.pM, Mv, rowpart, dgA, dL, c.err, c.s);
  if (gM) {
    const int64_t lanes = c.pA.n * kMapLanes;
    const dim3 grid((unsigned)((lanes + 255) / 256)), bs(256);
    hipLaunchKernelGGL(k_transpose<T>, grid, bs, 0, c.s, c.pA, (int64_t*)nullptr, Av, Atv, c.err);
    hipLaunchKernelGGL(k_transpose<T>, grid, bs, 0, c.s, c.pM, tM, (const T*)nullptr, (T*)nullptr,
                       c.err);
    launch_cols<T>(c.pA, Av, Atv, c.pM, Mv, tM, rowpart, dgM, dL, c.err, c.s);
  }
  HIPCHK(hipGetLastError());
  int herr = 0;
  HIPCHK(hipMemcpyAsync(&herr, c.err, sizeof(int), hipMemcpyDeviceToHost, c.s));
  if (host_out) {
    if (gA) HIPCHK(hipMemcpyAsync(gA, dgA, 8 * c.nnzA, hipMemcpyDeviceToHost, c.s));
    if (gM) HIPCHK(hipMemcpyAsync(gM, dgM, 8 * c.nnzM, hipMemcpyDeviceToHost, c.s));
  }
  HIPCHK(hipStreamSynchronize(c.s));
  if (herr & 2) return fail(SPAI_ERR_ARG, "loss: the pattern of A or M is not symmetric");
  if (herr) return fail(SPAI_ERR_CAPACITY, "loss: a row or column exceeded the per-column tile");
  return SPAI_OK;
}

// ---- allocation-free forward loss ---------------------------------------------------
// Scratch of spai_loss_fwd_noalloc: the per-row partial sums (at most kNoAllocRows rows)
// and the chunk sums of the fixed-order reduction, in a file-scope device array (each
// GPU holds its own copy until the process ends).  Host code never passes the array's
// name to a kernel: it takes the array's device address from hipGetSymbolAddress, once
// per device, and uses that address.
constexpr int64_t kNoAllocRows = (int64_t)1 << 21;
constexpr int kNoAllocChunks = 512;
__device__ __align__(256) double scratch[kNoAllocRows + kNoAllocChunks];

std::mutex g_scratch_mu;
std::map<int, double*> g_scratch_ptr;   // device -> address of its scratch array

int noalloc_scratch(double** out) {
  int dev = 0;
  HIPCHK(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  auto it = g_scratch_ptr.find(dev);
  if (it == g_scratch_ptr.end()) {
    void* p = nullptr;
    HIPCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    it = g_scratch_ptr.emplace(dev, (double*)p).first;
  }
  *out = it->second;
  return SPAI_OK;
}

__global__ void k_zero_flag(int* p) { *p = 0; }

}  // namespace
}  // namespace spai

using namespace spai;

extern "C" int spai_loss_fwd(const spai_csr_t* A, const spai_csr_t* M, double* L,
                             const spai_opts_t* opts) {
  try {
    if (!L) return fail(SPAI_ERR_ARG, "loss: null output");
    LossCall c;
    int rc = c.load(A, M, opts, false);
    if (rc) return rc;
    const bool f32 = opts && opts->precision == SPAI_PREC_MIXED;
    return f32 ? loss_fwd_t<float>(c, L) : loss_fwd_t<double>(c, L);
  } catch (...) {
    return fail(SPAI_ERR_HIP, "unexpected exception");
  }
}

extern "C" int spai_loss_bwd(const spai_csr_t* A, const spai_csr_t* M, double dL, double* gA,
                             double* gM, const spai_opts_t* opts) {
  try {
    LossCall c;
    int rc = c.load(A, M, opts, false);
    if (rc) return rc;
    const bool f32 = opts && opts->precision == SPAI_PREC_MIXED;
    const bool host_out = !A->on_device;
    return f32 ? loss_bwd_t<float>(c, dL, gA, gM, host_out) : loss_bwd_t<double>(c, dL, gA, gM, host_out);
  } catch (...) {
    return fail(SPAI_ERR_HIP, "unexpected exception");
  }
}

extern "C" int spai_loss_fwd_noalloc(const spai_csr_t* A, const spai_csr_t* M, double* L, int* err,
                                     const spai_opts_t* opts) {
  try {
    if (!A || !M || !L || !err) return fail(SPAI_ERR_ARG, "loss_fwd_noalloc: null argument");
    if (A->n != M->n || A->n < 1) return fail(SPAI_ERR_ARG, "loss_fwd_noalloc: bad shapes");
    if (!A->on_device || !M->on_device)
      return fail(SPAI_ERR_ARG, "loss_fwd_noalloc: A and M must be on the device");
    if (A->n > kNoAllocRows)
      return fail(SPAI_ERR_ARG, "loss_fwd_noalloc: more than 2^21 rows (the scratch holds 2^21)");
    if (opts && opts->precision != SPAI_PREC_F64)
      return fail(SPAI_ERR_ARG, "loss_fwd_noalloc: float64 only (the float32 copies would need "
                                "scratch of the matrices' size)");
    hipStream_t s = opts ? (hipStream_t)opts->stream : nullptr;
    double* scr = nullptr;
    int rc = noalloc_scratch(&scr);
    if (rc) return rc;
    double* rowpart = scr;
    double* chunks = scr + kNoAllocRows;
    const Pat pA{A->n, A->rowptr, A->colind}, pM{M->n, M->rowptr, M->colind};
    // the flag is cleared by a kernel (no memset node), so the call can be captured
    hipLaunchKernelGGL(k_zero_flag, dim3(1), dim3(1), 0, s, err);
    launch_rows<double>(pA, A->val, pM, M->val, rowpart, nullptr, 1.0, err, s);
    const int64_t chunk = (A->n + kNoAllocChunks - 1) / kNoAllocChunks;
    const int nb = (int)((A->n + chunk - 1) / chunk);
    hipLaunchKernelGGL(k_sum_chunks, dim3(nb), dim3(256), 0, s, rowpart, A->n, chunk, chunks);
    hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(256), 0, s, chunks, (int64_t)nb, L);
    HIPCHK(hipGetLastError());
    return SPAI_OK;
  } catch (...) {
    return fail(SPAI_ERR_HIP, "unexpected exception");
  }
}
