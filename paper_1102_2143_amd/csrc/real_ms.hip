// Multishift CG for a real symmetric positive-definite A (the paper's own benchmark
// matrix, the 2-D 5-point Poisson operator of Section 4 / Table 1, is real): the same
// shifted recurrences as the complex solve (Section 2, Algorithm 1 with the re-derived
// constants), on real vectors and a real copy of the sliced ELLPACK matrix, so every
// matrix value and vector element moves half the bytes of the complex path.  T = double
// (FP64) or float (the matrix, the residuals and the shifted directions in single
// precision, products and scalars in FP64: the paper's "single" column).
//
// One iteration is one kernel.  A is given, so with w_n = A r_n the iteration needs a single
// reduction point: g_n = r_n.r_n and d_n = r_n.(A + sigma0) r_n give
//   b_n = g_n / g_{n-1},  a_n = g_n / (d_n - b_n g_n / a_{n-1}),
//   s_n = w_n + sigma0 r_n + b_n s_{n-1},  r_{n+1} = r_n - a_n s_n,
// and w_{n+1} = A r_{n+1} follows in the same kernel, r_{n+1} being formed from r, w and s
// at every gathered column as its owner forms it (Chronopoulos and Gear's arrangement of
// CG).  Every workgroup sums the previous kernel's partials itself, in one order.  The
// shifted vectors take
//   p_k <- zeta_k r_n + b_k p_k,  x_k += a_k p_k
// (k = 0, the driving system, with zeta = 1); nothing else reads them, so up to eight steps
// are composed against the first one's p_k and the residuals of the steps, which stay in a
// ring, and applied in one pass.
//
// P = d_n - b_n g_n / a_{n-1} and the recurred s suppose that r_n is orthogonal to s_{n-1}.  Where A
// has eigenvalues far above the rest, rounding breaks that (multishift.hip).  The kernel also sums
// c_n = r_n.s_{n-1}, so that P = d_n + b_n (2 c_n + b_n P_{n-1}) is that of the vectors held, and
// once P leaves its short form, or x_0 misses the tolerance that its recursive residual has met,
// the sequence goes on with its direction, in two kernels (k_r_dir, k_r_step), s_n and P from p_n
// and x_0 updated step by step.  In single precision it does so from the start: a penalty of 100
// on one edge of a grid is too much for the residuals' rounding without it.
//
// Bound by memory: a row moves its matrix entries (10 bytes each), r, w and s in and out
// (w and s in FP64 always: recurred in single precision, s would add an error of its own),
// and an eighth of 32 bytes per live shift.  1000 x 1000 points, 15 shifts: 62.6 us an
// iteration in FP64 and 49.8 in single precision with three kernels (t = A p; r; the
// shifts' step, unfolded), 28.7 and (with the direction) 32.0 here; 60 x 50 points 24.0 and 24.0,
// 10.0 and 13.4.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "dev_common.h"
#include "msc_internal.h"

namespace msc {

namespace {

template <class T> __device__ __forceinline__ SellReal<T> rmat(const RealArgs& a);
template <> __device__ __forceinline__ SellReal<double> rmat<double>(const RealArgs& a) { return a.m64; }
template <> __device__ __forceinline__ SellReal<float> rmat<float>(const RealArgs& a) { return a.m32; }

__device__ __forceinline__ int32_t ld_uniform(const int32_t* p, int64_t i) {
  using cptr_t = const __attribute__((address_space(4))) int32_t*;
  return ((cptr_t)p)[i];
}

// Columns of pair q = c kSlice + lane of pair column c (32-bit or narrow 16-bit offsets).
template <class T>
__device__ __forceinline__ int2 r_cols(const SellReal<T>& m, int32_t c, int64_t q) {
  if (m.col16) {
    const uint32_t w = m.col16[q];
    return int2{ld_uniform(m.cbase, 2 * int64_t(c)) + int32_t(w & 0xffffu),
                ld_uniform(m.cbase, 2 * int64_t(c) + 1) + int32_t(w >> 16)};
  }
  return int2{m.col[2 * q], m.col[2 * q + 1]};
}

// One sliced ELLPACK row per lane times x (off-diagonal part plus the diagonal); four
// pairs per round trip, all their loads issued before the first multiply-add.
template <class T>
__device__ __forceinline__ T r_row(const SellReal<T>& m, const T* __restrict__ x, int64_t sl,
                                   int lane, int64_t row) {
  int32_t c, c1;
  if (m.wp > 0) {
    c = int32_t(sl) * m.wp;
    c1 = c + m.wp;
  } else {
    c = ld_uniform(m.cptr, sl);
    c1 = ld_uniform(m.cptr, sl + 1);
  }
  T acc = m.diag[row] * x[row];
  constexpr int KP = 4;
  for (; c < c1; c += KP) {
    int2 cc[KP];
    T v0[KP], v1[KP], g0[KP], g1[KP];
#pragma unroll
    for (int u = 0; u < KP; ++u) {
      if (c + u < c1) {
        const int64_t q = int64_t(c + u) * kSlice + lane;
        cc[u] = r_cols(m, c + u, q);
        v0[u] = m.val[2 * q];
        v1[u] = m.val[2 * q + 1];
      } else {
        cc[u] = int2{int32_t(row), int32_t(row)};
        v0[u] = v1[u] = T(0);
      }
    }
#pragma unroll
    for (int u = 0; u < KP; ++u) {
      g0[u] = x[cc[u].x];
      g1[u] = x[cc[u].y];
    }
#pragma unroll
    for (int u = 0; u < KP; ++u) acc = fma(v1[u], g1[u], fma(v0[u], g0[u], acc));
  }
  return acc;
}

__device__ double r_sum(const double* partial, int count, int stride, int k) {
  constexpr int kPer = kMaxGrid / kBlock;
  double v[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int i = threadIdx.x + u * kBlock;
    v[u] = i < count ? load_agent(&partial[i * stride + k]) : 0.0;
  }
  double s = 0.0;
#pragma unroll
  for (int u = 0; u < kPer; ++u) s += v[u];
  return block_sum<kBlock>(s);
}

// One row of slice `sl` times the vector val(column), off-diagonal part plus diagonal, in FP64.
template <class T, class F>
__device__ __forceinline__ double r_row_f(const SellReal<T>& m, F val, T own, int64_t sl, int lane,
                                     int64_t row) {
  int32_t c, c1;
  if (m.wp > 0) {
    c = int32_t(sl) * m.wp;
    c1 = c + m.wp;
  } else {
    c = ld_uniform(m.cptr, sl);
    c1 = ld_uniform(m.cptr, sl + 1);
  }
  double acc = double(m.diag[row]) * double(own);
  constexpr int KP = 2;
  for (; c < c1; c += KP) {
    int2 cc[KP];
    T v0[KP], v1[KP], g0[KP], g1[KP];
#pragma unroll
    for (int u = 0; u < KP; ++u) {
      if (c + u < c1) {
        const int64_t q = int64_t(c + u) * kSlice + lane;
        cc[u] = r_cols(m, c + u, q);
        v0[u] = m.val[2 * q];
        v1[u] = m.val[2 * q + 1];
      } else {
        cc[u] = int2{int32_t(row), int32_t(row)};
        v0[u] = v1[u] = T(0);
      }
    }
#pragma unroll
    for (int u = 0; u < KP; ++u) {
      g0[u] = val(cc[u].x);
      g1[u] = val(cc[u].y);
    }
#pragma unroll
    for (int u = 0; u < KP; ++u) acc = fma(double(v1[u]), double(g1[u]), fma(double(v0[u]), double(g0[u]), acc));
  }
  return acc;
}

// Partials of g (0), d (1) and c (2) of the kernel of parity par (their reader's parity).
__device__ __forceinline__ double* r_region(const RealArgs& a, int par, int which) {
  return a.partial + (3 * par + which) * kMaxGrid;
}

__device__ __forceinline__ void r_store_partials(const RealArgs& a, int par, double g, double d, double c) {
  double v[3] = {g, d, c};
  block_sum_k<kBlock, 3>(v);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < 3; ++k) store_agent(&r_region(a, par, k)[blockIdx.x], v[k]);
  }
}
__device__ __forceinline__ void r_store_one(const RealArgs& a, int par, int which, double v) {
  v = block_sum<kBlock>(v);
  if (threadIdx.x == 0) store_agent(&r_region(a, par, which)[blockIdx.x], v);
}

// The sums of the first K of them (a.par's), in every thread: plain loads, which the XCD's L2
// serves to all but its first workgroup.
template <int K> __device__ __forceinline__ void r_sums(const RealArgs& a, double (&tot)[K]) {
  __shared__ double sh[K];
  constexpr int kPer = kRealGrid / kBlock;
  double v[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    double w[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int i = threadIdx.x + u * kBlock;
      w[u] = i < int(gridDim.x) ? r_region(a, a.par, k)[i] : 0.0;
    }
    v[k] = 0.0;
#pragma unroll
    for (int u = 0; u < kPer; ++u) v[k] += w[u];
  }
  block_sum_k<kBlock, K>(v);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) sh[k] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) tot[k] = sh[k];
}

// r_0 = b in ring slot 0, s = 0, w_0 = A r_0 and the partials of g_0 and d_0.
template <class T>
__global__ __launch_bounds__(kBlock) void k_r_start(RealArgs a) {
  const SellReal<T> m = rmat<T>(a);
  T* __restrict__ r = static_cast<T*>(a.r);
  double* __restrict__ w = a.w[0];
  double* __restrict__ s = a.s[0];
  const double sigma0 = a.st->sigma0;
  constexpr int SPB = kBlock / kSlice;
  const int lane = threadIdx.x % kSlice;
  const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kSlice));
  int64_t beg, end;
  block_range(a.nslices, SPB, beg, end);
  double g = 0.0, d = 0.0;
  for (int64_t sl = beg + wv; sl < end; sl += SPB) {
    const int64_t row = sl * kSlice + lane;
    const int64_t rr = row < a.n ? row : a.n - 1;  // lanes past n read a valid row, unused
    const T own = T(a.b[rr]);
    const double v = r_row_f<T>(m, [&](int32_t c) { return T(a.b[c]); }, own, sl, lane, rr);
    if (row < a.n) {
      r[row] = own;
      w[row] = v;
      s[row] = 0.0;
      const double rd = double(own);
      g = fma(rd, rd, g);
      d += rd * v + sigma0 * rd * rd;
    }
  }
  r_store_partials(a, 0, g, d, 0.0);
}

// What an iteration's kernel does, shared through LDS.
struct RealPlan {
  double a, b;         // a_n, b_n (live only)
  int live;            // 1: this kernel takes step n
  int apply;           // 1: the composed steps go into x_k and p_k
  int m;               // composed steps (the last one step n when live)
  int fresh;           // 1: first application (x_k and p_k start from zero, unread)
  int nact;            // systems listed
  double cx[kMaxSteps + 1][kMaxShifts], cp[kMaxSteps + 1][kMaxShifts];
  int64_t xo[kMaxShifts], po[kMaxShifts];
};

__device__ __forceinline__ double r_b(const RealArgs& a, const RealRot& rs, double g) {
  return rs.iter == 0 ? 0.0 : (a.resume ? a.st->ru_g : g) / rs.g;
}
// Converged, at the limit, or |r|^2 not finite.
__device__ __forceinline__ bool r_ends(const RealArgs& a, const RealRot& rs, double g) {
  const double bn2 = rs.iter == 0 ? g : a.st->bnorm2;
  return !isfinite(g) || g <= a.st->tol2 * bn2 || rs.iter >= a.st->max_iter;
}

// Every workgroup derives a_n, b_n and whether step n runs; the shifts' scalars (wave 0,
// lane j) are needed by workgroup 0, which writes the next state, and by all where the
// composed steps are applied.  d: r_n.(A + sigma0) r_n, with the direction P itself.
__device__ void r_plan(const RealArgs& a, double g, double d, double c, RealPlan& pl) {
  RealState* st = a.st;
  const RealRot& rs = st->rot[a.par];
  const int j = threadIdx.x;
  if (j >= kWave) return;
  const bool head = blockIdx.x == 0;
  const int n = rs.iter, m0 = rs.m;
  const double bn2 = n == 0 ? g : st->bnorm2, eps2 = st->tol2 * bn2;
  const double b = r_b(a, rs, g);
  double P = d, off = 0.0;
  if (!a.dir && n > 0) {
    P = d + b * (2.0 * c + b * rs.P);
    off = fabs(P - (d - b * g / rs.a));
  }
  // |r|^2 first: an infinite |b|^2 would pass for its own limit
  const bool done = isfinite(g) && (g <= eps2 || n >= st->max_iter);
  const bool ok = done || (isfinite(g) && P > 0.0 && isfinite(P) && off <= kDevLimit64 * P);
  const bool take = !ok && isfinite(g) && !a.dir && n > 0;  // the direction is to be taken up
  const bool live = !done && ok;
  const double step = live ? g / P : 0.0;
  const int m = m0 + (live ? 1 : 0);
  const bool apply = live ? m >= a.steps : (m0 > 0 || rs.fresh != 0);
  int listed = 0;
  if (head || apply) {
    const bool mine = j < st->ns;
    double z = 1.0, zp = 1.0, cx[kMaxSteps + 1], cp[kMaxSteps + 1];
    int act = 0, took = 0;
#pragma unroll
    for (int i = 0; i <= kMaxSteps; ++i) cx[i] = cp[i] = 0.0;
    if (mine) {
      z = rs.zeta[j];
      zp = rs.zeta_prev[j];
      act = rs.active[j];
      if (m0 > 0) {
        took = rs.took[j];
#pragma unroll
        for (int i = 0; i <= kMaxSteps; ++i) {
          if (i <= m0) {
            cx[i] = rs.cx[i][j];
            cp[i] = rs.cp[i][j];
          }
        }
      } else {
        cp[0] = 1.0;
      }
    }
    const bool freeze = act && j > 0 && st->freeze && z * z * g <= eps2;
    if (freeze) act = 0;
    double zn = z;
    if (live && act) {
      // step n of system j: zeta^(n+1), a_j, b_j, composed with the pending ones
      if (j > 0)
        zn = n == 0 ? z / (1.0 + st->s[j] * step)
                    : z * zp * rs.a / (step * b * (zp - z) + zp * rs.a * (1.0 + st->s[j] * step));
      const double ratio = z / zp, aj = step * zn / z, bj = b * ratio * ratio;
#pragma unroll
      for (int i = 0; i <= kMaxSteps; ++i)
        if (i <= m0) cp[i] *= bj;
#pragma unroll
      for (int i = 1; i <= kMaxSteps; ++i)
        if (i == m) cp[i] = z;
#pragma unroll
      for (int i = 0; i <= kMaxSteps; ++i)
        if (i <= m) cx[i] = fma(aj, cp[i], cx[i]);
      took = 1;
    }
    const bool list = apply && mine && (took || rs.fresh) && !(a.dir && j == 0);
    const uint64_t mask = __ballot(list);
    if (list) {
      const int pos = __popcll(mask & ((uint64_t(1) << j) - 1));
#pragma unroll
      for (int i = 0; i <= kMaxSteps; ++i) {
        pl.cx[i][pos] = i <= m ? cx[i] : 0.0;
        pl.cp[i][pos] = i <= m ? cp[i] : 0.0;
      }
      pl.xo[pos] = int64_t(st->orig[j]) * a.n;
      pl.po[pos] = int64_t(j) * a.n;
    }
    listed = __popcll(mask);
    if (head) {
      RealRot& nx = st->rot[a.par ^ 1];
      if (mine) {
        if (freeze) st->freeze_iter[j] = n;
        nx.zeta_prev[j] = live && act ? z : zp;
        nx.zeta[j] = zn;
        nx.active[j] = act;
        nx.took[j] = apply ? 0 : took;
        if (!apply) {
#pragma unroll
          for (int i = 0; i <= kMaxSteps; ++i) {
            nx.cx[i][j] = i <= m ? cx[i] : 0.0;
            nx.cp[i][j] = i <= m ? cp[i] : 0.0;
          }
        }
      }
      if (j == 0) {
        // of the last step taken
        nx.g = live ? g : rs.g;
        nx.a = live ? step : rs.a;
        nx.P = live ? P : rs.P;
        nx.iter = live ? n + 1 : n;
        nx.m = apply ? 0 : m;
        nx.fresh = apply ? 0 : rs.fresh;
        nx.halt = live ? 0 : 1;
        if (n == 0) st->bnorm2 = g;
        if (apply) {
          st->n_upd += listed;
          st->n_kept += m;
        }
        if (!live) {
          st->iter = n;
          st->R = g;
          st->eps2 = eps2;
          st->status = ok || take ? 0 : 1;
          st->fin = a.par ^ 1;
          store_host_flag(a.hflag, take ? 5 : 1);
        }
      }
    }
  }
  if (j == 0) {
    pl.a = step;
    pl.b = b;
    pl.live = live ? 1 : 0;
    pl.apply = apply ? 1 : 0;
    pl.m = m;
    pl.fresh = rs.fresh;
    pl.nact = listed;
  }
}

// The composed steps of one row: the listed systems' x_k and p_k.
template <class T>
__device__ __forceinline__ void r_apply_row(const RealArgs& a, const RealPlan& pl, int n, int64_t i) {
  const T* __restrict__ ring = static_cast<const T*>(a.r);
  T* __restrict__ pk = static_cast<T*>(a.pk);
  double* __restrict__ x = a.x;
  const int m = pl.m;
  // residuals of the m steps, the last one n (live) or n - 1
  const int last = pl.live ? n : n - 1;
  double rk[kMaxSteps];
#pragma unroll
  for (int k = 0; k < kMaxSteps; ++k)
    rk[k] = k < m ? double(ring[int64_t((last - m + 1 + k) % kRealRing) * a.n + i]) : 0.0;
  constexpr int G = 4;  // systems whose loads are issued together
  auto group = [&](int q, int cnt) {
    double xv[G], pv[G];
#pragma unroll
    for (int u = 0; u < G; ++u) {
      xv[u] = pv[u] = 0.0;
      if (u < cnt && !pl.fresh) {
        pv[u] = double(__builtin_nontemporal_load(&pk[pl.po[q + u] + i]));
        xv[u] = __builtin_nontemporal_load(&x[pl.xo[q + u] + i]);
      }
    }
#pragma unroll
    for (int u = 0; u < G; ++u) {
      if (u < cnt) {
        double dx = pl.cx[0][q + u] * pv[u], np = pl.cp[0][q + u] * pv[u];
#pragma unroll
        for (int k = 0; k < kMaxSteps; ++k) {
          if (k < m) {
            dx = fma(pl.cx[k + 1][q + u], rk[k], dx);
            np = fma(pl.cp[k + 1][q + u], rk[k], np);
          }
        }
        __builtin_nontemporal_store(xv[u] + dx, &x[pl.xo[q + u] + i]);
        __builtin_nontemporal_store(T(np), &pk[pl.po[q + u] + i]);
      }
    }
  };
  for (int q = 0; q < pl.nact; q += G) group(q, min(G, pl.nact - q));
}

// ---- one iteration --------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_r_iter(RealArgs a) {
  RealState* st = a.st;
  const RealRot& rs = st->rot[a.par];
  if (rs.halt) {
    if (blockIdx.x == 0 && threadIdx.x == 0) st->rot[a.par ^ 1].halt = 1;
    return;
  }
  double tot[3];
  r_sums(a, tot);
  __shared__ RealPlan pl;
  const int n = rs.iter;
  r_plan(a, tot[0], tot[1], tot[2], pl);
  __syncthreads();
  const bool live = pl.live != 0, apply = pl.apply != 0;
  if (!live && !apply) return;
  const SellReal<double> m = rmat<double>(a);
  double* ring = static_cast<double*>(a.r);
  const double* __restrict__ r = ring + int64_t(n % kRealRing) * a.n;
  double* __restrict__ rn = ring + int64_t((n + 1) % kRealRing) * a.n;
  const double* __restrict__ w = a.w[a.par];
  const double* __restrict__ s = a.s[a.par];
  double* __restrict__ wn = a.w[a.par ^ 1];
  double* __restrict__ sn = a.s[a.par ^ 1];
  const double step = pl.a, b = pl.b, sigma0 = st->sigma0;
  // s_n and r_{n+1} at a row, rounded once each: the same bits wherever they are formed
  auto s_of = [&](int64_t c) {
    return fma(b, s[c], fma(sigma0, r[c], w[c]));
  };
  auto r_of = [&](int64_t c) { return fma(-step, s_of(c), r[c]); };
  constexpr int SPB = kBlock / kSlice;
  const int lane = threadIdx.x % kSlice;
  const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kSlice));
  int64_t beg, end;
  block_range(a.nslices, SPB, beg, end);
  double g = 0.0, d = 0.0, cs = 0.0;
  for (int64_t sl = beg + wv; sl < end; sl += SPB) {
    const int64_t row = sl * kSlice + lane;
    const int64_t rr = row < a.n ? row : a.n - 1;  // lanes past n read a valid row, unused
    if (live) {
      const double sv = s_of(rr);
      const double own = fma(-step, sv, r[rr]);
      const double v = r_row_f<double>(m, [&](int32_t c) { return r_of(c); }, own, sl, lane, rr);
      if (row < a.n) {
        rn[row] = own;
        sn[row] = sv;
        wn[row] = v;
        g = fma(own, own, g);
        d += own * v + sigma0 * own * own;
        cs = fma(own, sv, cs);
      }
    }
    if (apply && row < a.n) r_apply_row<double>(a, pl, n, row);
  }
  if (live) r_store_partials(a, a.par ^ 1, g, d, cs);
}

// ---- one iteration with the direction ---------------------------------------------------
// p_n = r_n + b_n p_{n-1}, t = A p_n (into w) and P's partials.  p, rounded to T, is formed at
// every gathered column as its owner forms it.
template <class T>
__global__ __launch_bounds__(kBlock) void k_r_dir(RealArgs a) {
  RealState* st = a.st;
  const RealRot& rs = st->rot[a.par];
  if (rs.halt) return;
  double g[1];
  r_sums(a, g);
  if (r_ends(a, rs, g[0])) return;
  const double b = r_b(a, rs, g[0]), sigma0 = st->sigma0;
  const SellReal<T> m = rmat<T>(a);
  const T* __restrict__ r = static_cast<const T*>(a.r) + int64_t(rs.iter % kRealRing) * a.n;
  const double* __restrict__ p = a.s[a.par];
  double* __restrict__ pn = a.s[a.par ^ 1];
  double* __restrict__ t = a.w[a.par ^ 1];
  auto p_of = [&](int64_t c) { return T(fma(b, p[c], double(r[c]))); };
  constexpr int SPB = kBlock / kSlice;
  const int lane = threadIdx.x % kSlice;
  const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kSlice));
  int64_t beg, end;
  block_range(a.nslices, SPB, beg, end);
  double P = 0.0;
  for (int64_t sl = beg + wv; sl < end; sl += SPB) {
    const int64_t row = sl * kSlice + lane;
    const int64_t rr = row < a.n ? row : a.n - 1;  // lanes past n read a valid row, unused
    const T own = p_of(rr);
    const double v = r_row_f<T>(m, [&](int32_t c) { return p_of(c); }, own, sl, lane, rr);
    if (row < a.n) {
      const double pd = double(own);
      pn[row] = pd;
      t[row] = v;
      P += pd * v + sigma0 * pd * pd;
    }
  }
  r_store_one(a, a.par, 1, P);
}

// r_{n+1} = r_n - a_n (t + sigma0 p_n), x_0 += a_n p_n and the other systems' composed steps.
template <class T>
__global__ __launch_bounds__(kBlock) void k_r_step(RealArgs a) {
  RealState* st = a.st;
  const RealRot& rs = st->rot[a.par];
  if (rs.halt) {
    if (blockIdx.x == 0 && threadIdx.x == 0) st->rot[a.par ^ 1].halt = 1;
    return;
  }
  double tot[2];
  r_sums(a, tot);
  __shared__ RealPlan pl;
  const int n = rs.iter;
  r_plan(a, tot[0], tot[1], 0.0, pl);
  __syncthreads();
  const bool live = pl.live != 0, apply = pl.apply != 0;
  if (!live && !apply) return;
  T* ring = static_cast<T*>(a.r);
  const T* __restrict__ r = ring + int64_t(n % kRealRing) * a.n;
  T* __restrict__ rn = ring + int64_t((n + 1) % kRealRing) * a.n;
  const double* __restrict__ p = a.s[a.par ^ 1];
  const double* __restrict__ t = a.w[a.par ^ 1];
  double* __restrict__ x0 = a.x + int64_t(st->orig[0]) * a.n;
  const double step = pl.a, sigma0 = st->sigma0;
  int64_t beg, end;
  block_range(a.n, kBlock, beg, end);
  double g = 0.0;
  for (int64_t i = beg + threadIdx.x; i < end; i += kBlock) {
    if (live) {
      const double pv = p[i];
      const T v = T(fma(-step, fma(sigma0, pv, t[i]), double(r[i])));
      rn[i] = v;
      x0[i] = fma(step, pv, n == 0 ? 0.0 : x0[i]);
      g = fma(double(v), double(v), g);
    } else if (n == 0) {
      x0[i] = 0.0;
    }
    if (apply) r_apply_row<T>(a, pl, n, i);
  }
  if (live) r_store_one(a, a.par ^ 1, 0, g);
}

// Go on after a halt: r_n = b - (A + sigma0) x_0 in FP64, its g's partials, and p_{n-1} in s[a.par]
// (load: from the driving system's direction, else from the other buffer where it lies there).
template <class T>
__global__ __launch_bounds__(kBlock) void k_r_load(RealArgs a, int load) {
  const RealState* st = a.st;
  const RealRot& fin = st->rot[st->fin];
  const SellReal<double> m = rmat<double>(a);
  T* __restrict__ r = static_cast<T*>(a.r) + int64_t(fin.iter % kRealRing) * a.n;
  const double* __restrict__ x0 = a.x + int64_t(st->orig[0]) * a.n;
  const T* __restrict__ pk = static_cast<const T*>(a.pk);
  const double* from = a.s[st->fin ^ 1];
  double* to = a.s[a.par];
  const double sigma0 = st->sigma0;
  constexpr int SPB = kBlock / kSlice;
  const int lane = threadIdx.x % kSlice;
  const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kSlice));
  int64_t beg, end;
  block_range(a.nslices, SPB, beg, end);
  double g = 0.0;
  for (int64_t sl = beg + wv; sl < end; sl += SPB) {
    const int64_t row = sl * kSlice + lane;
    const int64_t rr = row < a.n ? row : a.n - 1;
    const double v = r_row<double>(m, x0, sl, lane, rr);
    if (row < a.n) {
      const T o = T(a.b[row] - v - sigma0 * x0[row]);
      r[row] = o;
      g = fma(double(o), double(o), g);
      to[row] = load ? double(pk[row]) : from[row];
    }
  }
  r_store_one(a, a.par, 0, g);
}

// Its state (which may be the halted one's: a lane reads before it writes).
__global__ __launch_bounds__(kBlock) void k_r_go_on(RealArgs a) {
  RealState* st = a.st;
  const RealRot& fin = st->rot[st->fin];
  RealRot& rs = st->rot[a.par];
  const int j = threadIdx.x;
  if (j < kMaxShifts) {
    rs.zeta[j] = fin.zeta[j];
    rs.zeta_prev[j] = fin.zeta_prev[j];
    // repeats of the driving shift stopped with it and go on with it
    rs.active[j] = fin.active[j] || (j < st->ns && st->s[j] == 0.0);
    rs.took[j] = 0;
  }
  if (j == 0) {
    rs.g = fin.g;
    rs.a = fin.a;
    rs.P = fin.P;
    rs.iter = fin.iter;
    rs.m = 0;
    rs.fresh = 0;
    rs.halt = 0;
    st->ru_g = st->R;
  }
}

// ---- FP64 true residuals |b - (A + sigma_k) x_k|^2 of up to kRealCheck systems ----------
__global__ __launch_bounds__(kBlock) void k_r_verify(RealArgs a, const double* __restrict__ x,
                                                     RealSigma sg, int cnt, double* out) {
  const SellReal<double> m = rmat<double>(a);
  constexpr int SPB = kBlock / kSlice;
  const int lane = threadIdx.x % kSlice;
  const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kSlice));
  int64_t beg, end;
  block_range(a.nslices, SPB, beg, end);
  double acc[kRealCheck];
#pragma unroll
  for (int q = 0; q < kRealCheck; ++q) acc[q] = 0.0;
  for (int64_t sl = beg + wv; sl < end; sl += SPB) {
    const int64_t row = sl * kSlice + lane;
    const int64_t rr = row < a.n ? row : a.n - 1;
#pragma unroll
    for (int q = 0; q < kRealCheck; ++q) {
      if (q < cnt) {
        const double* __restrict__ xq = x + int64_t(q) * a.n;
        const double v = r_row<double>(m, xq, sl, lane, rr);
        if (row < a.n) {
          const double e = a.b[row] - v - sg.v[q] * xq[row];
          acc[q] = fma(e, e, acc[q]);
        }
      }
    }
  }
  block_sum_k<kBlock, kRealCheck>(acc);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < kRealCheck; ++q) store_agent(&a.partial[blockIdx.x * kRealCheck + q], acc[q]);
  }
  if (!arrive_last(a.tickets)) return;
  for (int q = 0; q < cnt; ++q) {
    const double t = r_sum(a.partial, gridDim.x, kRealCheck, q);
    if (threadIdx.x == 0) out[q] = t;
  }
}

// Real parts of the complex sliced copy (values and diagonal) and the largest imaginary
// part seen (atomic max on its bits: non-negative doubles order like their bit patterns).
__global__ void k_r_extract(const double2* __restrict__ v64, double* __restrict__ r64,
                            float* __restrict__ r32, int64_t count,
                            unsigned long long* __restrict__ imax) {
  unsigned long long local = 0;
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < count;
       i += int64_t(gridDim.x) * blockDim.x) {
    const double2 v = v64[i];
    r64[i] = v.x;
    r32[i] = float(v.x);
    const double ai = fabs(v.y);
    const unsigned long long bits = __double_as_longlong(ai);
    local = bits > local ? bits : local;
  }
  if (local) atomicMax(imax, local);
}

// Workgroups for the rows, a multiple of the XCD count, at most kRealGrid: more of them wait
// on longer sums of partials (1000 x 1000: 21.5 / 14.8 / 12.5 / 14.6 ms a solve with 256 /
// 512 / 1024 / 2048).
int r_grid(int64_t nslices) {
  const int64_t g = (nslices + kBlock / kSlice - 1) / (kBlock / kSlice);
  return int((std::min<int64_t>(std::max<int64_t>(g, 1), kRealGrid) + kXcds - 1) / kXcds * kXcds);
}

}  // namespace

hipError_t launch_real_extract(const double2* v64, double* r64, float* r32, int64_t count,
                               unsigned long long* imax, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  int64_t g = (count + 255) / 256;
  if (g > 8192) g = 8192;
  k_r_extract<<<unsigned(g), 256, 0, s>>>(v64, r64, r32, count, imax);
  return hipGetLastError();
}

hipError_t launch_real_start(int prec, const RealArgs& a, hipStream_t s) {
  const int g = r_grid(a.nslices);
  if (prec == MSC_PREC_MIXED)
    k_r_start<float><<<g, kBlock, 0, s>>>(a);
  else
    k_r_start<double><<<g, kBlock, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t launch_real_iteration(int prec, const RealArgs& a, hipStream_t s) {
  const int g = r_grid(a.nslices);
  if (prec == MSC_PREC_MIXED) {  // always with the direction
    k_r_dir<float><<<g, kBlock, 0, s>>>(a);
    k_r_step<float><<<g, kBlock, 0, s>>>(a);
  } else if (a.dir) {
    k_r_dir<double><<<g, kBlock, 0, s>>>(a);
    k_r_step<double><<<g, kBlock, 0, s>>>(a);
  } else {
    k_r_iter<<<g, kBlock, 0, s>>>(a);
  }
  return hipGetLastError();
}

hipError_t launch_real_direction(int prec, const RealArgs& a, bool load, hipStream_t s) {
  const int g = r_grid(a.nslices);
  if (prec == MSC_PREC_MIXED)
    k_r_load<float><<<g, kBlock, 0, s>>>(a, load ? 1 : 0);
  else
    k_r_load<double><<<g, kBlock, 0, s>>>(a, load ? 1 : 0);
  k_r_go_on<<<1, kBlock, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t launch_real_verify(const RealArgs& a, const double* x, const RealSigma& sg, int cnt,
                              double* out, hipStream_t s) {
  k_r_verify<<<r_grid(a.nslices), kBlock, 0, s>>>(a, x, sg, cnt, out);
  return hipGetLastError();
}

}  // namespace msc
