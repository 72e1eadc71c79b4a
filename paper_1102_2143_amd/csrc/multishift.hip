// The multishift CG iteration (paper: Section 2, Algorithm 1; Section 3 design rules), in
// Chronopoulos and Gear's arrangement of CG: with w_n = A r_n,
//   g_n = |r_n|^2,  d_n = r_n^H (A + sigma0) r_n,
//   b_n = g_n / g_{n-1},  a_n = g_n / (d_n - b_n g_n / a_{n-1}),
//   s_n = w_n + sigma0 r_n + b_n s_{n-1},  r_{n+1} = r_n - a_n s_n,
// the steps and residuals of Algorithm 1 without its direction p: the driving system's p
// and x are updated with the other shifts',
//   p_j <- zeta_j r_n + b_j p_j,  x_j += a_j p_j     (j = 0, the driving one: zeta = 1).
// For A = M^H M an iteration is two kernels:
//   K1  u = M r_n and the partials of |u|^2 (d_n = |u|^2 + sigma0 g_n): it needs no scalar
//   K2  a_n, b_n; w = M^H u, s_n, r_{n+1} and the partials of g_{n+1}
// For A given, on the sliced copy, it is one kernel, which forms r_{n+1} at every gathered
// column and the next w with it; on the CSR, K1 forms w and K2 is elementwise.
//
// What s_n = (A + sigma0) p_n and a_n's denominator P = p_n^H (A + sigma0) p_n suppose is that
// r_n is orthogonal to s's part of the direction before it.  Where A has eigenvalues far above
// the rest (a stiff constraint on few rows) rounding breaks that: s drifts from its product and
// P from its form (in complex64 from a condition of about 1e7 on, in FP64 far beyond).  K2
// therefore also sums c_n = Re(r_n^H s_{n-1}), from which
//   P = d_n + b_n (2 c_n + b_n P_{n-1})
// is the form of the vectors held, and the sequence takes the direction up as soon as P has
// left its short form: k_dir updates p_n = r_n + b_n p_{n-1} (from the driving system's p_0,
// which the applications keep), K1 and K2 form s_n and P from it, and a breakdown is reported
// only where that P is not positive.  So does an FP64 sequence whose x_0 misses the tolerance
// that its recursive residual has met.  Steps, shifts and their scalars go on as they were.
// Measured deviations |P - short form| / P: below 1e-13 in FP64 and 3e-4 in complex64 on lattices
// and grids of condition 1e6; a penalty of 1e4 on one edge of a 60 x 60 grid 4e-11 and above 1.
//
// Nothing reads x_j and p_j but their own update, so K2 only composes each step: the
// coefficients of x_j's increment and of p_j against the first pending step's p_j and the
// residuals of the steps, which stay in a ring.  Every update_steps-th iteration (eight), a
// kernel of its own (k_flush) applies the composed steps of every shift in one pass; so do
// a reliable update, which reads x_0, the switch to complex64 and the end of the sequence.
//
// The shift recurrences are the values forced by the collinearity r_j = zeta_j r:
//   zeta' = zeta zeta_prev a_prev / (a b (zeta_prev - zeta) + zeta_prev a_prev (1 + s a)),
//   a_j = a zeta'/zeta,  b_j = b (zeta/zeta_prev)^2,  with s = sigma_j - sigma0 >= 0.
// All scalar work stays on the device in FP64 (Section 3: the iteration constants are
// computed on the GPU to avoid host round trips).  Reductions are deterministic: each
// workgroup writes one partial, and every workgroup of the consuming kernel sums them in
// one fixed order (reliable update and verification: the last workgroup to arrive does).
// The shifts' scalars are the work of one workgroup more than the rows need.
#include <hip/hip_ext.h>

#include <map>
#include <mutex>
#include <type_traits>
#include <utility>

#include "dev_common.h"
#include "msc_internal.h"
#include "sell_load.h"
#include "stencil.h"

namespace msc {

namespace {

template <class R> __device__ __forceinline__ Csr<cplx<R>> pick_m(const MsArgs& a);
template <> __device__ __forceinline__ Csr<float2> pick_m<float>(const MsArgs& a) { return a.m32; }
template <> __device__ __forceinline__ Csr<double2> pick_m<double>(const MsArgs& a) { return a.m64; }
template <class R> __device__ __forceinline__ Csr<cplx<R>> pick_mh(const MsArgs& a);
template <> __device__ __forceinline__ Csr<float2> pick_mh<float>(const MsArgs& a) { return a.mh32; }
template <> __device__ __forceinline__ Csr<double2> pick_mh<double>(const MsArgs& a) { return a.mh64; }

template <class R> __device__ __forceinline__ Sell<cplx<R>> pick_sm(const MsArgs& a);
template <> __device__ __forceinline__ Sell<float2> pick_sm<float>(const MsArgs& a) { return a.s32; }
template <> __device__ __forceinline__ Sell<double2> pick_sm<double>(const MsArgs& a) { return a.s64; }
template <class R> __device__ __forceinline__ Stencil<cplx<R>> pick_w(const MsArgs& a);
template <> __device__ __forceinline__ Stencil<float2> pick_w<float>(const MsArgs& a) { return a.w32; }
template <> __device__ __forceinline__ Stencil<double2> pick_w<double>(const MsArgs& a) { return a.w64; }
template <class R> __device__ __forceinline__ Sell<cplx<R>> pick_shm(const MsArgs& a);
template <> __device__ __forceinline__ Sell<float2> pick_shm<float>(const MsArgs& a) { return a.sh32; }
template <> __device__ __forceinline__ Sell<double2> pick_shm<double>(const MsArgs& a) { return a.sh64; }

// Tuning knobs of the sliced ELLPACK SpMV (defaults measured best on MI355X):
//   MSC_SELL_KP32 / MSC_SELL_KP64: pairs per round trip for complex64 / complex128.
#ifndef MSC_SELL_KP32
#define MSC_SELL_KP32 12
#endif
#ifndef MSC_SELL_KP64
#define MSC_SELL_KP64 6
#endif

// The residual ring: launch l of the sequence reads its r_n from slot l % kRing (a.launch: a
// kernel argument, so the first gathers wait for no state) and writes r_{n+1} into the next.
template <class R> __device__ __forceinline__ cplx<R>* rslot(const MsArgs& a, int l) {
  return static_cast<cplx<R>*>(a.ring) + int64_t(l % kRing) * a.n;
}

// Pairs per round trip of the sliced ELLPACK row product (register budget: complex64
// keeps a 24-entry staggered row in flight at once, complex128 half of it).
template <class R> constexpr int sell_kp();
template <> constexpr int sell_kp<float>() { return MSC_SELL_KP32; }
template <> constexpr int sell_kp<double>() { return MSC_SELL_KP64; }

// NA: sums kept apart, entry e of a chunk in acc[e % NA].
template <class R, int KP, bool FULL, int NA>
__device__ __forceinline__ void sell_gather_fma(const cplx<R>* __restrict__ x, int np,
                                                const int2 (&cc)[KP], const cplx<R> (&v)[2 * KP],
                                                cplx<R> (&acc)[NA]) {
  cplx<R> xv[2 * KP];
#pragma unroll
  for (int u = 0; u < KP; ++u) {
    if (FULL || u < np) {
      xv[2 * u] = x[cc[u].x];
      xv[2 * u + 1] = x[cc[u].y];
    } else {
      xv[2 * u] = xv[2 * u + 1] = czero<R>();
    }
  }
#pragma unroll
  for (int u = 0; u < 2 * KP; ++u) cfma<R>(acc[u % NA], v[u], xv[u]);
}

// Off-diagonal part of the product of one sliced ELLPACK row per lane with x; slice `sl`
// is wavefront-uniform.  Pairs go KP at a time: a chunk's column and value loads, then
// its gathers, are all issued before its first multiply-add.  NA > 1 (a power of two): that
// many sums added in pairs at the end, for products that are results themselves (a row of 24
// entries in FP64: 1.4e-16 of rounding with eight, 2.6e-16 with one); init starts the last.
template <class R, bool NARROW, int NA>
__device__ __forceinline__ cplx<R> sell_row_cols(const Sell<cplx<R>>& m,
                                                 const cplx<R>* __restrict__ x, int64_t sl,
                                                 int lane, const cplx<R>& init) {
  constexpr int KP = NA > 1 ? NA / 2 : sell_kp<R>();  // an entry of a chunk per sum
  int32_t c, c1;
  if (m.wp > 0) {
    c = int32_t(sl) * m.wp;
    c1 = c + m.wp;
  } else {
    c = load_uniform(m.cptr, sl);
    c1 = load_uniform(m.cptr, sl + 1);
  }
  cplx<R> acc[NA];
#pragma unroll
  for (int k = 0; k < NA; ++k) acc[k] = k == NA - 1 ? init : czero<R>();
  int2 cc[KP];
  cplx<R> v[2 * KP];
  for (; c + KP <= c1; c += KP) {
    sell_load<R, KP, true, NARROW>(m, c, KP, lane, cc, v);
    sell_gather_fma<R, KP, true, NA>(x, KP, cc, v, acc);
  }
  if (c < c1) {
    const int np = c1 - c;
    sell_load<R, KP, false, NARROW>(m, c, np, lane, cc, v);
    sell_gather_fma<R, KP, false, NA>(x, np, cc, v, acc);
  }
#pragma unroll
  for (int o = NA / 2; o > 0; o /= 2) {
#pragma unroll
    for (int k = 0; k < o; ++k) {
      acc[k].x += acc[k + o].x;
      acc[k].y += acc[k + o].y;
    }
  }
  return acc[0];
}
template <class R, int NA = 1>
__device__ __forceinline__ cplx<R> sell_row(const Sell<cplx<R>>& m, const cplx<R>* __restrict__ x,
                                            int64_t sl, int lane,
                                            const cplx<R>& init = czero<R>()) {
  return m.col16 ? sell_row_cols<R, true, NA>(m, x, sl, lane, init)
                 : sell_row_cols<R, false, NA>(m, x, sl, lane, init);
}

// most t-slices per column of the march along t
constexpr int kK2March = 16;

// One CSR row times a vector, L lanes per row; the sum is returned in every lane.
// Entries of one row handled by a lane per chunk: the column and value loads of a chunk,
// then its gathers, are all issued before the first multiply-add, so a row of up to
// kChunk * L entries costs one round trip for the matrix and one for the gather.
constexpr int kChunk = 4;

template <class R, int L>
__device__ __forceinline__ cplx<R> row_dot(const Csr<cplx<R>>& m, const cplx<R>* __restrict__ x,
                                           int64_t row, int lane) {
  const int32_t beg = m.rowptr[row], end = m.rowptr[row + 1];
  cplx<R> acc = czero<R>();
  for (int32_t base = beg; base < end; base += kChunk * L) {
    int32_t c[kChunk];
    cplx<R> v[kChunk], xv[kChunk];
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      const int32_t j = base + lane + u * L;
      const bool ok = j < end;
      c[u] = ok ? m.col[j] : 0;
      v[u] = ok ? m.val[j] : czero<R>();
    }
#pragma unroll
    for (int u = 0; u < kChunk; ++u) xv[u] = x[c[u]];
#pragma unroll
    for (int u = 0; u < kChunk; ++u) cfma<R>(acc, v[u], xv[u]);
  }
  return group_sum_c<L, R>(acc);
}

// Two rows per row group at a time: both rows' loads share one round trip.  An empty
// second row (beg1 == end1) contributes zero.
template <class R, int L>
__device__ __forceinline__ void row_dot2(const Csr<cplx<R>>& m, const cplx<R>* __restrict__ x,
                                         int64_t row0, int64_t row1, bool has1, int lane,
                                         cplx<R>& out0, cplx<R>& out1) {
  const int32_t b0 = m.rowptr[row0], e0 = m.rowptr[row0 + 1];
  const int32_t b1 = has1 ? m.rowptr[row1] : 0, e1 = has1 ? m.rowptr[row1 + 1] : 0;
  const int32_t len = (e0 - b0) > (e1 - b1) ? (e0 - b0) : (e1 - b1);
  cplx<R> a0 = czero<R>(), a1 = czero<R>();
  for (int32_t base = 0; base < len; base += kChunk * L) {
    int32_t c0[kChunk], c1[kChunk];
    cplx<R> v0[kChunk], v1[kChunk], x0[kChunk], x1[kChunk];
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      const int32_t j0 = b0 + base + lane + u * L, j1 = b1 + base + lane + u * L;
      const bool ok0 = j0 < e0, ok1 = j1 < e1;
      c0[u] = ok0 ? m.col[j0] : 0;
      v0[u] = ok0 ? m.val[j0] : czero<R>();
      c1[u] = ok1 ? m.col[j1] : 0;
      v1[u] = ok1 ? m.val[j1] : czero<R>();
    }
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      x0[u] = x[c0[u]];
      x1[u] = x[c1[u]];
    }
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      cfma<R>(a0, v0[u], x0[u]);
      cfma<R>(a1, v1[u], x1[u]);
    }
  }
  out0 = group_sum_c<L, R>(a0);
  out1 = group_sum_c<L, R>(a1);
}

// The last workgroup sums `count` (<= kMaxGrid) partials (stride `stride`, offset `k`)
// in a fixed order; all loads are in flight together.  The result is valid in thread 0.
__device__ __forceinline__ double sum_partials(const double* partial, int count, int stride, int k) {
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

// ---- the iteration's reductions ------------------------------------------------------
// One partial per workgroup: of g_n in region n % 2, of d_n (|u|^2, or r^H w) in region
// 2 + n % 2, of c_n in 6 + n % 2; the reliable update's in 4 and 5.  The consuming kernel's workgroups each add
// all of them up in the same order; the producer was another kernel, so plain loads do.
__device__ __forceinline__ double* region(const MsArgs& a, int k) {
  return a.sc.partial + k * kMaxGrid;
}

__device__ __forceinline__ void store_partial(double* reg, double acc) {
  const double tot = block_sum<kBlock>(acc);
  if (threadIdx.x == 0) store_agent(&reg[blockIdx.x], tot);
}

// K2's: g_{n+1} and, without the direction, c_{n+1}.
template <bool DIR> __device__ __forceinline__ void store_k2(const MsArgs& a, double g, double c) {
  const int nx = a.par ^ 1;
  if constexpr (DIR) {
    store_partial(region(a, nx), g);
  } else {
    double v[2] = {g, c};
    block_sum_k<kBlock, 2>(v);
    if (threadIdx.x == 0) {
      store_agent(&region(a, nx)[blockIdx.x], v[0]);
      store_agent(&region(a, 6 + nx)[blockIdx.x], v[1]);
    }
  }
}

// The sums of `count` partials in each of K regions, in every thread (the same in every workgroup).
template <int K>
__device__ __forceinline__ void region_sums(const MsArgs& a, const int (&which)[K], int count,
                                            double (&v)[K]) {
  __shared__ double total[K];
  constexpr int U = 4;  // in flight together
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = 0.0;
  for (int i0 = threadIdx.x; i0 < count; i0 += U * kBlock) {
    double w[K][U];
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
      for (int u = 0; u < U; ++u) w[k][u] = i0 + u * kBlock < count ? region(a, which[k])[i0 + u * kBlock] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
      for (int u = 0; u < U; ++u) v[k] += w[k][u];
    }
  }
  block_sum_k<kBlock, K>(v);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) total[k] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = total[k];
}

// The work of K1's extra workgroup, the last: g_n and c_n for K2, which then sums d_n alone.
__device__ __forceinline__ bool k1_totals(const MsArgs& a) {
  if (int(blockIdx.x) != a.gd) return false;
  const int which[2] = {a.par, 6 + a.par};
  double v[2];
  region_sums(a, which, a.gg, v);
  if (threadIdx.x == 0) {
    a.st->g_n = v[0];
    a.st->c_n = v[1];
  }
  return true;
}

// K1's partials are loaded early (four per thread, covering grids of up to 1024 workgroups)
// so that their round trip overlaps the caller's own first loads.
constexpr int kEarly = 4;
struct Early {
  double d[kEarly];
};

__device__ __forceinline__ void load_early(const MsArgs& a, Early& e) {
  const double* rd = region(a, 2 + a.par);
#pragma unroll
  for (int u = 0; u < kEarly; ++u) {
    const int i = threadIdx.x + u * kBlock;
    e.d[u] = i < a.gd ? rd[i] : 0.0;
  }
}

// g_n, d_n of K1's vector and c_n (of no use with the direction).
struct Sums {
  double g, d, c;
};

// Step n's scalars, the same in every workgroup.
struct StepPlan {
  double a, b;  // a_n, b_n
  double P;     // p_n^H (A + sigma0) p_n
  double off;   // |P - its short form|
  int stop;     // 0: step n runs; 1: converged or at the limit; 2: end of the FP64 phase of
                // a mixed solve; 3: breakdown (P <= 0 or not finite: A + sigma0 not PD);
                // 4: the direction is to be taken up
};

// What the step needs of the state, read before the partials are summed.
struct StepIn {
  double g1, a1, P1;           // g_{n-1}, a_{n-1}, P_{n-1}
  double bn2, tol2, sw2, sigma0;
  double ru_g;
  int n, halt, max_iter, ru;
};

__device__ __forceinline__ StepIn step_in(const MsArgs& a) {
  const SolveState* st = a.st;
  const RotState& rs = st->rot[a.par];
  StepIn i;
  i.halt = rs.halt;
  i.n = rs.iter;
  i.g1 = rs.g;
  i.a1 = rs.a;
  i.P1 = rs.P;
  i.bn2 = st->bnorm2;
  i.tol2 = st->tol2;
  i.sw2 = st->sw2;
  i.sigma0 = st->sigma0;
  i.max_iter = st->max_iter;
  i.ru = a.ru_check || a.resume ? st->ru_flag : 0;
  i.ru_g = st->ru_g;
  return i;
}

// In every thread.  ONE: one kernel an iteration, which left all partials itself.
template <bool ONE>
__device__ __forceinline__ Sums all_sums(const MsArgs& a, const Early& e) {
  if constexpr (ONE) {
    const int which[3] = {a.par, 2 + a.par, 6 + a.par};
    double v[3];
    region_sums(a, which, a.gg, v);
    return Sums{v[0], v[1], v[2]};
  }
  __shared__ double total;
  // K1's totals are read here: held during K2's first product they cost it 15 us of 265 (FP64, 32^3 x
  // 64: its loads then go out in more parts)
  const double g = a.st->g_n, c = a.st->c_n;
  const double* rd = region(a, 2 + a.par);
  double d = 0.0;
#pragma unroll
  for (int u = 0; u < kEarly; ++u) d += e.d[u];
  for (int i = threadIdx.x + kEarly * kBlock; i < a.gd; i += kBlock) d += rd[i];
  d = block_sum<kBlock>(d);
  if (threadIdx.x == 0) total = d;
  __syncthreads();
  return Sums{g, total, c};
}

// b_n: where r_n was replaced it keeps the recursive residual's g_n (the direction is the
// sequence's).
__device__ __forceinline__ double step_b(const StepIn& i, double g) {
  return i.n == 0 ? 0.0 : (i.ru ? i.ru_g : g) / i.g1;
}

// Converged, at the limit, at the end of the FP64 phase, or |r|^2 not finite.
__device__ __forceinline__ bool step_ends(const StepIn& i, double g, double bn2) {
  return !isfinite(g) || g <= i.tol2 * bn2 || i.n >= i.max_iter || g <= i.sw2 * bn2;
}

// t.d: with the direction P itself, else r_n^H A r_n.  The short form of P supposes c_n = -b_n
// P_{n-1}, which a replaced r_n never fulfils; it is taken where c_n is not known (has_c).
__device__ __forceinline__ StepPlan step_plan(const MsArgs& a, const StepIn& i, const Sums& t,
                                              bool has_c = true) {
  const double g = t.g;
  const double bn2 = i.n == 0 ? g : i.bn2;
  StepPlan p;
  p.b = step_b(i, g);
  p.P = t.d;
  p.off = 0.0;
  if (!a.dir) {
    p.P += i.sigma0 * g;
    if (i.n > 0) {
      const double plain = p.P - p.b * g / i.a1;
      p.P = has_c ? p.P + p.b * (2.0 * t.c + p.b * i.P1) : plain;
      if (!i.ru) p.off = fabs(p.P - plain);
    }
  }
  p.a = g / p.P;
  const bool ok = p.P > 0.0 && isfinite(p.P);
  p.stop = 0;
  if (step_ends(i, g, bn2) || !ok || !(p.off <= a.dev_limit * p.P)) {
    // |r|^2 first: an infinite |b|^2 would pass for its own limit
    p.stop = !isfinite(g)                             ? 3
             : g <= i.tol2 * bn2 || i.n >= i.max_iter ? 1
             : (a.dir || i.n == 0) && !ok             ? 3
             : g <= i.sw2 * bn2                       ? 2
                                                      : 4;
  }
  return p;
}

// Shift j's scalars and its composed steps, in its lane.
struct ShiftSteps {
  double z = 1.0, zp = 1.0, s = 0.0, cx[kMaxSteps + 1], cp[kMaxSteps + 1];
  int act = 0, took = 0;

  __device__ __forceinline__ void load(const RotState& rs, double sj, int j) {
    z = rs.zeta[j];
    zp = rs.zeta_prev[j];
    act = rs.active[j];
    took = rs.took[j];
    s = sj;
#pragma unroll
    for (int i = 0; i <= kMaxSteps; ++i) {
      cx[i] = rs.cx[i][j];
      cp[i] = rs.cp[i][j];
    }
  }
  // Iteration n with m0 steps pending: freezing (true: j froze), then, when the step runs
  // (live), zeta^(n+1), a_j and b_j, composed with the pending steps.
  __device__ __forceinline__ bool step(int j, int n, int m0, bool live, bool freeze, double g,
                                       double eps2, double a, double b, double a1) {
    bool froze = false;
    double zn = z;
    if (m0 == 0) {
      took = 0;
      cp[0] = 1.0;
      cx[0] = 0.0;
    }
#pragma unroll
    for (int i = 1; i <= kMaxSteps; ++i)
      if (i > m0) cx[i] = cp[i] = 0.0;
    if (act && j > 0 && freeze && z * z * g <= eps2) {
      act = 0;
      froze = true;
    }
    if (live && act) {
      if (j > 0)
        zn = n == 0 ? z / (1.0 + s * a)
                    : z * zp * a1 / (a * b * (zp - z) + zp * a1 * (1.0 + s * a));
      const double ratio = z / zp, aj = a * zn / z, bj = b * ratio * ratio;
#pragma unroll
      for (int i = 0; i <= kMaxSteps; ++i) {
        if (i <= m0) cp[i] *= bj;
        if (i == m0 + 1) cp[i] = z;
        if (i <= m0 + 1) cx[i] = fma(aj, cp[i], cx[i]);
      }
      took = 1;
      zp = z;
      z = zn;
    }
    return froze;
  }
  __device__ __forceinline__ void store(RotState& nx, int j) const {
    nx.zeta_prev[j] = zp;
    nx.zeta[j] = z;
    nx.active[j] = act;
    nx.took[j] = took;
#pragma unroll
    for (int i = 0; i <= kMaxSteps; ++i) {
      nx.cx[i][j] = cx[i];
      nx.cp[i][j] = cp[i];
    }
  }
};

__device__ __forceinline__ void sequence_halts(const MsArgs& a, int fin, int n, const Sums& t,
                                               double eps2, int stop) {
  SolveState* st = a.st;
  st->fin = fin;
  st->iter = n;
  st->R = t.g;
  st->c = t.c;
  st->eps2 = eps2;
  st->status = stop == 3 ? 1 : 0;
  store_host_flag(a.hflag, 1 | (stop == 2 ? 2 : 0) | (stop == 4 ? 4 : 0));
}

// The work of K2's extra workgroup: the shifts' scalars of step n (wave 0, lane j: shift
// j): freezing, then, when the step runs, zeta^(n+1), a_j and b_j, composed with the
// pending steps; the state of iteration n + 1, or of the halted sequence.  On small
// operators it is the longest chain of the iteration: all it reads is read before the sums.
template <bool ONE>
__device__ __forceinline__ void plan_workgroup(const MsArgs& a, const StepIn& in, const Early& e) {
  SolveState* st = a.st;
  const RotState& rs = st->rot[a.par];
  RotState& nx = st->rot[a.par ^ 1];
  const int j = threadIdx.x, n = in.n;
  const bool mine = j < st->ns;
  ShiftSteps h;
  if (mine) h.load(rs, st->s[j], j);
  const int m = rs.m, fresh = rs.fresh, freeze = st->freeze;
  const Sums t = all_sums<ONE>(a, e);
  const double g = t.g;
  const StepPlan p = step_plan(a, in, t);
  if (j >= kWave) return;
  // a flush since the last step leaves nothing pending
  const bool flushed = a.flushed || in.ru;
  const int m0 = flushed ? 0 : m;
  const bool live = p.stop == 0;
  const double eps2 = in.tol2 * (n == 0 ? g : in.bn2);
  if (mine) {
    if (h.step(j, n, m0, live, freeze != 0, g, eps2, p.a, p.b, in.a1)) st->freeze_iter[j] = n;
    h.store(nx, j);
  }
  if (j == 0) {
    if (n == 0) st->bnorm2 = g;
    nx.g = live ? g : in.g1;
    nx.a = live ? p.a : in.a1;
    nx.P = live ? p.P : in.P1;
    nx.iter = live ? n + 1 : n;
    nx.launch = live ? a.launch + 1 : a.launch;
    nx.m = live ? m0 + 1 : m0;
    nx.fresh = flushed ? 0 : fresh;
    nx.halt = live ? 0 : 1;
    if (live && p.off > st->dev * p.P) st->dev = p.off / p.P;
    if (!live) sequence_halts(a, a.par ^ 1, n, t, eps2, p.stop);
  }
}

// K2's prologue: true in a workgroup that goes on to the rows (with e and in loaded); a
// halted iteration hands the halt on, the extra workgroup does the plan.
template <bool ONE = false>
__device__ __forceinline__ bool k2_begin(const MsArgs& a, Early& e, StepIn& in) {
  if (!ONE) load_early(a, e);
  in = step_in(a);
  if (int(blockIdx.x) != a.gg) return true;
  if (in.halt) {
    if (threadIdx.x == 0) a.st->rot[a.par ^ 1].halt = 1;
  } else {
    plan_workgroup<ONE>(a, in, e);
  }
  return false;
}

// The sums and the step in every other workgroup; false where no step runs.
template <bool ONE = false>
__device__ __forceinline__ bool k2_step(const MsArgs& a, const Early& e, const StepIn& in, StepPlan& p) {
  p.stop = 1;
  if (in.halt) return false;
  p = step_plan(a, in, all_sums<ONE>(a, e));
  return p.stop == 0;
}

// The march positions [beg, end) of this wave: its XCD's share of [0, n) (workgroups are
// dealt to the XCDs in turn), split evenly and contiguously over the XCD's waves.  g, the
// workgroups that share them, is a multiple of kXcds (grid_rows, resident_grid).
__device__ __forceinline__ void march_range(int64_t n, int wpb, int64_t& beg, int64_t& end,
                                            int g = gridDim.x) {
  const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kWave));
  const int x = int(blockIdx.x % kXcds);
  const int64_t lo = n * x / kXcds, hi = n * (x + 1) / kXcds;
  const int64_t nw = int64_t(g / kXcds) * wpb, w = int64_t(blockIdx.x / kXcds) * wpb + wv;
  beg = lo + (hi - lo) * w / nw;
  end = lo + (hi - lo) * (w + 1) / nw;
}

// s_n = q + sigma0 r + b s, r_{n+1} = r - a s_n at one row (q = (A r_n)_row), formed in FP64
// and rounded once each.  DIR: q = (A p_n)_row and s is p_n there, s_n = q + sigma0 p_n.
template <class R, bool DIR = false>
__device__ __forceinline__ void row_step(const StepPlan& p, double sigma0, const cplx<R>& q,
                                         const cplx<R>& r, const cplx<R>& s, cplx<R>& sn,
                                         cplx<R>& rn) {
  const double2 qd = to_d(q), rd = to_d(r), sd = to_d(s);
  const double2 v = DIR ? double2{fma(sigma0, sd.x, qd.x), fma(sigma0, sd.y, qd.y)}
                        : double2{fma(p.b, sd.x, fma(sigma0, rd.x, qd.x)),
                                  fma(p.b, sd.y, fma(sigma0, rd.y, qd.y))};
  sn = from_d<R>(v);
  rn = from_d<R>(double2{fma(-p.a, v.x, rd.x), fma(-p.a, v.y, rd.y)});
}

// K1's vector: r_n, or p_n.
template <class R, bool DIR> __device__ __forceinline__ const cplx<R>* k1_vec(const MsArgs& a) {
  return DIR ? static_cast<const cplx<R>*>(a.s[0]) : rslot<R>(a, a.launch);
}

// K1's term of one row, u = (M v)_row or (A v)_row: v^H A v's, with sigma0 |v|^2's where v = p_n.
template <class R, bool MHM, bool DIR>
__device__ __forceinline__ double k1_term(const cplx<R>& u, const cplx<R>& v, double sigma0) {
  const double t = MHM ? norm2d<R>(u) : double(v.x) * double(u.x) + double(v.y) * double(u.y);
  return DIR ? fma(sigma0, norm2d<R>(v), t) : t;
}

// x_0 += a_n p_n at one row: with the direction the driving system's own x takes each step as it
// is (composed, its increments would differ from A^-1 of s's by rounding that stiff rows blow up).
template <class R>
__device__ __forceinline__ void x0_step(double2* x0, int64_t row, double a, const cplx<R>& p) {
  const double2 pd = to_d(p), x = x0[row];
  x0[row] = double2{fma(a, pd.x, x.x), fma(a, pd.y, x.y)};
}
__device__ __forceinline__ double2* x0_of(const MsArgs& a) {
  return a.x + int64_t(a.st->orig[0]) * a.n;
}

// c's term of one row.
template <class R>
__device__ __forceinline__ double c_term(const cplx<R>& rn, const cplx<R>& sn) {
  return fma(double(rn.x), double(sn.x), double(rn.y) * double(sn.y));
}

// p_n = r_n + b_n p_{n-1}, in the order of the ring, where step n may run.
template <class R> __global__ __launch_bounds__(kBlock) void k_dir(MsArgs a) {
  const StepIn in = step_in(a);
  if (in.halt) return;
  const int which[1] = {a.par};
  double g[1];
  region_sums(a, which, a.gg, g);
  if (step_ends(in, g[0], in.n == 0 ? g[0] : in.bn2)) return;
  const double b = step_b(in, g[0]);
  const cplx<R>* __restrict__ r = rslot<R>(a, a.launch);
  cplx<R>* __restrict__ p = static_cast<cplx<R>*>(a.s[0]);
  for (int64_t i = blockIdx.x * int64_t(kBlock) + threadIdx.x; i < a.n; i += int64_t(gridDim.x) * kBlock) {
    const double2 rd = to_d(r[i]), pd = to_d(p[i]);
    p[i] = from_d<R>(double2{fma(b, pd.x, rd.x), fma(b, pd.y, rd.y)});
  }
}

// ---- A = M^H M or the CSR: K1 u = M r_n (A r_n for A given) and d_n's partials -----------
template <class R, int L, bool MHM, bool DIR>
__global__ __launch_bounds__(kBlock) void k1_csr(MsArgs a) {
  const RotState& rs = a.st->rot[a.par];
  if (rs.halt || k1_totals(a)) return;
  const Csr<cplx<R>> m = pick_m<R>(a);
  const cplx<R>* __restrict__ r = k1_vec<R, DIR>(a);
  const double sigma0 = a.st->sigma0;
  cplx<R>* __restrict__ u = static_cast<cplx<R>*>(a.u);
  constexpr int GPB = kBlock / L;
  const int lane = threadIdx.x % L, grp = threadIdx.x / L;
  int64_t beg, end;
  block_range(a.n, GPB, beg, end, a.gd);
  double acc = 0.0;
  auto epilogue = [&](int64_t row, const cplx<R>& v) {
    u[row] = v;
    acc += k1_term<R, MHM, DIR>(v, MHM && !DIR ? v : r[row], sigma0);
  };
  for (int64_t row = beg + grp; row < end; row += 2 * GPB) {
    const int64_t row1 = row + GPB;
    const bool has1 = row1 < end;
    cplx<R> v0, v1;
    row_dot2<R, L>(m, r, row, row1, has1, lane, v0, v1);
    if (lane == 0) {
      epilogue(row, v0);
      if (has1) epilogue(row1, v1);
    }
  }
  store_partial(region(a, 2 + a.par), acc);
}

// K2: w = M^H u (u itself for A given), s_n, r_{n+1}, g_{n+1}'s and c_{n+1}'s partials.
template <class R, int L, bool MHM, bool DIR>
__global__ __launch_bounds__(kBlock) void k2_csr(MsArgs a) {
  Early e;
  StepIn in;
  if (!k2_begin(a, e, in)) return;
  StepPlan p;
  if (!k2_step(a, e, in, p)) return;
  const cplx<R>* __restrict__ u = static_cast<const cplx<R>*>(a.u);
  const cplx<R>* __restrict__ r = rslot<R>(a, a.launch);
  cplx<R>* __restrict__ rn = rslot<R>(a, a.launch + 1);
  cplx<R>* __restrict__ s = static_cast<cplx<R>*>(a.s[0]);
  double2* __restrict__ x0 = x0_of(a);
  const double sigma0 = in.sigma0;
  int64_t beg, end;
  double acc = 0.0, ac = 0.0;
  auto epilogue = [&](int64_t row, const cplx<R>& q) {
    cplx<R> sv, nv;
    row_step<R, DIR>(p, sigma0, q, r[row], s[row], sv, nv);
    if (DIR)
      x0_step<R>(x0, row, p.a, s[row]);
    else
      s[row] = sv;
    rn[row] = nv;
    acc += norm2d<R>(nv);
    if (!DIR) ac += c_term<R>(nv, sv);
  };
  if constexpr (MHM) {
    const Csr<cplx<R>> mh = pick_mh<R>(a);
    constexpr int GPB = kBlock / L;
    const int lane = threadIdx.x % L, grp = threadIdx.x / L;
    block_range(a.n, GPB, beg, end, a.gg);
    for (int64_t row = beg + grp; row < end; row += 2 * GPB) {
      const int64_t row1 = row + GPB;
      const bool has1 = row1 < end;
      cplx<R> q0, q1;
      row_dot2<R, L>(mh, u, row, row1, has1, lane, q0, q1);
      if (lane == 0) {
        epilogue(row, q0);
        if (has1) epilogue(row1, q1);
      }
    }
  } else {
    block_range(a.n, kBlock, beg, end, a.gg);
    for (int64_t i = beg + threadIdx.x; i < end; i += kBlock) epilogue(i, u[i]);
  }
  store_k2<DIR>(a, acc, ac);
}

// ---- the sliced ELLPACK copies: one row per lane, one slice per wave ----------------------
// (A given, MHM false: with the direction only, with the CSR's K2; else k_herm below)
template <class R, bool MHM, bool DIR>
__global__ __launch_bounds__(kBlock) void k1_sell(MsArgs a) {
  const RotState& rs = a.st->rot[a.par];
  if (rs.halt || k1_totals(a)) return;
  const Sell<cplx<R>> m = pick_sm<R>(a);
  const cplx<R>* __restrict__ r = k1_vec<R, DIR>(a);
  const double sigma0 = a.st->sigma0;
  cplx<R>* __restrict__ u = static_cast<cplx<R>*>(a.u);
  const int lane = threadIdx.x % kSlice;
  double acc = 0.0;
  for (Sweep sw = make_sweep(a.nslices, a.ord, kBlock / kSlice, a.gd); sw.more(); sw.next()) {
    const int64_t sl = sw.slice();
    const int64_t row = sl * kSlice + lane;
    const int64_t rr = row < a.n ? row : a.n - 1;  // lanes past n read a valid row, unused
    const cplx<R> own = r[rr], d = m.diag[rr];
    cplx<R> v = sell_row<R>(m, r, sl, lane);
    cfma<R>(v, d, own);
    if (row < a.n) {
      u[row] = v;
      acc += k1_term<R, MHM, DIR>(v, own, sigma0);
    }
  }
  store_partial(region(a, 2 + a.par), acc);
}

template <class R, bool DIR>
__global__ __launch_bounds__(kBlock) void k2_sell(MsArgs a) {
  Early e;
  StepIn in;
  if (!k2_begin(a, e, in)) return;
  const Sell<cplx<R>> mh = pick_shm<R>(a);
  const cplx<R>* __restrict__ u = static_cast<const cplx<R>*>(a.u);
  const cplx<R>* __restrict__ r = rslot<R>(a, a.launch);
  cplx<R>* __restrict__ rn = rslot<R>(a, a.launch + 1);
  cplx<R>* __restrict__ s = static_cast<cplx<R>*>(a.s[0]);
  double2* __restrict__ x0 = x0_of(a);
  const double sigma0 = in.sigma0;
  const int lane = threadIdx.x % kSlice;
  struct Row {
    cplx<R> q, r, s;
  };
  auto product = [&](int64_t sl) {
    const int64_t row = sl * kSlice + lane;
    const int64_t rr = row < a.n ? row : a.n - 1;
    const cplx<R> ur = u[rr];
    Row o;
    o.r = ld_stream(&r[rr]);
    o.s = ld_stream(&s[rr]);
    const cplx<R> d = mh.diag[rr];
    o.q = sell_row<R>(mh, u, sl, lane);
    cfma<R>(o.q, d, ur);
    return o;
  };
  StepPlan p;
  double acc = 0.0, ac = 0.0;
  auto epilogue = [&](int64_t sl, const Row& o) {
    const int64_t row = sl * kSlice + lane;
    if (row >= a.n) return;
    cplx<R> sv, nv;
    row_step<R, DIR>(p, sigma0, o.q, o.r, o.s, sv, nv);
    if (DIR)
      x0_step<R>(x0, row, p.a, o.s);
    else
      st_stream(&s[row], sv);
    rn[row] = nv;
    acc += norm2d<R>(nv);
    if (!DIR) ac += c_term<R>(nv, sv);
  };
  // the first slice's product runs while the partials are on their way
  Sweep sw = make_sweep(a.nslices, a.ord, kBlock / kSlice, a.gg);
  const bool has0 = sw.more();
  const int64_t sl0 = has0 ? sw.slice() : 0;
  Row first{};
  if (has0) first = product(sl0);
  if (!k2_step(a, e, in, p)) return;
  if (has0) epilogue(sl0, first);
  for (sw.next(); sw.more(); sw.next()) {
    const int64_t sl = sw.slice();
    epilogue(sl, product(sl));
  }
  store_k2<DIR>(a, acc, ac);
}

// A given: one kernel.  r_{n+1} is formed at every gathered column from r, w and s, rounded
// as its owner rounds it, and w_{n+1} = A r_{n+1} with it.
template <class R, bool NARROW, class F>
__device__ __forceinline__ cplx<R> sell_row_f(const Sell<cplx<R>>& m, int64_t sl, int lane, F val) {
  constexpr int KP = std::is_same<R, float>::value ? 4 : 2;
  int32_t c, c1;
  if (m.wp > 0) {
    c = int32_t(sl) * m.wp;
    c1 = c + m.wp;
  } else {
    c = load_uniform(m.cptr, sl);
    c1 = load_uniform(m.cptr, sl + 1);
  }
  cplx<R> acc = czero<R>();
  for (; c < c1; c += KP) {
    const int np = c1 - c;
    int2 cc[KP];
    cplx<R> v[2 * KP], x[2 * KP];
    if (np >= KP)
      sell_load<R, KP, true, NARROW>(m, c, KP, lane, cc, v);
    else
      sell_load<R, KP, false, NARROW>(m, c, np, lane, cc, v);
#pragma unroll
    for (int u = 0; u < KP; ++u) {
      if (u < np) {
        x[2 * u] = val(cc[u].x);
        x[2 * u + 1] = val(cc[u].y);
      }
    }
#pragma unroll
    for (int u = 0; u < 2 * KP; ++u)
      if (u < 2 * np) cfma<R>(acc, v[u], x[u]);
  }
  return acc;
}

template <class R, class F>
__device__ __forceinline__ cplx<R> sell_row_any(const Sell<cplx<R>>& m, int64_t sl, int lane, F val) {
  return m.col16 ? sell_row_f<R, true>(m, sl, lane, val) : sell_row_f<R, false>(m, sl, lane, val);
}

template <class R> __global__ __launch_bounds__(kBlock) void k_herm(MsArgs a) {
  Early e;
  StepIn in;
  if (!k2_begin<true>(a, e, in)) return;
  StepPlan p;
  if (!k2_step<true>(a, e, in, p)) return;
  const Sell<cplx<R>> m = pick_sm<R>(a);
  const cplx<R>* __restrict__ r = rslot<R>(a, a.launch);
  cplx<R>* __restrict__ rn = rslot<R>(a, a.launch + 1);
  const cplx<R>* __restrict__ w = static_cast<const cplx<R>*>(a.w[a.par]);
  const cplx<R>* __restrict__ s = static_cast<const cplx<R>*>(a.s[a.par]);
  cplx<R>* __restrict__ wn = static_cast<cplx<R>*>(a.w[a.par ^ 1]);
  cplx<R>* __restrict__ sn = static_cast<cplx<R>*>(a.s[a.par ^ 1]);
  const double sigma0 = in.sigma0;
  const int lane = threadIdx.x % kSlice;
  auto next = [&](int32_t c) {
    cplx<R> sv, nv;
    row_step<R>(p, sigma0, w[c], r[c], s[c], sv, nv);
    return nv;
  };
  double ag = 0.0, ad = 0.0, ac = 0.0;
  for (Sweep sw = make_sweep(a.nslices, a.ord, kBlock / kSlice, a.gg); sw.more(); sw.next()) {
    const int64_t sl = sw.slice();
    const int64_t row = sl * kSlice + lane;
    const int64_t rr = row < a.n ? row : a.n - 1;
    cplx<R> sv, own;
    row_step<R>(p, sigma0, w[rr], r[rr], s[rr], sv, own);
    const cplx<R> dg = m.diag[rr];
    cplx<R> v = sell_row_any<R>(m, sl, lane, next);
    cfma<R>(v, dg, own);
    if (row < a.n) {
      rn[row] = own;
      sn[row] = sv;
      wn[row] = v;
      ag += norm2d<R>(own);
      ad += k1_term<R, false, false>(v, own, 0.0);
      ac += c_term<R>(own, sv);
    }
  }
  double v[3] = {ag, ad, ac};
  block_sum_k<kBlock, 3>(v);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < 3; ++k) store_agent(&region(a, (k < 2 ? 2 * k : 6) + (a.par ^ 1))[blockIdx.x], v[k]);
  }
}

// w_n = A r_n and d_n's partials for the iteration's first k_herm and after a reliable
// update (only_ru: where it ran).
template <class R> __global__ __launch_bounds__(kBlock) void k_herm_w(MsArgs a, int only_ru) {
  const RotState& rs = a.st->rot[a.par];
  if (rs.halt || (only_ru && !a.st->ru_flag)) return;
  const Sell<cplx<R>> m = pick_sm<R>(a);
  const cplx<R>* __restrict__ r = rslot<R>(a, a.launch);
  cplx<R>* __restrict__ w = static_cast<cplx<R>*>(a.w[a.par]);
  const int lane = threadIdx.x % kSlice;
  double acc = 0.0;
  for (Sweep sw = make_sweep(a.nslices, a.ord, kBlock / kSlice); sw.more(); sw.next()) {
    const int64_t sl = sw.slice();
    const int64_t row = sl * kSlice + lane;
    const int64_t rr = row < a.n ? row : a.n - 1;
    const cplx<R> own = r[rr], dg = m.diag[rr];
    cplx<R> v = sell_row_any<R>(m, sl, lane, [&](int32_t c) { return r[c]; });
    cfma<R>(v, dg, own);
    if (row < a.n) {
      w[row] = v;
      acc += double(own.x) * double(v.x) + double(own.y) * double(v.y);
    }
  }
  store_partial(region(a, 2 + a.par), acc);
}

// ---- the links: one lattice site (three rows) per lane --------------------------------------
// r, u and s lie colour by colour here, v(site, c) at c V + site: a wave's 64 consecutive
// sites then read and write each colour in one contiguous run, so that streaming hints can
// be given, and they are: a wave's own rows of r and s, and the t links it carries, are read
// once per launch, and the L2 is left to the links and values that neighbours read again.
// MARCH (a.march = tc >= 2 t-slices per column; the host checks that a t-slice holds whole
// blocks of 64 sites and that tc divides L_t): the blocks are taken in columns of tc
// consecutive t-slices, and each wave takes a contiguous run of them.  A lane's next site
// is then its last one moved one slice along t: the site's t link (the next one's backward
// t link), its values and its forward t neighbour's (the next one's own) stay in registers
// (TCarry); a run that enters a new column loads them.
// 32^3 x 64, K1 and K2 of an iteration: FP64 221 and 266 us, complex64 120 and 138 (with rows
// of three colours together and no hints 322 and 342, 184 and 175, of which the head's r,
// p and t and the applications, now apart, are a part).
constexpr int kSiteBlock = kWave;  // sites per wave pass

// The march's block at position q.
__device__ __forceinline__ uint32_t march_block(uint32_t q, uint32_t tc, uint32_t bs) {
  const uint32_t col = q / tc, chunk = col / bs;
  return (chunk * tc + (q - col * tc)) * bs + (col - chunk * bs);
}

// body(site, out, own) for this wave's sites, out = (m + sign D) v and own = v there; lanes past the volume
// are left out.  first(): called once by every wave of the workgroup, between its first
// product (if it has any) and the rest; false ends the work.  g: workgroups that share the
// sites.
template <class R, int LR, bool MARCH, class F0, class F>
__device__ __forceinline__ void for_sites(const MsArgs& a, const Stencil<cplx<R>>& w,
                                          const cplx<R>* __restrict__ v, int sign, int g, F0 first,
                                          F body) {
  const uint32_t vol = uint32_t(w.vol);
  const int64_t nblk = (int64_t(vol) + kSiteBlock - 1) / kSiteBlock;
  constexpr int WPB = kBlock / kWave;
  const int lane = threadIdx.x % kWave;
  auto at = [&](uint32_t s, int c) { return v[int64_t(c) * vol + s]; };
  cplx<R> own[3], out[3];
  if constexpr (MARCH) {
    const uint32_t tc = uint32_t(a.march);
    const uint32_t vol3 = vol / uint32_t(w.L[3]);
    const uint32_t bs = vol3 / uint32_t(kSiteBlock);
    constexpr int K = 3 * LR;
    TCarry<R, LR> car;
    int64_t qb, qe;
    march_range(nblk, WPB, qb, qe, g);
#pragma nounroll
    for (uint32_t q = uint32_t(qb);; ++q) {
      const bool has = q < uint32_t(qe);
      uint32_t site = 0;
      if (has) {
        site = march_block(q, tc, bs) * uint32_t(kSiteBlock) + uint32_t(lane);  // below vol
        if (q == uint32_t(qb) || q % tc == 0) {
          const uint32_t sb = site >= vol3 ? site - vol3 : site + (vol - vol3);  // periodic
          const cplx<R>* __restrict__ wt = w.w + int64_t(3) * K * vol;
#pragma unroll
          for (int k = 0; k < K; ++k) car.u[k] = wt[int64_t(k) * vol + sb];
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            car.own[c] = at(sb, c);
            car.fw[c] = at(site, c);
          }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) own[c] = car.fw[c];
        stencil_site_c<R, LR, true, false>(w, site, own, sign, at, out, &car);
#pragma unroll
        for (int c = 0; c < 3; ++c) car.own[c] = own[c];
      }
      if (q == uint32_t(qb) && !first()) return;
      if (!has) return;
      body(site, out, own);
    }
  } else {
    Sweep sw = make_sweep(nblk, a.ord, WPB, g);
#pragma nounroll
    for (bool begin = true;; begin = false, sw.next()) {
      const bool has = sw.more();
      uint32_t site = 0;
      if (has) {
        site = uint32_t(sw.slice() * kSiteBlock) + uint32_t(lane);
        const uint32_t ss = site < vol ? site : vol - 1;  // lanes past the volume: unused
#pragma unroll
        for (int c = 0; c < 3; ++c) own[c] = at(ss, c);
        stencil_site<R, LR>(w, ss, own, sign, at, out);
      }
      if (begin && !first()) return;
      if (!has) return;
      if (site < vol) body(site, out, own);
    }
  }
}

// STREAM (FP64): u goes out with streaming stores (32^3 x 64: 240 -> 235 us; in complex64
// they make no difference).
template <class R, int LR, bool STREAM, bool MARCH, bool DIR>
__global__ __launch_bounds__(kBlock, 2) void k1_site(MsArgs a) {
  static_assert(!MARCH || LR == 2, "the march carries two-row links");
  // looked at after the first block's product: its loads do not wait for the state
  const int halt = a.st->rot[a.par].halt;
  if (k1_totals(a)) return;
  const Stencil<cplx<R>> w = pick_w<R>(a);
  cplx<R>* __restrict__ u = static_cast<cplx<R>*>(a.u);
  const double sigma0 = a.st->sigma0;
  double acc = 0.0;
  for_sites<R, LR, MARCH>(
      a, w, k1_vec<R, DIR>(a), 1, a.gd, [&] { return halt == 0; },
      [&](uint32_t site, const cplx<R>(&out)[3], const cplx<R>(&own)[3]) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          if constexpr (STREAM)
            st_stream(&u[c * w.vol + site], out[c]);
          else
            u[c * w.vol + site] = out[c];
          acc += k1_term<R, true, DIR>(out[c], own[c], sigma0);
        }
      });
  if (!halt) store_partial(region(a, 2 + a.par), acc);
}

template <class R, int LR, bool MARCH, bool DIR>
__global__ __launch_bounds__(kBlock, 2) void k2_site(MsArgs a) {
  static_assert(!MARCH || LR == 2, "the march carries two-row links");
  Early e;
  StepIn in;
  if (!k2_begin(a, e, in)) return;
  const Stencil<cplx<R>> w = pick_w<R>(a);
  const cplx<R>* __restrict__ r = rslot<R>(a, a.launch);
  cplx<R>* __restrict__ rn = rslot<R>(a, a.launch + 1);
  cplx<R>* __restrict__ s = static_cast<cplx<R>*>(a.s[0]);
  double2* __restrict__ x0 = x0_of(a);
  const double sigma0 = in.sigma0;
  StepPlan p;
  double acc = 0.0, ac = 0.0;
  for_sites<R, LR, MARCH>(
      a, w, static_cast<const cplx<R>*>(a.u), -1, a.gg,
      // the first block's product runs while the partials are on their way
      [&] { return k2_step(a, e, in, p); },
      [&](uint32_t site, const cplx<R>(&out)[3], const cplx<R>(&)[3]) {
        cplx<R> ro[3], so[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          ro[c] = ld_stream(&r[c * w.vol + site]);
          so[c] = ld_stream(&s[c * w.vol + site]);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const int64_t i = c * w.vol + site;
          cplx<R> sv, nv;
          row_step<R, DIR>(p, sigma0, out[c], ro[c], so[c], sv, nv);
          if (DIR)
            x0_step<R>(x0, 3 * int64_t(site) + c, p.a, so[c]);
          else
            st_stream(&s[i], sv);
          st_stream(&rn[i], nv);
          acc += norm2d<R>(nv);
          if (!DIR) ac += c_term<R>(nv, sv);
        }
      });
  if (p.stop) return;
  store_k2<DIR>(a, acc, ac);
}

// ---- the links of small lattices: one direction per wave --------------------------------------
// A workgroup takes blocks of 64 sites, its four waves a direction each, so that all loads
// of a site are in flight at once, over four times the waves; the directions meet in LDS,
// and each row is then finished by a lane of its own.  Used while every block can have a
// workgroup (prepare_impl): there an iteration is a chain of latencies.
// An iteration in FP64, one lane per site and here: 4^4 16.8 and 12.2 us, 12^4 23.4 and 15.1,
// 16^4 30.2 and 26.9, 18^4 37.9 and 43.0 (since the sums go by DPP: 8^4 11.8 -> 11.3, 12x10x14x18
// 15.6 -> 14.9; with K1 summing g_n and c_n for K2 a whole solve of 311 steps there 5.05 -> 4.97
// ms; 4^4 now has a form of its own below).
template <class R> using DirParts = cplx<R>[4][3][kWave];

// (m + sign D) v, and v itself (own), at this thread's row of block `blk` (thread t < 192: colour t / 64 of site t %
// 64; live: the row exists), after a barrier of its own; the caller's rows are free to use
// `part` again once every thread has passed the next one.
template <class R, int LR>
__device__ __forceinline__ cplx<R> split_row(const Stencil<cplx<R>>& w, const cplx<R>* __restrict__ v,
                                             int sign, int64_t blk, DirParts<R>& part, cplx<R>& own) {
  const uint32_t vol = uint32_t(w.vol);
  const int lane = threadIdx.x % kWave;
  const int mu = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kWave));
  const uint32_t site = uint32_t(blk * kSiteBlock) + uint32_t(lane);
  const uint32_t ss = site < vol ? site : vol - 1;  // lanes past the volume: unused
  const int c = mu < 3 ? mu : 0;
  own = v[int64_t(c) * vol + ss];
  cplx<R> h[3];
  stencil_dir<R, LR>(w, ss, mu, [&](uint32_t s, int k) { return v[int64_t(k) * vol + s]; }, h);
#pragma unroll
  for (int k = 0; k < 3; ++k) part[mu][k][lane] = h[k];
  __syncthreads();
  cplx<R> o = czero<R>();
  if (mu < 3) {
    const cplx<R> a = part[0][c][lane], b = part[1][c][lane], d = part[2][c][lane], e = part[3][c][lane];
    const R hx = (a.x + b.x) + (d.x + e.x), hy = (a.y + b.y) + (d.y + e.y), m = R(w.mass);
    o.x = fma(m, own.x, sign > 0 ? hx : -hx);
    o.y = fma(m, own.y, sign > 0 ? hy : -hy);
  }
  return o;
}

// This thread's row of a block, or -1.
__device__ __forceinline__ int64_t split_index(int64_t vol, int64_t blk) {
  const int64_t site = blk * kSiteBlock + int64_t(threadIdx.x % kWave);
  return threadIdx.x < 3 * kWave && site < vol ? int64_t(threadIdx.x / kWave) * vol + site : -1;
}

template <class R, int LR, bool DIR>
__global__ __launch_bounds__(kBlock) void k1_split(MsArgs a) {
  const int halt = a.st->rot[a.par].halt;
  if (k1_totals(a)) return;
  const Stencil<cplx<R>> w = pick_w<R>(a);
  const cplx<R>* __restrict__ r = k1_vec<R, DIR>(a);
  const double sigma0 = a.st->sigma0;
  cplx<R>* __restrict__ u = static_cast<cplx<R>*>(a.u);
  const int64_t nblk = (w.vol + kSiteBlock - 1) / kSiteBlock;
  __shared__ DirParts<R> part;
  double acc = 0.0;
  for (int64_t blk = logical_block(a.gd); blk < nblk; blk += a.gd) {
    cplx<R> own;
    const cplx<R> v = split_row<R, LR>(w, r, 1, blk, part, own);
    if (halt) return;
    const int64_t i = split_index(w.vol, blk);
    if (i >= 0) {
      u[i] = v;
      acc += k1_term<R, true, DIR>(v, own, sigma0);
    }
    __syncthreads();
  }
  store_partial(region(a, 2 + a.par), acc);
}

template <class R, int LR, bool DIR>
__global__ __launch_bounds__(kBlock) void k2_split(MsArgs a) {
  Early e;
  StepIn in;
  if (!k2_begin(a, e, in)) return;
  const Stencil<cplx<R>> w = pick_w<R>(a);
  const cplx<R>* __restrict__ u = static_cast<const cplx<R>*>(a.u);
  const cplx<R>* __restrict__ r = rslot<R>(a, a.launch);
  cplx<R>* __restrict__ rn = rslot<R>(a, a.launch + 1);
  cplx<R>* __restrict__ s = static_cast<cplx<R>*>(a.s[0]);
  double2* __restrict__ x0 = x0_of(a);
  const int64_t nblk = (w.vol + kSiteBlock - 1) / kSiteBlock;
  __shared__ DirParts<R> part;
  StepPlan p;
  p.stop = -1;
  double acc = 0.0, ac = 0.0;
  for (int64_t blk = logical_block(a.gg); blk < nblk; blk += a.gg) {
    const int64_t i = split_index(w.vol, blk);
    const cplx<R> rv = i >= 0 ? r[i] : czero<R>(), sv = i >= 0 ? s[i] : czero<R>();
    cplx<R> own;
    const cplx<R> q = split_row<R, LR>(w, u, -1, blk, part, own);
    if (p.stop < 0 && !k2_step(a, e, in, p)) return;
    if (i >= 0) {
      cplx<R> sn, nv;
      row_step<R, DIR>(p, in.sigma0, q, rv, sv, sn, nv);
      if (DIR)  // i is colour by colour
        x0_step<R>(x0, 3 * (i % w.vol) + i / w.vol, p.a, sv);
      else
        s[i] = sn;
      rn[i] = nv;
      acc += norm2d<R>(nv);
      if (!DIR) ac += c_term<R>(nv, sn);
    }
    __syncthreads();
  }
  store_k2<DIR>(a, acc, ac);
}

// ---- the smallest lattices: several iterations in one workgroup ---------------------------------
// Four lanes a site, a direction each: a lane keeps its link and forms both products with
// it; r and u lie in LDS, so an iteration's halves and sums are four barriers apart instead
// of two kernels.  c_n is summed at the end of a launch (in every step it costs registers that
// are not there, and the direction from the start a barrier: 2.53 and 2.10 ms for a solve at
// 4^4 that takes 2.04, and 1.97 without c_n), so P's form is looked at once in up to eight steps; where it is not
// positive in between, the direction is taken up there, by the pair of kernels.  The shifts' scalars of all a.span steps follow at the end, a shift per
// lane; the state goes on as from a.span launches of the pair.  For lattices whose sites one
// workgroup holds (256): an iteration in FP64 and mixed at 4^4 11.2 and 11.8 us with the
// pair, 7.0 and 7.6 here, of which 1.6 are the launches and the applications; two sites a
// lane, 4^3 x 6, took 27.8 (the links do not fit the registers) for 11.5.
constexpr int kSmallBlock = 1024;
constexpr int kSmallSites = kSmallBlock / 4;

// Sum over the workgroup, in every thread; a barrier.  Callers alternate between two `part`s.
__device__ __forceinline__ double small_sum(double v, double* part) {
  constexpr int W = kSmallBlock / kWave;
  v = group_sum<kWave>(v);
  if (threadIdx.x % kWave == 0) part[threadIdx.x / kWave] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < W; ++i) s += part[i];
  return s;
}

template <class R, int LR>
__global__ __launch_bounds__(kSmallBlock) void k_small(MsArgs a) {
  constexpr int K = 3 * LR;
  __shared__ cplx<R> rl[3][kSmallSites], ul[3][kSmallSites], back[3][kSmallBlock];
  __shared__ double part[2][kSmallBlock / kWave], hist[kMaxSteps][3];
  SolveState* st = a.st;
  StepIn in = step_in(a);
  const int pe = (a.launch + a.span) & 1;  // the state this launch leaves
  const int tid = threadIdx.x;
  if (in.halt) {
    if (tid == 0) st->rot[pe].halt = 1;
    return;
  }
  const Stencil<cplx<R>> w = pick_w<R>(a);
  const uint32_t vol = uint32_t(w.vol);
  const int mu = tid % 4;
  const cplx<R>* __restrict__ wm = w.w + int64_t(mu) * K * vol;
  cplx<R>* __restrict__ sg = static_cast<cplx<R>*>(a.s[0]);
  const uint32_t site = min(uint32_t(tid) / 4, vol - 1);
  const bool row = uint32_t(tid) / 4 < vol && mu < 3;  // this lane finishes the row of colour mu
  const int64_t i0 = int64_t(mu) * vol + site;
  uint32_t fwd = site, bwd = site;
  R te = R(2);
  {
    uint32_t rem = site, par = 0;
#pragma unroll
    for (int nu = 0; nu < 4; ++nu) {
      const uint32_t L = uint32_t(w.L[nu]), sd = uint32_t(w.stride[nu]);
      const uint32_t q = rem / L, xm = rem - q * L;
      rem = q;
      if (nu == mu) {
        te = (par & 1u) ? R(-2) : R(2);
        fwd = xm == L - 1 ? site - (L - 1) * sd : site + sd;
        bwd = xm == 0 ? site + (L - 1) * sd : site - sd;
      }
      par += xm;
    }
  }
  cplx<R> U[9], rr = czero<R>(), ss = czero<R>();
#pragma unroll
  for (int k = 0; k < K; ++k) U[k] = wm[k * vol + site];
  if (row) {
    rr = rslot<R>(a, a.launch)[i0];
    ss = sg[i0];
    rl[mu][site] = rr;
  }
  if constexpr (LR == 2) third_row<R>(U, te);
  // This lane's row of (m + sign D) v, v in LDS and own its value there.  A lane forms both
  // products with its one link, U v(s + mu) for its site and U^H v(s) for the site ahead.
  auto product = [&](const cplx<R>(&v)[3][kSmallSites], int sign, const cplx<R>& own) {
    cplx<R> h[3], g[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) h[c] = g[c] = czero<R>();
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const cplx<R> f = v[j][fwd], o = v[j][site];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        cfma<R>(h[c], U[3 * c + j], f);
        cfma_conj<R>(g[c], U[3 * j + c], o);
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) back[c][tid] = g[c];
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const cplx<R> b = back[c][4 * bwd + mu];
      h[c].x = group_sum<4>(h[c].x - b.x);
      h[c].y = group_sum<4>(h[c].y - b.y);
    }
    const cplx<R> q = mu == 0 ? h[0] : mu == 1 ? h[1] : h[2];
    const R m = R(w.mass);
    return cplx<R>{fma(m, own.x, sign > 0 ? q.x : -q.x), fma(m, own.y, sign > 0 ? q.y : -q.y)};
  };
  double v = 0.0, c = 0.0;
  for (int i = tid; i < a.gg; i += kSmallBlock) {
    v += region(a, a.par)[i];
    c += region(a, 6 + a.par)[i];
  }
  c = group_sum<kWave>(c);
  if (tid % kWave == 0) part[0][tid / kWave] = c;
  double g = small_sum(v, part[1]);  // and r is in LDS
  c = 0.0;
#pragma unroll
  for (int i = 0; i < kSmallBlock / kWave; ++i) c += part[0][i];
  const int n0 = in.n;
  int done = 0, stop = 0;
  double a1 = in.a1, dev = 0.0;
  for (; done < a.span; ++done) {
    double acc = 0.0;
    const cplx<R> uu = product(rl, 1, rr);
    if (row) {
      ul[mu][site] = uu;
      acc = norm2d<R>(uu);
    }
    const double d = small_sum(acc, part[0]);
    const StepPlan p = step_plan(a, in, Sums{g, d, c}, done == 0);
    if (in.n == 0) in.bn2 = g;
    stop = p.stop;
    if (stop) break;
    if (done == 0) dev = p.off / p.P;
    cplx<R>* __restrict__ rn = rslot<R>(a, a.launch + done + 1);
    const cplx<R> q = product(ul, -1, uu);
    acc = 0.0;
    if (row) {
      cplx<R> sn, nv;
      row_step<R>(p, in.sigma0, q, rr, ss, sn, nv);
      ss = sn;
      rr = nv;
      rl[mu][site] = nv;
      rn[i0] = nv;
      acc = norm2d<R>(nv);
    }
    if (tid == 0) {
      hist[done][0] = g;
      hist[done][1] = p.a;
      hist[done][2] = p.b;
    }
    in.g1 = g;
    in.a1 = p.a;
    in.P1 = p.P;
    in.n += 1;
    g = small_sum(acc, part[1]);
    in.ru = 0;
  }
  if (row) sg[i0] = ss;
  if (done > 0) c = small_sum(row ? c_term<R>(rr, ss) : 0.0, part[stop ? 1 : 0]);
  for (int i = tid; i < a.gg; i += kSmallBlock) {
    region(a, pe)[i] = i == 0 ? g : 0.0;
    region(a, 6 + pe)[i] = i == 0 ? c : 0.0;
  }
  if (tid >= kWave) return;
  const int j = tid;
  const RotState& rs = st->rot[a.par];
  RotState& nx = st->rot[pe];
  const int m = rs.m, fresh = rs.fresh;
  const bool flushed = a.flushed || (a.ru_check && st->ru_flag);
  const int m0 = flushed ? 0 : m;
  const double eps2 = in.tol2 * in.bn2;
  if (j < st->ns) {
    ShiftSteps h;
    h.load(rs, st->s[j], j);
    for (int k = 0; k < done; ++k) {
      const double ak = hist[k][1];
      if (h.step(j, n0 + k, m0 + k, true, st->freeze != 0, hist[k][0], eps2, ak, hist[k][2], a1))
        st->freeze_iter[j] = n0 + k;
      a1 = ak;
    }
    if (stop && h.step(j, in.n, m0 + done, false, st->freeze != 0, g, eps2, 0.0, 0.0, a1))
      st->freeze_iter[j] = in.n;
    h.store(nx, j);
  }
  if (j == 0) {
    if (n0 == 0) st->bnorm2 = in.bn2;
    nx.g = in.g1;
    nx.a = in.a1;
    nx.P = in.P1;
    nx.iter = in.n;
    nx.launch = a.launch + done;
    nx.m = m0 + done;
    nx.fresh = flushed ? 0 : fresh;
    nx.halt = stop ? 1 : 0;
    if (dev > st->dev) st->dev = dev;
    if (stop) sequence_halts(a, pe, in.n, Sums{g, 0.0, c}, eps2, stop);
  }
}

// ---- the composed steps of every shift: x_j and p_j -------------------------------------------
// x_j += cx[0] p_j + sum_{k<m} cx[k+1] r_k, p_j <- cp[0] p_j + sum_{k<m} cp[k+1] r_k, the r_k
// being the m composed steps' residuals; before the first application x_j and p_j are zero
// and are not read.  One pass for all shifts, one row per lane (x and p_j in the caller's
// row order).  Bound by memory: 64 bytes a row and shift in FP64, 16 a kept residual.
// when: 0 always (unless the sequence has halted), 1 for a reliable update that is due
// (r_n's g has fallen by kRuDelta2 since the last one, or a.ru_force), 2 at the end.
struct FlushPlan {
  double cx[kMaxSteps + 1][kMaxShifts], cp[kMaxSteps + 1][kMaxShifts];
  int64_t xo[kMaxShifts], po[kMaxShifts];
  int nact, m, first, fresh;
};

// Shifts whose x_j and p_j loads are issued together.
constexpr int kUpdGroup = 4;

template <class R, bool COLOURS>
__global__ __launch_bounds__(kBlock) void k_flush(MsArgs a, int par, int when) {
  SolveState* st = a.st;
  const int at = when == 2 ? st->fin : par;
  const RotState& rs = st->rot[at];
  if (when != 2 && rs.halt) {
    if (when == 1 && blockIdx.x == 0 && threadIdx.x == 0) st->ru_flag = 0;
    return;
  }
  int flushed = a.flushed;
  if (when == 1) {
    const int which[1] = {a.par};
    double sum[1];
    region_sums(a, which, a.gg, sum);
    const double g = sum[0];
    const bool due = a.ru_force || g < kRuDelta2 * st->R_ru;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      st->ru_flag = due ? 1 : 0;
      st->ru_g = g;
    }
    if (!due) return;
  } else {
    flushed = 0;
  }
  if (flushed || (rs.m == 0 && !rs.fresh)) return;
  __shared__ FlushPlan pl;
  const int j = threadIdx.x;
  if (j < kWave) {
    // with the direction K2 keeps x_0 and p_0
    const bool list = j < st->ns && ((rs.m > 0 && rs.took[j]) || rs.fresh) && !(a.dir && j == 0);
    const uint64_t mask = __ballot(list);
    if (list) {
      const int pos = __popcll(mask & ((uint64_t(1) << j) - 1));
#pragma unroll
      for (int i = 0; i <= kMaxSteps; ++i) {
        pl.cx[i][pos] = rs.cx[i][j];
        pl.cp[i][pos] = rs.cp[i][j];
      }
      pl.xo[pos] = int64_t(st->orig[j]) * a.n;
      pl.po[pos] = int64_t(j) * a.n;
    }
    if (j == 0) {
      pl.nact = __popcll(mask);
      pl.m = rs.m;
      pl.first = rs.launch - rs.m;
      pl.fresh = rs.fresh;
      if (blockIdx.x == 0) {
        constexpr int ph = sizeof(R) == 4 ? 1 : 0;
        st->n_upd[ph] += pl.nact;
        st->n_kept[ph] += pl.m;
        if (a.sample >= 0 && a.sample < kMaxSamples) {
          st->smp_nact[a.sample] = pl.nact;
          st->smp_m[a.sample] = pl.m;
        }
      }
    }
  }
  __syncthreads();
  const int m = pl.m, nact = pl.nact, fresh = pl.fresh;
  cplx<R>* __restrict__ pk = static_cast<cplx<R>*>(a.pk);
  double2* __restrict__ x = a.x;
  const cplx<R>* rk[kMaxSteps];
#pragma unroll
  for (int k = 0; k < kMaxSteps; ++k) rk[k] = rslot<R>(a, pl.first + (k < m ? k : 0));
  const int64_t vol = a.n / 3;
  int64_t beg, end;
  block_range(a.n, kBlock, beg, end);
  for (int64_t i = beg + threadIdx.x; i < end; i += kBlock) {
    const int64_t ri = COLOURS ? (i % 3) * vol + i / 3 : i;  // the residuals' row
    double2 rv[kMaxSteps];
#pragma unroll
    for (int k = 0; k < kMaxSteps; ++k)
      rv[k] = k < m ? to_d(ld_stream(&rk[k][ri])) : double2{0.0, 0.0};
    auto group = [&](int q, int cnt, auto full) {
      cplx<R> pj[kUpdGroup];
      double2 xj[kUpdGroup];
#pragma unroll
      for (int u = 0; u < kUpdGroup; ++u) {
        pj[u] = czero<R>();
        xj[u] = double2{0.0, 0.0};
        if ((decltype(full)::value || u < cnt) && !fresh) {
          pj[u] = ld_stream(&pk[pl.po[q + u] + i]);
          xj[u] = ld_stream(&x[pl.xo[q + u] + i]);
        }
      }
#pragma unroll
      for (int u = 0; u < kUpdGroup; ++u) {
        if (decltype(full)::value || u < cnt) {
          const int c = q + u;
          const double2 pd = to_d(pj[u]);
          double2 xv{fma(pl.cx[0][c], pd.x, xj[u].x), fma(pl.cx[0][c], pd.y, xj[u].y)};
          double2 np{pl.cp[0][c] * pd.x, pl.cp[0][c] * pd.y};
#pragma unroll
          for (int k = 0; k < kMaxSteps; ++k) {
            if (k < m) {
              const double cx = pl.cx[k + 1][c], cp = pl.cp[k + 1][c];
              xv.x = fma(cx, rv[k].x, xv.x);
              xv.y = fma(cx, rv[k].y, xv.y);
              np.x = fma(cp, rv[k].x, np.x);
              np.y = fma(cp, rv[k].y, np.y);
            }
          }
          st_stream(&x[pl.xo[c] + i], xv);
          st_stream(&pk[pl.po[c] + i], from_d<R>(np));
        }
      }
    };
    int q = 0;
    for (; q + kUpdGroup <= nact; q += kUpdGroup) group(q, kUpdGroup, std::true_type{});
    if (q < nact) group(q, nact - q, std::false_type{});
  }
}

// ---- start: r_0 = b, s = 0 and g_0's partials (x_j and p_j start unwritten) ----------------
template <bool COLOURS>
__global__ __launch_bounds__(kBlock) void k_init(MsArgs a) {
  double2* __restrict__ r = rslot<double>(a, a.launch);
  double2* __restrict__ s = static_cast<double2*>(a.s[0]);
  const int64_t vol = a.n / 3;
  int64_t beg, end;
  block_range(a.n, kBlock, beg, end);
  double acc = 0.0;
  for (int64_t i = beg + threadIdx.x; i < end; i += kBlock) {
    const double2 bv = a.b[i];
    r[COLOURS ? (i % 3) * vol + i / 3 : i] = bv;
    s[i] = double2{0.0, 0.0};
    acc += fma(bv.x, bv.x, bv.y * bv.y);
  }
  store_partial(region(a, a.par), acc);
}

// ---- end of the FP64 phase of a mixed solve: r, s and the p_j to complex64 --------------------
__global__ __launch_bounds__(kBlock) void k_switch(MsArgs a64, MsArgs a32, int ns, int herm) {
  SolveState* st = a64.st;
  const RotState& fin = st->rot[st->fin];
  const int64_t n = a64.n;
  const double2* __restrict__ r = rslot<double>(a64, fin.launch);
  // the buffer of s the halted iteration would have read: A given alternates two
  const int from = herm ? st->fin ^ 1 : 0, to = herm ? a64.par : 0;
  const double2* __restrict__ s = static_cast<const double2*>(a64.s[from]);
  const double2* __restrict__ pk = static_cast<const double2*>(a64.pk);
  float2* __restrict__ r32 = rslot<float>(a32, a32.launch);
  float2* __restrict__ s32 = static_cast<float2*>(a32.s[to]);
  float2* __restrict__ pk32 = static_cast<float2*>(a32.pk);
  const int64_t total = int64_t(ns + 1) * n;  // r and s, then ns directions
  for (int64_t idx = blockIdx.x * int64_t(kBlock) + threadIdx.x; idx < total;
       idx += int64_t(gridDim.x) * kBlock) {
    if (idx < n) {
      r32[idx] = from_d<float>(r[idx]);
      s32[idx] = from_d<float>(s[idx]);
    } else {
      pk32[idx - n] = from_d<float>(pk[idx - n]);
    }
  }
  // partials of g and c: the sums the halted iteration formed
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < kMaxGrid; i += kBlock) {
      region(a64, a64.par)[i] = i ? 0.0 : st->R;
      region(a64, 6 + a64.par)[i] = i ? 0.0 : st->c;
    }
  }
}

// The state of the halted sequence's next iteration, a.launch of parity a.par, from the halted
// one's (which may be the same of the two: a lane reads before it writes): the complex64
// phase's first, or (`replaced`) one with the direction taken up, whose r_n may differ from
// the recursive one.
__global__ __launch_bounds__(kBlock) void k_go_on(MsArgs a, int replaced) {
  SolveState* st = a.st;
  const RotState& fin = st->rot[st->fin];
  RotState& rs = st->rot[a.par];
  const int j = threadIdx.x;
  if (j < kMaxShifts) {
    rs.zeta[j] = fin.zeta[j];
    rs.zeta_prev[j] = fin.zeta_prev[j];
    // repeats of the driving shift stopped with it and go on with it
    rs.active[j] = fin.active[j] || (replaced && j < st->ns && st->s[j] == 0.0);
    rs.took[j] = 0;
  }
  if (j == 0) {
    rs.g = fin.g;
    rs.a = fin.a;
    rs.P = fin.P;
    rs.iter = fin.iter;
    rs.launch = a.launch;
    rs.m = 0;
    rs.fresh = 0;
    rs.halt = 0;
    if (replaced) {
      st->ru_flag = 1;
      st->ru_g = st->R;
    } else {
      st->sw2 = 0.0;
      st->R_ru = st->R;
    }
  }
}

// p_{n-1}, kept as the driving system's direction until now, in the order of the ring.
template <class R, bool COLOURS> __global__ __launch_bounds__(kBlock) void k_load_p(MsArgs a) {
  const cplx<R>* __restrict__ pk = static_cast<const cplx<R>*>(a.pk);
  cplx<R>* __restrict__ p = static_cast<cplx<R>*>(a.s[0]);
  const int64_t vol = a.n / 3;
  for (int64_t i = blockIdx.x * int64_t(kBlock) + threadIdx.x; i < a.n; i += int64_t(gridDim.x) * kBlock)
    p[COLOURS ? (i % 3) * vol + i / 3 : i] = pk[i];
}

// r_n = b - ax into the ring slot of launch a.launch; its g's partials.
template <class R, bool COLOURS>
__global__ __launch_bounds__(kBlock) void k_load_r(MsArgs a, const double2* __restrict__ ax) {
  cplx<R>* __restrict__ r = rslot<R>(a, a.launch);
  const int64_t vol = a.n / 3;
  int64_t beg, end;
  block_range(a.n, kBlock, beg, end);
  double acc = 0.0;
  for (int64_t i = beg + threadIdx.x; i < end; i += kBlock) {
    const double2 bv = a.b[i], av = ax[i];
    const cplx<R> v = from_d<R>(double2{bv.x - av.x, bv.y - av.y});
    r[COLOURS ? (i % 3) * vol + i / 3 : i] = v;
    acc += norm2d<R>(v);
  }
  store_partial(region(a, a.par), acc);
}

// ---- reliable update: r_n = b - (A + sigma0) x_0 in FP64, before iteration n ------------------
// k_flush has brought x_0 up to date and decided whether it runs (st->ru_flag).  The last
// workgroup replaces g_n's partials and c_n's (with the direction, which s then is, unused); a
// non-finite residual ends the sequence in iteration n (breakdown).
__device__ __forceinline__ bool ru_runs(const MsArgs& a) {
  return a.st->ru_flag != 0 && !a.st->rot[a.par].halt;
}

__device__ void ru_finish(const MsArgs& a, double acc, double dot) {
  SolveState* st = a.st;
  double v[2] = {acc, dot};
  block_sum_k<kBlock, 2>(v);
  if (threadIdx.x == 0) {
    store_agent(&region(a, 4)[blockIdx.x], v[0]);
    store_agent(&region(a, 5)[blockIdx.x], v[1]);
  }
  if (!arrive_last(a.sc.tickets + 2 * kTicketSite)) return;
  const double Rt = sum_partials(region(a, 4), gridDim.x, 1, 0);
  const double ct = sum_partials(region(a, 5), gridDim.x, 1, 0);
  for (int i = threadIdx.x; i < a.gg; i += kBlock) {
    region(a, a.par)[i] = i ? 0.0 : Rt;
    region(a, 6 + a.par)[i] = i ? 0.0 : ct;
  }
  if (threadIdx.x == 0) {
    st->R_ru = Rt;
    st->n_reliable += 1;
  }
}

// One row: r_n from b, (A x_0)_row and x_0; |r_n|^2 and Re(r_n^H s).
template <class R>
__device__ __forceinline__ cplx<R> ru_row(const double2& bv, const double2& q, const double2& xv,
                                          double sigma0, const cplx<R>& s, double& acc, double& dot) {
  const double2 rt{bv.x - q.x - sigma0 * xv.x, bv.y - q.y - sigma0 * xv.y};
  const double2 sd = to_d(s);
  acc += fma(rt.x, rt.x, rt.y * rt.y);
  dot += rt.x * sd.x + rt.y * sd.y;
  return from_d<R>(rt);
}

template <class R> __device__ __forceinline__ const cplx<R>* ru_s(const MsArgs& a) {
  return static_cast<const cplx<R>*>(a.s[a.s[1] ? a.par : 0]);
}

template <int L>
__global__ __launch_bounds__(kBlock) void k_ru_first(MsArgs a) {
  // t64 = M x_0 (A = M^H M) -- first half of the FP64 operator
  if (!ru_runs(a)) return;
  const double2* __restrict__ x0 = a.x + int64_t(a.st->orig[0]) * a.n;
  constexpr int GPB = kBlock / L;
  const int lane = threadIdx.x % L, grp = threadIdx.x / L;
  int64_t beg, end;
  block_range(a.n, GPB, beg, end);
  for (int64_t row = beg + grp; row < end; row += GPB) {
    const double2 v = row_dot<double, L>(a.m64, x0, row, lane);
    if (lane == 0) a.t64[row] = v;
  }
}

template <class R, int L, bool MHM>
__global__ __launch_bounds__(kBlock) void k_ru_second(MsArgs a) {
  if (!ru_runs(a)) return;
  const double2* __restrict__ x0 = a.x + int64_t(a.st->orig[0]) * a.n;
  cplx<R>* __restrict__ r = rslot<R>(a, a.launch);
  const cplx<R>* __restrict__ s = ru_s<R>(a);
  constexpr int GPB = kBlock / L;
  const int lane = threadIdx.x % L, grp = threadIdx.x / L;
  int64_t beg, end;
  block_range(a.n, GPB, beg, end);
  double acc = 0.0, dot = 0.0;
  for (int64_t row = beg + grp; row < end; row += GPB) {
    const double2 q = MHM ? row_dot<double, L>(a.mh64, a.t64, row, lane)
                          : row_dot<double, L>(a.m64, x0, row, lane);
    if (lane == 0) r[row] = ru_row<R>(a.b[row], q, x0[row], a.st->sigma0, s[row], acc, dot);
  }
  ru_finish(a, acc, dot);
}

// The same on the sliced ELLPACK copies: one row per lane, one slice per wavefront.
__global__ __launch_bounds__(kBlock) void k_ru_first_s(MsArgs a) {
  if (!ru_runs(a)) return;
  const double2* __restrict__ x0 = a.x + int64_t(a.st->orig[0]) * a.n;
  constexpr int SPB = kBlock / kSlice;
  const int lane = threadIdx.x % kSlice;
  const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kSlice));
  int64_t beg, end;
  block_range(a.nslices, SPB, beg, end);
  for (int64_t sl = beg + wv; sl < end; sl += SPB) {
    const int64_t row = sl * kSlice + lane;
    const int64_t rr = row < a.n ? row : a.n - 1;
    double2 v = sell_row<double>(a.s64, x0, sl, lane);
    cfma<double>(v, a.s64.diag[rr], x0[rr]);
    if (row < a.n) a.t64[row] = v;
  }
}

template <class R, bool MHM>
__global__ __launch_bounds__(kBlock) void k_ru_second_s(MsArgs a) {
  if (!ru_runs(a)) return;
  const double2* __restrict__ x0 = a.x + int64_t(a.st->orig[0]) * a.n;
  cplx<R>* __restrict__ r = rslot<R>(a, a.launch);
  const cplx<R>* __restrict__ s = ru_s<R>(a);
  const Sell<double2> m = MHM ? a.sh64 : a.s64;
  const double2* __restrict__ in = MHM ? a.t64 : x0;
  constexpr int SPB = kBlock / kSlice;
  const int lane = threadIdx.x % kSlice;
  const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kSlice));
  int64_t beg, end;
  block_range(a.nslices, SPB, beg, end);
  double acc = 0.0, dot = 0.0;
  for (int64_t sl = beg + wv; sl < end; sl += SPB) {
    const int64_t row = sl * kSlice + lane;
    const int64_t rr = row < a.n ? row : a.n - 1;
    double2 q = sell_row<double>(m, in, sl, lane);
    cfma<double>(q, m.diag[rr], in[rr]);
    if (row < a.n) r[row] = ru_row<R>(a.b[row], q, x0[row], a.st->sigma0, s[row], acc, dot);
  }
  ru_finish(a, acc, dot);
}

// The same on the links (LR rows per link), one site per lane: t64 = M x_0 (in the caller's
// row order, as x_0 and b), then r_n = b - M^H t64 - sigma0 x_0 (colour by colour).
template <class F>
__device__ __forceinline__ void ru_sites(uint32_t vol, F body) {
  constexpr int WPB = kBlock / kWave;
  const int lane = threadIdx.x % kWave;
  const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kWave));
  int64_t beg, end;
  block_range((int64_t(vol) + kSiteBlock - 1) / kSiteBlock, WPB, beg, end);
  for (int64_t blk = beg + wv; blk < end; blk += WPB) {
    const uint32_t site = uint32_t(blk * kSiteBlock) + uint32_t(lane);
    body(site < vol ? site : vol - 1, site < vol);  // lanes past the volume: unused
  }
}

template <int LR>
__global__ __launch_bounds__(kBlock) void k_ru_first_site(MsArgs a) {
  if (!ru_runs(a)) return;
  const double2* __restrict__ x0 = a.x + int64_t(a.st->orig[0]) * a.n;
  const Stencil<double2> w = a.w64;
  ru_sites(uint32_t(w.vol), [&](uint32_t site, bool live) {
    const int64_t r0 = 3 * int64_t(site);
    double2 own[3], v[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) own[c] = x0[r0 + c];
    stencil_site<double, LR>(w, site, own, 1,
                             [&](uint32_t t, int c) { return x0[3 * int64_t(t) + c]; }, v);
    if (live) {
#pragma unroll
      for (int c = 0; c < 3; ++c) a.t64[r0 + c] = v[c];
    }
  });
}

template <class R, int LR>
__global__ __launch_bounds__(kBlock) void k_ru_second_site(MsArgs a) {
  if (!ru_runs(a)) return;
  const double2* __restrict__ x0 = a.x + int64_t(a.st->orig[0]) * a.n;
  const double2* __restrict__ u = a.t64;
  cplx<R>* __restrict__ r = rslot<R>(a, a.launch);
  const cplx<R>* __restrict__ s = ru_s<R>(a);
  const Stencil<double2> w = a.w64;
  double acc = 0.0, dot = 0.0;
  ru_sites(uint32_t(w.vol), [&](uint32_t site, bool live) {
    const int64_t r0 = 3 * int64_t(site);
    double2 own[3], q[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) own[c] = u[r0 + c];
    stencil_site<double, LR>(w, site, own, -1,
                             [&](uint32_t t, int c) { return u[3 * int64_t(t) + c]; }, q);
    if (live) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const int64_t i = c * w.vol + site;
        r[i] = ru_row<R>(a.b[r0 + c], q[c], x0[r0 + c], a.st->sigma0, s[i], acc, dot);
      }
    }
  });
  ru_finish(a, acc, dot);
}

// ---- verification: FP64 true residual norms of up to 8 solutions ---------------------
constexpr int kVerifyChunk = 8;

template <int L>
__device__ __forceinline__ void row_dot_multi(const Csr<double2>& m, const double2* __restrict__ x,
                                              int64_t n, int kc, int64_t row, int lane,
                                              double2 (&acc)[kVerifyChunk]) {
#pragma unroll
  for (int q = 0; q < kVerifyChunk; ++q) acc[q] = double2{0.0, 0.0};
  const int32_t beg = m.rowptr[row], end = m.rowptr[row + 1];
  for (int32_t j = beg + lane; j < end; j += L) {
    const int32_t c = m.col[j];
    const double2 v = m.val[j];
#pragma unroll
    for (int q = 0; q < kVerifyChunk; ++q)
      if (q < kc) cfma<double>(acc[q], v, x[int64_t(q) * n + c]);
  }
#pragma unroll
  for (int q = 0; q < kVerifyChunk; ++q) acc[q] = group_sum_c<L, double>(acc[q]);
}

template <int L>
__global__ __launch_bounds__(kBlock) void k_verify_first(Csr<double2> m, const double2* x, int64_t n,
                                                         int kc, double2* u) {
  constexpr int GPB = kBlock / L;
  const int lane = threadIdx.x % L, grp = threadIdx.x / L;
  int64_t beg, end;
  block_range(n, GPB, beg, end);
  double2 acc[kVerifyChunk];
  for (int64_t row = beg + grp; row < end; row += GPB) {
    row_dot_multi<L>(m, x, n, kc, row, lane, acc);
    if (lane == 0) {
#pragma unroll
      for (int q = 0; q < kVerifyChunk; ++q)
        if (q < kc) u[int64_t(q) * n + row] = acc[q];
    }
  }
}

struct VerifyArgs {
  Csr<double2> m;        // M^H (MHM) or A (HERM)
  Sell<double2> s;       // its sliced ELLPACK copy (the SELL kernels)
  int64_t nslices;
  const double2* in;     // U = M X (MHM) or X (HERM), chunk of kc vectors
  const double2* x;      // X, chunk of kc vectors
  const double2* b;
  double sig[kVerifyChunk];
  int64_t n;
  int kc;
  double* partial;
  unsigned* ticket;
  double* out;           // res2 of the chunk
};

// Per-chunk norms: workgroup partials, then the last workgroup's totals in out[0..kc).
__device__ void verify_finish(const VerifyArgs& v, double (&nrm)[kVerifyChunk]) {
  block_sum_k<kBlock, kVerifyChunk>(nrm);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < kVerifyChunk; ++q) store_agent(&v.partial[blockIdx.x * kVerifyChunk + q], nrm[q]);
  }
  if (!arrive_last(v.ticket)) return;
  for (int q = 0; q < v.kc; ++q) {
    const double s = sum_partials(v.partial, gridDim.x, kVerifyChunk, q);
    if (threadIdx.x == 0) v.out[q] = s;
  }
}

template <int L>
__global__ __launch_bounds__(kBlock) void k_verify_second(VerifyArgs v) {
  constexpr int GPB = kBlock / L;
  const int lane = threadIdx.x % L, grp = threadIdx.x / L;
  int64_t beg, end;
  block_range(v.n, GPB, beg, end);
  double2 acc[kVerifyChunk];
  double nrm[kVerifyChunk];
#pragma unroll
  for (int q = 0; q < kVerifyChunk; ++q) nrm[q] = 0.0;
  for (int64_t row = beg + grp; row < end; row += GPB) {
    row_dot_multi<L>(v.m, v.in, v.n, v.kc, row, lane, acc);
    if (lane == 0) {
      const double2 bv = v.b[row];
#pragma unroll
      for (int q = 0; q < kVerifyChunk; ++q) {
        if (q < v.kc) {
          const double2 xv = v.x[int64_t(q) * v.n + row];
          const double rx = bv.x - acc[q].x - v.sig[q] * xv.x;
          const double ry = bv.y - acc[q].y - v.sig[q] * xv.y;
          nrm[q] += fma(rx, rx, ry * ry);
        }
      }
    }
  }
  verify_finish(v, nrm);
}

// One row per lane on the sliced ELLPACK copies: u_q = M x_q, then the residual norms.
__global__ __launch_bounds__(kBlock) void k_verify_first_s(Sell<double2> m, const double2* x,
                                                           int64_t n, int64_t nslices, int kc,
                                                           double2* u) {
  constexpr int SPB = kBlock / kSlice;
  const int lane = threadIdx.x % kSlice;
  const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kSlice));
  const double2* xs[kVerifyChunk];
#pragma unroll
  for (int q = 0; q < kVerifyChunk; ++q) xs[q] = x + int64_t(q < kc ? q : 0) * n;
  int64_t beg, end;
  block_range(nslices, SPB, beg, end);
  for (int64_t sl = beg + wv; sl < end; sl += SPB) {
    const int64_t row = sl * kSlice + lane;
    const int64_t rr = row < n ? row : n - 1;
    double2 acc[kVerifyChunk];
    sell_row_multi<double, kVerifyChunk, 1>(m, xs, kc, sl, lane, acc);
    const double2 d = m.diag[rr];
#pragma unroll
    for (int q = 0; q < kVerifyChunk; ++q) {
      if (q < kc) {
        cfma<double>(acc[q], d, xs[q][rr]);
        if (row < n) u[int64_t(q) * n + row] = acc[q];
      }
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_verify_second_s(VerifyArgs v) {
  constexpr int SPB = kBlock / kSlice;
  const int lane = threadIdx.x % kSlice;
  const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kSlice));
  const double2* ins[kVerifyChunk];
#pragma unroll
  for (int q = 0; q < kVerifyChunk; ++q) ins[q] = v.in + int64_t(q < v.kc ? q : 0) * v.n;
  double nrm[kVerifyChunk];
#pragma unroll
  for (int q = 0; q < kVerifyChunk; ++q) nrm[q] = 0.0;
  int64_t beg, end;
  block_range(v.nslices, SPB, beg, end);
  for (int64_t sl = beg + wv; sl < end; sl += SPB) {
    const int64_t row = sl * kSlice + lane;
    const int64_t rr = row < v.n ? row : v.n - 1;
    double2 acc[kVerifyChunk];
    sell_row_multi<double, kVerifyChunk, 1>(v.s, ins, v.kc, sl, lane, acc);
    const double2 d = v.s.diag[rr];
    if (row < v.n) {
      const double2 bv = v.b[row];
#pragma unroll
      for (int q = 0; q < kVerifyChunk; ++q) {
        if (q < v.kc) {
          cfma<double>(acc[q], d, ins[q][row]);
          const double2 xv = v.x[int64_t(q) * v.n + row];
          const double rx = bv.x - acc[q].x - v.sig[q] * xv.x;
          const double ry = bv.y - acc[q].y - v.sig[q] * xv.y;
          nrm[q] += fma(rx, rx, ry * ry);
        }
      }
    }
  }
  verify_finish(v, nrm);
}

// ---- the operator applied on its own: out = (A + shift) in ----------------------------
// One kernel per half of A.  The first half reads the caller's vector (converted to the
// working precision where it is gathered), the last one adds shift * in and writes
// complex128.  `in` and `out` may be the same buffer: for A = M^H M the last half gathers
// the product of the first and reads `in` at its own rows only, before it writes them;
// for a given A the launcher keeps the product apart when the two overlap.

// Sizes from which FP64 products read the links (sites) and the sliced copy (rows) instead
// of the CSR.  Below, the product is a chain of latencies, and the CSR's eight lanes per
// row have the most of them in flight: per call, links / CSR 44 / 49 us at 16^3 x 8, 46 / 49 at
// 20 x 18 x 12 x 9, 47 / 61 at 16^4, 125 / 317 at 24^4; sliced copy / CSR 28.4 / 27.5 at 8^4,
// 28.2 / 29.1 at 8^3 x 16, 34.3 / 38.3 at 12^4.
#ifndef MSC_APPLY_SITES_MIN
#define MSC_APPLY_SITES_MIN 16384
#endif
#ifndef MSC_APPLY_SELL_MIN
#define MSC_APPLY_SELL_MIN 16384
#endif
constexpr int64_t kApplySitesMin = MSC_APPLY_SITES_MIN;
constexpr int64_t kApplySellMin = MSC_APPLY_SELL_MIN;

// x at a gathered column, in the working precision R.
template <class R, class V>
__device__ __forceinline__ cplx<R> in_prec(const V& v) { return from_d<R>(to_d(v)); }

__device__ __forceinline__ double2 with_shift(const double2& q, double shift, const double2& xv) {
  return double2{q.x + shift * xv.x, q.y + shift * xv.y};
}

// One CSR row times x, L lanes per row, as row_dot but with x in its own precision.
template <class R, int L, class V>
__device__ __forceinline__ cplx<R> row_dot_in(const Csr<cplx<R>>& m, const V* __restrict__ x,
                                              int64_t row, int lane) {
  const int32_t beg = m.rowptr[row], end = m.rowptr[row + 1];
  cplx<R> acc = czero<R>();
  for (int32_t base = beg; base < end; base += kChunk * L) {
    int32_t c[kChunk];
    cplx<R> v[kChunk], xv[kChunk];
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      const int32_t j = base + lane + u * L;
      const bool ok = j < end;
      c[u] = ok ? m.col[j] : 0;
      v[u] = ok ? m.val[j] : czero<R>();
    }
#pragma unroll
    for (int u = 0; u < kChunk; ++u) xv[u] = in_prec<R>(x[c[u]]);
#pragma unroll
    for (int u = 0; u < kChunk; ++u) cfma<R>(acc, v[u], xv[u]);
  }
  return group_sum_c<L, R>(acc);
}

// y = m x (LAST false), or out = m x + shift in (LAST true), from the CSR.
template <class R, int L, bool LAST, class V>
__global__ __launch_bounds__(kBlock) void k_apply_csr(Csr<cplx<R>> m, const V* x, cplx<R>* y,
                                                      const double2* in, double2* out,
                                                      double shift, int64_t n) {
  constexpr int GPB = kBlock / L;
  const int lane = threadIdx.x % L, grp = threadIdx.x / L;
  int64_t beg, end;
  block_range(n, GPB, beg, end);
  for (int64_t row = beg + grp; row < end; row += GPB) {
    const cplx<R> v = row_dot_in<R, L>(m, x, row, lane);
    if (lane == 0) {
      if constexpr (LAST)
        out[row] = with_shift(to_d(v), shift, in[row]);
      else
        y[row] = v;
    }
  }
}

// The same in FP64 from the sliced copy, one row per lane.
template <bool LAST>
__global__ __launch_bounds__(kBlock) void k_apply_sell(Sell<double2> m, const double2* x,
                                                       const double2* in, double2* out,
                                                       double shift, int64_t n, int64_t nslices) {
  constexpr int SPB = kBlock / kSlice;
  const int lane = threadIdx.x % kSlice;
  const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kSlice));
  int64_t beg, end;
  block_range(nslices, SPB, beg, end);
  for (int64_t sl = beg + wv; sl < end; sl += SPB) {
    const int64_t row = sl * kSlice + lane;
    const int64_t rr = row < n ? row : n - 1;
    double2 own = czero<double>();
    cfma<double>(own, m.diag[rr], x[rr]);
    const double2 v = sell_row<double, 8>(m, x, sl, lane, own);
    if (row < n) out[row] = LAST ? with_shift(v, shift, in[row]) : v;
  }
}

template <class R>
__global__ __launch_bounds__(kBlock) void k_apply_shift(const cplx<R>* q, const double2* in,
                                                        double2* out, double shift, int64_t n) {
  for (int64_t i = blockIdx.x * int64_t(kBlock) + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * kBlock)
    out[i] = with_shift(to_d(q[i]), shift, in[i]);
}

// One half of A = M^H M on the links in FP64, one site per lane: t = M in (LAST false), or
// out = M^H t + shift in (LAST true), from all nine values of a link (a third row rebuilt from
// two adds its own rounding: 3.4e-16 of the product for 1.4e-16).  Bound by the links and the
// gathers, as K2 is; where a t-slice holds whole blocks of 64 sites it marches along t (tc >= 2
// t-slices per column) with the same carry, two workgroups per CU.  A call at 32^3 x 64 takes
// 725 us (803 without the march; 828 with three per CU; two rows 553; CSR 1870).
template <bool LAST, bool MARCH>
__global__ __launch_bounds__(kBlock, 2) void k_apply_site(Stencil<double2> w, SweepOrder ord,
                                                          uint32_t tc, const double2* x,
                                                          const double2* in, double2* out,
                                                          double shift) {
  constexpr int LR = 3;
  const uint32_t vol = uint32_t(w.vol);
  const int64_t nblk = (int64_t(vol) + kSiteBlock - 1) / kSiteBlock;
  constexpr int WPB = kBlock / kWave;
  const int lane = threadIdx.x % kWave;
  auto store = [&](uint32_t site, const double2 (&v)[3]) {
    const int64_t r0 = 3 * int64_t(site);
#pragma unroll
    for (int c = 0; c < 3; ++c)
      out[r0 + c] = LAST ? with_shift(v[c], shift, in[r0 + c]) : v[c];
  };
  auto gather = [&](uint32_t t, int c) { return x[3 * int64_t(t) + c]; };
  if constexpr (MARCH) {
    const uint32_t vol3 = vol / uint32_t(w.L[3]);
    const uint32_t bs = vol3 / uint32_t(kSiteBlock);
    constexpr int K = 3 * LR;
    TCarry<double, LR> car;
    int64_t qb, qe;
    march_range(nblk, WPB, qb, qe);
    for (uint32_t q = uint32_t(qb); q < uint32_t(qe); ++q) {
      const uint32_t site = march_block(q, tc, bs) * uint32_t(kSiteBlock) + uint32_t(lane);  // below vol
      if (q == uint32_t(qb) || q % tc == 0) {
        const uint32_t sb = site >= vol3 ? site - vol3 : site + (vol - vol3);  // periodic
        const double2* __restrict__ wt = w.w + int64_t(3) * K * vol;
#pragma unroll
        for (int k = 0; k < K; ++k) car.u[k] = wt[int64_t(k) * vol + sb];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          car.own[c] = x[3 * int64_t(sb) + c];
          car.fw[c] = x[3 * int64_t(site) + c];
        }
      }
      double2 own[3], v[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) own[c] = car.fw[c];
      stencil_site_c<double, LR, true, true>(w, site, own, LAST ? -1 : 1, gather, v, &car);
#pragma unroll
      for (int c = 0; c < 3; ++c) car.own[c] = own[c];
      store(site, v);
    }
  } else {
    for (Sweep sw = make_sweep(nblk, ord, WPB); sw.more(); sw.next()) {
      const uint32_t site = uint32_t(sw.slice() * kSiteBlock) + uint32_t(lane);
      const uint32_t ss = site < vol ? site : vol - 1;  // lanes past the volume: unused
      double2 own[3], v[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) own[c] = x[3 * int64_t(ss) + c];
      stencil_site_c<double, LR, false, true>(w, ss, own, LAST ? -1 : 1, gather, v,
                                              static_cast<TCarry<double, LR>*>(nullptr));
      if (site < vol) store(site, v);
    }
  }
}

// Workgroups for `n` items processed `rows_per_pass` at a time: one pass each when that
// fits under the cap (kMaxGrid, or a smaller tuning value), a multiple of the XCD count.
int grid_rows(int64_t n, int rows_per_pass, int cap = kMaxGrid) {
  if (cap <= 0 || cap > kMaxGrid) cap = kMaxGrid;
  int64_t g = (n + rows_per_pass - 1) / rows_per_pass;
  if (g > cap) g = cap;
  if (g < kXcds) g = kXcds;
  g = (g + kXcds - 1) / kXcds * kXcds;
  if (g > kMaxGrid) g = kMaxGrid;
  return int(g);
}

// Workgroups of kernel `kern` (kBlock threads) that the device holds resident at once,
// rounded down to a multiple of the XCD count: the grid of a launch whose waves sweep a
// lattice order in step (a larger grid would leave the later workgroups' positions to a
// second round).  Cached per device and kernel.
int resident_grid(const void* kern, int cap) {
  static std::mutex mu;
  static std::map<std::pair<int, const void*>, int> cache;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return cap;
  std::lock_guard<std::mutex> lk(mu);
  const auto key = std::make_pair(dev, kern);
  auto it = cache.find(key);
  if (it == cache.end()) {
    int per_cu = 0, cus = 0;
    int g = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kBlock, 0) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess)
      g = per_cu * cus / kXcds * kXcds;
    it = cache.emplace(key, g).first;
  }
  const int g = it->second;
  return g >= kXcds && g < cap ? g : cap;
}

// Dispatch on lanes per row.
#define MSC_LANES_SWITCH(LANES, CALL) \
  switch (LANES) {                    \
    case 4: { constexpr int LL = 4; CALL; } break;   \
    case 8: { constexpr int LL = 8; CALL; } break;   \
    case 16: { constexpr int LL = 16; CALL; } break;  \
    case 32: { constexpr int LL = 32; CALL; } break;  \
    default: return hipErrorInvalidValue;            \
  }

// Launch one kernel of an iteration.  With `ev`, the start/stop events of pair `k` are
// attached to the dispatch itself (their timestamps are the kernel's own begin and
// end), so the elapsed time excludes the queue gap between kernels.
template <class K, class... A>
void launch_timed(K kern, int grid, hipStream_t s, hipEvent_t* ev, int k, const A&... args) {
  if (ev)
    hipExtLaunchKernelGGL(kern, dim3(grid), dim3(kBlock), 0, s, ev[2 * k], ev[2 * k + 1], 0, args...);
  else
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kBlock), 0, s, args...);
}

// t-slices per column of the march along t that this lattice allows (1: none): a t-slice holds
// whole blocks of 64 sites and some power of two up to kK2March divides L_t.
int march_columns(const Stencil<double2>& w) {
  const int64_t lt = w.L[3];
  if (lt <= 0 || (w.vol / lt) % kSiteBlock != 0) return 1;
  for (int c = kK2March; c >= 2; c /= 2)
    if (lt % c == 0) return c;
  return 1;
}

// Workgroups of a links' kernel that sweeps or marches in order, at most: two per CU in FP64,
// four in complex64.  More waves in flight than that outrun the L2 (32^3 x 64: FP64 K1 + applications 355 us, 396 with
// three workgroups per CU, 447 with one and a half; complex64 180, 187 with five, 186 with
// three; K2 264 / 261 / 348 and 141 / 141 / 144).
template <class R> constexpr int site_cap() { return std::is_same<R, double>::value ? 512 : 1024; }

template <class R, int LR, bool MARCH> const void* site_kernel(int half) {
  constexpr bool STREAM = std::is_same<R, double>::value;
  return half == 1 ? reinterpret_cast<const void*>(k1_site<R, LR, STREAM, MARCH, false>)
                   : reinterpret_cast<const void*>(k2_site<R, LR, MARCH, false>);
}

// The grid of a links' half, and whether it marches: it does when every resident wave gets
// a run of at least 4 blocks.
template <class R> int site_grid(const MsArgs& a, int half, int& march) {
  const int64_t nblk = (a.w64.vol + kSiteBlock - 1) / kSiteBlock;
  constexpr int WPB = kBlock / kWave;
  const int cap = std::min(a.grid, a.ord.on ? site_cap<R>() : kMaxGrid);
  const int all = grid_rows(nblk, WPB, cap);
  march = 0;
  if (a.stencil == 2 && a.ord.on && a.march > 1) {
    const int g = resident_grid(site_kernel<R, 2, true>(half), all);
    if (nblk >= int64_t(g) * WPB * 4) {
      march = 1;
      return g;
    }
  }
  if (!a.ord.on) return all;
  return resident_grid(a.stencil == 2 ? site_kernel<R, 2, false>(half) : site_kernel<R, 3, false>(half),
                       all);
}

template <class R> void prepare_impl(MsArgs& a) {
  const bool mhm = a.kind == MSC_A_MHM;
  a.m1 = a.m2 = a.split = a.small = 0;
  if (a.sell && mhm && a.stencil) {
    // a direction per wave while every block of 64 sites gets a workgroup of its own (up to
    // 65536 sites; k1_split has the times on both sides)
    a.split = (a.w64.vol + kSiteBlock - 1) / kSiteBlock <= a.grid ? 1 : 0;
    a.small = a.split && a.w64.vol <= kSmallSites ? 1 : 0;
    if (a.split) {
      a.gd = a.gg = grid_rows(a.w64.vol, kSiteBlock, a.grid);
      return;
    }
    a.march = a.ord.on ? march_columns(a.w64) : 1;
    a.gd = site_grid<R>(a, 1, a.m1);
    a.gg = site_grid<R>(a, 2, a.m2);
  } else if (a.sell) {
    auto grid = [&](const void* kern) {
      const int g = grid_rows(a.n, kBlock, a.grid);
      return a.ord.on ? resident_grid(kern, g) : g;
    };
    if (mhm) {
      a.gd = grid(reinterpret_cast<const void*>(k1_sell<R, true, false>));
      a.gg = grid(reinterpret_cast<const void*>(k2_sell<R, false>));
    } else {
      a.gd = a.gg = grid(reinterpret_cast<const void*>(k_herm<R>));
    }
  } else {
    a.gd = grid_rows(a.n, kBlock / a.lanes, a.grid);
    a.gg = mhm ? a.gd : grid_rows(a.n, kBlock, a.grid);
  }
}

template <class R> hipError_t flush_impl(const MsArgs& a, int par, int when, hipStream_t s, hipEvent_t* ev) {
  const int g = grid_rows(a.n, kBlock);
  if (a.sell && a.stencil)
    launch_timed(k_flush<R, true>, g, s, ev, 2, a, par, when);
  else
    launch_timed(k_flush<R, false>, g, s, ev, 2, a, par, when);
  return hipGetLastError();
}

template <class R>
hipError_t reliable_impl(const MsArgs& a, hipStream_t s) {
  if (const hipError_t e = flush_impl<R>(a, a.par, 1, s, nullptr); e != hipSuccess) return e;
  if (a.sell && a.kind == MSC_A_MHM && a.stencil != 0) {
    // the links: the same FP64 operator as the stored copies, a third of their bytes
    const int gs = grid_rows((a.w64.vol + kSiteBlock - 1) / kSiteBlock, kBlock / kWave);
    if (a.stencil == 2) {
      k_ru_first_site<2><<<gs, kBlock, 0, s>>>(a);
      k_ru_second_site<R, 2><<<gs, kBlock, 0, s>>>(a);
    } else {
      k_ru_first_site<3><<<gs, kBlock, 0, s>>>(a);
      k_ru_second_site<R, 3><<<gs, kBlock, 0, s>>>(a);
    }
    return hipGetLastError();
  }
  if (a.sell) {
    const int gs = grid_rows(a.nslices, kBlock / kSlice);
    if (a.kind == MSC_A_MHM) {
      k_ru_first_s<<<gs, kBlock, 0, s>>>(a);
      k_ru_second_s<R, true><<<gs, kBlock, 0, s>>>(a);
    } else {
      k_ru_second_s<R, false><<<gs, kBlock, 0, s>>>(a);
      if (!a.dir) k_herm_w<R><<<a.gd, kBlock, 0, s>>>(a, 1);
    }
    return hipGetLastError();
  }
  const int g1 = grid_rows(a.n, kBlock / a.lanes);
  if (a.kind == MSC_A_MHM) {
    MSC_LANES_SWITCH(a.lanes, (k_ru_first<LL><<<g1, kBlock, 0, s>>>(a)));
    MSC_LANES_SWITCH(a.lanes, (k_ru_second<R, LL, true><<<g1, kBlock, 0, s>>>(a)));
  } else {
    MSC_LANES_SWITCH(a.lanes, (k_ru_second<R, LL, false><<<g1, kBlock, 0, s>>>(a)));
  }
  return hipGetLastError();
}

template <class R, int LR, bool DIR> void launch_sites(const MsArgs& a, hipStream_t s, hipEvent_t* ev) {
  constexpr bool STREAM = std::is_same<R, double>::value;
  if (a.split) {
    launch_timed(k1_split<R, LR, DIR>, a.gd + 1, s, ev, 0, a);
    launch_timed(k2_split<R, LR, DIR>, a.gg + 1, s, ev, 1, a);
    return;
  }
  if constexpr (LR == 2) {
    if (a.m1)
      launch_timed(k1_site<R, 2, STREAM, true, DIR>, a.gd + 1, s, ev, 0, a);
    else
      launch_timed(k1_site<R, 2, STREAM, false, DIR>, a.gd + 1, s, ev, 0, a);
    if (a.m2)
      launch_timed(k2_site<R, 2, true, DIR>, a.gg + 1, s, ev, 1, a);
    else
      launch_timed(k2_site<R, 2, false, DIR>, a.gg + 1, s, ev, 1, a);
  } else {
    launch_timed(k1_site<R, LR, STREAM, false, DIR>, a.gd + 1, s, ev, 0, a);
    launch_timed(k2_site<R, LR, false, DIR>, a.gg + 1, s, ev, 1, a);
  }
}

// The operator halves (each has a workgroup more than the rows need); with the direction its
// update goes first.
template <class R, bool DIR>
hipError_t halves_impl(const MsArgs& a, hipStream_t s, hipEvent_t* ev) {
  const bool mhm = a.kind == MSC_A_MHM;
  if (DIR) k_dir<R><<<grid_rows(a.n, kBlock), kBlock, 0, s>>>(a);
  if (a.sell && mhm && a.stencil) {
    if (a.stencil == 2)
      launch_sites<R, 2, DIR>(a, s, ev);
    else
      launch_sites<R, 3, DIR>(a, s, ev);
  } else if (a.sell && mhm) {
    launch_timed(k1_sell<R, true, DIR>, a.gd + 1, s, ev, 0, a);
    launch_timed(k2_sell<R, DIR>, a.gg + 1, s, ev, 1, a);
  } else if (a.sell) {
    if constexpr (DIR) {
      launch_timed(k1_sell<R, false, true>, a.gd + 1, s, ev, 0, a);
      launch_timed(k2_csr<R, 4, false, true>, a.gg + 1, s, ev, 1, a);
    } else {
      launch_timed(k_herm<R>, a.gg + 1, s, ev, 0, a);
    }
  } else if (mhm) {
    MSC_LANES_SWITCH(a.lanes, (launch_timed(k1_csr<R, LL, true, DIR>, a.gd + 1, s, ev, 0, a)));
    MSC_LANES_SWITCH(a.lanes, (launch_timed(k2_csr<R, LL, true, DIR>, a.gg + 1, s, ev, 1, a)));
  } else {
    MSC_LANES_SWITCH(a.lanes, (launch_timed(k1_csr<R, LL, false, DIR>, a.gd + 1, s, ev, 0, a)));
    launch_timed(k2_csr<R, 4, false, DIR>, a.gg + 1, s, ev, 1, a);
  }
  return hipGetLastError();
}

// One iteration: the reliable update where one is due, the operator halves, then with `flush`
// the composed steps.
template <class R>
hipError_t iteration_impl(const MsArgs& a, hipStream_t s, hipEvent_t* ev, bool flush) {
  hipError_t e = a.ru_check ? reliable_impl<R>(a, s) : hipSuccess;
  if (e != hipSuccess) return e;
  if (a.span > 0) {
    if (a.stencil == 2)
      k_small<R, 2><<<1, kSmallBlock, 0, s>>>(a);
    else
      k_small<R, 3><<<1, kSmallBlock, 0, s>>>(a);
    e = hipGetLastError();
  } else {
    e = a.dir ? halves_impl<R, true>(a, s, ev) : halves_impl<R, false>(a, s, ev);
  }
  if (e != hipSuccess) return e;
  return flush ? flush_impl<R>(a, (a.launch + std::max(1, a.span)) & 1, 0, s, ev) : hipSuccess;
}

template <class R, bool COLOURS>
void direction_impl(const MsArgs& a, bool load, const double2* ax, hipStream_t s) {
  if (load) k_load_p<R, COLOURS><<<grid_rows(a.n, kBlock), kBlock, 0, s>>>(a);
  if (!ax) return;
  k_load_r<R, COLOURS><<<a.gg, kBlock, 0, s>>>(a, ax);
  k_go_on<<<1, kBlock, 0, s>>>(a, 1);
}
void load_direction(int prec, const MsArgs& a, bool load, const double2* ax, hipStream_t s) {
  const bool colours = a.sell && a.stencil;
  if (prec == MSC_PREC_MIXED)
    colours ? direction_impl<float, true>(a, load, ax, s) : direction_impl<float, false>(a, load, ax, s);
  else
    colours ? direction_impl<double, true>(a, load, ax, s) : direction_impl<double, false>(a, load, ax, s);
}

}  // namespace

void prepare_iteration(int prec, MsArgs& a) {
  prec == MSC_PREC_MIXED ? prepare_impl<float>(a) : prepare_impl<double>(a);
}

hipError_t launch_init(const MsArgs& a, hipStream_t s) {
  if (a.sell && a.stencil)
    k_init<true><<<a.gg, kBlock, 0, s>>>(a);
  else
    k_init<false><<<a.gg, kBlock, 0, s>>>(a);
  if (a.sell && a.kind != MSC_A_MHM) k_herm_w<double><<<a.gd, kBlock, 0, s>>>(a, 0);
  return hipGetLastError();
}

hipError_t launch_iteration(int prec, const MsArgs& a, hipStream_t s, hipEvent_t* ev, bool flush) {
  return prec == MSC_PREC_MIXED ? iteration_impl<float>(a, s, ev, flush)
                                : iteration_impl<double>(a, s, ev, flush);
}

hipError_t launch_final_flush(int prec, const MsArgs& a, hipStream_t s) {
  return prec == MSC_PREC_MIXED ? flush_impl<float>(a, 0, 2, s, nullptr)
                                : flush_impl<double>(a, 0, 2, s, nullptr);
}

hipError_t launch_switch_to_mixed(const MsArgs& a64, const MsArgs& a32, int ns, hipStream_t s) {
  const bool herm = a64.sell && a64.kind != MSC_A_MHM && !a64.dir;
  const int g = grid_rows(int64_t(ns + 1) * a64.n, kBlock);
  k_switch<<<g, kBlock, 0, s>>>(a64, a32, ns, herm ? 1 : 0);
  k_go_on<<<1, kBlock, 0, s>>>(a32, 0);
  if (a32.dir)
    load_direction(MSC_PREC_MIXED, a32, !a64.dir, nullptr, s);
  else if (herm)
    k_herm_w<float><<<a32.gd, kBlock, 0, s>>>(a32, 0);
  return hipGetLastError();
}

hipError_t launch_direction(int prec, const MsArgs& a, bool load, const double2* ax, hipStream_t s) {
  load_direction(prec, a, load, ax, s);
  return hipGetLastError();
}

hipError_t launch_verify(const MsArgs& a, const double* sigma_by_caller_index, int k0, int kc,
                         double2* u64, hipStream_t s) {
  if (kc < 1 || kc > kVerifyChunk) return hipErrorInvalidValue;
  const int g1 = grid_rows(a.n, kBlock / a.lanes);
  const double2* xc = a.x + int64_t(k0) * a.n;
  VerifyArgs v;
  v.in = xc;
  v.x = xc;
  v.b = a.b;
  for (int q = 0; q < kVerifyChunk; ++q) v.sig[q] = q < kc ? sigma_by_caller_index[k0 + q] : 0.0;
  v.n = a.n;
  v.kc = kc;
  v.partial = a.sc.partial;
  v.ticket = a.sc.tickets + 4 * kTicketSite;
  v.out = a.sc.res2 + k0;
  if (a.sell) {
    const int gs = grid_rows(a.nslices, kBlock / kSlice);
    v.nslices = a.nslices;
    if (a.kind == MSC_A_MHM) {
      k_verify_first_s<<<gs, kBlock, 0, s>>>(a.s64, xc, a.n, a.nslices, kc, u64);
      v.s = a.sh64;
      v.in = u64;
    } else {
      v.s = a.s64;
    }
    k_verify_second_s<<<gs, kBlock, 0, s>>>(v);
    return hipGetLastError();
  }
  if (a.kind == MSC_A_MHM) {
    MSC_LANES_SWITCH(a.lanes, (k_verify_first<LL><<<g1, kBlock, 0, s>>>(a.m64, xc, a.n, kc, u64)));
    v.m = a.mh64;
    v.in = u64;
  } else {
    v.m = a.m64;
  }
  MSC_LANES_SWITCH(a.lanes, (k_verify_second<LL><<<g1, kBlock, 0, s>>>(v)));
  return hipGetLastError();
}

namespace {
hipError_t apply_links(const ApplyArgs& a, hipStream_t s) {
  const Stencil<double2>& w = a.w64;
  double2* t = static_cast<double2*>(a.tmp);
  const int64_t nblk = (w.vol + kSiteBlock - 1) / kSiteBlock;
  constexpr int WPB = kBlock / kWave;
  int g = grid_rows(nblk, WPB);
  const int tc = a.ord.on ? march_columns(w) : 1;
  const int gm = std::min(g, site_cap<double>());
  // as K2: runs of at least 4 blocks, or there is little to carry
  if (tc > 1 && nblk >= int64_t(gm) * WPB * 4) {
    k_apply_site<false, true><<<gm, kBlock, 0, s>>>(w, a.ord, uint32_t(tc), a.in, a.in, t, 0.0);
    k_apply_site<true, true><<<gm, kBlock, 0, s>>>(w, a.ord, uint32_t(tc), t, a.in, a.out, a.shift);
    return hipGetLastError();
  }
  if (a.ord.on) g = resident_grid(reinterpret_cast<const void*>(k_apply_site<true, false>), g);
  k_apply_site<false, false><<<g, kBlock, 0, s>>>(w, a.ord, 1u, a.in, a.in, t, 0.0);
  k_apply_site<true, false><<<g, kBlock, 0, s>>>(w, a.ord, 1u, t, a.in, a.out, a.shift);
  return hipGetLastError();
}

// Stored matrix, FP64: the sliced copy from kApplySellMin rows on (one row per lane: below,
// too few waves hide its chain of loads), else the CSR.
hipError_t apply_stored64(const ApplyArgs& a, hipStream_t s) {
  double2* t = static_cast<double2*>(a.tmp);
  const int g1 = grid_rows(a.n, kBlock / a.lanes);
  const bool sell = a.sell && a.n >= kApplySellMin;
  const int gs = sell ? grid_rows(a.nslices, kBlock / kSlice) : 0;
  if (a.kind == MSC_A_MHM) {
    if (sell) {
      k_apply_sell<false><<<gs, kBlock, 0, s>>>(a.s64, a.in, a.in, t, 0.0, a.n, a.nslices);
      k_apply_sell<true><<<gs, kBlock, 0, s>>>(a.sh64, t, a.in, a.out, a.shift, a.n, a.nslices);
      return hipGetLastError();
    }
    MSC_LANES_SWITCH(a.lanes, (k_apply_csr<double, LL, false, double2><<<g1, kBlock, 0, s>>>(
                                  a.m64, a.in, t, a.in, a.out, 0.0, a.n)));
    MSC_LANES_SWITCH(a.lanes, (k_apply_csr<double, LL, true, double2><<<g1, kBlock, 0, s>>>(
                                  a.mh64, t, t, a.in, a.out, a.shift, a.n)));
    return hipGetLastError();
  }
  // A given: one pass, unless it would gather rows that it has overwritten
  const bool apart = a.in + a.n <= a.out || a.out + a.n <= a.in;
  if (sell) {
    if (apart)
      k_apply_sell<true><<<gs, kBlock, 0, s>>>(a.s64, a.in, a.in, a.out, a.shift, a.n, a.nslices);
    else
      k_apply_sell<false><<<gs, kBlock, 0, s>>>(a.s64, a.in, a.in, t, 0.0, a.n, a.nslices);
  } else if (apart) {
    MSC_LANES_SWITCH(a.lanes, (k_apply_csr<double, LL, true, double2><<<g1, kBlock, 0, s>>>(
                                  a.m64, a.in, t, a.in, a.out, a.shift, a.n)));
  } else {
    MSC_LANES_SWITCH(a.lanes, (k_apply_csr<double, LL, false, double2><<<g1, kBlock, 0, s>>>(
                                  a.m64, a.in, t, a.in, a.out, 0.0, a.n)));
  }
  if (!apart)
    k_apply_shift<double><<<grid_rows(a.n, kBlock), kBlock, 0, s>>>(t, a.in, a.out, a.shift, a.n);
  return hipGetLastError();
}

// complex64 arithmetic: the CSR, whose products are the same bits at every size.
hipError_t apply_stored32(const ApplyArgs& a, hipStream_t s) {
  float2* t = static_cast<float2*>(a.tmp);
  const int g1 = grid_rows(a.n, kBlock / a.lanes);
  if (a.kind == MSC_A_MHM) {
    MSC_LANES_SWITCH(a.lanes, (k_apply_csr<float, LL, false, double2><<<g1, kBlock, 0, s>>>(
                                  a.m32, a.in, t, a.in, a.out, 0.0, a.n)));
    MSC_LANES_SWITCH(a.lanes, (k_apply_csr<float, LL, true, float2><<<g1, kBlock, 0, s>>>(
                                  a.mh32, t, t, a.in, a.out, a.shift, a.n)));
    return hipGetLastError();
  }
  if (a.in + a.n <= a.out || a.out + a.n <= a.in) {
    MSC_LANES_SWITCH(a.lanes, (k_apply_csr<float, LL, true, double2><<<g1, kBlock, 0, s>>>(
                                  a.m32, a.in, t, a.in, a.out, a.shift, a.n)));
    return hipGetLastError();
  }
  MSC_LANES_SWITCH(a.lanes, (k_apply_csr<float, LL, false, double2><<<g1, kBlock, 0, s>>>(
                                a.m32, a.in, t, a.in, a.out, 0.0, a.n)));
  k_apply_shift<float><<<grid_rows(a.n, kBlock), kBlock, 0, s>>>(t, a.in, a.out, a.shift, a.n);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_apply(const ApplyArgs& a, hipStream_t s) {
  if (a.prec == MSC_PREC_MIXED) return apply_stored32(a, s);
  if (a.links != 0 && a.w64.vol >= kApplySitesMin) return apply_links(a, s);
  return apply_stored64(a, s);
}

// ---- operator application without allocation ------------------------------------------
// The temporary of the no-allocation apply lives in a file-scope device array: each
// GPU the library runs on holds its own copy, until the process ends.  In host code the
// name `scratch` is only a host-side stand-in, so it is never passed to a kernel: the
// array's address on each device comes from hipGetSymbolAddress, looked up once per
// device with that device current, and kept in scratch_addr.
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex scratch_mutex;
void* scratch_addr[kMaxDevices] = {};
}  // namespace

size_t apply_scratch_bytes(int kind, int prec, int64_t n) {
  // The product uses one temporary, a vector of the working precision; the count leaves room
  // for two (one for a given A in FP64).  It is the documented limit of the entry point, and
  // what lies beyond it is refused.
  const size_t elem = prec == MSC_PREC_MIXED ? sizeof(float2) : sizeof(double2);
  const int count = (prec == MSC_PREC_MIXED || kind == MSC_A_MHM) ? 2 : 1;
  const size_t one = (elem * size_t(n) + 255) / 256 * 256;
  return one * count;
}

hipError_t noalloc_scratch(int device, void** ptr) {
  *ptr = nullptr;
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (!scratch_addr[device]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    scratch_addr[device] = p;
  }
  *ptr = scratch_addr[device];
  return hipSuccess;
}

hipError_t launch_apply_noalloc(ApplyArgs a, void* base, hipStream_t s) {
  if (apply_scratch_bytes(a.kind, a.prec, a.n) > kNoAllocScratchBytes) return hipErrorInvalidValue;
  a.tmp = base;
  return launch_apply(a, s);
}

}  // namespace msc
