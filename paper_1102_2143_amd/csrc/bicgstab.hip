// Multishift BiCGStab (BiCGStab-M) for a general, non-Hermitian sparse A: the family
// (A + sigma_k I) x_k = b (paper: Section 2, eq. linprob) from one BiCGStab sequence of
// the driving matrix B = A + sigma0 I (the paper's second shifted solver, Sections 1
// and 3).  The shifted constants follow from the BiCG polynomials: the shifted BiCG
// residuals are multiples of the driving one (the zeta recurrence of CG-M), and the
// shifted stabilising steps om / (1 + s om) keep the whole shifted residual a multiple
// of the driving one, r_n(s) = (z_n / tau_n) r_n, so every shift is advanced from r_n,
// s_n and r_{n+1} with no extra operator product.
//
// One iteration is two kernels, one per product.  Each workgroup sums the previous kernel's
// partials itself, in one order, and derives the scalars; vectors that the other kernel
// left to be formed are formed at every gathered column as their owner forms them:
//   BA   om_{n-1} = t^H s / t^H t, rho_n = w^H s - om w^H t, |r_n|^2 = |s|^2 - |t^H s|^2 /
//        t^H t (both summed over r_n itself where they cancel), be_n;  r_n = s - om t, p_n = r_n + be (p - om v), v_n = B p_n;  w^H v_n
//   BB   al_n = rho_n / w^H v_n;  s_n = r_n - al v_n, t_n = B s_n;  t^H s, t^H t, w^H s,
//        w^H t, |s|^2
// The shifts take, per step,
//   x(s) += al(s) p(s) + om(s) (z'/tau) s,
//   p(s) <- (z'/tau') r' + be(s) [p(s) - (om(s)/al(s)) ((z/tau) r - (z'/tau) s)];
// nothing else reads them, so msc_params::update_steps steps, at most kBcgSteps, are composed
// against the first one's p(s) and the r and s of the steps, which stay in rings, and BA
// applies them in one pass.
// Complex scalars are FP64 throughout; the shadow vector is b.
//
// Bound by memory and, on grids that fit the caches, by latency.  64 x 48 x 50 points, 8
// shifts, a solve of 42 steps: 3.60 ms with four kernels on the CSR, 1.71 ms here.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "dev_common.h"
#include "msc_internal.h"
#include "sell_load.h"

namespace msc {

namespace {

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return double2{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
__device__ __forceinline__ double2 cdiv(double2 a, double2 b) {
  // Smith's scaling keeps the quotient finite for any finite non-zero b
  if (fabs(b.x) >= fabs(b.y)) {
    const double r = b.y / b.x, d = b.x + b.y * r;
    return double2{(a.x + a.y * r) / d, (a.y - a.x * r) / d};
  }
  const double r = b.x / b.y, d = b.x * r + b.y;
  return double2{(a.x * r + a.y) / d, (a.y * r - a.x) / d};
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return double2{a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return double2{a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ double cabs2(double2 a) { return a.x * a.x + a.y * a.y; }
__device__ __forceinline__ bool cfinite(double2 a) { return isfinite(a.x) && isfinite(a.y); }
// acc += conj(a) b
__device__ __forceinline__ void cdot_acc(double2& acc, double2 a, double2 b) {
  acc.x = fma(a.x, b.x, acc.x);
  acc.x = fma(a.y, b.y, acc.x);
  acc.y = fma(a.x, b.y, acc.y);
  acc.y = fma(-a.y, b.x, acc.y);
}
// c += a b
__device__ __forceinline__ void cmad(double2& c, double2 a, double2 b) {
  c.x = fma(a.x, b.x, c.x);
  c.x = fma(-a.y, b.y, c.x);
  c.y = fma(a.x, b.y, c.y);
  c.y = fma(a.y, b.x, c.y);
}

// s = r - al v, written so that the owner of a row and every lane that gathers it form
// the same bits.
__device__ __forceinline__ double2 s_of(double2 r, double2 v, double2 al) {
  double2 s;
  s.x = fma(-al.x, v.x, fma(al.y, v.y, r.x));
  s.y = fma(-al.x, v.y, fma(-al.y, v.x, r.y));
  return s;
}

// One CSR row of A times a vector read through gather(col); L lanes per row, the sum in
// every lane.  All loads of a chunk are issued before its first multiply-add.
constexpr int kBcgChunk = 4;
template <int L, class G>
__device__ __forceinline__ double2 row_f(const Csr<double2>& m, int64_t row, int lane, G gather) {
  const int32_t beg = m.rowptr[row], end = m.rowptr[row + 1];
  double2 acc{0.0, 0.0};
  for (int32_t base = beg; base < end; base += kBcgChunk * L) {
    int32_t c[kBcgChunk];
    double2 v[kBcgChunk], xv[kBcgChunk];
#pragma unroll
    for (int u = 0; u < kBcgChunk; ++u) {
      const int32_t j = base + lane + u * L;
      const bool ok = j < end;
      c[u] = ok ? m.col[j] : 0;
      v[u] = ok ? m.val[j] : double2{0.0, 0.0};
    }
#pragma unroll
    for (int u = 0; u < kBcgChunk; ++u) xv[u] = gather(c[u]);
#pragma unroll
    for (int u = 0; u < kBcgChunk; ++u) cmad(acc, v[u], xv[u]);
  }
  return group_sum_c<L, double>(acc);
}

// One sliced row of A (off-diagonal part and diagonal) times gather(col), own at the row.
template <bool NARROW, class G>
__device__ __forceinline__ double2 sell_f(const Sell<double2>& m, int64_t sl, int lane, int64_t row,
                                          double2 own, G gather) {
  int32_t c, c1;
  if (m.wp > 0) {
    c = int32_t(sl) * m.wp;
    c1 = c + m.wp;
  } else {
    c = load_uniform(m.cptr, sl);
    c1 = load_uniform(m.cptr, sl + 1);
  }
  double2 acc{0.0, 0.0};
  cmad(acc, m.diag[row], own);
  constexpr int KP = 2;
  for (; c < c1; c += KP) {
    const int np = c1 - c;
    int2 cc[KP];
    double2 v[2 * KP], xv[2 * KP];
    if (np >= KP)
      sell_load<double, KP, true, NARROW>(m, c, KP, lane, cc, v);
    else
      sell_load<double, KP, false, NARROW>(m, c, np, lane, cc, v);
#pragma unroll
    for (int u = 0; u < KP; ++u) {
      if (u < np) {
        xv[2 * u] = gather(cc[u].x);
        xv[2 * u + 1] = gather(cc[u].y);
      }
    }
#pragma unroll
    for (int u = 0; u < 2 * KP; ++u)
      if (u < 2 * np) cmad(acc, v[u], xv[u]);
  }
  return acc;
}

// Partials: component k of a kernel's workgroup i at reg[k kBcgGrid + i]; BA's two in region
// 0, BB's eight in 1 and a checking BA's three in 2 (the BA that reads them writes region 0).
__device__ __forceinline__ double* bcg_region(const BcgArgs& a, int which) {
  return a.partial + (which == 0 ? 0 : which == 1 ? 2 : 10) * kBcgGrid;
}

// |r_n|^2 = |s|^2 - |t^H s|^2 / |t|^2 and w^H r_n = w^H s - om w^H t carry the rounding of their
// larger terms, about 1e-15 of them.  Where the first falls below this part of |s|^2, BA sums
// both over r_n itself (a pass of its own) and the step ends in the next BA, so that no shift
// stops, and no be follows, from rounding alone: |r_n| is then known to 1e-5 of itself.
constexpr double kBcgCancel = 1e-10;

template <int K> __device__ __forceinline__ void bcg_store(double* reg, double (&v)[K]) {
  block_sum_k<kBlock, K>(v);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) store_agent(&reg[k * kBcgGrid + blockIdx.x], v[k]);
  }
}

// The sums of all workgroups' K components, in every thread.  The previous kernel wrote
// them, so plain loads do, and the XCD's L2 serves all but its first workgroup's.
template <int K> __device__ __forceinline__ void bcg_sums(const double* reg, double (&tot)[K]) {
  __shared__ double sh[K];
  constexpr int kPer = kBcgGrid / kBlock;
  double v[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    double w[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int i = threadIdx.x + u * kBlock;
      w[u] = i < int(gridDim.x) ? reg[k * kBcgGrid + i] : 0.0;
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

__device__ __forceinline__ double2* ring(double2* v, int64_t n, int i, int slots) {
  return v + int64_t(i % slots) * n;
}

// ---- start: what BA turns into r_0 = p_0 = b (om = be = 0); |b|^2 --------------------------
__global__ __launch_bounds__(kBlock) void k_bcg_start(BcgArgs a) {
  double2* __restrict__ s = ring(a.s, a.n, kBcgSteps - 1, kBcgSteps);
  int64_t beg, end;
  block_range(a.n, kBlock, beg, end);
  double v[8] = {};
  for (int64_t i = beg + threadIdx.x; i < end; i += kBlock) {
    const double2 bv = a.b[i];
    s[i] = bv;
    a.t[i] = a.p[0][i] = a.v[0][i] = double2{0.0, 0.0};
    v[7] += cabs2(bv);
  }
  bcg_store<8>(bcg_region(a, 1), v);
}

// What BA does, shared through LDS.
struct BcgPlan {
  double2 om, be;
  int check;           // 1: this BA only sums r_n
  int live, apply, m, first, fresh, nact;  // composed steps: first .. first + m - 1
  double2 cx[kBcgTerms][kMaxShifts], cp[kBcgTerms][kMaxShifts];
  int64_t xo[kMaxShifts], po[kMaxShifts];
};

// BA's prologue (wave 0, lane j: shift j).  Step n - 1 (s, t, alpha, z', al(s) known)
// ends here; every workgroup derives the same, workgroup 0 writes the next state.  exact:
// w^H r_n and |r_n|^2 where the BA before summed them (rs.check).
__device__ void bcg_plan(const BcgArgs& a, const double (&tot)[8], const double (&exact)[3], BcgPlan& pl) {
  BcgState* st = a.st;
  const BcgRot& rs = st->rot[a.par];
  const int j = threadIdx.x;
  if (j >= kWave) return;
  const bool head = blockIdx.x == 0, mine = j < st->ns;
  const int n = rs.iter, m0 = rs.m;
  const double2 ts{tot[0], tot[1]}, ws{tot[3], tot[4]}, wt{tot[5], tot[6]};
  const double tt = tot[2], ss = tot[7];
  const double bn2 = n == 0 ? ss : st->bnorm2, eps2 = st->tol2 * bn2;
  int act = mine ? rs.active[j] : 0;
  double2 om{0.0, 0.0}, be{0.0, 0.0}, rho{ss, 0.0};
  double R = ss;
  // 0: go on, 1: halt, 2: breakdown
  int stop = 0;
  const bool step = n > 0;      // a step ends here
  bool took = mine && m0 > 0 ? rs.took[j] != 0 : false;
  double2 z{1.0, 0.0}, zn{1.0, 0.0}, tau{1.0, 0.0}, taun{1.0, 0.0};
  double2 cx[kBcgTerms], cp[kBcgTerms];
#pragma unroll
  for (int e = 0; e < kBcgTerms; ++e) cx[e] = cp[e] = double2{0.0, 0.0};
  // p(s) before the first composed step: itself, or r_0 = b where it was never written
  if (rs.fresh)
    cp[1].x = 1.0;
  else
    cp[0].x = 1.0;
  if (mine && m0 > 0) {
#pragma unroll
    for (int e = 0; e < kBcgTerms; ++e) {
      cx[e] = rs.cx[e][j];
      cp[e] = rs.cp[e][j];
    }
  }
  if (mine) {
    z = zn = rs.z[j];
    tau = taun = rs.tau[j];
  }
  int m = m0;
  const bool check = step && !st->bad && !rs.check && tt > 0.0 && isfinite(tt) && cfinite(ts) &&
                     ss - cabs2(ts) / tt <= kBcgCancel * ss;
  if (check) {  // the state goes on as it is, with om for the sums
    if (j == 0) {
      pl.om = double2{ts.x / tt, ts.y / tt};
      pl.check = 1;
      pl.live = pl.apply = 0;
    }
    if (!head) return;
    BcgRot& nx = st->rot[a.par ^ 1];
    if (mine) {
      nx.z[j] = rs.z[j];
      nx.zo[j] = rs.zo[j];
      nx.tau[j] = rs.tau[j];
      nx.active[j] = rs.active[j];
      nx.took[j] = rs.took[j];
#pragma unroll
      for (int e = 0; e < kBcgTerms; ++e) {
        nx.cx[e][j] = rs.cx[e][j];
        nx.cp[e][j] = rs.cp[e][j];
      }
    }
    if (j == 0) {
      nx.rho = rs.rho;
      nx.be = rs.be;
      nx.al = rs.al;
      nx.iter = n;
      nx.m = m0;
      nx.fresh = rs.fresh;
      nx.halt = 0;
      nx.check = 1;
    }
    return;
  }
  if (step && st->bad) {
    stop = 2;  // BB found w^H v = 0: no step n - 1
  } else if (step) {
    const bool ok = tt > 0.0 && isfinite(tt) && cfinite(ts);
    if (ok) om = double2{ts.x / tt, ts.y / tt};
    const double sj = mine ? st->s[j] : 0.0;
    const double2 g{1.0 + sj * om.x, sj * om.y};
    const bool bad = !ok || (act && g.x == 0.0 && g.y == 0.0);
    if (__ballot(bad)) {
      stop = 2;
      act = 0;
    } else {
      const double2 al = st->alpha;
      rho = rs.check ? double2{exact[0], exact[1]} : csub(ws, cmul(om, wt));
      R = rs.check ? exact[2] : ss - cabs2(ts) / tt;
      const bool rho_ok = rho.x != 0.0 || rho.y != 0.0, om_ok = om.x != 0.0 || om.y != 0.0;
      // be = (rho' / rho)(al / om); a vanishing rho' or om ends the sequence after this step
      if (rho_ok && om_ok) be = cmul(cdiv(rho, rs.rho), cdiv(al, om));
      int next = act;
      if (act) {
        zn = st->zn[j];
        taun = cmul(tau, g);
        const double2 als = st->als[j], oms = cdiv(om, g);
        const double2 c1 = cdiv(zn, tau);    // s_n(s) = c1 s_n
        const double2 c2 = cdiv(zn, taun);   // r_{n+1}(s) = c2 r_{n+1}
        const double2 c3 = cdiv(z, tau);     // r_n(s) = c3 r_n
        const double2 ratio = cdiv(zn, z), bes = cmul(be, cmul(ratio, ratio));
        const double2 q = cmul(bes, cdiv(oms, als)), qc3 = cmul(q, c3);
        const double2 xs = cmul(oms, c1), ps = cmul(q, c1);
        // x += als p + xs s;  p <- bes p + c2 r' - q c3 r + q c1 s, composed as step m0
#pragma unroll
        for (int e = 0; e < kBcgTerms; ++e) {
          cmad(cx[e], als, cp[e]);
          cp[e] = cmul(bes, cp[e]);
          if (e == 1 + m0) cp[e] = csub(cp[e], qc3);
          if (e == 2 + m0) cp[e] = cadd(cp[e], c2);
          if (e == 2 + kBcgSteps + m0) {
            cx[e] = cadd(cx[e], xs);
            cp[e] = cadd(cp[e], ps);
          }
        }
        took = true;
        const double res2 = cabs2(c2) * R;   // this shift's residual after the step
        if (res2 <= eps2) {
          next = 0;
          if (head) st->freeze_iter[j] = n;
        }
        if (!isfinite(res2)) next = 0;
      }
      act = next;
      m = m0 + 1;
      const bool finite = isfinite(R) && cfinite(rho);
      if (!finite)
        stop = 2;
      else if (__ballot(act != 0) == 0 || !rho_ok || !om_ok || n >= st->max_iter)
        stop = 1;
    }
  } else if (!(bn2 > 0.0) || !isfinite(bn2)) {
    stop = isfinite(bn2) ? 1 : 2;
  } else if (st->max_iter <= 0) {
    stop = 1;
  }
  const bool live = stop == 0;
  const bool apply = live ? m >= a.steps : (m > 0 || rs.fresh);
  const bool list = apply && mine && (took || rs.fresh);
  const uint64_t mask = __ballot(list);
  if (list) {
    const int pos = __popcll(mask & ((uint64_t(1) << j) - 1));
#pragma unroll
    for (int e = 0; e < kBcgTerms; ++e) {
      pl.cx[e][pos] = cx[e];
      pl.cp[e][pos] = cp[e];
    }
    pl.xo[pos] = int64_t(st->orig[j]) * a.n;
    pl.po[pos] = int64_t(j) * a.n;
  }
  if (j == 0) {
    pl.om = om;
    pl.be = be;
    pl.check = 0;
    pl.live = live ? 1 : 0;
    pl.apply = apply ? 1 : 0;
    pl.m = m;
    pl.first = (step && m == m0 ? n - 1 : n) - m;
    pl.fresh = rs.fresh;
    pl.nact = __popcll(mask);
  }
  if (!head) return;
  BcgRot& nx = st->rot[a.par ^ 1];
  if (mine) {
    nx.zo[j] = took && step ? z : rs.zo[j];
    nx.z[j] = zn;
    nx.tau[j] = taun;
    nx.active[j] = act;
    nx.took[j] = apply ? 0 : (took ? 1 : 0);
    if (!apply) {
#pragma unroll
      for (int e = 0; e < kBcgTerms; ++e) {
        nx.cx[e][j] = cx[e];
        nx.cp[e][j] = cp[e];
      }
    }
    if (!live) st->at_end[j] = act;
  }
  if (j == 0) {
    nx.rho = rho;
    nx.be = be;
    nx.al = step ? st->alpha : double2{1.0, 0.0};
    nx.iter = live ? n + 1 : n;
    nx.m = apply ? 0 : m;
    nx.fresh = apply ? 0 : rs.fresh;
    nx.halt = live ? 0 : 1;
    nx.check = 0;
    if (n == 0) st->bnorm2 = ss;
    if (!live) {
      // a step that broke down before its end does not count
      st->iter = stop == 2 && step && m == m0 ? n - 1 : n;
      st->status = stop == 2 ? 1 : 0;
      store_host_flag(a.hflag, 1);
    }
  }
}

enum { kBcgCsr = 0, kBcgSell = 1 };

// This workgroup's rows [beg, end): whole slices on the sliced copy.
template <int ST, int L>
__device__ __forceinline__ void bcg_rows(const BcgArgs& a, int64_t& beg, int64_t& end) {
  if constexpr (ST == kBcgSell) {
    block_range(a.nslices, kBlock / kSlice, beg, end);
    beg *= kSlice;
    end *= kSlice;
  } else {
    block_range(a.n, kBlock / L, beg, end);
  }
}

// The product B x (x = gather(col)) at the workgroup's rows: body(row, own, (B x)_row) in
// the one lane that owns the row.
template <int ST, int L, class G, class F>
__device__ __forceinline__ void bcg_product(const BcgArgs& a, int64_t beg, int64_t end,
                                            double sigma0, G gather, F body) {
  if constexpr (ST == kBcgSell) {
    const int lane = threadIdx.x % kSlice;
    const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kSlice));
    for (int64_t sl = beg / kSlice + wv; sl * kSlice < end; sl += kBlock / kSlice) {
      const int64_t row = sl * kSlice + lane;
      const int64_t rr = row < a.n ? row : a.n - 1;  // lanes past n read a valid row, unused
      const double2 own = gather(int32_t(rr));
      double2 q = a.sm.col16 ? sell_f<true>(a.sm, sl, lane, rr, own, gather)
                             : sell_f<false>(a.sm, sl, lane, rr, own, gather);
      q.x = fma(sigma0, own.x, q.x);
      q.y = fma(sigma0, own.y, q.y);
      if (row < a.n) body(row, own, q);
    }
  } else {
    const int lane = threadIdx.x % L;
    for (int64_t row = beg + threadIdx.x / L; row < end; row += kBlock / L) {
      double2 q = row_f<L>(a.m, row, lane, gather);
      const double2 own = gather(int32_t(row));
      q.x = fma(sigma0, own.x, q.x);
      q.y = fma(sigma0, own.y, q.y);
      if (lane == 0) body(row, own, q);
    }
  }
}

// ---- BA: r_n, p_n, v_n = B p_n and w^H v_n; the shifts' composed steps --------------------
template <int ST, int L>
__global__ __launch_bounds__(kBlock) void k_bcg_a(BcgArgs a) {
  BcgState* st = a.st;
  const BcgRot& rs = st->rot[a.par];
  if (rs.halt) {
    if (blockIdx.x == 0 && threadIdx.x == 0) st->rot[a.par ^ 1].halt = 1;
    return;
  }
  double tot[8], exact[3] = {0.0, 0.0, 0.0};
  bcg_sums<8>(bcg_region(a, 1), tot);
  if (rs.check) bcg_sums<3>(bcg_region(a, 2), exact);
  __shared__ BcgPlan pl;
  bcg_plan(a, tot, exact, pl);
  __syncthreads();
  const int n = rs.iter;
  const bool live = pl.live != 0, check = pl.check != 0;
  if (!live && !pl.apply && !check) return;
  const double2 om = pl.om, be = pl.be;
  const double2* __restrict__ s = ring(a.s, a.n, n + kBcgSteps - 1, kBcgSteps);  // s_{n-1}
  const double2* __restrict__ t = a.t;
  const double2* __restrict__ p = a.p[a.par];
  const double2* __restrict__ v = a.v[a.par];
  double2* __restrict__ pn = a.p[a.par ^ 1];
  double2* __restrict__ vn = a.v[a.par ^ 1];
  double2* __restrict__ rn = ring(a.r, a.n, n, kBcgRing);
  auto r_of = [&](int64_t c) { return s_of(s[c], t[c], om); };
  auto p_of = [&](int64_t c) {
    double2 o = r_of(c);
    cmad(o, be, s_of(p[c], v[c], om));
    return o;
  };
  int64_t beg, end;
  bcg_rows<ST, L>(a, beg, end);
  if (check) {  // p and v move on with the parity
    double c[3] = {0.0, 0.0, 0.0};
    const int64_t stop = end < a.n ? end : a.n;
    for (int64_t i = beg + threadIdx.x; i < stop; i += kBlock) {
      const double2 r = r_of(i);
      double2 wr{0.0, 0.0};
      cdot_acc(wr, a.b[i], r);
      c[0] += wr.x;
      c[1] += wr.y;
      c[2] += cabs2(r);
      pn[i] = p[i];
      vn[i] = v[i];
    }
    bcg_store<3>(bcg_region(a, 2), c);
    return;
  }
  if (live) {
    double2 wv{0.0, 0.0};
    bcg_product<ST, L>(a, beg, end, st->sigma0, [&](int32_t c) { return p_of(c); },
                       [&](int64_t row, const double2& own, const double2& q) {
                         pn[row] = own;
                         vn[row] = q;
                         rn[row] = r_of(row);
                         cdot_acc(wv, a.b[row], q);
                       });
    double c[2] = {wv.x, wv.y};
    bcg_store<2>(bcg_region(a, 0), c);
  }
  if (!pl.apply) return;
  // x(s) and p(s) from p(s) and the r and s of the composed steps; the last r, r_n, goes
  // into p(s) only, which a sequence that halts here no longer needs
  const int m = pl.m, first = pl.first, nact = pl.nact, fresh = pl.fresh;
  const int64_t stop = end < a.n ? end : a.n;
  for (int64_t i = beg + threadIdx.x; i < stop; i += kBlock) {
    double2 b[kBcgTerms];  // b[1 + k] = r_{first + k}, b[2 + kBcgSteps + k] = s_{first + k}
#pragma unroll
    for (int k = 0; k < kBcgSteps; ++k) {
      const bool in = k < m;
      b[1 + k] = in ? ring(a.r, a.n, first + k, kBcgRing)[i] : double2{0.0, 0.0};
      b[2 + kBcgSteps + k] = in ? ring(a.s, a.n, first + k, kBcgSteps)[i] : double2{0.0, 0.0};
    }
    b[1 + kBcgSteps] = double2{0.0, 0.0};
    const double2 last = live ? r_of(i) : double2{0.0, 0.0};
#pragma unroll
    for (int k = 0; k <= kBcgSteps; ++k)
      if (k == m) b[1 + k] = last;
    for (int q = 0; q < nact; ++q) {
      double2* __restrict__ xj = a.x + pl.xo[q];
      double2* __restrict__ pj = a.pk + pl.po[q];
      double2 xv{0.0, 0.0}, np{0.0, 0.0};
      if (!fresh) {
        xv = ld_stream(&xj[i]);
        const double2 pv = ld_stream(&pj[i]);
        cmad(xv, pl.cx[0][q], pv);
        cmad(np, pl.cp[0][q], pv);
      }
#pragma unroll
      for (int e = 1; e < kBcgTerms; ++e) {
        cmad(xv, pl.cx[e][q], b[e]);
        cmad(np, pl.cp[e][q], b[e]);
      }
      st_stream(&xj[i], xv);
      st_stream(&pj[i], np);
    }
  }
}

// ---- BB: al; s_n and t_n = B s_n with their products ---------------------------------------
template <int ST, int L>
__global__ __launch_bounds__(kBlock) void k_bcg_b(BcgArgs a) {
  BcgState* st = a.st;
  const BcgRot& rs = st->rot[a.par ^ 1];  // written by this iteration's BA
  if (rs.halt || rs.check) return;
  double wv[2];
  bcg_sums<2>(bcg_region(a, 0), wv);
  const double2 wvc{wv[0], wv[1]};
  const bool ok = cfinite(wvc) && (wvc.x != 0.0 || wvc.y != 0.0);
  const double2 al = ok ? cdiv(rs.rho, wvc) : double2{0.0, 0.0};
  const int j = threadIdx.x, n = rs.iter - 1;  // this is step n
  if (blockIdx.x == 0 && j < kWave) {
    if (ok && j < st->ns && rs.active[j]) {
      const double2 z = rs.z[j], zo = rs.zo[j], alp = rs.al, bep = rs.be;
      const double s = st->s[j];
      // z' = z zo alp / (al bep (zo - z) + zo alp (1 + s al))
      const double2 one_sal{1.0 + s * al.x, s * al.y};
      const double2 den = cadd(cmul(cmul(al, bep), csub(zo, z)), cmul(cmul(zo, alp), one_sal));
      const double2 zn = cdiv(cmul(cmul(z, zo), alp), den);
      st->zn[j] = zn;
      st->als[j] = cdiv(cmul(al, zn), z);
    }
    if (j == 0) {
      st->alpha = al;
      st->bad = ok ? 0 : 1;
    }
  }
  if (!ok) return;  // every workgroup sees the same sum; the next BA halts
  const double2* __restrict__ r = ring(a.r, a.n, n, kBcgRing);
  const double2* __restrict__ v = a.v[a.par ^ 1];
  double2* __restrict__ s = ring(a.s, a.n, n, kBcgSteps);
  int64_t beg, end;
  bcg_rows<ST, L>(a, beg, end);
  double2 ts{0.0, 0.0}, ws{0.0, 0.0}, wt{0.0, 0.0};
  double tt = 0.0, ss = 0.0;
  bcg_product<ST, L>(a, beg, end, st->sigma0, [&](int32_t c) { return s_of(r[c], v[c], al); },
                     [&](int64_t row, const double2& own, const double2& q) {
                       s[row] = own;
                       a.t[row] = q;
                       const double2 w = a.b[row];
                       cdot_acc(ts, q, own);
                       cdot_acc(ws, w, own);
                       cdot_acc(wt, w, q);
                       tt += cabs2(q);
                       ss += cabs2(own);
                     });
  double c[8] = {ts.x, ts.y, tt, ws.x, ws.y, wt.x, wt.y, ss};
  bcg_store<8>(bcg_region(a, 1), c);
}

// Workgroups for the rows, a multiple of the XCD count (at most kBcgGrid: the case above
// takes 2.35 / 2.26 / 1.96 / 1.95 / 2.02 ms with 256 / 512 / 768 / 1024 / 2048).
int bcg_grid(int64_t items, int per_pass) {
  const int64_t g = (items + per_pass - 1) / per_pass;
  return int((std::min<int64_t>(std::max<int64_t>(g, 1), kBcgGrid) + kXcds - 1) / kXcds * kXcds);
}

template <int ST, int L> void bcg_launch(const BcgArgs& a, int g, hipStream_t s) {
  k_bcg_a<ST, L><<<g, kBlock, 0, s>>>(a);
  k_bcg_b<ST, L><<<g, kBlock, 0, s>>>(a);
}

int bcg_grid_of(const BcgArgs& a) {
  return a.sell ? bcg_grid(a.nslices, kBlock / kSlice) : bcg_grid(a.n, kBlock / a.lanes);
}

}  // namespace

hipError_t launch_bcg_start(const BcgArgs& a, hipStream_t s) {
  // the first BA reads as many partials as it has workgroups
  k_bcg_start<<<bcg_grid_of(a), kBlock, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t launch_bcg_iteration(const BcgArgs& a, hipStream_t s) {
  const int g = bcg_grid_of(a);
  if (a.sell) {
    bcg_launch<kBcgSell, 1>(a, g, s);
  } else {
    switch (a.lanes) {
      case 4: bcg_launch<kBcgCsr, 4>(a, g, s); break;
      case 8: bcg_launch<kBcgCsr, 8>(a, g, s); break;
      case 16: bcg_launch<kBcgCsr, 16>(a, g, s); break;
      case 32: bcg_launch<kBcgCsr, 32>(a, g, s); break;
      default: return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

}  // namespace msc
