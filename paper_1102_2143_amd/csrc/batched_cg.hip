// Batched single-shift CG: m <= 16 systems (A + sigma_j) e_j = f_j that share one
// operator, advanced together so every iteration reads the matrix once for all of them.
//
// Used for the per-shift refinement after a mixed-precision multishift sequence (each
// shift's FP64 true residual becomes the right-hand side of a correction solve) and for
// adjoint solves with unrelated right-hand sides.  The vectors of the batch lie one system
// after the other, v[j n + i], as the caller's do, so that a wave's gathers for one system
// read neighbouring rows together.
//
// Systems still iterating are kept in a list on the device; the two operator halves take
// it in groups of a few systems, one group per workgroup.  A wave reads the matrix
// (or the links) of its rows once for its group and gathers each system's values in turn;
// the workgroups of the other groups on the same rows follow one another on one XCD, whose
// L2 then serves the matrix to all but the first.  A system that has converged costs
// nothing from the next iteration on.  Ten systems at 16^4 in FP64, an iteration's halves:
// 155 and 162 us with 16 interleaved systems on the CSR (10 padded to 16, all of them to
// the end); 38 and 44 us on the sliced copy, 31 and 38 us on the links on average here.
//
// An outer defect-correction cycle recomputes f_j - (A + sigma_j) x_j in FP64 (the
// multi-vector kernels below), the inner CG runs in the working precision from e = 0,
// and x_j += e_j is accumulated in FP64.
#include <algorithm>
#include <type_traits>

#include "dev_common.h"
#include "msc_internal.h"
#include "sell_load.h"
#include "stencil.h"

namespace msc {

namespace {

template <class R> __device__ __forceinline__ Csr<cplx<R>> pick_a(const BssArgs& a, bool second);
template <> __device__ __forceinline__ Csr<float2> pick_a<float>(const BssArgs& a, bool second) {
  return second ? a.mh32 : a.m32;
}
template <> __device__ __forceinline__ Csr<double2> pick_a<double>(const BssArgs& a, bool second) {
  return second ? a.mh64 : a.m64;
}
template <class R> __device__ __forceinline__ Sell<cplx<R>> pick_s(const BssArgs& a, bool second);
template <> __device__ __forceinline__ Sell<float2> pick_s<float>(const BssArgs& a, bool second) {
  return second ? a.sh32 : a.s32;
}
template <> __device__ __forceinline__ Sell<double2> pick_s<double>(const BssArgs& a, bool second) {
  return second ? a.sh64 : a.s64;
}
template <class R> __device__ __forceinline__ Stencil<cplx<R>> pick_l(const BssArgs& a);
template <> __device__ __forceinline__ Stencil<float2> pick_l<float>(const BssArgs& a) { return a.w32; }
template <> __device__ __forceinline__ Stencil<double2> pick_l<double>(const BssArgs& a) { return a.w64; }

enum { kCsr = 0, kSell = 1, kLinks3 = 2, kLinks2 = 3 };  // what an operator half reads

// Most systems of one group, and most workgroups, by storage.  A wave of the links' halves
// holds a direction's two links beside its group's accumulators (252 VGPRs at five
// systems), and two waves per SIMD with little each beat fewer, longer ones; the sliced
// rows need few registers, and a larger group reads the matrix less often.  Ten systems at
// 16^4 in FP64, whole solve: links, groups of 1 / 2 / 3 / 5 / 8: 33.0 / 28.7 / 29.7 / 33.4 /
// 45.2 ms, and 30.8 ms with 768 workgroups (vectors colour by colour: 28.9 / 28.3 / 28.2 ms
// with 1 on 768, 2 and 3; in row order 29.0 with 2; own rows past the caches 30.4); sliced copy (a gradient), groups of 2 / 3 / 4 /
// 5 / 8 on 512: 61.1 / 59.6 / 58.4 / 55.9 / 58.2 ms; 5 on 768 and 1024: 51.3 and 53.8 ms.
template <int ST> constexpr int group_max() { return ST == kCsr || ST == kSell ? 5 : 2; }
template <int ST> constexpr int half_grid() { return ST == kCsr || ST == kSell ? 768 : 512; }

// This workgroup's share of an operator half: systems list[lo, lo + cnt) and, in units of
// `step` items (rows, slices or blocks of sites), the contiguous range [beg, end).  The
// grid is a multiple of the XCD count; XCD x owns an eighth of the items, its workgroups
// are dealt to the groups in turn and the workgroups of a group split its items evenly.
struct Share {
  int groups, group, lo, cnt;
  int64_t beg, end;
};

__device__ __forceinline__ int group_lo(int nact, int groups, int g) { return nact * g / groups; }

template <int G> __device__ __forceinline__ Share make_share(int nact, int64_t items, int step) {
  Share h;
  const int x = int(blockIdx.x) % kXcds, xb = int(blockIdx.x) / kXcds, nb = int(gridDim.x) / kXcds;
  h.groups = (nact + G - 1) / G;  // nact >= 1 while the batch runs; at most nb
  h.group = xb % h.groups;
  h.lo = group_lo(nact, h.groups, h.group);
  h.cnt = group_lo(nact, h.groups, h.group + 1) - h.lo;
  const int mates = (nb - h.group + h.groups - 1) / h.groups, me = xb / h.groups;
  const int64_t units = (items + step - 1) / step;
  const int64_t u0 = units * x / kXcds, u1 = units * (x + 1) / kXcds;
  h.beg = (u0 + (u1 - u0) * me / mates) * step;
  h.end = min((u0 + (u1 - u0) * (me + 1) / mates) * step, items);
  return h;
}

// The workgroup's sums of its group's systems, then (in the last workgroup) the totals of
// all systems of the list into out[0..nact).
template <int G>
__device__ __forceinline__ void store_group_partials(double (&v)[G], double* partial) {
  block_sum_k<kBlock, G>(v);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < G; ++q) store_agent(&partial[blockIdx.x * G + q], v[q]);
  }
}

template <int G>
__device__ __forceinline__ void sum_group_partials(const double* partial, int nact, int groups,
                                                   double* out) {
  // thread -> (position in the list tid / 16, sub-lane tid % 16)
  const int li = threadIdx.x / 16, s = threadIdx.x % 16;
  double acc = 0.0;
  if (li < nact) {
    int g = 0;
    while (group_lo(nact, groups, g + 1) <= li) ++g;
    const int u = li - group_lo(nact, groups, g);
    const int nb = int(gridDim.x) / kXcds, mates = (nb - g + groups - 1) / groups;
    const int count = mates * kXcds;  // workgroups of the group, sixteen at a time
    constexpr int kAhead = 8;
    for (int b = s; b < count; b += 16 * kAhead) {
      double w[kAhead];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) {
        const int c = b + 16 * k;
        const int blk = ((c / kXcds) * groups + g) * kXcds + c % kXcds;
        w[k] = c < count ? load_agent(&partial[blk * G + u]) : 0.0;
      }
#pragma unroll
      for (int k = 0; k < kAhead; ++k) acc += w[k];
    }
  }
  acc = group_sum<16>(acc);
  if (s == 0) out[li] = acc;
  __syncthreads();
}

// After the partials of half 1 are stored: the last workgroup forms a_j = R_j / P_j.
template <int G> __device__ void ik1_finish(const BssArgs& a, int groups) {
  BssState* st = a.st;
  if (!arrive_last(a.tickets + 8 * kTicketSite)) return;
  __shared__ double tot[kBssMax];
  const int nact = st->nlist[a.par];
  sum_group_partials<G>(a.partial, nact, groups, tot);
  if (int(threadIdx.x) < nact) {
    const int q = st->list[a.par][threadIdx.x];
    const double P = tot[threadIdx.x];
    if (P > 0.0 && isfinite(P)) {
      st->a[q] = st->R[q] / P;
    } else {
      st->a[q] = 0.0;
      st->active[q] = 0;
      st->bad[q] = 1;
    }
  }
}

// After the partials of half 2 are stored: the last workgroup forms b_j and R_j, retires
// converged systems, lists the others for the next iteration and decides whether the
// batch halts.
template <int G> __device__ void ik2_finish(const BssArgs& a, int groups) {
  BssState* st = a.st;
  if (!arrive_last(a.tickets + 9 * kTicketSite)) return;
  __shared__ double tot[kBssMax];
  const int nact = st->nlist[a.par];
  sum_group_partials<G>(a.partial, nact, groups, tot);
  if (threadIdx.x < kWave) {
    const int li = threadIdx.x;
    const int q = li < nact ? st->list[a.par][li] : 0;
    bool act = false;
    if (li < nact) {
      bool upd = false;
      if (st->active[q]) {
        const double Rn = tot[li];
        if (!isfinite(Rn)) {
          st->bad[q] = 1;
          st->active[q] = 0;
        } else {
          upd = true;
          st->b[q] = Rn / st->R[q];
          st->R[q] = Rn;
          st->iters[q] += 1;
          act = !(Rn <= st->target2[q]);
          st->active[q] = act ? 1 : 0;
        }
      }
      st->upd[q] = upd ? 1 : 0;
    }
    const uint64_t am = __ballot(act);
    if (act) st->list[a.par ^ 1][__popcll(am & ((uint64_t(1) << li) - 1))] = q;
    if (li == 0) {
      st->nlist[a.par ^ 1] = __popcll(am);
      st->iter += 1;
      if (am == 0 || st->iter >= st->max_iter) {
        st->halt = 1;
        store_host_flag(a.hflag, 1);
      }
      st->k3_enable = 1;
    }
  }
}

// The group's vectors of one array: system list[lo + u] starts at v + list[lo + u] n (the
// last one repeated past cnt, so that every pointer is valid).
template <int G, class T>
__device__ __forceinline__ void group_ptrs(const BssArgs& a, const Share& h, T* v, T* (&o)[G]) {
  const int* list = a.st->list[a.par];
#pragma unroll
  for (int u = 0; u < G; ++u)
    o[u] = v + int64_t(list[h.lo + (u < h.cnt ? u : h.cnt - 1)]) * a.n;
}

// P's term of one row: v = (A1 p)_i of system sig, p its direction there.
template <class R, bool MHM>
__device__ __forceinline__ double p_term(const cplx<R>& v, const cplx<R>& p, double sig) {
  if (MHM) return norm2d<R>(v) + sig * norm2d<R>(p);
  return double(p.x) * double(v.x) + double(p.y) * double(v.y) + sig * norm2d<R>(p);
}

// r - a (q + sig p) at one row.
template <class R>
__device__ __forceinline__ cplx<R> r_next(const cplx<R>& r, const cplx<R>& q, const cplx<R>& p,
                                          double step, double sig) {
  const double2 qd = to_d(q), pd = to_d(p), rd = to_d(r);
  return from_d<R>(double2{rd.x - step * (qd.x + sig * pd.x), rd.y - step * (qd.y + sig * pd.y)});
}

// Off-diagonal entries of one sliced row times the group's vectors (KP pairs a round trip).
template <class R, int G, int KP, bool NARROW>
__device__ __forceinline__ void sell_row_group(const Sell<cplx<R>>& m,
                                               const cplx<R>* const (&xs)[G], int cnt,
                                               int64_t sl, int lane, cplx<R> (&acc)[G]) {
  int32_t c, c1;
  if (m.wp > 0) {
    c = int32_t(sl) * m.wp;
    c1 = c + m.wp;
  } else {
    c = load_uniform(m.cptr, sl);
    c1 = load_uniform(m.cptr, sl + 1);
  }
  for (; c < c1; c += KP) {
    const int np = c1 - c;
    int2 cc[KP];
    cplx<R> v[2 * KP];
    if (np >= KP)
      sell_load<R, KP, true, NARROW>(m, c, KP, lane, cc, v);
    else
      sell_load<R, KP, false, NARROW>(m, c, np, lane, cc, v);
#pragma unroll
    for (int q = 0; q < G; ++q) {
      if (q < cnt) {
        cplx<R> g[2 * KP];
#pragma unroll
        for (int u = 0; u < KP; ++u) {  // a missing pair: column 0, values 0
          g[2 * u] = xs[q][cc[u].x];
          g[2 * u + 1] = xs[q][cc[u].y];
        }
#pragma unroll
        for (int u = 0; u < 2 * KP; ++u)
          if (u < 2 * np) cfma<R>(acc[q], v[u], g[u]);
      }
    }
  }
}

// One half of the operator for this workgroup's systems and rows: body(row, out) with the
// products out[u] of every system u < cnt at `row` of the vectors (on the links colour by
// colour); lanes with nothing to do skip it.
template <class R, int G, int ST, int L, class F>
__device__ __forceinline__ void half(const BssArgs& a, bool second, const Share& h,
                                     const cplx<R>* const (&xs)[G], F body) {
  if constexpr (ST == kCsr) {
    const Csr<cplx<R>> m = pick_a<R>(a, second);
    constexpr int GPB = kBlock / L;
    const int lane = threadIdx.x % L;
    for (int64_t row = h.beg + threadIdx.x / L; row < h.end; row += GPB) {
      cplx<R> o[G];
#pragma unroll
      for (int q = 0; q < G; ++q) o[q] = czero<R>();
      const int32_t e1 = m.rowptr[row + 1];
      for (int32_t e = m.rowptr[row] + lane; e < e1; e += L) {
        const int32_t c = m.col[e];
        const cplx<R> v = m.val[e];
#pragma unroll
        for (int q = 0; q < G; ++q)
          if (q < h.cnt) cfma<R>(o[q], v, xs[q][c]);
      }
#pragma unroll
      for (int q = 0; q < G; ++q)
        if (q < h.cnt) o[q] = group_sum_c<L, R>(o[q]);
      if (lane == 0) body(row, o);
    }
  } else if constexpr (ST == kSell) {
    const Sell<cplx<R>> m = pick_s<R>(a, second);
    constexpr int KP = std::is_same<R, float>::value ? 4 : 2;
    const int lane = threadIdx.x % kSlice;
    const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kSlice));
    for (int64_t sl = h.beg + wv; sl < h.end; sl += kBlock / kSlice) {
      const int64_t row = sl * kSlice + lane;
      const int64_t rr = row < a.n ? row : a.n - 1;  // lanes past n read a valid row, unused
      cplx<R> o[G];
      const cplx<R> d = m.diag[rr];
#pragma unroll
      for (int q = 0; q < G; ++q) {
        o[q] = czero<R>();
        if (q < h.cnt) cfma<R>(o[q], d, xs[q][rr]);
      }
      if (m.col16)
        sell_row_group<R, G, KP, true>(m, xs, h.cnt, sl, lane, o);
      else
        sell_row_group<R, G, KP, false>(m, xs, h.cnt, sl, lane, o);
      if (row < a.n) body(row, o);
    }
  } else {
    constexpr int LR = ST == kLinks2 ? 2 : 3;
    const Stencil<cplx<R>> w = pick_l<R>(a);
    const uint32_t vol = uint32_t(w.vol);
    const int lane = threadIdx.x % kWave;
    const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kWave));
    for (int64_t blk = h.beg + wv; blk < h.end; blk += kBlock / kWave) {
      const uint32_t site = uint32_t(blk * kWave) + uint32_t(lane);
      const uint32_t ss = site < vol ? site : vol - 1;  // lanes past the volume: unused
      cplx<R> o[G][3];
      stencil_site_group<R, LR, G>(w, ss, second ? -1 : 1, xs, h.cnt, o);
      if (site < vol) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          cplx<R> oc[G];
#pragma unroll
          for (int q = 0; q < G; ++q) oc[q] = o[q][c];
          body(int64_t(c) * vol + site, oc);
        }
      }
    }
  }
}

template <int ST, int L> __device__ __forceinline__ int64_t half_items(const BssArgs& a) {
  return ST == kCsr ? a.n : (ST == kSell ? a.nslices : (a.w64.vol + kWave - 1) / kWave);
}
template <int ST, int L> constexpr int half_step() {
  return ST == kCsr ? kBlock / L : kBlock / kWave;
}

// ---- half 1: t_j = A1 p_j and P_j = p_j^H (A + sigma_j) p_j --------------------------
template <class R, int ST, int L, bool MHM>
__global__ __launch_bounds__(kBlock, 2) void ik1(BssArgs a) {
  constexpr int G = group_max<ST>();
  BssState* st = a.st;
  if (st->halt) {
    if (blockIdx.x == 0 && threadIdx.x == 0) st->k3_enable = 0;
    return;
  }
  const Share h = make_share<G>(st->nlist[a.par], half_items<ST, L>(a), half_step<ST, L>());
  const cplx<R>* p[G];
  cplx<R>* t[G];
  group_ptrs<G, const cplx<R>>(a, h, static_cast<const cplx<R>*>(a.p), p);
  group_ptrs<G, cplx<R>>(a, h, static_cast<cplx<R>*>(a.t), t);
  double sig[G], acc[G];
#pragma unroll
  for (int u = 0; u < G; ++u) {
    sig[u] = st->sigma[st->list[a.par][h.lo + (u < h.cnt ? u : 0)]];
    acc[u] = 0.0;
  }
  half<R, G, ST, L>(a, false, h, p, [&](int64_t row, const cplx<R>(&o)[G]) {
#pragma unroll
    for (int u = 0; u < G; ++u) {
      if (u < h.cnt) {
        t[u][row] = o[u];
        acc[u] += p_term<R, MHM>(o[u], p[u][row], sig[u]);
      }
    }
  });
  store_group_partials(acc, a.partial);
  ik1_finish<G>(a, h.groups);
}

// ---- half 2: r_j <- r_j - a_j (A2 t_j + sigma_j p_j), R_j = |r_j|^2 --------------------
template <class R, int ST, int L, bool MHM>
__global__ __launch_bounds__(kBlock, 2) void ik2(BssArgs a) {
  constexpr int G = group_max<ST>();
  BssState* st = a.st;
  if (st->halt) return;
  const Share h = make_share<G>(st->nlist[a.par], half_items<ST, L>(a), half_step<ST, L>());
  const cplx<R>* p[G];
  const cplx<R>* t[G];
  cplx<R>* r[G];
  group_ptrs<G, const cplx<R>>(a, h, static_cast<const cplx<R>*>(a.p), p);
  group_ptrs<G, const cplx<R>>(a, h, static_cast<const cplx<R>*>(a.t), t);
  group_ptrs<G, cplx<R>>(a, h, static_cast<cplx<R>*>(a.r), r);
  double sig[G], step[G], acc[G];
#pragma unroll
  for (int u = 0; u < G; ++u) {
    const int j = st->list[a.par][h.lo + (u < h.cnt ? u : 0)];
    sig[u] = st->sigma[j];
    step[u] = st->active[j] ? st->a[j] : 0.0;
    acc[u] = 0.0;
  }
  auto row_step = [&](int64_t row, const cplx<R>(&o)[G]) {
#pragma unroll
    for (int u = 0; u < G; ++u) {
      if (u < h.cnt) {
        const cplx<R> nr = r_next<R>(r[u][row], o[u], p[u][row], step[u], sig[u]);
        r[u][row] = nr;
        acc[u] += norm2d<R>(nr);
      }
    }
  };
  if constexpr (MHM) {
    half<R, G, ST, L>(a, true, h, t, row_step);
  } else {  // A given: t is A p already
    const int64_t rows = ST == kCsr ? 1 : kSlice, end = min(h.end * rows, a.n);
    for (int64_t row = h.beg * rows + threadIdx.x; row < end; row += kBlock) {
      cplx<R> o[G];
#pragma unroll
      for (int u = 0; u < G; ++u) o[u] = u < h.cnt ? t[u][row] : czero<R>();
      row_step(row, o);
    }
  }
  store_group_partials(acc, a.partial);
  ik2_finish<G>(a, h.groups);
}

// ---- IK3: e_j += a_j p_j; p_j <- r_j + b_j p_j for the systems of this iteration ---------
template <class R>
__global__ __launch_bounds__(kBlock) void ik3(BssArgs a) {
  const BssState* st = a.st;
  if (!st->k3_enable) return;
  int64_t beg, end;
  block_range(a.n, kBlock, beg, end);
  const int nact = st->nlist[a.par];
  for (int li = 0; li < nact; ++li) {
    const int j = st->list[a.par][li];
    if (!st->upd[j]) continue;
    const cplx<R>* __restrict__ r = static_cast<const cplx<R>*>(a.r) + int64_t(j) * a.n;
    cplx<R>* __restrict__ p = static_cast<cplx<R>*>(a.p) + int64_t(j) * a.n;
    cplx<R>* __restrict__ ev = static_cast<cplx<R>*>(a.e) + int64_t(j) * a.n;
    const double aj = st->a[j], bj = st->b[j];
    const bool more = st->active[j] != 0;
    for (int64_t i = beg + threadIdx.x; i < end; i += kBlock) {
      const double2 pd = to_d(p[i]);
      double2 ed = to_d(ev[i]);
      ed.x = fma(aj, pd.x, ed.x);
      ed.y = fma(aj, pd.y, ed.y);
      ev[i] = from_d<R>(ed);
      if (more) {
        const double2 rd = to_d(r[i]);
        p[i] = from_d<R>(double2{fma(bj, pd.x, rd.x), fma(bj, pd.y, rd.y)});
      }
    }
  }
}

// ---- FP64 residual of up to 8 systems: r_j = f_j - (A + sigma_j) x_j ---------------------
template <int L>
__device__ __forceinline__ void row_dot_ptrs(const Csr<double2>& m, const double2* const* xs, int kc,
                                             int64_t row, int lane, double2 (&acc)[kResChunk]) {
#pragma unroll
  for (int q = 0; q < kResChunk; ++q) acc[q] = double2{0.0, 0.0};
  const int32_t beg = m.rowptr[row], end = m.rowptr[row + 1];
  for (int32_t e = beg + lane; e < end; e += L) {
    const int32_t c = m.col[e];
    const double2 v = m.val[e];
#pragma unroll
    for (int q = 0; q < kResChunk; ++q)
      if (q < kc) cfma<double>(acc[q], v, xs[q][c]);
  }
#pragma unroll
  for (int q = 0; q < kResChunk; ++q) acc[q] = group_sum_c<L, double>(acc[q]);
}

template <int L>
__global__ __launch_bounds__(kBlock) void k_res_first(ResArgs v) {
  constexpr int GPB = kBlock / L;
  const int lane = threadIdx.x % L, grp = threadIdx.x / L;
  int64_t beg, end;
  block_range(v.n, GPB, beg, end);
  double2 acc[kResChunk];
  for (int64_t row = beg + grp; row < end; row += GPB) {
    row_dot_ptrs<L>(v.m1, v.x, v.kc, row, lane, acc);
    if (lane == 0) {
#pragma unroll
      for (int q = 0; q < kResChunk; ++q)
        if (q < v.kc) v.u[int64_t(q) * v.n + row] = acc[q];
    }
  }
}

// Per-system norms: workgroup partials, then the last workgroup's totals in out[0..kc).
__device__ void res_finish(const ResArgs& v, double (&nrm)[kResChunk]) {
  block_sum_k<kBlock, kResChunk>(nrm);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < kResChunk; ++q) store_agent(&v.partial[blockIdx.x * kResChunk + q], nrm[q]);
  }
  if (!arrive_last(v.ticket)) return;
  for (int q = 0; q < v.kc; ++q) {
    double s = 0.0;
    for (int i = threadIdx.x; i < int(gridDim.x); i += kBlock) s += load_agent(&v.partial[i * kResChunk + q]);
    s = block_sum<kBlock>(s);
    if (threadIdx.x == 0) v.out[q] = s;
  }
}

// Row `row`'s residuals from the products acc_q = (A x_q)[row]: norms, and the
// system's r = p = residual, e = 0 when r is set.
template <class R>
__device__ __forceinline__ void res_row(const ResArgs& v, int64_t row, const double2 (&acc)[kResChunk],
                                        double (&nrm)[kResChunk]) {
  cplx<R>* __restrict__ r = static_cast<cplx<R>*>(v.r);
  cplx<R>* __restrict__ p = static_cast<cplx<R>*>(v.p);
  cplx<R>* __restrict__ e = static_cast<cplx<R>*>(v.e);
#pragma unroll
  for (int q = 0; q < kResChunk; ++q) {
    if (q < v.kc) {
      const double2 fv = v.f[q][row], xv = v.x[q][row];
      double2 rt;
      rt.x = fv.x - acc[q].x - v.sig[q] * xv.x;
      rt.y = fv.y - acc[q].y - v.sig[q] * xv.y;
      nrm[q] += fma(rt.x, rt.x, rt.y * rt.y);
      if (r) {
        const int64_t idx = int64_t(v.j0 + q) * v.n + (v.vol ? (row % 3) * v.vol + row / 3 : row);
        const cplx<R> rc = from_d<R>(rt);
        r[idx] = rc;
        p[idx] = rc;
        e[idx] = czero<R>();
      }
    }
  }
}

template <class R, int L>
__global__ __launch_bounds__(kBlock) void k_res_second(ResArgs v) {
  constexpr int GPB = kBlock / L;
  const int lane = threadIdx.x % L, grp = threadIdx.x / L;
  int64_t beg, end;
  block_range(v.n, GPB, beg, end);
  double2 acc[kResChunk];
  double nrm[kResChunk];
#pragma unroll
  for (int q = 0; q < kResChunk; ++q) nrm[q] = 0.0;
  const double2* in[kResChunk];
#pragma unroll
  for (int q = 0; q < kResChunk; ++q) in[q] = v.mhm ? v.u + int64_t(q) * v.n : v.x[q];
  for (int64_t row = beg + grp; row < end; row += GPB) {
    row_dot_ptrs<L>(v.m2, in, v.kc, row, lane, acc);
    if (lane == 0) res_row<R>(v, row, acc, nrm);
  }
  res_finish(v, nrm);
}

// The same two steps on the sliced ELLPACK copies: one row per lane.
__global__ __launch_bounds__(kBlock) void k_res_first_s(ResArgs v) {
  constexpr int SPB = kBlock / kSlice;
  const int lane = threadIdx.x % kSlice;
  const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kSlice));
  const double2* xs[kResChunk];
#pragma unroll
  for (int q = 0; q < kResChunk; ++q) xs[q] = v.x[q < v.kc ? q : 0];
  int64_t beg, end;
  block_range(v.nslices, SPB, beg, end);
  for (int64_t sl = beg + wv; sl < end; sl += SPB) {
    const int64_t row = sl * kSlice + lane;
    const int64_t rr = row < v.n ? row : v.n - 1;
    double2 acc[kResChunk];
    sell_row_multi<double, kResChunk, 1>(v.s1, xs, v.kc, sl, lane, acc);
    const double2 d = v.s1.diag[rr];
#pragma unroll
    for (int q = 0; q < kResChunk; ++q) {
      if (q < v.kc) {
        cfma<double>(acc[q], d, xs[q][rr]);
        if (row < v.n) v.u[int64_t(q) * v.n + row] = acc[q];
      }
    }
  }
}

template <class R>
__global__ __launch_bounds__(kBlock) void k_res_second_s(ResArgs v) {
  constexpr int SPB = kBlock / kSlice;
  const int lane = threadIdx.x % kSlice;
  const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kSlice));
  const double2* in[kResChunk];
#pragma unroll
  for (int q = 0; q < kResChunk; ++q) {
    const int qq = q < v.kc ? q : 0;
    in[q] = v.mhm ? v.u + int64_t(qq) * v.n : v.x[qq];
  }
  double nrm[kResChunk];
#pragma unroll
  for (int q = 0; q < kResChunk; ++q) nrm[q] = 0.0;
  int64_t beg, end;
  block_range(v.nslices, SPB, beg, end);
  for (int64_t sl = beg + wv; sl < end; sl += SPB) {
    const int64_t row = sl * kSlice + lane;
    const int64_t rr = row < v.n ? row : v.n - 1;
    double2 acc[kResChunk];
    sell_row_multi<double, kResChunk, 1>(v.s2, in, v.kc, sl, lane, acc);
    const double2 d = v.s2.diag[rr];
#pragma unroll
    for (int q = 0; q < kResChunk; ++q)
      if (q < v.kc) cfma<double>(acc[q], d, in[q][rr]);
    if (row < v.n) res_row<R>(v, row, acc, nrm);
  }
  res_finish(v, nrm);
}

// x_j += e_j (FP64 accumulation of the correction)
template <class R>
__global__ __launch_bounds__(kBlock) void k_accum(BssArgs a, XPtrs xp) {
  const int m = a.st->m;
  const int64_t vol = a.links ? a.n / 3 : 0;  // colour by colour on the links
  for (int j = 0; j < m; ++j) {
    const cplx<R>* __restrict__ ev = static_cast<const cplx<R>*>(a.e) + int64_t(j) * a.n;
    double2* __restrict__ x = xp.x[j];
    for (int64_t i = blockIdx.x * int64_t(kBlock) + threadIdx.x; i < a.n; i += int64_t(gridDim.x) * kBlock) {
      const double2 d = to_d(ev[vol ? (i % 3) * vol + i / 3 : i]);
      double2 v = x[i];
      v.x += d.x;
      v.y += d.y;
      x[i] = v;
    }
  }
}

int grid_for(int64_t items, int per_pass) {
  int64_t g = (items + per_pass - 1) / per_pass;
  if (g > kMaxGrid) g = kMaxGrid;
  if (g < kXcds) g = kXcds;
  return int((g + kXcds - 1) / kXcds * kXcds);
}

#define MSC_L_SWITCH(LANES, CALL)                        \
  switch (LANES) {                                       \
    case 4: { constexpr int LL = 4; CALL; } break;       \
    case 8: { constexpr int LL = 8; CALL; } break;       \
    case 16: { constexpr int LL = 16; CALL; } break;     \
    case 32: { constexpr int LL = 32; CALL; } break;     \
    default: return hipErrorInvalidValue;                \
  }

template <class R, int ST, int L>
void launch_halves(const BssArgs& a, int64_t items, int step, hipStream_t s) {
  // at least one workgroup per XCD and group
  const int groups = (a.m + group_max<ST>() - 1) / group_max<ST>();
  const int grid = std::max(kXcds * groups, std::min(half_grid<ST>(), grid_for(items * groups, step)));
  if (a.kind == MSC_A_MHM) {
    ik1<R, ST, L, true><<<grid, kBlock, 0, s>>>(a);
    ik2<R, ST, L, true><<<grid, kBlock, 0, s>>>(a);
  } else if constexpr (ST == kCsr || ST == kSell) {  // links are M's
    ik1<R, ST, L, false><<<grid, kBlock, 0, s>>>(a);
    ik2<R, ST, L, false><<<grid, kBlock, 0, s>>>(a);
  }
}

template <class R>
hipError_t bss_iteration_impl(const BssArgs& a, hipStream_t s) {
  const int gw = kBlock / kWave;
  const int64_t blocks = (a.w64.vol + kWave - 1) / kWave;
  if (a.links == 2) {
    launch_halves<R, kLinks2, 1>(a, blocks, gw, s);
  } else if (a.links == 3) {
    launch_halves<R, kLinks3, 1>(a, blocks, gw, s);
  } else if (a.sell) {
    launch_halves<R, kSell, 1>(a, a.nslices, gw, s);
  } else {
    MSC_L_SWITCH(a.lanes, (launch_halves<R, kCsr, LL>(a, a.n, kBlock / LL, s)));
  }
  ik3<R><<<grid_for(a.n, kBlock), kBlock, 0, s>>>(a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_bss_iteration(int prec, const BssArgs& a, hipStream_t s) {
  return prec == MSC_PREC_MIXED ? bss_iteration_impl<float>(a, s) : bss_iteration_impl<double>(a, s);
}

hipError_t launch_residual(int prec, int lanes, const ResArgs& v, hipStream_t s) {
  if (v.kc < 1 || v.kc > kResChunk) return hipErrorInvalidValue;
  if (v.sell) {
    const int gs = grid_for(v.nslices, kBlock / kSlice);
    if (v.mhm) k_res_first_s<<<gs, kBlock, 0, s>>>(v);
    if (prec == MSC_PREC_MIXED)
      k_res_second_s<float><<<gs, kBlock, 0, s>>>(v);
    else
      k_res_second_s<double><<<gs, kBlock, 0, s>>>(v);
    return hipGetLastError();
  }
  const int g1 = grid_for(v.n, kBlock / lanes);
  if (v.mhm) MSC_L_SWITCH(lanes, (k_res_first<LL><<<g1, kBlock, 0, s>>>(v)));
  if (prec == MSC_PREC_MIXED) {
    MSC_L_SWITCH(lanes, (k_res_second<float, LL><<<g1, kBlock, 0, s>>>(v)));
  } else {
    MSC_L_SWITCH(lanes, (k_res_second<double, LL><<<g1, kBlock, 0, s>>>(v)));
  }
  return hipGetLastError();
}

hipError_t launch_accum(int prec, const BssArgs& a, const XPtrs& xp, hipStream_t s) {
  const int g = grid_for(a.n, kBlock);
  if (prec == MSC_PREC_MIXED)
    k_accum<float><<<g, kBlock, 0, s>>>(a, xp);
  else
    k_accum<double><<<g, kBlock, 0, s>>>(a, xp);
  return hipGetLastError();
}

}  // namespace msc
