// Batched multishift solves: many independent systems of uneven size, each with up to
// four right-hand sides and up to sixteen shifts, advanced together -- one launch of
// each iteration kernel covers every row of every unfinished system.
//
// Work is split into chunks of rows (each chunk belongs to one system); the kernels are
// persistent (a bounded grid loops over the chunk list), one launch for the systems of each
// precision.  Every system has its own scalar state.  The sequence is the single solve's
// (multishift.hip): BK1 u = M r, BS1 the scalars of the step (one workgroup per system, one
// lane per (rhs, shift)), BK2 the step of s and r, BS2 the stopping rules.  The shifts' steps
// are composed and applied by a kernel of its own (BF) every few iterations, which also
// converts a system whose right-hand sides have all reached switch_tol to complex64 (it
// waits for that BF); reliable updates run between BFs.
//
// As there, BK2 also sums c = Re r^H s, and a system whose P leaves its short form (or whose FP64
// phase says that it would in complex64) waits for the next BF, which hands its right-hand sides
// their directions; from then on BP updates p, BK1 and BK2 form P and s from it and BK2 keeps x_0.
//
// Operators made from links read them: a wave takes 64 sites of one right-hand side, whose
// vectors lie apart, colour by colour; the waves of the other right-hand sides on the same
// sites share its links in the caches.  Stored matrices: the right-hand sides of a system
// are interleaved, v[i R + q], so that one read of a matrix row serves all of them.
//
// The iteration kernels are bound by the round trips of a wave's task (about 28000 tasks of 64
// sites or rows), so what counts is how many are in flight and how few they are: with each
// system's last chunk finalising its scalars (a ticket that every chunk waits for), both
// precisions in one kernel (216 registers) and the descriptors read as vectors, 48 lattices
// of 4^4 to 12^4 and 16 grids of 32^3, four right-hand sides and ten shifts each, took
// 122 + 140 us an iteration in complex64; without the tickets 83 + 104; a kernel per
// precision 66 + 78; descriptors and state through the scalar cache (164 and 98 registers)
// 53 + 70, FP64 83 + 111 (the vectors and links alone at 5.5 TB/s: 35 + 54 and 70 + 108); with
// c_n summed besides, 53 + 74 and 84 + 115.
// The solve in mixed precision: 172 -> 87 ms; as stored matrices 175 -> 122.
#include <type_traits>

#include "dev_common.h"
#include "msc_internal.h"
#include "sell_load.h"
#include "stencil.h"

namespace msc {

namespace {

constexpr int kQK = kBatchMaxRhs * kBatchMaxShifts;  // 64 lanes of the finalising wave

// What no kernel of a launch writes (descriptors; the state, in BK1 and BK2), read through the
// scalar cache: addresses are uniform over the workgroup.
template <class T> __device__ __forceinline__ T load_const(const T* p) {
  static_assert(sizeof(T) % 4 == 0, "words");
  using cword = const __attribute__((address_space(4))) uint32_t;
  uint32_t w[sizeof(T) / 4];
  cword* c = (cword*)(reinterpret_cast<uintptr_t>(p));
#pragma unroll
  for (unsigned i = 0; i < sizeof(T) / 4; ++i) w[i] = c[i];
  T v;
  __builtin_memcpy(&v, w, sizeof(T));
  return v;
}

template <class R> struct BVec;  // a system's vectors of one precision
template <> struct BVec<double> {
  static __device__ __forceinline__ double2* slot(const BatchSys& S, int k, int64_t len) {
    return S.ring64 + k * len;
  }
  static __device__ __forceinline__ double2* u(const BatchSys& S) { return S.u64; }
  static __device__ __forceinline__ double2* s(const BatchSys& S) { return S.s64v; }
  static __device__ __forceinline__ double2* pk(const BatchSys& S) { return S.pk64; }
  static __device__ __forceinline__ Stencil<double2> w(const BatchSys& S) { return S.w64; }
};
template <> struct BVec<float> {
  static __device__ __forceinline__ float2* slot(const BatchSys& S, int k, int64_t len) {
    return k == 0 ? S.slot32 : S.ring32 + (k - 1) * len;
  }
  static __device__ __forceinline__ float2* u(const BatchSys& S) { return S.u32; }
  static __device__ __forceinline__ float2* s(const BatchSys& S) { return S.s32v; }
  static __device__ __forceinline__ float2* pk(const BatchSys& S) { return S.pk32; }
  static __device__ __forceinline__ Stencil<float2> w(const BatchSys& S) { return S.w32; }
};
template <class R> __device__ __forceinline__ Csr<cplx<R>> mat1(const BatchSys& S);
template <> __device__ __forceinline__ Csr<double2> mat1<double>(const BatchSys& S) { return S.m64; }
template <> __device__ __forceinline__ Csr<float2> mat1<float>(const BatchSys& S) { return S.m32; }
template <class R> __device__ __forceinline__ Csr<cplx<R>> mat2(const BatchSys& S);
template <> __device__ __forceinline__ Csr<double2> mat2<double>(const BatchSys& S) { return S.mh64; }
template <> __device__ __forceinline__ Csr<float2> mat2<float>(const BatchSys& S) { return S.mh32; }


// Slot of the residual ring: step l of a system's phase reads slot l % ring, writes the next.
template <class R, int RR>
__device__ __forceinline__ cplx<R>* bslot(const BatchSys& S, int l) {
  return BVec<R>::slot(S, l % S.ring, S.n * RR);
}

// Where (row i, rhs q) lies in a system's vectors.
template <int RR> __device__ __forceinline__ int64_t bidx(const BatchSys& S, int64_t i, int q) {
  return S.links ? int64_t(q) * S.n + (i % 3) * (S.n / 3) + i / 3 : i * RR + q;
}

// Row i of a CSR times the RHS-interleaved vector x (RR right-hand sides), L lanes per
// row; sums returned in every lane of the row group.
template <class R, int L, int RR>
__device__ __forceinline__ void row_dot_rhs(const Csr<cplx<R>>& m, const cplx<R>* __restrict__ x,
                                            int64_t row, int lane, cplx<R> (&acc)[RR]) {
#pragma unroll
  for (int q = 0; q < RR; ++q) acc[q] = czero<R>();
  const int32_t beg = m.rowptr[row], end = m.rowptr[row + 1];
  for (int32_t base = beg; base < end; base += 4 * L) {
    int32_t c[4];
    cplx<R> v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int32_t j = base + lane + u * L;
      const bool ok = j < end;
      c[u] = ok ? m.col[j] : 0;
      v[u] = ok ? m.val[j] : czero<R>();
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
#pragma unroll
      for (int q = 0; q < RR; ++q) cfma<R>(acc[q], v[u], x[int64_t(c[u]) * RR + q]);
    }
  }
#pragma unroll
  for (int q = 0; q < RR; ++q) acc[q] = group_sum_c<L, R>(acc[q]);
}

template <class R> __device__ __forceinline__ Sell<cplx<R>> sell1(const BatchSys& S);
template <> __device__ __forceinline__ Sell<double2> sell1<double>(const BatchSys& S) { return S.s64; }
template <> __device__ __forceinline__ Sell<float2> sell1<float>(const BatchSys& S) { return S.s32; }
template <class R> __device__ __forceinline__ Sell<cplx<R>> sell2(const BatchSys& S);
template <> __device__ __forceinline__ Sell<double2> sell2<double>(const BatchSys& S) { return S.sh64; }
template <> __device__ __forceinline__ Sell<float2> sell2<float>(const BatchSys& S) { return S.sh32; }

// Pairs per round trip of the RR-rhs product (the 64 systems as stored matrices, mixed and
// FP64: one 145 and 179 ms, two 140 and 174, four 148 and 192).
template <int RR> constexpr int kp_rhs() { return RR >= 4 ? 2 : 4; }

// Workgroup partials of a chunk (K values): store, take the system's ticket; true in the
// last chunk of the system, which then holds the totals in tot[].
template <int K>
__device__ __forceinline__ bool chunk_reduce(double (&v)[K], const BatchSys& S, int cidx, int ticket,
                                             double* tot) {
  block_sum_k<kBlock, K>(v);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < K; ++q) store_agent(&S.partial[cidx * K + q], v[q]);
  }
  if (!arrive_last(S.tickets + ticket * kTicketSite, unsigned(S.nchunks), unsigned(cidx))) return false;
  // thread -> (value q, sub-lane): all loads of a value in flight together
  constexpr int LN = kBlock / K;
  const int q = threadIdx.x / LN, s = threadIdx.x % LN;
  double acc = 0.0;
  for (int c = s; c < S.nchunks; c += LN) acc += load_agent(&S.partial[c * K + q]);
  acc = group_sum<LN>(acc);
  if (s == 0) tot[q] = acc;
  __syncthreads();
  return true;
}

// The iteration kernels' partial sums, one set per wave and chunk, added by the system's
// workgroup of the next kernel: no wave waits for another.  On links a wave has one
// right-hand side's (wave % RR), else all of them; either way entry % RR is its q.  set: 0 for
// d_n and g_{n+1}, 1 for c_{n+1}.
__device__ __forceinline__ double* partial_set(const BatchSys& S, int set) {
  return S.partial + int64_t(set) * S.nchunks * (kBatchPartial / 2);
}
template <int RR>
__device__ __forceinline__ void wave_partial(const BatchSys& S, const int4& ch, int set, double (&v)[RR]) {
  const int wv = threadIdx.x / kWave;
  double* __restrict__ to = partial_set(S, set);
  if (S.links) {
    const double t = group_sum<kWave>(v[0]);
    if (threadIdx.x % kWave == 0) to[ch.w * (kBlock / kWave) + wv] = t;
    return;
  }
#pragma unroll
  for (int q = 0; q < RR; ++q) v[q] = group_sum<kWave>(v[q]);
  if (threadIdx.x % kWave == 0) {
#pragma unroll
    for (int q = 0; q < RR; ++q) to[(ch.w * (kBlock / kWave) + wv) * RR + q] = v[q];
  }
}

// The totals of the first SETS sets per rhs, in every thread's view of tot[set][] (kBatchMaxRhs).
template <int RR, int SETS>
__device__ __forceinline__ void system_totals(const BatchSys& S, double (*tot)[kBatchMaxRhs]) {
  constexpr int U = 16;  // in flight together: all of a system of 4096 partials (with 4, and the
                         // state read after the sums, the 64 systems took 86.8 for 85.0 ms)
  const int np = S.nchunks * (kBlock / kWave) * (S.links ? 1 : RR);
  double v[SETS];
#pragma unroll
  for (int t = 0; t < SETS; ++t) v[t] = 0.0;
  for (int i = threadIdx.x; i < np; i += U * kBlock) {
    double a[SETS][U];
#pragma unroll
    for (int t = 0; t < SETS; ++t) {
#pragma unroll
      for (int u = 0; u < U; ++u) a[t][u] = i + u * kBlock < np ? partial_set(S, t)[i + u * kBlock] : 0.0;
    }
#pragma unroll
    for (int t = 0; t < SETS; ++t) {
#pragma unroll
      for (int u = 0; u < U; ++u) v[t] += a[t][u];
    }
  }
  __shared__ double part[SETS][kBlock / kWave][kBatchMaxRhs];
#pragma unroll
  for (int t = 0; t < SETS; ++t) {
    // lanes of one rhs: those equal mod RR
#pragma unroll
    for (int o = kWave / 2; o >= RR; o /= 2) v[t] += __shfl_xor(v[t], o, kWave);
    if (int(threadIdx.x % kWave) < RR) part[t][threadIdx.x / kWave][threadIdx.x % kWave] = v[t];
  }
  __syncthreads();
  if (threadIdx.x < SETS * kBatchMaxRhs) {
    const int t = threadIdx.x / kBatchMaxRhs, q = threadIdx.x % kBatchMaxRhs;
    double s = 0.0;
    if (q < RR)
      for (int w = 0; w < kBlock / kWave; ++w) s += part[t][w][q];
    tot[t][q] = s;
  }
  __syncthreads();
}

// One wave's share of a links' chunk: 64 sites (from `site`) of right-hand side q.  out = (m +
// sign D) v there, v and out colour by colour.
struct SiteTask {
  int q;
  uint32_t site;   // this lane's, or the last one of the system where it has none
  bool live;
};
template <int RR> __device__ __forceinline__ SiteTask site_task(const int4& ch) {
  SiteTask t;
  const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kWave));
  t.q = wv % RR;
  const uint32_t s0 = uint32_t(ch.y) / 3u, s1 = uint32_t(ch.z) / 3u;
  const uint32_t s = s0 + uint32_t(wv / RR) * uint32_t(kWave) + threadIdx.x % kWave;
  t.live = s < s1;
  t.site = t.live ? s : s1 - 1;
  return t;
}
template <class R>
__device__ __forceinline__ void site_product(const BatchSys& S, const cplx<R>* __restrict__ v,
                                             const SiteTask& t, int sign, cplx<R> (&own)[3],
                                             cplx<R> (&out)[3]) {
  const Stencil<cplx<R>> w = BVec<R>::w(S);
  const cplx<R>* __restrict__ vq = v + int64_t(t.q) * S.n;
  const int64_t vol = w.vol;
#pragma unroll
  for (int c = 0; c < 3; ++c) own[c] = vq[c * vol + t.site];
  auto at = [&](uint32_t s, int c) { return vq[c * vol + s]; };
  if ((std::is_same<R, float>::value ? S.links32 : S.links) == 2)
    stencil_site<R, 2>(w, t.site, own, sign, at, out);
  else
    stencil_site<R, 3>(w, t.site, own, sign, at, out);
}

// ---- BK1: u = M r (A r for A given) for every rhs and d's share: |u|^2 or Re r^H u (with the
// direction of p instead, and sigma0 |p|^2 besides) ------------------------------------------
template <class R, int L, int RR>
__device__ __forceinline__ void bk1_chunk(const BatchSys& S, const BatchState* st, const int4& ch) {
  const bool dir = load_const(&st->dir) != 0;
  const cplx<R>* __restrict__ r = dir ? BVec<R>::s(S) : bslot<R, RR>(S, load_const(&st->slot));
  const double sd = dir ? load_const(&st->sigma0) : 0.0;
  cplx<R>* __restrict__ u = BVec<R>::u(S);
  const bool mhm = S.kind == MSC_A_MHM;
  double acc[RR];
#pragma unroll
  for (int q = 0; q < RR; ++q) acc[q] = 0.0;
  auto epilogue = [&](int64_t row, const cplx<R> (&v)[RR], const cplx<R> (&rr)[RR]) {
#pragma unroll
    for (int q = 0; q < RR; ++q) {
      u[row * RR + q] = v[q];
      acc[q] += mhm ? norm2d<R>(v[q])
                    : double(rr[q].x) * double(v[q].x) + double(rr[q].y) * double(v[q].y);
      acc[q] = fma(sd, norm2d<R>(rr[q]), acc[q]);
    }
  };
  if (S.links) {
    const SiteTask t = site_task<RR>(ch);
    cplx<R> own[3], v[3];
    site_product<R>(S, r, t, 1, own, v);
    double sum = 0.0;
    if (t.live) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        u[int64_t(t.q) * S.n + c * S.w64.vol + t.site] = v[c];
        sum += norm2d<R>(v[c]);
      }
      if (dir) {  // read again: the registers are full
#pragma unroll
        for (int c = 0; c < 3; ++c)
          sum = fma(sd, norm2d<R>(r[int64_t(t.q) * S.n + c * S.w64.vol + t.site]), sum);
      }
    }
    acc[0] = sum;
  } else if (S.sell) {
    // one row per lane: the chunk's four slices, one per wave
    const Sell<cplx<R>> ms = sell1<R>(S);
    const int lane = threadIdx.x % kSlice;
    const int64_t sl = ch.y / kSlice + __builtin_amdgcn_readfirstlane(int(threadIdx.x / kSlice));
    if (sl * kSlice < ch.z) {
      const int64_t row = sl * kSlice + lane;
      const int64_t rr = row < ch.z ? row : ch.z - 1;
      cplx<R> pr[RR], v[RR];
      load_rhs<R, RR>(r, rr, pr);
      const cplx<R> d = ms.diag[rr];
      sell_row_rhs<R, RR, kp_rhs<RR>()>(ms, r, sl, lane, v);
#pragma unroll
      for (int q = 0; q < RR; ++q) cfma<R>(v[q], d, pr[q]);
      if (row < ch.z) epilogue(row, v, pr);
    }
  } else {
    constexpr int GPB = kBlock / L;
    const int lane = threadIdx.x % L, grp = threadIdx.x / L;
    const Csr<cplx<R>> m = mat1<R>(S);
    for (int64_t row = ch.y + grp; row < ch.z; row += GPB) {
      cplx<R> v[RR];
      row_dot_rhs<R, L, RR>(m, r, row, lane, v);
      if (lane == 0) {
        cplx<R> pr[RR];
#pragma unroll
        for (int q = 0; q < RR; ++q) pr[q] = r[row * RR + q];
        epilogue(row, v, pr);
      }
    }
  }
  wave_partial<RR>(S, ch, 0, acc);
}

// The scalars of the step, one workgroup per system.
template <int RR>
__device__ __forceinline__ void bs1_system(const BatchSys& S, BatchState* st,
                                           double (*tot)[kBatchMaxRhs]) {
  // lane = q * 16 + k: the scalars of step n of rhs q, and shift k's, composed with
  // the pending steps; every lane reads the state before any lane writes it, and
  // before the sums, whose round trip it shares
  const int lk = threadIdx.x;
  const int q = lk / kBatchMaxShifts, k = lk % kBatchMaxShifts, ns = st->ns;
  const bool live = lk < kQK && q < st->nrhs && !st->halt[q];
  const int n = live ? st->iter[q] : 0, ru = live ? st->ru[q] : 0, m = live ? st->m[q] : 0;
  const double g = live ? st->R[q] : 1.0, g1 = live ? st->g1[q] : 1.0, a1 = live ? st->a1[q] : 1.0;
  const double P1 = live ? st->P1[q] : 1.0, rg = live ? st->ru_g[q] : 0.0, rc = live ? st->c[q] : 0.0;
  const int dir = st->dir;
  const double limit = st->phase32 ? kDevLimit32 : kDevLimit64, dev = live ? st->dev[q] : 0.0;
  const bool act = live && k < ns && (k == 0 || st->active[lk]);
  const double z = live && k ? st->zeta[lk] : 1.0, zp = live && k ? st->zeta_prev[lk] : 1.0;
  const double sigma0 = st->sigma0, sk = live ? st->s[k] : 0.0;
  const int slot = st->slot;
  const bool had = m > 0 && st->took[lk];
  double cx[kMaxSteps + 1], cp[kMaxSteps + 1];
#pragma unroll
  for (int i = 0; i <= kMaxSteps; ++i) {
    cx[i] = m > 0 && i <= m ? st->cx[i][lk] : 0.0;
    cp[i] = m > 0 && i <= m ? st->cp[i][lk] : 0.0;
  }
  if (m == 0) cp[0] = 1.0;
  system_totals<RR, 1>(S, tot);
  if (lk >= kQK) return;
  const double d = dir ? tot[0][q] : tot[0][q] + sigma0 * g;
  const double b = n == 0 ? 0.0 : (ru ? rg : g) / g1;
  const double P = n == 0 || dir ? d : d + b * (2.0 * rc + b * P1);
  const double off = n == 0 || dir || ru ? 0.0 : fabs(P - (d - b * g / a1));
  const bool ok = P > 0.0 && isfinite(P);
  // a right-hand side that needs its direction: none of the system steps until BF has
  // handed them out
  if (__ballot(live && !dir && n > 0 && (!ok || !(off <= limit * P)))) {
    if (k == 0 && q < kBatchMaxRhs) st->step[q] = 0;
    if (lk == 0) st->wait |= 2;
    return;
  }
  const double a = g / P;
  if (k == 0 && q < kBatchMaxRhs) st->step[q] = live && ok ? 1 : 0;
  if (live && !ok && k == 0) {
    st->status[q] = 1;
    st->halt[q] = 1;
  }
  if (!live || !ok) return;
  bool took = had;
  if (act) {
    const double zn = k == 0   ? 1.0
                      : n == 0 ? z / (1.0 + sk * a)
                               : z * zp * a1 / (a * b * (zp - z) + zp * a1 * (1.0 + sk * a));
    const double ratio = z / zp, aj = a * zn / z, bj = b * ratio * ratio;
#pragma unroll
    for (int i = 0; i <= kMaxSteps; ++i) {
      if (i <= m) cp[i] *= bj;
      if (i == m + 1) cp[i] = z;
      if (i <= m + 1) cx[i] = fma(aj, cp[i], cx[i]);
    }
    st->zeta_prev[lk] = z;
    st->zeta[lk] = zn;
    took = true;
  }
  st->took[lk] = took ? 1 : 0;
#pragma unroll
  for (int i = 0; i <= kMaxSteps; ++i) {
    st->cx[i][lk] = cx[i];
    st->cp[i][lk] = cp[i];
  }
  if (k == 0) {
    st->a[q] = st->a1[q] = a;
    st->b[q] = b;
    st->P1[q] = P;
    st->g1[q] = g;
    st->m[q] = m + 1;
    st->last[q] = slot;  // the newest of the composed steps
    st->ru[q] = 0;
    if (off > dev * P) st->dev[q] = off / P;
  }
}

// ---- BK2: s <- w + s0 r + b s, r' = r - a s, R' = |r'|^2; freezing, halting, switching -----
template <class R, int L, int RR>
__device__ __forceinline__ void bk2_chunk(const BatchSys& S, const BatchState* st, const int4& ch) {
  const int slot = load_const(&st->slot);
  const cplx<R>* __restrict__ u = BVec<R>::u(S);
  const cplx<R>* __restrict__ r = bslot<R, RR>(S, slot);
  cplx<R>* __restrict__ rn = bslot<R, RR>(S, slot + 1);
  cplx<R>* __restrict__ sv = BVec<R>::s(S);
  const double s0 = load_const(&st->sigma0);
  const bool mhm = S.kind == MSC_A_MHM, dir = load_const(&st->dir) != 0;
  const double cr = dir ? 0.0 : s0;  // s = w + cr r + cs s_old, s_old being p with the direction
  double2* __restrict__ x0 = S.x + int64_t(load_const(&st->orig[0])) * S.n;
  const int64_t xq = int64_t(load_const(&st->ns)) * S.n;
  double acc[RR], ac[RR];
#pragma unroll
  for (int q = 0; q < RR; ++q) acc[q] = ac[q] = 0.0;
  // one element's step (row i of right-hand side q in the caller's order); `stream` where a wave's s is one run (else its lines, shared by the
  // right-hand sides of a row, would leave the caches between them)
  auto element = [&](int64_t idx, int64_t i, int q, const cplx<R>& w, double a, double cs, auto stream,
                     double& g, double& c) {
    const double2 wd = to_d(w), rd = to_d(r[idx]), sd = to_d(stream ? ld_stream(&sv[idx]) : sv[idx]);
    const double2 t{fma(cs, sd.x, fma(cr, rd.x, wd.x)), fma(cs, sd.y, fma(cr, rd.y, wd.y))};
    const cplx<R> nr = from_d<R>(double2{fma(-a, t.x, rd.x), fma(-a, t.y, rd.y)}), ts = from_d<R>(t);
    if (dir) {
      double2* x = x0 + (q * xq + i);
      *x = double2{fma(a, sd.x, x->x), fma(a, sd.y, x->y)};
    } else if (stream) {
      st_stream(&sv[idx], ts);
    } else {
      sv[idx] = ts;
    }
    rn[idx] = nr;
    g += norm2d<R>(nr);
    c = fma(double(nr.x), double(ts.x), fma(double(nr.y), double(ts.y), c));
  };
  if (S.links) {
    const SiteTask t = site_task<RR>(ch);
    if (t.q < load_const(&st->nrhs) && load_const(&st->step[t.q])) {
      cplx<R> own[3], w[3];
      site_product<R>(S, u, t, -1, own, w);
      const double a = load_const(&st->a[t.q]), cs = dir ? s0 : load_const(&st->b[t.q]);
      if (t.live) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
          element(int64_t(t.q) * S.n + c * S.w64.vol + t.site, 3 * int64_t(t.site) + c, t.q, w[c], a,
                  cs, std::true_type{}, acc[0], ac[0]);
      }
    }
  } else {
    double a[RR], b[RR];
    bool go[RR];
#pragma unroll
    for (int q = 0; q < RR; ++q) {
      go[q] = q < load_const(&st->nrhs) && load_const(&st->step[q]);
      a[q] = go[q] ? load_const(&st->a[q]) : 0.0;
      b[q] = dir ? s0 : go[q] ? load_const(&st->b[q]) : 0.0;
    }
    auto epilogue = [&](int64_t row, const cplx<R> (&w)[RR]) {
#pragma unroll
      for (int q = 0; q < RR; ++q)
        if (go[q])
          element(row * RR + q, row, q, w[q], a[q], b[q], std::false_type{}, acc[q], ac[q]);
    };
    if (S.sell && mhm) {
      // one row per lane: the chunk's four slices, one per wave
      const Sell<cplx<R>> ms = sell2<R>(S);
      const int lane = threadIdx.x % kSlice;
      const int64_t sl = ch.y / kSlice + __builtin_amdgcn_readfirstlane(int(threadIdx.x / kSlice));
      if (sl * kSlice < ch.z) {
        const int64_t row = sl * kSlice + lane;
        const int64_t rr = row < ch.z ? row : ch.z - 1;
        cplx<R> tr[RR], w[RR];
        load_rhs<R, RR>(u, rr, tr);
        const cplx<R> d = ms.diag[rr];
        sell_row_rhs<R, RR, kp_rhs<RR>()>(ms, u, sl, lane, w);
#pragma unroll
        for (int q = 0; q < RR; ++q) cfma<R>(w[q], d, tr[q]);
        if (row < ch.z) epilogue(row, w);
      }
    } else if (mhm) {
      constexpr int GPB = kBlock / L;
      const int lane = threadIdx.x % L, grp = threadIdx.x / L;
      for (int64_t row = ch.y + grp; row < ch.z; row += GPB) {
        cplx<R> w[RR];
        row_dot_rhs<R, L, RR>(mat2<R>(S), u, row, lane, w);
        if (lane == 0) epilogue(row, w);
      }
    } else {  // A given: u is A r already
      const int q = threadIdx.x % RR;  // kBlock is a multiple of RR: this thread's rhs
      double sum = 0.0, sc = 0.0, aq = 0.0, bq = 0.0;
      bool gq = false;
#pragma unroll
      for (int k = 0; k < RR; ++k) {
        if (k == q) {
          aq = a[k];
          bq = b[k];
          gq = go[k];
        }
      }
      const int64_t end = int64_t(ch.z) * RR;
      if (gq)
        for (int64_t e = int64_t(ch.y) * RR + threadIdx.x; e < end; e += kBlock)
          element(e, e / RR, q, u[e], aq, bq, std::true_type{}, sum, sc);
#pragma unroll
      for (int k = 0; k < RR; ++k) {
        acc[k] = k == q ? sum : 0.0;
        ac[k] = k == q ? sc : 0.0;
      }
    }
  }
  wave_partial<RR>(S, ch, 0, acc);
  wave_partial<RR>(S, ch, 1, ac);
}

// ---- BP: p <- r + b p of a system with directions, before BK1 --------------------------------
template <class R, int RR>
__device__ __forceinline__ void bp_chunk(const BatchSys& S, const BatchState* st, const int4& ch) {
  const cplx<R>* __restrict__ r = bslot<R, RR>(S, st->slot);
  cplx<R>* __restrict__ p = BVec<R>::s(S);
  const int rows = ch.z - ch.y, elems = rows * st->nrhs;
  for (int e = threadIdx.x; e < elems; e += kBlock) {
    const int q = e / rows;
    if (st->halt[q]) continue;
    const double b = (st->ru[q] ? st->ru_g[q] : st->R[q]) / st->g1[q];
    const int64_t idx = bidx<RR>(S, ch.y + e % rows, q);
    const double2 rd = to_d(r[idx]), pd = to_d(p[idx]);
    p[idx] = from_d<R>(double2{fma(b, pd.x, rd.x), fma(b, pd.y, rd.y)});
  }
}

template <int RR>
__device__ __forceinline__ void bs2_system(const BatchSys& S, BatchState* st,
                                           double (*tot)[kBatchMaxRhs],
                                           int* active_systems) {
  // one wave: lane = q * 16 + k; every lane reads the state before any lane
  // writes it, and system-wide decisions travel by ballot, not through memory
  const int lk = threadIdx.x;
  const int q = lk / kBatchMaxShifts, k = lk % kBatchMaxShifts;
  const bool live = lk < kWave && q < st->nrhs && st->step[q] && !st->halt[q];
  const int it = live ? st->iter[q] + 1 : 0;
  const double eps2 = live ? st->eps2[q] : 0.0, sw2 = live ? st->sw_eps2[q] : 0.0;
  const int phase32 = st->phase32, max_iter = st->max_iter;
  const bool act = live && k >= 1 && k < st->ns && st->active[lk];
  const double z = act ? st->zeta[lk] : 0.0;
  const int dir = st->dir;
  const double dev = fmax(fmax(st->dev[0], st->dev[1]), fmax(st->dev[2], st->dev[3]));
  system_totals<RR, 2>(S, tot);
  if (lk >= kWave) return;
  const double Rn = live ? tot[0][q] : 0.0;
  if (act && z * z * Rn <= eps2) {
    st->active[lk] = 0;
    st->freeze_iter[lk] = it;
  }
  bool halted_after = true, below = true;
  if (k == 0 && live) {
    st->R[q] = Rn;
    st->c[q] = tot[1][q];
    st->iter[q] = it;
    if (!isfinite(Rn)) {
      st->status[q] = 1;
      st->halt[q] = 1;
    } else if (Rn <= eps2 || it >= max_iter) {
      st->halt[q] = 1;
    } else {
      halted_after = false;
      below = Rn <= sw2;
    }
  }
  // the iterations of the right-hand sides that stepped: the same number
  int most = it;
  most = max(most, __shfl_xor(most, 16, kWave));
  most = max(most, __shfl_xor(most, 32, kWave));
  const bool all_halted = __ballot(!halted_after) == 0;
  const bool all_below = __ballot(!halted_after && !below) == 0;
  if (lk == 0) {
    st->slot += 1;
    if (all_halted) {
      st->done = 1;
      atomicSub(&active_systems[phase32], 1);
      if (dir) atomicSub(&active_systems[2], 1);
    } else if (!phase32 && all_below) {
      st->wait = !dir && dev > kDevSwitch ? 3 : 1;
      st->iters_fp64 = most;
    }
  }
}

// ---- BF: the composed steps of every shift; the switch to complex64 ----------------------
// Bound by the bytes: 8 steps folded, FP64 10 * 64 + 8 * 16 per row and rhs, 940 us at 5.9 M
// of them = 4.8 TB/s (four steps folded and p read and written besides: 198 us each step).
// x_k += cx[0] p_k + sum_{i<m} cx[i+1] r_i, p_k likewise with cp (k = 0, the driving system,
// too); before a system's first BF its x_k and p_k are zero and are not read.  One row per
// thread, p_k in the caller's row order, [k][q][row].  W != R: r, s and p_k go to complex64.
struct BFlush {
  double cx[kMaxSteps + 1][kQK], cp[kMaxSteps + 1][kQK];
  int took[kQK], orig[kBatchMaxShifts];
  int m[kBatchMaxRhs], last[kBatchMaxRhs];
  int nrhs, ns, fresh, slot;
  int dir, take;  // with directions (BK2 keeps x_0 and p_0); they are handed out here
};

template <class R, class W, int RR>
__device__ __forceinline__ void bf_chunk(const BatchSys& S, BatchState* st, const int4& ch, BFlush& f, int* active) {
  const int tid = threadIdx.x;
  __syncthreads();  // the previous chunk of this workgroup is done with f
  if (tid < kQK) {
#pragma unroll
    for (int i = 0; i <= kMaxSteps; ++i) {
      f.cx[i][tid] = st->cx[i][tid];
      f.cp[i][tid] = st->cp[i][tid];
    }
    f.took[tid] = st->took[tid];
  }
  if (tid < kBatchMaxShifts) f.orig[tid] = st->orig[tid];
  if (tid < kBatchMaxRhs) {
    f.m[tid] = st->m[tid];
    f.last[tid] = st->last[tid];
  }
  if (tid == 0) {
    f.nrhs = st->nrhs;
    f.ns = st->ns;
    f.fresh = st->fresh;
    f.slot = st->slot;
    f.dir = st->dir;
    f.take = st->wait & 2;
  }
  __syncthreads();
  constexpr bool same = std::is_same<R, W>::value;
  const int64_t n = S.n;
  const int ns = f.ns, fresh = f.fresh, kf = f.dir ? 1 : 0;
  cplx<R>* __restrict__ pk = BVec<R>::pk(S);
  cplx<W>* __restrict__ pw = BVec<W>::pk(S);
  // one (row, rhs) per thread: fewer vectors of the others between two of its loads
  const int rows = ch.z - ch.y, elems = rows * f.nrhs;
  for (int e = tid; e < elems; e += kBlock) {
    const int q = e / rows;
    const int64_t i = ch.y + e % rows;
    const int64_t idx = bidx<RR>(S, i, q);
    if (!same) {
      bslot<W, RR>(S, 0)[idx] = from_d<W>(to_d(bslot<R, RR>(S, f.slot)[idx]));
      BVec<W>::s(S)[idx] = from_d<W>(to_d(BVec<R>::s(S)[idx]));
    }
    const int m = f.m[q];
    if (same && m == 0 && !fresh && !f.take) continue;
    double2 rv[kMaxSteps];
#pragma unroll
    for (int k = 0; k < kMaxSteps; ++k)
      rv[k] = k < m ? to_d(bslot<R, RR>(S, f.last[q] - m + 1 + k)[idx]) : double2{0.0, 0.0};
    constexpr int G = 2;  // shifts whose loads are issued together
    for (int k0 = 0; k0 < ns; k0 += G) {
      double2 pj[G], xv[G];
      bool ux[G], ld[G];
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const int k = k0 + u;
        ux[u] = k >= kf && k < ns && ((m > 0 && f.took[q * kBatchMaxShifts + k]) || fresh);
        ld[u] = k >= kf && k < ns && (ux[u] || !same || (f.take && k == 0));
        pj[u] = xv[u] = double2{0.0, 0.0};
        if (ld[u] && !fresh) pj[u] = to_d(ld_stream(&pk[(int64_t(k) * RR + q) * n + i]));
        if (ux[u] && !fresh) xv[u] = ld_stream(&S.x[(int64_t(q) * ns + f.orig[k]) * n + i]);
      }
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const int k = k0 + u;
        if (!ld[u]) continue;
        double2 np = pj[u];
        if (ux[u]) {
          const int lk = q * kBatchMaxShifts + k;
          const bool some = m > 0 && f.took[lk];
          double2 xs = xv[u];
          np = double2{0.0, 0.0};
          if (some) {
            xs.x = fma(f.cx[0][lk], pj[u].x, xs.x);
            xs.y = fma(f.cx[0][lk], pj[u].y, xs.y);
            np = double2{f.cp[0][lk] * pj[u].x, f.cp[0][lk] * pj[u].y};
#pragma unroll
            for (int j = 0; j < kMaxSteps; ++j) {
              if (j < m) {
                xs.x = fma(f.cx[j + 1][lk], rv[j].x, xs.x);
                xs.y = fma(f.cx[j + 1][lk], rv[j].y, xs.y);
                np.x = fma(f.cp[j + 1][lk], rv[j].x, np.x);
                np.y = fma(f.cp[j + 1][lk], rv[j].y, np.y);
              }
            }
          }
          st_stream(&S.x[(int64_t(q) * ns + f.orig[k]) * n + i], xs);
        }
        st_stream(&pw[(int64_t(k) * RR + q) * n + i], from_d<W>(np));
        if (f.take && k == 0) BVec<W>::s(S)[idx] = from_d<W>(np);
      }
    }
  }
  if (!arrive_last(S.tickets + 2 * kTicketSite, unsigned(S.nchunks), unsigned(ch.w))) return;
  // every chunk has read the state: nothing is pending any more
  if (tid < kBatchMaxRhs) {
    const int ph = sizeof(R) == 4 ? 1 : 0, m = f.m[tid];
    int upd = 0;
    for (int k = kf; k < ns; ++k)
      upd += (m > 0 && f.took[tid * kBatchMaxShifts + k]) || fresh ? 1 : 0;
    if (tid < f.nrhs) {
      st->n_upd[tid][ph] += upd;
      st->n_kept[tid][ph] += m;
    }
    st->m[tid] = 0;
  }
  if (tid == 0) {
    st->fresh = 0;
    st->wait = 0;
    if (f.take) {
      st->dir = 1;
      if (!st->done) atomicAdd(&active[2], 1);
    }
    if (!same) {
      st->phase32 = 1;
      st->slot = 0;
      if (!st->done) {
        atomicSub(&active[0], 1);
        atomicAdd(&active[1], 1);
      }
    }
  }
}

// ---- init: r = b_q, s = 0, |b_q|^2 ---------------------------------------------------------
template <int RR>
__device__ __forceinline__ void binit_chunk(const BatchSys& S, BatchState* st, const int4& ch) {
  const int64_t n = S.n;
  double acc[kBatchMaxRhs] = {0.0, 0.0, 0.0, 0.0};
  double2* __restrict__ r = bslot<double, RR>(S, 0);
  for (int64_t i = ch.y + threadIdx.x; i < ch.z; i += kBlock) {
#pragma unroll
    for (int q = 0; q < RR; ++q) {
      const int64_t idx = bidx<RR>(S, i, q);
      const double2 bv = q < st->nrhs ? S.b[int64_t(q) * n + i] : double2{0.0, 0.0};
      r[idx] = bv;
      S.s64v[idx] = double2{0.0, 0.0};
      acc[q] += fma(bv.x, bv.x, bv.y * bv.y);
    }
  }
  __shared__ double tot[kBatchMaxRhs];
  if (!chunk_reduce(acc, S, ch.w, 2, tot)) return;
  if (threadIdx.x < st->nrhs) {
    const int q = threadIdx.x;
    const double B2 = tot[q];
    st->bnorm2[q] = B2;
    st->R[q] = B2;
    st->eps2[q] *= B2;
    st->sw_eps2[q] *= B2;
    if (!(B2 > 0.0) || !isfinite(B2)) {
      st->halt[q] = 1;
      if (!isfinite(B2)) st->status[q] = 1;
    }
  }
}

// ---- FP64 products with several vectors (reliable update, verification) ------------------
// out(row, v, value) in the lane that owns the row, of vectors in + v step (row order), v <
// nv <= NV: M in, or M^H in where `second` (A = M^H M's other half; A in for A given).
template <int L, int NV, class OUT>
__device__ __forceinline__ void product64(const BatchSys& S, const int4& ch, bool second, int nv,
                                          const double2* __restrict__ in, int64_t step, OUT out) {
  const bool mh = second && S.kind == MSC_A_MHM;
  if (S.links) {
    // a wave per 64 sites and vector
    const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kWave));
    const uint32_t s0 = uint32_t(ch.y) / 3u, s1 = uint32_t(ch.z) / 3u;
    const int blocks = int((s1 - s0 + kWave - 1) / kWave);
    for (int task = wv; task < blocks * nv; task += kBlock / kWave) {
      const int v = task % nv;
      const uint32_t s = s0 + uint32_t(task / nv) * uint32_t(kWave) + threadIdx.x % kWave;
      const bool live = s < s1;
      const uint32_t ss = live ? s : s1 - 1;
      const double2* __restrict__ x = in + v * step;
      double2 own[3], o[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) own[c] = x[3 * int64_t(ss) + c];
      auto at = [&](uint32_t t, int c) { return x[3 * int64_t(t) + c]; };
      stencil_site<double, 3>(S.v64, ss, own, mh ? -1 : 1, at, o);
      if (live) {
#pragma unroll
        for (int c = 0; c < 3; ++c) out(3 * int64_t(s) + c, v, o[c]);
      }
    }
    return;
  }
  if (S.sell) {
    // a row per lane, KV vectors at a time
    constexpr int KV = NV < 4 ? NV : 4;
    const Sell<double2> ms = mh ? S.sh64 : S.s64;
    const int lane = threadIdx.x % kSlice;
    const int64_t sl = ch.y / kSlice + __builtin_amdgcn_readfirstlane(int(threadIdx.x / kSlice));
    if (sl * kSlice >= ch.z) return;
    const int64_t row = sl * kSlice + lane;
    const bool live = row < ch.z;
    const double2 d = ms.diag[live ? row : ch.z - 1];
#pragma unroll
    for (int v0 = 0; v0 < NV; v0 += KV) {
      if (v0 >= nv) break;
      const int kc = min(KV, nv - v0);
      const double2* xs[KV];
      double2 acc[KV];
#pragma unroll
      for (int q = 0; q < KV; ++q) {
        xs[q] = in + int64_t(min(v0 + q, nv - 1)) * step;
        acc[q] = double2{0.0, 0.0};
      }
      sell_row_multi<double, KV, 1>(ms, xs, kc, sl, lane, acc);
      if (live) {
#pragma unroll
        for (int q = 0; q < KV; ++q) {
          if (q < kc) {
            cfma<double>(acc[q], d, xs[q][row]);
            out(row, v0 + q, acc[q]);
          }
        }
      }
    }
    return;
  }
  constexpr int GPB = kBlock / L;
  const int lane = threadIdx.x % L, grp = threadIdx.x / L;
  const Csr<double2> m = mh ? S.mh64 : S.m64;
  for (int64_t row = ch.y + grp; row < ch.z; row += GPB) {
    double2 acc[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = double2{0.0, 0.0};
    const int32_t end = m.rowptr[row + 1];
    for (int32_t j = m.rowptr[row] + lane; j < end; j += L) {
      const int32_t c = m.col[j];
      const double2 a = m.val[j];
#pragma unroll
      for (int v = 0; v < NV; ++v)
        if (v < nv) cfma<double>(acc[v], a, in[v * step + c]);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      acc[v] = group_sum_c<L, double>(acc[v]);
      if (lane == 0 && v < nv) out(row, v, acc[v]);
    }
  }
}

// ---- reliable update of a system in its complex64 phase: r_q = b_q - (A + s0) x_q0 -------
template <int L, int RR>
__device__ __forceinline__ void bru1_chunk(const BatchSys& S, const BatchState* st, const int4& ch) {
  // u = M x_q0 (FP64), vector q at ru64 + q n
  const int64_t n = S.n;
  const double2* __restrict__ x0 = S.x + int64_t(st->orig[0]) * n;
  const int64_t step = int64_t(st->ns) * n;
  product64<L, RR>(S, ch, false, st->nrhs, x0, step,
                   [&](int64_t i, int v, const double2& o) { S.ru64[v * n + i] = o; });
}

template <int L, int RR>
__device__ __forceinline__ void bru2_chunk(const BatchSys& S, BatchState* st, const int4& ch) {
  const int64_t n = S.n;
  const bool mhm = S.kind == MSC_A_MHM;
  const double s0 = st->sigma0;
  const double2* __restrict__ x0 = S.x + int64_t(st->orig[0]) * n;
  const int64_t step = int64_t(st->ns) * n;
  const double2* __restrict__ in = mhm ? S.ru64 : x0;
  const int64_t istep = mhm ? n : step;
  float2* __restrict__ r = bslot<float, RR>(S, st->slot);
  double acc[2 * kBatchMaxRhs];  // |r_q|^2, then Re r_q^H s_q
#pragma unroll
  for (int q = 0; q < 2 * kBatchMaxRhs; ++q) acc[q] = 0.0;
  product64<L, RR>(S, ch, true, st->nrhs, in, istep,
                   [&](int64_t i, int v, const double2& o) {
                     const double2 bv = S.b[v * n + i], xv = x0[v * step + i];
                     const double2 rt{bv.x - o.x - s0 * xv.x, bv.y - o.y - s0 * xv.y};
                     const int64_t idx = bidx<RR>(S, i, v);
                     const double2 sd = to_d(S.s32v[idx]);
                     r[idx] = from_d<float>(rt);
#pragma unroll
                     for (int q = 0; q < RR; ++q) {
                       if (q == v) {
                         acc[q] += fma(rt.x, rt.x, rt.y * rt.y);
                         acc[kBatchMaxRhs + q] += rt.x * sd.x + rt.y * sd.y;
                       }
                     }
                   });
  __shared__ double tot[2 * kBatchMaxRhs];
  if (!chunk_reduce<2 * kBatchMaxRhs>(acc, S, ch.w, 3, tot)) return;
  if (threadIdx.x < st->nrhs) {
    const int q = threadIdx.x;
    if (!st->halt[q]) {
      if (!st->ru[q]) st->ru_g[q] = st->R[q];
      st->ru[q] = 1;
      st->c[q] = tot[kBatchMaxRhs + q];
      st->R[q] = tot[q];
      if (!isfinite(tot[q])) {
        st->status[q] = 1;
        st->halt[q] = 1;
      } else if (tot[q] <= st->eps2[q]) {
        st->halt[q] = 1;
      }
    }
    if (q == 0) st->n_reliable += 1;
  }
}

// ---- FP64 true residuals of shifts [k0, k0 + 8) of right-hand side q, every system ----------
// (a launch for all systems in place of one each: 13 -> 3.5 ms for the 64 systems)
constexpr int kBvShifts = 8;
template <int L>
__device__ __forceinline__ void bv1_chunk(const BatchSys& S, const BatchState* st, const int4& ch, int q, int k0) {
  const int64_t n = S.n;
  const int nv = min(kBvShifts, st->ns - k0);
  const double2* __restrict__ x = S.x + (int64_t(q) * st->ns + k0) * n;
  double2* __restrict__ u = S.pk64;  // the sequence has ended: its vectors are free
  product64<L, kBvShifts>(S, ch, false, nv, x, n,
                          [&](int64_t i, int v, const double2& o) { u[v * n + i] = o; });
}

template <int L>
__device__ __forceinline__ void bv2_chunk(const BatchSys& S, const BatchState* st, const int4& ch, int q, int k0,
                          const double* sig, double* out) {
  const int64_t n = S.n;
  const int nv = min(kBvShifts, st->ns - k0);
  const double2* __restrict__ x = S.x + (int64_t(q) * st->ns + k0) * n;
  const double2* __restrict__ in = S.kind == MSC_A_MHM ? S.pk64 : x;
  const double2* __restrict__ b = S.b + int64_t(q) * n;
  double acc[kBvShifts];
#pragma unroll
  for (int v = 0; v < kBvShifts; ++v) acc[v] = 0.0;
  product64<L, kBvShifts>(S, ch, true, nv, in, n,
                          [&](int64_t i, int v, const double2& o) {
                            const double2 bv = b[i], xv = x[v * n + i];
                            const double ex = bv.x - o.x - sig[k0 + v] * xv.x;
                            const double ey = bv.y - o.y - sig[k0 + v] * xv.y;
#pragma unroll
                            for (int w = 0; w < kBvShifts; ++w)
                              if (w == v) acc[w] += fma(ex, ex, ey * ey);
                          });
  __shared__ double tot[kBvShifts];
  if (!chunk_reduce<kBvShifts>(acc, S, ch.w, 0, tot)) return;
  if (threadIdx.x < nv) out[k0 + threadIdx.x] = tot[threadIdx.x];
}

// ---- persistent drivers over the chunk list ---------------------------------------------
// Waves per SIMD that the registers are kept to: FP64 3 (at most 168), complex64 4 (128; 5,
// with 96, is no faster).
template <class R> constexpr int waves_per_simd() { return sizeof(R) == 4 ? 4 : 3; }

template <class R, int L, int RR>
__global__ __launch_bounds__(kBlock, waves_per_simd<R>()) void bk1(BatchArgs a) {
  for (int c = blockIdx.x; c < a.nchunks; c += gridDim.x) {
    const int4 ch = load_const(a.chunks + c);
    const BatchSys S = load_const(a.sys + ch.x);
    const BatchState* st = S.st;
    if (load_const(&st->phase32) != int(sizeof(R) == 4) || load_const(&st->done) ||
        load_const(&st->wait) || (load_const(&st->dir) && !(a.phases & 4)))
      continue;
    bk1_chunk<R, L, RR>(S, st, ch);
  }
}

// A system with no step in this launch: finished, waiting for the next BF, or in a phase or
// with directions that the launch leaves out.
__device__ __forceinline__ bool idle(const BatchArgs& a, const BatchState* st) {
  return st->done || st->wait || !(a.phases & (st->phase32 ? 2 : 1)) || (st->dir && !(a.phases & 4));
}

template <int RR> __global__ __launch_bounds__(kBlock) void bp(BatchArgs a) {
  for (int c = blockIdx.x; c < a.nchunks; c += gridDim.x) {
    const int4 ch = load_const(a.chunks + c);
    const BatchSys S = load_const(a.sys + ch.x);
    const BatchState* st = S.st;
    if (!st->dir || idle(a, st)) continue;
    if (st->phase32)
      bp_chunk<float, RR>(S, st, ch);
    else
      bp_chunk<double, RR>(S, st, ch);
  }
}

template <int RR> __global__ __launch_bounds__(kBlock) void bs1(BatchArgs a) {
  const BatchSys S = load_const(a.sys + blockIdx.x);
  if (idle(a, S.st)) return;
  __shared__ double tot[1][kBatchMaxRhs];
  bs1_system<RR>(S, S.st, tot);  // its barriers come after every thread has looked
}

template <class R, int L, int RR>
__global__ __launch_bounds__(kBlock, waves_per_simd<R>()) void bk2(BatchArgs a) {
  for (int c = blockIdx.x; c < a.nchunks; c += gridDim.x) {
    const int4 ch = load_const(a.chunks + c);
    const BatchSys S = load_const(a.sys + ch.x);
    const BatchState* st = S.st;
    if (load_const(&st->phase32) != int(sizeof(R) == 4) || load_const(&st->done) ||
        load_const(&st->wait) || (load_const(&st->dir) && !(a.phases & 4)))
      continue;
    bk2_chunk<R, L, RR>(S, st, ch);
  }
}

template <int RR> __global__ __launch_bounds__(kBlock) void bs2(BatchArgs a) {
  const BatchSys S = load_const(a.sys + blockIdx.x);
  if (idle(a, S.st)) return;
  __shared__ double tot[2][kBatchMaxRhs];
  bs2_system<RR>(S, S.st, tot, a.active_systems);
}

template <int RR>
__global__ __launch_bounds__(kBlock, 4) void bf(BatchArgs a) {
  __shared__ BFlush f;
  for (int c = blockIdx.x; c < a.nchunks; c += gridDim.x) {
    const int4 ch = load_const(a.chunks + c);
    const BatchSys S = load_const(a.sys + ch.x);
    BatchState* st = S.st;
    const int any = st->m[0] | st->m[1] | st->m[2] | st->m[3] | st->fresh;
    if (!any && !st->wait) continue;
    if (st->phase32)
      bf_chunk<float, float, RR>(S, st, ch, f, a.active_systems);
    else if (st->wait & 1)
      bf_chunk<double, float, RR>(S, st, ch, f, a.active_systems);
    else
      bf_chunk<double, double, RR>(S, st, ch, f, a.active_systems);
  }
}

template <int RR>
__global__ __launch_bounds__(kBlock) void binit(BatchArgs a) {
  for (int c = blockIdx.x; c < a.nchunks; c += gridDim.x) {
    const int4 ch = load_const(a.chunks + c);
    const BatchSys S = load_const(a.sys + ch.x);
    binit_chunk<RR>(S, S.st, ch);
  }
}

template <int L, int RR>
__global__ __launch_bounds__(kBlock) void bru1(BatchArgs a) {
  for (int c = blockIdx.x; c < a.nchunks; c += gridDim.x) {
    const int4 ch = load_const(a.chunks + c);
    const BatchSys S = load_const(a.sys + ch.x);
    if (S.st->done || !S.st->phase32 || S.kind != MSC_A_MHM) continue;
    bru1_chunk<L, RR>(S, S.st, ch);
  }
}

template <int L, int RR>
__global__ __launch_bounds__(kBlock) void bru2(BatchArgs a) {
  for (int c = blockIdx.x; c < a.nchunks; c += gridDim.x) {
    const int4 ch = load_const(a.chunks + c);
    const BatchSys S = load_const(a.sys + ch.x);
    if (S.st->done || !S.st->phase32) continue;
    bru2_chunk<L, RR>(S, S.st, ch);
  }
}

// sig and out: kMaxShifts per (system, rhs), in the caller's order; slot of (s, q) = first[s] + q.
template <int L>
__global__ __launch_bounds__(kBlock) void bv1(BatchArgs a, int q, int k0) {
  for (int c = blockIdx.x; c < a.nchunks; c += gridDim.x) {
    const int4 ch = load_const(a.chunks + c);
    const BatchSys S = load_const(a.sys + ch.x);
    if (q >= S.st->nrhs || k0 >= S.st->ns || S.kind != MSC_A_MHM) continue;
    bv1_chunk<L>(S, S.st, ch, q, k0);
  }
}

template <int L>
__global__ __launch_bounds__(kBlock) void bv2(BatchArgs a, int q, int k0) {
  for (int c = blockIdx.x; c < a.nchunks; c += gridDim.x) {
    const int4 ch = load_const(a.chunks + c);
    const BatchSys S = load_const(a.sys + ch.x);
    if (q >= S.st->nrhs || k0 >= S.st->ns) continue;
    bv2_chunk<L>(S, S.st, ch, q, k0, S.sig, S.res2 + int64_t(q) * kMaxShifts);
  }
}

#define MSC_BATCH_LANES(CALL)                       \
  switch (a.lanes) {                                \
    case 4: { constexpr int LL = 4; CALL; } break;  \
    case 8: { constexpr int LL = 8; CALL; } break;  \
    case 16: { constexpr int LL = 16; CALL; } break; \
    default: return hipErrorInvalidValue;           \
  }
#define MSC_BATCH_RHS(CALL)                         \
  switch (a.rr) {                                   \
    case 1: { constexpr int RP = 1; CALL; } break;  \
    case 2: { constexpr int RP = 2; CALL; } break;  \
    case 4: { constexpr int RP = 4; CALL; } break;  \
    default: return hipErrorInvalidValue;           \
  }

}  // namespace

hipError_t launch_batch_init(const BatchArgs& a, hipStream_t s) {
  MSC_BATCH_RHS((binit<RP><<<a.grid, kBlock, 0, s>>>(a)));
  return hipGetLastError();
}

hipError_t launch_batch_iteration(const BatchArgs& a, bool flush, hipStream_t s) {
  if (a.phases & 4) MSC_BATCH_RHS((bp<RP><<<a.grid, kBlock, 0, s>>>(a)));
  if (a.phases & 1) MSC_BATCH_RHS(MSC_BATCH_LANES((bk1<double, LL, RP><<<a.grid, kBlock, 0, s>>>(a))));
  if (a.phases & 2) MSC_BATCH_RHS(MSC_BATCH_LANES((bk1<float, LL, RP><<<a.grid, kBlock, 0, s>>>(a))));
  MSC_BATCH_RHS((bs1<RP><<<a.nsys, kBlock, 0, s>>>(a)));
  if (a.phases & 1) MSC_BATCH_RHS(MSC_BATCH_LANES((bk2<double, LL, RP><<<a.grid, kBlock, 0, s>>>(a))));
  if (a.phases & 2) MSC_BATCH_RHS(MSC_BATCH_LANES((bk2<float, LL, RP><<<a.grid, kBlock, 0, s>>>(a))));
  MSC_BATCH_RHS((bs2<RP><<<a.nsys, kBlock, 0, s>>>(a)));
  if (flush) MSC_BATCH_RHS((bf<RP><<<a.grid, kBlock, 0, s>>>(a)));
  return hipGetLastError();
}

hipError_t launch_batch_reliable(const BatchArgs& a, hipStream_t s) {
  MSC_BATCH_RHS(MSC_BATCH_LANES((bru1<LL, RP><<<a.grid, kBlock, 0, s>>>(a))));
  MSC_BATCH_RHS(MSC_BATCH_LANES((bru2<LL, RP><<<a.grid, kBlock, 0, s>>>(a))));
  return hipGetLastError();
}

hipError_t launch_batch_verify(const BatchArgs& a, int nrhs, int ns, hipStream_t s) {
  for (int q = 0; q < nrhs; ++q) {
    for (int k0 = 0; k0 < ns; k0 += kBvShifts) {
      MSC_BATCH_LANES((bv1<LL><<<a.grid, kBlock, 0, s>>>(a, q, k0)));
      MSC_BATCH_LANES((bv2<LL><<<a.grid, kBlock, 0, s>>>(a, q, k0)));
    }
  }
  return hipGetLastError();
}

}  // namespace msc
