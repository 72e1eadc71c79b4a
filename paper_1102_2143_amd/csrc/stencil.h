// Matrix-free staggered operator: M = m + D and M^H = m - D computed from the link field
// (Stencil in msc_internal.h) instead of a stored matrix, one lattice site per lane.
//
// D v at site s, colour c, reads row c of the four forward links W_mu(s) and column c of
// the four backward links W_mu(s - mu), and the three colours of the eight neighbours.  A
// lane computes all three colours of its site, so it reads each of its eight links once,
// whole, and each neighbour's three values once (paper: Section 3, where the library
// leaves room for a custom linear operator kernel in place of the stored matrix when an
// application warrants one).
//
// The links are stored value-major: entry k (row-major within the 3 x 3 matrix) of W_mu
// at site s is w[(mu K + k) vol + s], K = 9, or K = 6 when only rows 0 and 1 are kept.
// The 64 lanes of a wave hold 64 consecutive sites, so each of their link loads reads
// one contiguous run of 64 values.
#pragma once

#include "dev_common.h"
#include "msc_internal.h"

namespace msc {

// acc += conj(a) * b
template <class R>
__device__ __forceinline__ void cfma_conj(cplx<R>& acc, const cplx<R>& a, const cplx<R>& b) {
  acc.x = fma(a.x, b.x, acc.x);
  acc.x = fma(a.y, b.y, acc.x);
  acc.y = fma(a.x, b.y, acc.y);
  acc.y = fma(-a.y, b.x, acc.y);
}

// conj(a b - c d)
template <class R>
__device__ __forceinline__ cplx<R> conj_diff(const cplx<R>& a, const cplx<R>& b, const cplx<R>& c,
                                             const cplx<R>& d) {
  const R re = fma(a.x, b.x, fma(-a.y, b.y, fma(-c.x, d.x, c.y * d.y)));
  const R im = fma(a.x, b.y, fma(a.y, b.x, fma(-c.x, d.y, -c.y * d.x)));
  return cplx<R>{re, -im};
}

// Row 2 of an SU(3) link W = (eta/2) U from its rows 0 and 1 (u[0..2], u[3..5]): the third
// row of U is conj(u0 x u1), so that of W is conj(w0 x w1) / (eta/2) = 2 eta conj(w0 x w1).
// te = 2 eta, equal for a site and its backward neighbour in direction mu (eta_mu does
// not depend on x_mu).
template <class R>
__device__ __forceinline__ void third_row(cplx<R> (&u)[9], R te) {
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int j1 = (j + 1) % 3, j2 = (j + 2) % 3;
    cplx<R> r2 = conj_diff<R>(u[j1], u[3 + j2], u[j2], u[3 + j1]);
    r2.x *= te;
    r2.y *= te;
    u[6 + j] = r2;
  }
}

// What a wave marching along t (one site per lane, the next site one t-slice further on)
// keeps from one site to the next: the stored entries of the site's t link, which are
// the next site's backward t link, and the values at the site and at its forward t
// neighbour, which are the next site's backward t neighbour and its own values.
template <class R, int LR> struct TCarry {
  cplx<R> u[3 * LR];
  cplx<R> own[3];
  cplx<R> fw[3];
};

// out[c] = m own[c] + sign (D v)(s, c), c = 0, 1, 2, with v read through gather(site, colour)
// and own[c] = v(s, c).  LR: link rows stored (3, or 2 for SU(3) links).
// CAR: car->u and car->own stand in for the backward t link and the backward t
// neighbour's values, and must hold exactly those (the previous site's t link and values
// when the site lies one t-slice past it, else loaded for the site); on return car->u
// holds this site's t link and car->fw the forward t neighbour's values (car->own is the
// caller's to set).  The arithmetic is the same either way.
// TREE: the eight half directions' three terms are summed by themselves and then in pairs,
// which halves the rounding of a product (relative to it 1.4e-16 in FP64, 2.6e-16 in one chain
// of 24 terms); for products that are results themselves.
template <class R, int LR, bool CAR, bool TREE, class G>
__device__ __forceinline__ void stencil_site_c(const Stencil<cplx<R>>& op, uint32_t s,
                                               const cplx<R> (&own)[3], int sign, G gather,
                                               cplx<R> (&out)[3], TCarry<R, LR>* car) {
  static_assert(LR == 2 || LR == 3, "link rows");
  constexpr int K = 3 * LR;
  // neighbours and the sign mask in 32 bits (the volume is below 2^31, checked at
  // creation)
  const uint32_t vol = uint32_t(op.vol);
  uint32_t rem = s;
  uint32_t fwd[4], bwd[4];
  uint32_t neg = 0;  // bit mu: eta_mu(x) = -1
  uint32_t par = 0;
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    const uint32_t L = uint32_t(op.L[mu]);
    const uint32_t q = rem / L;
    const uint32_t xm = rem - q * L;
    rem = q;
    neg |= (par & 1u) << mu;
    par += xm;
    const uint32_t st = uint32_t(op.stride[mu]);
    fwd[mu] = xm == L - 1 ? s - (L - 1) * st : s + st;
    bwd[mu] = xm == 0 ? s + (L - 1) * st : s - st;
  }
  cplx<R> h[3], even[3];  // even: TREE, directions 0 and 2
#pragma unroll
  for (int c = 0; c < 3; ++c) h[c] = czero<R>();
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    const cplx<R>* __restrict__ wm = op.w + int64_t(mu) * K * vol;
    cplx<R> U[9], B[9], gf[3], gb[3];
    const bool kept = CAR && mu == 3;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      // a carried t link is read this once: the streaming hint leaves the L2 to the links
      // and values that the neighbours read again
      U[k] = kept ? ld_stream(&wm[int64_t(k) * vol + s]) : wm[int64_t(k) * vol + s];
      if (kept)
        B[k] = car->u[k];
      else
        B[k] = wm[int64_t(k) * vol + bwd[mu]];
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      gf[j] = gather(fwd[mu], j);
      if (kept)
        gb[j] = car->own[j];
      else
        gb[j] = gather(bwd[mu], j);
    }
    if constexpr (CAR) {
      if (mu == 3) {
#pragma unroll
        for (int k = 0; k < K; ++k) car->u[k] = U[k];
#pragma unroll
        for (int j = 0; j < 3; ++j) car->fw[j] = gf[j];
      }
    }
    if constexpr (LR == 2) {
      const R te = ((neg >> mu) & 1u) ? R(-2) : R(2);
      third_row<R>(U, te);
      third_row<R>(B, te);
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      gb[j].x = -gb[j].x;
      gb[j].y = -gb[j].y;
    }
    if constexpr (TREE) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        // the mass term starts a sum of its own size rather than ending the whole one
        const R mo = mu > 0 ? R(0) : sign > 0 ? R(op.mass) : -R(op.mass);
        cplx<R> f{mo * own[c].x, mo * own[c].y}, b = czero<R>();
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          cfma<R>(f, U[3 * c + j], gf[j]);
          cfma_conj<R>(b, B[3 * j + c], gb[j]);
        }
        const cplx<R> d{f.x + b.x, f.y + b.y};
        if (mu % 2 == 0) {
          even[c] = d;
        } else {
          h[c].x += even[c].x + d.x;
          h[c].y += even[c].y + d.y;
        }
      }
    } else {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          cfma<R>(h[c], U[3 * c + j], gf[j]);
          cfma_conj<R>(h[c], B[3 * j + c], gb[j]);
        }
      }
    }
  }
  const R m = TREE ? R(0) : R(op.mass);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if constexpr (TREE) {
      out[c] = sign > 0 ? h[c] : cplx<R>{-h[c].x, -h[c].y};
      continue;
    }
    out[c].x = fma(m, own[c].x, sign > 0 ? h[c].x : -h[c].x);
    out[c].y = fma(m, own[c].y, sign > 0 ? h[c].y : -h[c].y);
  }
}

template <class R, int LR, class G>
__device__ __forceinline__ void stencil_site(const Stencil<cplx<R>>& op, uint32_t s,
                                             const cplx<R> (&own)[3], int sign, G gather,
                                             cplx<R> (&out)[3]) {
  stencil_site_c<R, LR, false, false>(op, s, own, sign, gather, out,
                                      static_cast<TCarry<R, LR>*>(nullptr));
}

// Direction mu's share of (D v)(s, .): the forward and the backward term of one direction.
template <class R, int LR, class G>
__device__ __forceinline__ void stencil_dir(const Stencil<cplx<R>>& op, uint32_t s, int mu, G gather,
                                            cplx<R> (&h)[3]) {
  constexpr int K = 3 * LR;
  const uint32_t vol = uint32_t(op.vol);
  uint32_t rem = s, par = 0, fwd = s, bwd = s;
#pragma unroll
  for (int nu = 0; nu < 4; ++nu) {
    if (nu <= mu) {  // mu is uniform
      const uint32_t L = uint32_t(op.L[nu]), st = uint32_t(op.stride[nu]);
      const uint32_t q = rem / L, xm = rem - q * L;
      rem = q;
      if (nu < mu) {
        par += xm;
      } else {
        fwd = xm == L - 1 ? s - (L - 1) * st : s + st;
        bwd = xm == 0 ? s + (L - 1) * st : s - st;
      }
    }
  }
  const cplx<R>* __restrict__ wm = op.w + int64_t(mu) * K * vol;
  cplx<R> U[9], B[9], gf[3], gb[3];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    U[k] = wm[int64_t(k) * vol + s];
    B[k] = wm[int64_t(k) * vol + bwd];
  }
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    gf[j] = gather(fwd, j);
    gb[j] = gather(bwd, j);
    gb[j].x = -gb[j].x;
    gb[j].y = -gb[j].y;
  }
  if constexpr (LR == 2) {
    const R te = (par & 1u) ? R(-2) : R(2);
    third_row<R>(U, te);
    third_row<R>(B, te);
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    h[c] = czero<R>();
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      cfma<R>(h[c], U[3 * c + j], gf[j]);
      cfma_conj<R>(h[c], B[3 * j + c], gb[j]);
    }
  }
}

// M (sign 1) or M^H (sign -1) times several vectors at one site: out[q][c] of xs[q] (colour by
// colour: value (s, c) at c vol + s), q < cnt <= G.  A direction's two links are read and completed once for all of them.
template <class R, int LR, int G>
__device__ __forceinline__ void stencil_site_group(const Stencil<cplx<R>>& op, uint32_t s, int sign,
                                                   const cplx<R>* const (&xs)[G], int cnt,
                                                   cplx<R> (&out)[G][3]) {
  constexpr int K = 3 * LR;
  const uint32_t vol = uint32_t(op.vol);
  uint32_t rem = s, par = 0;
  cplx<R> h[G][3];
#pragma unroll
  for (int q = 0; q < G; ++q)
#pragma unroll
    for (int c = 0; c < 3; ++c) h[q][c] = czero<R>();
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    const uint32_t L = uint32_t(op.L[mu]), st = uint32_t(op.stride[mu]);
    const uint32_t qt = rem / L, xm = rem - qt * L;
    rem = qt;
    const R te = (par & 1u) ? R(-2) : R(2);  // 2 eta_mu
    par += xm;
    const uint32_t fwd = xm == L - 1 ? s - (L - 1) * st : s + st;
    const uint32_t bwd = xm == 0 ? s + (L - 1) * st : s - st;
    const cplx<R>* __restrict__ wm = op.w + int64_t(mu) * K * vol;
    cplx<R> U[9], B[9];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      U[k] = wm[int64_t(k) * vol + s];
      B[k] = wm[int64_t(k) * vol + bwd];
    }
    if constexpr (LR == 2) {
      third_row<R>(U, te);
      third_row<R>(B, te);
    }
#pragma unroll
    for (int q = 0; q < G; ++q) {
      if (q < cnt) {
        cplx<R> gf[3], gb[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          gf[j] = xs[q][int64_t(j) * vol + fwd];
          gb[j] = xs[q][int64_t(j) * vol + bwd];
          gb[j].x = -gb[j].x;
          gb[j].y = -gb[j].y;
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            cfma<R>(h[q][c], U[3 * c + j], gf[j]);
            cfma_conj<R>(h[q][c], B[3 * j + c], gb[j]);
          }
        }
      }
    }
  }
  const R m = R(op.mass);
#pragma unroll
  for (int q = 0; q < G; ++q) {
    if (q < cnt) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const cplx<R> own = xs[q][int64_t(c) * vol + s];
        out[q][c].x = fma(m, own.x, sign > 0 ? h[q][c].x : -h[q][c].x);
        out[q][c].y = fma(m, own.y, sign > 0 ? h[q][c].y : -h[q][c].y);
      }
    }
  }
}

}  // namespace msc
