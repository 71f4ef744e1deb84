// Per-ring algebra of the electron rings and the beam-table count, shared by
// the one-species marcher and the two-species (mobile-ion) marcher.
#pragma once
#include "wake_device.h"

// ---------------------------------------------------------------------------
// per-ring algebra
// ---------------------------------------------------------------------------
// The recursion of eq. ai_bi at ring i in the form the marchers step it.  The
// transfer matrix is M_i = 1 + (A_i / 2) p q^T with p = (1, -rho^2) and q =
// (rho, 1/rho), q.p = 0, so with m(x) = rho^2 x_a + x_b (= rho q.x, the same
// before and after the step)
//   M_i x = x + (A_i m / (2 rho)) p,  M_i^-1 x = x - (A_i m / (2 rho)) p,
// and the offset is s_i = (s_a, rho C_i - rho^2 s_a) with s_a = (2 B_i + A_i
// C_i) / 4, so that det[x, s_i] = x_a rho C_i - s_a m(x).  B_i / A_i and C_i
// (eqs. b_coeffs_1-3 for an electron ring, q = -1, m = 1):
//   B / A = B^(b) + (d_rho psi (u^2 / psibar - gamma) + d_rho|a|^2 / 4
//           + u (u / rho - d_zeta psi)) / psibar
//   rho C = (w / 2) cc,  cc = 1 + (u^2 - 1 - |a|^2 / 2) / psibar^2.
// About 60 operations per ring and pass where the coefficients, the matrix
// and its products written out took 100 (7900 rings on one workgroup, rings
// in order: 53.5 -> 49.4 us per slice).
struct Local {
  double pb, ipb, gm, cu, A;    // psibar, 1/psibar, gamma, u/(rho psibar), A_i
};

__device__ __forceinline__ Local local_of(double irho, double u, double w, double psi, double a2) {
  Local L;
  L.pb = 1.0 + psi;
  L.ipb = rcp_nr(L.pb);
  const double t = __builtin_fma(0.5, a2, __builtin_fma(u, u, 1.0));
  L.gm = 0.5 * L.ipb * __builtin_fma(L.pb, L.pb, t);
  const double i = irho * L.ipb;
  L.cu = u * i;
  L.A = w * i;
  return L;
}

// cc and the first component s_a of the ring's offset
__device__ __forceinline__ void ring_source(double irho, double u, double w, const Local& L, double a2, double dpsi,
                                            double dz, double bb, double da2, double& cc, double& sa) {
  const double u2 = u * u;
  cc = __builtin_fma(L.ipb * L.ipb, __builtin_fma(-0.5, a2, u2 - 1.0), 1.0);
  double t = __builtin_fma(dpsi, __builtin_fma(u2, L.ipb, -L.gm), 0.25 * da2);
  t = __builtin_fma(u, __builtin_fma(u, irho, -dz), t);
  const double hb = __builtin_fma(L.ipb, t, bb);              // B / A
  sa = L.A * __builtin_fma(0.125 * w * irho, cc, 0.5 * hb);    // C / 4 = w cc / (8 rho)
}

__device__ __forceinline__ Pack<4> mat_adj(const Pack<4>& m) {
  return {{m.v[3], -m.v[1], -m.v[2], m.v[0]}};
}

// a / b for double-double a with a precomputed reciprocal ib = 1/b
__device__ __forceinline__ dd dd_div_rcp(dd a, double b, double ib) {
  _Pragma("clang fp contract(off)")
  const double q1 = a.hi * ib;
  const dd r = dd_sub(a, two_prod(q1, b));
  const double q2 = r.hi * ib;
  return fast_two_sum(q1, q2);
}

// The other species' field at a ring, as the interpolation leaves it:
// psi = (ph + pl) + t ps, d_rho psi = (dh + dl) + t ds with ph + pl and
// dh + dl the lower node's double-doubles and ps, ds the steps to the next.
struct Lerp {
  double ph, pl, ps, dh, dl, ds, t;
};

// PT + lnr w: the running sum of w ln rho, one ring further.
__device__ __forceinline__ dd psi_next(dd PT, dd lnr, double w) {
  _Pragma("clang fp contract(off)")
  const dd p = two_prod(lnr.hi, w);
  dd s = two_sum(PT.hi, p.hi);
  s.lo += PT.lo + __builtin_fma(lnr.lo, w, p.lo);
  return fast_two_sum(s.hi, s.lo);
}

// psi - psi(0) and d_rho psi at a ring (eqs. psi, dpsi_dr; the ring itself
// with its modified weight wh in the Gauss sum): S the weights below it, Sn
// those through it, PTn the sum of w ln rho through it, X the other
// species' share.  The sums cancel to psi, so their high parts are added
// with two_sum and every low part in binary64 (error a few 2^-104 of the
// terms, as from double-double additions); nothing is renormalised on the
// way, since both results are rounded at the end: 40 operations where the
// chain of double-double calls took 94 (7900 rings on one workgroup, rings
// in order: 58.3 -> 53.5 us per slice together with ion_find's one round of
// reads).
__device__ __forceinline__ void psi_family(dd S, dd Sn, dd PTn, dd lnr, double rho, double irho, double wh,
                                           const Lerp& X, double& psi, double& dpsi) {
  _Pragma("clang fp contract(off)")
  const dd p = two_prod(Sn.hi, lnr.hi);
  const double pe = __builtin_fma(Sn.hi, lnr.lo, __builtin_fma(Sn.lo, lnr.hi, p.lo));
  const dd a = two_sum(p.hi, -PTn.hi);
  const dd b = two_sum(a.hi, X.ph);
  const double lo = ((pe - PTn.lo) + X.pl) + (a.lo + b.lo);
  psi = b.hi + __builtin_fma(X.t, X.ps, lo);
  const dd g = two_sum(S.hi, wh);
  const double q1 = g.hi * irho;
  const double q2 = (__builtin_fma(-q1, rho, g.hi) + (g.lo + S.lo)) * irho;
  const dd d = two_sum(q1, X.dh);
  dpsi = d.hi + __builtin_fma(X.t, X.ds, (q2 + X.dl) + d.lo);
}

// Number of entries of the ascending table br[0..m) below r, given that
// the first lo entries are below r: galloping from lo (gallop) or a plain
// binary search of [lo, m).
template <class P>
__device__ __forceinline__ int count_below(P br, int lo, int m, double r, bool gallop) {
  int a, b;
  if (gallop) {
    if (lo >= m || !(br[lo] < r)) return lo;
    a = lo;                            // br[a] < r
    int step = 1;
    for (;;) {
      b = a + step;
      if (b >= m) { b = m; break; }
      if (!(br[b] < r)) break;
      a = b;
      step <<= 1;
    }
    a += 1;                            // answer in [a, b]
  } else {
    a = lo;
    b = m;
  }
  while (a < b) {
    const int mid = (a + b) >> 1;
    if (br[mid] < r) a = mid + 1; else b = mid;
  }
  return a;
}
// The same count for radii met in descending order: hi is the count of the
// previous (larger) radius when gallop is set.
template <class P>
__device__ __forceinline__ int count_below_down(P br, int hi, int m, double r, bool gallop) {
  int a, b;
  if (gallop) {
    if (hi <= 0 || br[hi - 1] < r) return hi;
    b = hi - 1;                        // br[b] >= r: the answer is at most b
    int step = 1;
    for (;;) {
      a = b - step;
      if (a < 0) { a = 0; break; }
      if (br[a] < r) { a += 1; break; }
      b = a;
      step <<= 1;
    }
  } else {
    a = 0;
    b = m;
  }
  while (a < b) {
    const int mid = (a + b) >> 1;
    if (br[mid] < r) a = mid + 1; else b = mid;
  }
  return a;
}
