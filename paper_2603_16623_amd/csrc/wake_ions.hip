// gfx950 marcher of the two-species gridless model: plasma electrons and
// mobile ions, each discretised into rings (paper, Sec. "Gridless
// quasistatic model" and "Key algorithmic adjustments": every species is
// summed on its own at its own rings, the fields of the other species are
// interpolated linearly between that species' rings, and the ion currents
// are left out of B_theta^(p)).
//
// One workgroup of 1024 threads marches one instance through its slices.
// Per species, thread t owns the C = ceil(N / 1024) consecutive sorted
// positions [tC, tC + C); per-position arrays are stored by slot
// (p % C) * 1024 + p / C and per-ring ones by the slot of the ring's initial
// position, so the k-th positions of a wave are contiguous.  The sorted radii
// of both species sit in LDS (by position, the low bits exchanged so that
// lanes C apart meet different banks), where the interval searches of the
// gathers run; node tables, per-position work and ring state live in device
// memory as planes of 16-B chunks.
//
// What bounds it: with one instance the chain of phases (a barrier and a
// round of loads each), with a device full of instances the bytes of the
// planes.  Before the planes, constants, state and order were read by ring id
// or position, one line per lane: 256 cycles of the load path per wave for
// the four constants of ln rho alone.
//
// The sums and the interpolated fields are double-doubles with both low parts
// added exactly (dd_add: about 2^-105 of the result) and every quotient is
// rounded to nearest: the two species' sums cancel to psi, and the form with
// low parts added in binary64 (dd_add_fast: some 2^-104 of the operands) and
// uncorrected reciprocals would hold less, though measured errors against 64
// bits are the same.  (1500 rings 48.7 us per slice where that form takes 42.7,
// 4000 89.1 and 78.9, a batch of 256 102 ms and 98.)
//
// Per slice:
//   order    each species' (rho, id) order: the previous one if it still
//            holds, else rounds of wave blocks of 256 positions sorted in
//            LDS and the blocks between them merged (the bitonic network
//            over all positions after three rounds that leave disorder);
//   sums     ln rho and the chunk sums of w and w ln rho; after their scans
//            own psi and d_rho psi at each species' rings (eqs. psi,
//            dpsi_dr; double-double prefix of w and suffix of w ln rho, the
//            ring itself with w^), its axis value, outer edge and exterior
//            field: the node tables;
//   gather   the other species' psi and d_rho psi interpolated at every
//            ring; psibar with the species' q and m; beam and laser sources;
//            own d_zeta psi (eq. dpsi_dzeta, suffix of q w u / (rho psibar));
//   B^(p)    electrons only, forward: the ions' d_zeta psi interpolated, the
//            ring's offset and transfer (eqs. b_coeffs_1-3, ai_bi), the
//            chunk's product G and lambda = sum of G_i^T J s_i; scans of the
//            transfers and then of the det-sums g.lambda, h.lambda (the
//            one-species marcher's Green's-function form);
//   push     electrons, backward: g and h stepped back, B^(p) (eq.
//            b_theta_plasma), fields out, Adams-Bashforth-2 push into the
//            other state buffer; then the ions: d_zeta psi and B^(p)
//            interpolated between the electron rings, fields out, push.
#include "wake_common.h"
#include "wake_device.h"
#include "wake_ring.h"
#include "wake_ions.h"

#include <math.h>

namespace {

constexpr int NT = WAKE_IONS_NT;
constexpr int NW = NT / 64;
constexpr int NMAX = WAKE_IONS_NMAX;

// dynamic LDS: sorted radii of both species, sort ids, scan area, slice
// constants (analytic source factors, then 16 scalars per species), the
// slice's beam table
struct IonsLds {
  static constexpr size_t r_off = 0;
  static constexpr size_t id_off = r_off + (size_t)2 * NMAX * sizeof(double);
  static constexpr size_t scan_off = id_off + (size_t)NMAX * sizeof(uint16_t);
  static constexpr size_t misc_off = scan_off + (size_t)NW * 16 * sizeof(double);
  static constexpr size_t br_off = misc_off + 64 * sizeof(double);
  // the slice's beam table: radii and cumulative charges of up to BOTH
  // entries, radii alone of up to 2 BOTH
  static constexpr int BOTH = 832;
  static constexpr size_t bytes = br_off + (size_t)2 * BOTH * sizeof(double);
};
static_assert(IonsLds::bytes <= 160 * 1024, "two-species LDS");

// per-species scalars of a slice (at s_misc + 32 + 16 s): psi(0) of the
// species alone (dd), total weight (dd), outer edge, exterior psi at the
// edge (dd), exterior d_rho psi at the edge (dd), d_zeta psi(0) of the species
// alone (dd)
enum { SC_PAH = 0, SC_PAL, SC_QH, SC_QL, SC_EDGE, SC_EPH, SC_EPL, SC_EDP, SC_EDL, SC_DZH, SC_DZL,
       SC_N = 16 };

// Slot of position p (home slot of ring p): p / C as a multiply and shift,
// exact for p < 8192 and C <= 8 (div = 65536 / C rounded up).
__device__ __forceinline__ unsigned pslot(int p, int C, unsigned div) {
  const unsigned q = ((unsigned)p * div) >> 16;
  return ((unsigned)p - q * (unsigned)C) * NT + q;
}
__device__ __forceinline__ unsigned slot_div(int C) { return (65536u + (unsigned)C - 1u) / (unsigned)C; }

// Where the radius of position p sits in LDS: the lanes of a wave own
// positions C apart, which for even C would meet in a few banks (at C = 8
// sixteen lanes in one); the block of eight is kept, so the index stays
// inside the array.
__device__ __forceinline__ unsigned rx(int p) { return (unsigned)p ^ (((unsigned)p >> 5) & 7u); }

// Bitonic sort of the keys (kr, ki) of n positions in place (n <= NMAX),
// padded with +inf keys to the next power of two.
__device__ void bitonic_ions(double* kr, uint16_t* ki, int n) {
  int P = 1;
  while (P < n) P <<= 1;
  for (int i = n + (int)threadIdx.x; i < P; i += NT) { kr[rx(i)] = INFINITY; ki[i] = 0xFFFF; }
  __syncthreads();
  for (int k = 2; k <= P; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = threadIdx.x; i < P; i += NT) {
        const int l = i ^ j;
        if (l > i) {
          const double a = kr[rx(i)], b = kr[rx(l)];
          const uint16_t ia = ki[i], ib = ki[l];
          const bool up = (i & k) == 0;
          const bool sw = up ? key_lt(b, (int32_t)ib, a, (int32_t)ia) : key_lt(a, (int32_t)ia, b, (int32_t)ib);
          if (sw) { kr[rx(i)] = b; kr[rx(l)] = a; ki[i] = ib; ki[l] = ia; }
        }
      }
      __syncthreads();
    }
  }
}

// (rho, id) order of keys with the id in k (no short-circuit: straight-line
// selects)
__device__ __forceinline__ bool ik_lt(double ra, uint32_t ka, double rb, uint32_t kb) {
  return (ra < rb) | ((ra == rb) & (ka < kb));
}
// One wave puts positions [b0, b0 + 256) (clipped at n) of the keys in LDS
// in order, in place.  MERGE: the two halves are each in order.
template <bool MERGE>
__device__ void ions_sort_block(double* kr, uint16_t* ki, int b0, int n) {
  double r[4];
  uint32_t k[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int p = b0 + wave_place<MERGE>(j);
    r[j] = p < n ? kr[rx(p)] : INFINITY;
    k[j] = p < n ? (uint32_t)ki[p] : ~0u;
  }
  if (!wave_sort256<MERGE>(r, k, [](uint32_t i) { return i; })) return;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int p = b0 + 4 * (threadIdx.x & 63) + j;
    if (p < n) { kr[rx(p)] = r[j]; ki[p] = (uint16_t)k[j]; }
  }
}

// Order of n nearly sorted keys in LDS (position order), in place, in
// rounds: the wave blocks of 256 positions at 0, 256, ... sorted, those at
// 128, 384, ... (two sorted halves) merged, and the order checked at the
// junctions of the second blocks (every segment between them is sorted).
// A ring that moved more than 128 positions leaves a junction out of order
// for the next round; after three rounds the bitonic network sorts all
// positions.
__device__ void ions_fix_order(double* kr, uint16_t* ki, int n) {
  constexpr int NW = NT / 64;
  static_assert(NMAX <= 64 * 256, "a junction per lane");
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  #pragma unroll 1
  for (int round = 0; round < 3; ++round) {
    #pragma unroll 1
    for (int b = wave; b * 256 < n; b += NW) ions_sort_block<false>(kr, ki, b * 256, n);
    __syncthreads();
    #pragma unroll 1
    for (int b = wave; 256 * (b + 1) < n; b += NW) ions_sort_block<true>(kr, ki, 128 + b * 256, n);
    __syncthreads();
    bool out = false;
    const int q = 128 + 256 * lane;
    if (q < n) out = ik_lt(kr[rx(q)], ki[q], kr[rx(q - 1)], ki[q - 1]);
    if (!__syncthreads_or(out)) return;     // also: every wave has read its junction keys
  }
  bitonic_ions(kr, ki, n);
}

// a / b with y = rcp_nr(b): the remainder of the first quotient (one fma) goes
// back through y, which leaves the sum within 2^-50 ulp of a / b before its
// rounding, as near as the division sequence comes, in two thirds of its
// operations.  b = 0, infinite or subnormal gives NaN: the slice breaks down
// there by its fields.
__device__ __forceinline__ double quot(double a, double b, double y) {
  const double q = a * y;
  return __builtin_fma(__builtin_fma(-q, b, a), y, q);
}
// a / b for double-double a, both quotients rounded to nearest
__device__ __forceinline__ dd dd_quot(dd a, double b, double y) {
  _Pragma("clang fp contract(off)")
  const double q1 = quot(a.hi, b, y);
  const dd r = dd_sub(a, two_prod(q1, b));
  return fast_two_sum(q1, quot(r.hi, b, y));
}

// The node interval of radius r of one species seen from the other (node 0
// the axis, node j = its ring j-1, node N+1 its edge): the lower node is j =
// the number of its rings below r; t the fraction of the way to node j+1,
// exactly 1 at the upper node, so that a ring at a node takes that node's value
// whole and the two species' sums cancel at rest.
__device__ __forceinline__ double interval_t(const double* ro, int N, double edge, double r, int j) {
  const double rl = j == 0 ? 0.0 : ro[rx(j - 1)];
  const double rh = j < N ? ro[rx(j)] : edge;
  return quot(r - rl, rh - rl, rcp_nr(rh - rl));
}

// Number of the sorted radii ro[0..n) below r, the first lo of which are:
// four at once (the answer for the next ring in order is a step or two
// away), then galloping and bisection.
__device__ __forceinline__ int rings_below(const double* ro, int lo, int n, double r) {
  const int last = n - 1;
  const double x0 = ro[rx(min(lo, last))], x1 = ro[rx(min(lo + 1, last))], x2 = ro[rx(min(lo + 2, last))],
               x3 = ro[rx(min(lo + 3, last))];
  const int c = (x0 < r ? 1 : 0) + (x1 < r ? 1 : 0) + (x2 < r ? 1 : 0) + (x3 < r ? 1 : 0);
  int a = min(lo + c, n);
  if (c < 4 || a == n) return a;
  int b, step = 4;                       // ro[a - 1] < r
  for (;;) {
    b = a + step;
    if (b > n) { b = n + 1; break; }
    if (!(ro[rx(b - 1)] < r)) break;
    a = b;
    step <<= 1;
  }
  // the answer is in [a, b)
  while (b - a > 1) {
    const int m = (a + b) >> 1;
    if (ro[rx(m - 1)] < r) a = m; else b = m;
  }
  return a;
}

// a + t (b - a) of two double-doubles
__device__ __forceinline__ dd dd_lerp(dd a, dd b, double t) {
  return dd_add(a, dd_mul_d(dd_sub(b, a), t));
}

__global__ __launch_bounds__(NT) void ions_march_kernel(const WakeIons* __restrict__ insts) {
  const WakeIons& I = insts[blockIdx.x];
  double* const s_r = reinterpret_cast<double*>(wake_lds + IonsLds::r_off);
  uint16_t* const s_id = reinterpret_cast<uint16_t*>(wake_lds + IonsLds::id_off);
  double* const s_scan = reinterpret_cast<double*>(wake_lds + IonsLds::scan_off);
  double* const s_misc = reinterpret_cast<double*>(wake_lds + IonsLds::misc_off);
  double* const s_sc = s_misc + 32;
  double* const s_br = reinterpret_cast<double*>(wake_lds + IonsLds::br_off);

  const int tid = threadIdx.x;
  const int N = I.N, C = I.C;
  const unsigned S = (unsigned)C * NT, div = slot_div(C);
  const int p0 = tid * C;
  const int cnt = N - p0 < 0 ? 0 : (N - p0 < C ? N - p0 : C);
  const int aw = __builtin_amdgcn_readfirstlane(((N + C - 1) / C + 63) >> 6);   // waves with rings
  if (I.ctl[CTL_BREAK] >= 0) return;
  int cur = I.ctl[CTL_CUR];
  const int end = I.first + I.count;
  const int n_an = I.n_an;
  const double dxi = I.dxi;
  const double m_ion = I.m_i;
  const bool has_laser = I.has_laser != 0;   // else |a|^2 and its gradient are 0 (not stored)
  const GA<D2> K = uview(reinterpret_cast<const D2*>(I.cst));
  const GA<D2> W = uview(reinterpret_cast<const D2*>(I.work));
  const GA<double> Wh = uview(reinterpret_cast<const double*>(I.work));   // its halves
  const GA<int32_t> ORD = uview(I.ord), SID = uview(I.sid), JX = uview(I.jx);
  unsigned long long fixups = 0;
  int n = I.first;
  for (; n < end; ++n) {
    const double xi = n * dxi;
    if (tid < n_an) {             // this slice's analytic source factors
      const WakeAnalytic& A = I.an[tid];
      if (A.kind == 2) {
        const double s2 = A.sigma_r * A.sigma_r;
        const double dl = xi - A.xi_c;
        s_misc[3 * tid] = 2.0;
        s_misc[3 * tid + 1] = A.q * A.n_peak * exp(-(dl * dl) / (2.0 * A.sigma_xi * A.sigma_xi)) * s2;
        s_misc[3 * tid + 2] = 1.0 / (2.0 * s2);
      } else {
        const double dl = xi - A.xi_l;
        s_misc[3 * tid] = 3.0;
        s_misc[3 * tid + 1] = A.a0 * A.a0 * exp(-2.0 * dl * dl / (A.L * A.L));
        s_misc[3 * tid + 2] = 2.0 / (A.w0 * A.w0);
      }
    }
    // this slice's beam table into LDS (read after the order phase's
    // barriers; the previous slice's reads ended at its last barrier): a
    // ring's charge read from device memory behind its search kept the waves
    // in the beam 15 us behind the others at 7900 rings
    const int bt0 = I.nb ? I.boff[n] : 0;
    const int bm = I.nb ? I.boff[n + 1] - bt0 : 0;
    const bool b_both = bm <= IonsLds::BOTH, b_lds = bm <= 2 * IonsLds::BOTH;
    if (b_lds)
      for (int i = tid; i < bm; i += NT) s_br[i] = gptr(I.br)[bt0 + i];
    if (b_both)
      for (int i = tid; i < bm; i += NT) s_br[IonsLds::BOTH + i] = gptr(I.bcum)[bt0 + i];
    const GA<D2> Sc = uview(reinterpret_cast<const D2*>(I.st[cur]));
    const GA<D2> Sn = uview(reinterpret_cast<const D2*>(I.st[cur ^ 1]));

    // ---- order of each species ----
    int bad_order = 0;
    #pragma unroll 1
    for (int s = 0; s < 2; ++s) {
      double* const sr = s_r + s * NMAX;
      const unsigned so = s * S, st = (unsigned)(s * IS_N + IS_RU) * S;
      int dis = 0, pi = -1;
      double pr = -INFINITY;
      #pragma unroll 2
      for (int k = 0; k < cnt; ++k) {
        const int p = p0 + k;
        const unsigned sl = so + k * NT + tid;
        const int id = ORD[sl];
        const unsigned hs = pslot(id, C, div);
        const double r = Sc[st + hs].x;
        SID.st(sl, (int32_t)hs);
        sr[rx(p)] = r;
        s_id[p] = (uint16_t)id;
        if (!key_lt(pr, pi, r, id)) dis = 1;
        pr = r;
        pi = id;
      }
      __syncthreads();
      if (cnt > 0 && p0 > 0 && !key_lt(sr[rx(p0 - 1)], (int32_t)s_id[p0 - 1], sr[rx(p0)], (int32_t)s_id[p0])) dis = 1;
      if (__syncthreads_or(dis)) {
        ions_fix_order(sr, s_id, N);
        ++fixups;
        #pragma unroll 2
        for (int k = 0; k < cnt; ++k) {
          const unsigned sl = so + k * NT + tid;
          int id = s_id[p0 + k];
          // a padding key among the first N positions: a radius that is not a
          // finite number (state injected from device memory) -- stop there
          if (id >= N) { id = 0; bad_order = 1; }
          ORD.st(sl, id);
          SID.st(sl, (int32_t)pslot(id, C, div));
        }
      }
    }

    // ---- own sums: ln rho, chunk sums of w and w ln rho ----
    dd sw[2], swl[2];
    #pragma unroll
    for (int s = 0; s < 2; ++s) {
      const unsigned wo = (unsigned)(s * IW_N) * S;
      const double* const sr = s_r + s * NMAX;
      sw[s] = dd_make(0.0);
      swl[s] = dd_make(0.0);
      #pragma unroll 2
      for (int k = 0; k < cnt; ++k) {
        const unsigned sl = k * NT + tid;
        const unsigned hs = (unsigned)SID[s * S + sl];
        const D2 w = K[IK_W * S + hs], r0 = K[IK_R0 * S + hs], l0 = K[IK_LN * S + hs];
        const double r = sr[rx(p0 + k)];
        // ln rho as ln r0 + log1p((r - r0)/r0): its rounding scales with the
        // ring's displacement, not with |ln rho|
        const dd lnr = dd_add_d({l0.x, l0.y}, log1p_fast((r - r0.x) * r0.y));
        W.st(wo + IW_W * S + sl, w);
        W.st(wo + IW_LN * S + sl, d2(lnr.hi, lnr.lo));
        sw[s] = dd_add_d(sw[s], w.x);
        swl[s] = dd_add(swl[s], dd_mul_d(lnr, w.x));
      }
    }
    Pack<4> exP, totP, exS, totS;
    block_prefix_suffix<NT, 4, 4, DD2Op, DD2Op, true>(
        Pack<4>{{sw[0].hi, sw[0].lo, sw[1].hi, sw[1].lo}}, Pack<4>{{0.0, 0.0, 0.0, 0.0}}, DD2Op(),
        Pack<4>{{swl[0].hi, swl[0].lo, swl[1].hi, swl[1].lo}}, Pack<4>{{0.0, 0.0, 0.0, 0.0}}, DD2Op(),
        s_scan, exP, totP, exS, totS, aw);
    // node tables: psi and d_rho psi of each species at its own rings
    #pragma unroll 1
    for (int s = 0; s < 2; ++s) {
      const bool neg = s == 1;              // psi = -q (...): the electrons' q is -1
      const unsigned wo = (unsigned)(s * IW_N) * S;
      double* const sc = s_sc + SC_N * s;
      const double* sr = s_r + s * NMAX;
      const dd Q = s ? dd{totP.v[2], totP.v[3]} : dd{totP.v[0], totP.v[1]};
      dd below = s ? dd{exP.v[2], exP.v[3]} : dd{exP.v[0], exP.v[1]};
      // sum over positions >= p
      dd rest = dd_add(s ? dd{exS.v[2], exS.v[3]} : dd{exS.v[0], exS.v[1]}, s ? swl[1] : swl[0]);
      #pragma unroll 2
      for (int k = 0; k < cnt; ++k) {
        const unsigned sl = k * NT + tid;
        const D2 w = W[wo + IW_W * S + sl], l = W[wo + IW_LN * S + sl];
        const dd lnr = {l.x, l.y};
        const double r = sr[rx(p0 + k)];
        rest = dd_sub(rest, dd_mul_d(lnr, w.x));     // sum over positions > p
        // psi = -q ((sum_{k<i} w_k + w_i) ln rho_i + sum_{k>i} w_k ln rho_k)
        // d_rho psi = -q (sum_{k<i} w_k + w^_i) / rho_i
        const dd Sn_ = dd_add_d(below, w.x);
        dd ps = dd_add(dd_mul(Sn_, lnr), rest);
        dd dp = dd_quot(dd_add_d(below, w.y), r, rcp_nr(r));
        below = Sn_;
        if (neg) { ps = dd_neg(ps); dp = dd_neg(dp); }
        W.st(wo + IW_T0 * S + sl, d2(ps.hi, ps.lo));
        W.st(wo + IW_T1 * S + sl, d2(dp.hi, dp.lo));
      }
      if (cnt > 0 && p0 + cnt == N) {
        // outer edge: the outermost ring plus half its initial extent, and
        // the exterior field there (-q Q ln r, -q Q / r)
        const unsigned sl = (cnt - 1) * NT + tid;
        const D2 l = W[wo + IW_LN * S + sl];
        const double r = sr[rx(N - 1)];
        const double edge = r + gptr(I.cst)[2 * IK_DR * S + (unsigned)SID[s * S + sl]] / 2.0;
        const dd lne = dd_add_d({l.x, l.y}, log1p_fast((edge - r) / r));
        dd eps = dd_mul(Q, lne);
        dd edp = dd_div_d(Q, edge);
        if (neg) { eps = dd_neg(eps); edp = dd_neg(edp); }
        sc[SC_EDGE] = edge;
        sc[SC_EPH] = eps.hi;
        sc[SC_EPL] = eps.lo;
        sc[SC_EDP] = edp.hi;
        sc[SC_EDL] = edp.lo;
      }
      if (tid == 0) {
        dd pa = s ? dd{totS.v[2], totS.v[3]} : dd{totS.v[0], totS.v[1]};
        if (neg) pa = dd_neg(pa);
        sc[SC_PAH] = pa.hi;
        sc[SC_PAL] = pa.lo;
        sc[SC_QH] = Q.hi;
        sc[SC_QL] = Q.lo;
      }
    }
    __syncthreads();

    // ---- gather psi, d_rho psi; sources; d_zeta psi sums ----
    int bad = bad_order;
    const WAKE_GLOBAL double* const brg = gptr(I.br) + bt0;
    const WAKE_GLOBAL double* const bcq = gptr(I.bcum) + bt0;
    dd szc0 = dd_make(0.0), szc1 = dd_make(0.0);
    #pragma unroll 1
    for (int s = 0; s < 2; ++s) {
      const int o = s ^ 1;
      const double q = s ? 1.0 : -1.0, m = s ? m_ion : 1.0;
      const double qm = q / m;
      const unsigned wo = (unsigned)(s * IW_N) * S, wx = (unsigned)(o * IW_N) * S;
      const double* sr = s_r + s * NMAX;
      const double* ro = s_r + o * NMAX;
      const double* sco = s_sc + SC_N * o;
      const double edge_o = sco[SC_EDGE];
      dd szc = dd_make(0.0);
      int lo = 0, blo = 0;
      #pragma unroll 1
      for (int k = 0; k < cnt; ++k) {
        const unsigned sl = k * NT + tid;
        const unsigned hs = (unsigned)SID[s * S + sl];
        const double r = sr[rx(p0 + k)];
        if (k == 0) {
          int a = 0, b = N;
          while (a < b) {
            const int c = (a + b) >> 1;
            if (ro[rx(c)] < r) a = c + 1; else b = c;
          }
          lo = a;
        } else {
          lo = rings_below(ro, lo, N, r);
        }
        // both tables' nodes (clamped; the end nodes put in below)
        const unsigned u0 = pslot(max(lo - 1, 0), C, div), u1 = pslot(min(lo, N - 1), C, div);
        const D2 a0 = W[wx + IW_T0 * S + u0], a1 = W[wx + IW_T1 * S + u0];
        const D2 b0 = W[wx + IW_T0 * S + u1], b1 = W[wx + IW_T1 * S + u1];
        const D2 t0 = W[wo + IW_T0 * S + sl], t1 = W[wo + IW_T1 * S + sl];
        const double w = W[wo + IW_W * S + sl].x;
        const double u = Sc[(unsigned)(s * IS_N + IS_RU) * S + hs].y;
        dd pg, dg;
        if (lo < N || !(r > edge_o)) {
          // both in double-double: at a ring of the other species (t = 0 or
          // 1) its node value is taken whole, so the two species' sums
          // cancel there as exactly as they do at rest
          dd pl = {a0.x, a0.y}, dl = {a1.x, a1.y}, ph = {b0.x, b0.y}, dh = {b1.x, b1.y};
          if (lo == 0) { pl = {sco[SC_PAH], sco[SC_PAL]}; dl = dd_make(0.0); }
          if (lo == N) { ph = {sco[SC_EPH], sco[SC_EPL]}; dh = {sco[SC_EDP], sco[SC_EDL]}; }
          const double t = interval_t(ro, N, edge_o, r, lo);
          pg = dd_lerp(pl, ph, t);
          dg = dd_lerp(dl, dh, t);
          JX.st(s * S + sl, lo);
        } else {                  // beyond the other species' edge: its exterior field
          const dd Qo = {sco[SC_QH], sco[SC_QL]};
          const D2 l = W[wo + IW_LN * S + sl];
          pg = dd_mul(Qo, {l.x, l.y});
          dg = dd_div_d(Qo, r);
          if (o) { pg = dd_neg(pg); dg = dd_neg(dg); }
          JX.st(s * S + sl, -1);
        }
        const double psi = dd_round(dd_add(pg, {t0.x, t0.y}));
        const double dpsi = dd_round(dd_add(dg, {t1.x, t1.y}));
        // beam charge inside r (table entries strictly below), analytic beams, lasers
        double lam = 0.0;
        if (bm > 0) {
          blo = b_lds ? count_below(s_br, blo, bm, r, k > 0) : count_below(brg, blo, bm, r, k > 0);
          if (blo > 0) {
            if (b_both) lam = s_br[IonsLds::BOTH + blo - 1];
            else lam = bcq[blo - 1];
          }
        }
        double a2 = 0.0, da2 = 0.0;
        #pragma unroll 1
        for (int si = 0; si < n_an; ++si) {
          const double kind = s_misc[3 * si], c0 = s_misc[3 * si + 1], c1 = s_misc[3 * si + 2];
          if (kind == 2.0) {
            lam += c0 * (-expm1(-r * r * c1));
          } else {
            const double x = c0 * exp(-r * r * c1);
            a2 += x;
            da2 += -(2.0 * r * c1) * x;
          }
        }
        const double pb = 1.0 - qm * psi;
        if (!(pb > 0.0) || !isfinite(pb)) bad = 1;
        const double rpb = r * pb;
        const double c = quot(q * u, rpb, rcp_nr(rpb));
        szc = dd_add_d(szc, w * c);
        W.st(wo + IW_F * S + sl, d2(psi, dpsi));
        W.st(wo + IW_UC * S + sl, d2(u, c));
        Wh.st(2 * (wo + IW_BB * S + sl), quot(lam, r, rcp_nr(r)));
        if (has_laser) W.st(wo + IW_A2 * S + sl, d2(a2, da2));
      }
      if (s) szc1 = szc; else szc0 = szc;
    }
    Pack<4> dzs, dzt;
    dzs = block_suffix<NT, 4>(Pack<4>{{szc0.hi, szc0.lo, szc1.hi, szc1.lo}},
                              Pack<4>{{0.0, 0.0, 0.0, 0.0}}, DD2Op(), s_scan, dzt, aw);
    // own d_zeta psi at each ring: the rings outside with w, the ring itself
    // with w - w^
    #pragma unroll
    for (int s = 0; s < 2; ++s) {
      const unsigned wo = (unsigned)(s * IW_N) * S;
      dd above = s ? dd{dzs.v[2], dzs.v[3]} : dd{dzs.v[0], dzs.v[1]};
      #pragma unroll 2
      for (int k = cnt - 1; k >= 0; --k) {
        const unsigned sl = k * NT + tid;
        const D2 w = W[wo + IW_W * S + sl];
        const double c = W[wo + IW_UC * S + sl].y;
        Wh.st(2 * (wo + IW_ZB * S + sl), dd_round(dd_add_d(above, (w.x - w.y) * c)));
        above = dd_add_d(above, w.x * c);
      }
      if (tid == 0) {
        s_sc[SC_N * s + SC_DZH] = s ? dzt.v[2] : dzt.v[0];
        s_sc[SC_N * s + SC_DZL] = s ? dzt.v[3] : dzt.v[1];
      }
    }
    __syncthreads();

    // ---- electrons: the ions' d_zeta psi; offsets, chunk transfer and lambda ----
    const unsigned wi = (unsigned)IW_N * S;      // the ions' planes (the electrons' start at 0)
    const double* const sre = s_r;
    const double* const sri = s_r + NMAX;
    Pack<4> G = mat_ident();
    double la = 0.0, lb = 0.0;
    {
      const double edge_i = s_sc[SC_N + SC_EDGE];
      const double dza_i = dd_round({s_sc[SC_N + SC_DZH], s_sc[SC_N + SC_DZL]});
      #pragma unroll 1
      for (int k = 0; k < cnt; ++k) {
        const unsigned sl = k * NT + tid;
        const int j = JX[sl];
        const D2 w = W[IW_W * S + sl], f = W[IW_F * S + sl];
        const double u = W[IW_UC * S + sl].x;
        const double bb = Wh[2 * (IW_BB * S + sl)];
        double dz = Wh[2 * (IW_ZB * S + sl)];
        const double r = sre[rx(p0 + k)];
        if (j >= 0) {
          const double dlo = Wh[2 * (wi + IW_ZB * S + pslot(max(j - 1, 0), C, div))];
          const double dhi = Wh[2 * (wi + IW_ZB * S + pslot(min(j, N - 1), C, div))];
          const double t = interval_t(sri, N, edge_i, r, j);
          const double dl = j == 0 ? dza_i : dlo, dh = j < N ? dhi : 0.0;
          dz += (1.0 - t) * dl + t * dh;
        }
        D2 a2 = d2(0.0, 0.0);
        if (has_laser) a2 = W[IW_A2 * S + sl];
        const double ir = rcp_nr(r);
        const Local L = local_of(ir, u, w.x, f.x, a2.x);
        double cc, sa;
        ring_source(ir, u, w.x, L, a2.x, f.y, dz, bb, a2.y, cc, sa);
        const double r2 = r * r, hAi = 0.5 * L.A * ir, rC = 0.5 * w.x * cc;
        const double m0 = __builtin_fma(r2, G.v[0], G.v[2]), m1 = __builtin_fma(r2, G.v[1], G.v[3]);
        const double y0 = hAi * m0, y1 = hAi * m1;
        G.v[0] += y0;
        G.v[1] += y1;
        G.v[2] = __builtin_fma(-r2, y0, G.v[2]);
        G.v[3] = __builtin_fma(-r2, y1, G.v[3]);
        la = __builtin_fma(-sa, m0, __builtin_fma(G.v[0], rC, la));
        lb = __builtin_fma(-sa, m1, __builtin_fma(G.v[1], rC, lb));
        W.st(IW_E * S + sl, d2(L.A, sa));
        W.st(IW_DC * S + sl, d2(dz, cc));
      }
    }
    // growing mode at the chunk start, decaying mode at the chunk end
    Pack<4> gp, gt, hx, ht;
    block_prefix_suffix<NT, 4, 4, FwdMatOp, BwdMatOp, true>(
        G, mat_ident(), FwdMatOp(), mat_adj(G), mat_ident(), BwdMatOp(), s_scan, gp, gt, hx, ht, aw);
    const double W_ = gt.v[0];                // det[g_N, (0, 1)]
    const double iW = 1.0 / W_;
    const double gsa = gp.v[0], gsb = gp.v[2], hea = hx.v[1], heb = hx.v[3];
    // the chunk's sums of det[g_i, s_i] and det[s_i, h_i]
    const double le = gsa * la + gsb * lb;
    const double ld = -((G.v[3] * hea - G.v[1] * heb) * la + (G.v[0] * heb - G.v[2] * hea) * lb);
    Pack<1> ep, et, dsf, dt;
    block_prefix_suffix<NT, 1, 1, SumOp<1>, SumOp<1>, true>(Pack<1>{{le}}, Pack<1>{{0.0}}, SumOp<1>(),
                                                           Pack<1>{{ld}}, Pack<1>{{0.0}}, SumOp<1>(),
                                                           s_scan, ep, et, dsf, dt, aw);
    const double bN = et.v[0] * iW;           // b_N = E_N / W (a_N = 0)

    // ---- fields out, push: electrons (backward), then ions ----
    const bool do_push = n < I.n_xi - 1;
    const bool rec_snap = I.stride > 0 && (n % I.stride) == 0;
    const bool rec_last = n == end - 1;
    auto finish = [&](int s, unsigned sl, unsigned hs, double r, double u, D2 f, double dz, double bt, D2 a2,
                      D2 fp) {
      const double q = s ? 1.0 : -1.0, m = s ? m_ion : 1.0;
      const double qm = q / m, q24 = (q * q) / (4.0 * m * m), qq2 = (q * q) / (2.0 * m * m);
      const double psi = f.x, dpsi = f.y, ez = -dz;
      if (!(isfinite(psi) && isfinite(dpsi) && isfinite(ez) && isfinite(bt))) bad = 1;
      if (rec_snap || rec_last) {
        const unsigned id = (hs & (NT - 1)) * (unsigned)C + hs / NT;      // the ring of home slot hs
        if (rec_snap) {
          WAKE_GLOBAL double* o = gptr(I.snap[s]) + (size_t)(n / I.stride) * OUT_N * N + id;
          o[OUT_PSI * N] = psi; o[OUT_ERBT * N] = -dpsi; o[OUT_EZ * N] = ez; o[OUT_BT * N] = bt;
          o[OUT_RHO * N] = r; o[OUT_UR * N] = u;
        }
        if (rec_last) {
          WAKE_GLOBAL double* o = gptr(I.last[s]) + id;
          o[OUT_PSI * N] = psi; o[OUT_ERBT * N] = -dpsi; o[OUT_EZ * N] = ez; o[OUT_BT * N] = bt;
          o[OUT_RHO * N] = r; o[OUT_UR * N] = u;
        }
      }
      if (do_push) {
        const double pb = 1.0 - qm * psi;
        const double ipb = rcp_nr(pb);
        const double gm = 0.5 * quot(1.0 + u * u + pb * pb + qq2 * a2.x, pb, ipb);   // eq. motion_4
        const double f_r = quot(u, pb, ipb);
        const double f_u = -(qm * (quot(gm * dpsi, pb, ipb) - bt) + quot(q24 * a2.y, pb, ipb));
        double pr = f_r, pu = f_u;
        if (n > 0) { pr = fp.x; pu = fp.y; }
        double rn = r + dxi * (1.5 * f_r - 0.5 * pr);
        double un = u + dxi * (1.5 * f_u - 0.5 * pu);
        double sr_ = f_r, su = f_u;
        if (rn < 0.0) { rn = -rn; un = -un; sr_ = -sr_; su = -su; }
        if (!(isfinite(rn) && isfinite(un))) bad = 1;
        Sn.st((unsigned)(s * IS_N + IS_RU) * S + hs, d2(rn, un));
        Sn.st((unsigned)(s * IS_N + IS_F) * S + hs, d2(sr_, su));
      }
    };
    {
      double ga = G.v[0] * gsa + G.v[1] * gsb, gb = G.v[2] * gsa + G.v[3] * gsb;   // at the chunk end
      double ha = hea, hb = heb;
      double E = ep.v[0] + le, D = dsf.v[0];
      #pragma unroll 1
      for (int k = cnt - 1; k >= 0; --k) {
        const unsigned sl = k * NT + tid;
        const unsigned hs = (unsigned)SID[sl];
        const D2 w = W[IW_W * S + sl], f = W[IW_F * S + sl], As = W[IW_E * S + sl], dc = W[IW_DC * S + sl];
        const double u = W[IW_UC * S + sl].x, bb = Wh[2 * (IW_BB * S + sl)];
        D2 a2 = d2(0.0, 0.0);
        if (has_laser) a2 = W[IW_A2 * S + sl];
        const D2 fp = Sc[(unsigned)IS_F * S + hs];
        const double r = sre[rx(p0 + k)];
        const double ir = rcp_nr(r), r2 = r * r, hAi = 0.5 * As.x * ir, rC = 0.5 * w.x * dc.y;
        const double mg = __builtin_fma(r2, ga, gb), mh = __builtin_fma(r2, ha, hb);
        D = __builtin_fma(As.y, mh, __builtin_fma(-rC, ha, D));   // D_{i-1}
        E = __builtin_fma(As.y, mg, __builtin_fma(-rC, ga, E));   // E_{i-1}
        const double yg = hAi * mg, yh = hAi * mh;
        ga -= yg;
        gb = __builtin_fma(r2, yg, gb);
        ha -= yh;
        hb = __builtin_fma(r2, yh, hb);
        // a_{i-1} rho + b_{i-1} / rho and the ring's own share w^ C / w
        const double bp = ir * __builtin_fma(iW, __builtin_fma(E, mh, -(D * mg)), 0.5 * w.y * dc.y);
        Wh.st(2 * (IW_ZB * S + sl) + 1, bp);
        finish(0, sl, hs, r, u, f, dc.x, bb + bp, a2, fp);
      }
    }
    __syncthreads();
    {
      const double edge_e = s_sc[SC_EDGE];
      const double dza_e = dd_round({s_sc[SC_DZH], s_sc[SC_DZL]});
      #pragma unroll 1
      for (int k = 0; k < cnt; ++k) {
        const unsigned sl = k * NT + tid;
        const unsigned hs = (unsigned)SID[S + sl];
        const int j = JX[S + sl];
        const D2 f = W[wi + IW_F * S + sl];
        const double u = W[wi + IW_UC * S + sl].x, bb = Wh[2 * (wi + IW_BB * S + sl)];
        double dz = Wh[2 * (wi + IW_ZB * S + sl)];
        D2 a2 = d2(0.0, 0.0);
        if (has_laser) a2 = W[wi + IW_A2 * S + sl];
        const D2 fp = Sc[(unsigned)(IS_N + IS_F) * S + hs];
        const double r = sri[rx(p0 + k)];
        double bp;
        if (j >= 0) {
          // the electrons' d_zeta psi and B^(p) between their rings
          D2 zl = W[IW_ZB * S + pslot(max(j - 1, 0), C, div)], zh = W[IW_ZB * S + pslot(min(j, N - 1), C, div)];
          if (j == 0) zl = d2(dza_e, 0.0);
          if (j == N) zh = d2(0.0, bN / edge_e);
          const double t = interval_t(sre, N, edge_e, r, j);
          dz += (1.0 - t) * zl.x + t * zh.x;
          bp = (1.0 - t) * zl.y + t * zh.y;
        } else {
          bp = bN / r;
        }
        finish(1, sl, hs, r, u, f, dz, bb + bp, a2, fp);
      }
    }
    if (tid == 0) {
      const dd pa = dd_add({s_sc[SC_PAH], s_sc[SC_PAL]}, {s_sc[SC_N + SC_PAH], s_sc[SC_N + SC_PAL]});
      const dd za = dd_add({s_sc[SC_DZH], s_sc[SC_DZL]}, {s_sc[SC_N + SC_DZH], s_sc[SC_N + SC_DZL]});
      gptr(I.axis)[2 * n] = dd_round(pa);
      gptr(I.axis)[2 * n + 1] = -dd_round(za);
    }
    if (__syncthreads_or(bad)) {      // breakdown: stop at this slice, its state kept
      if (tid == 0) { I.ctl[CTL_BREAK] = n; I.ctl[CTL_NEXT] = n; I.ctl[CTL_CUR] = cur; }
      break;
    }
    if (do_push) cur ^= 1;
  }
  if (tid == 0) {
    if (n == end) {
      I.ctl[CTL_CUR] = cur;
      I.ctl[CTL_NEXT] = end;
    }
    atomicAdd(I.cnt + CNT_SLICES, (unsigned long long)(n - I.first));
    atomicAdd(I.cnt + CNT_FIXUPS, fixups);
  }
}

// constants (when asked) and the rest state of both species in buffer 0
__global__ void ions_init_kernel(WakeIons J, const double* __restrict__ r0, const double* __restrict__ dr,
                                 const double* __restrict__ dens, int constants) {
  const int N = J.N, C = J.C;
  const size_t S = (size_t)C * NT;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j == 0) {
    J.ctl[CTL_CUR] = 0;
    J.ctl[CTL_BREAK] = -1;
    J.ctl[CTL_NEXT] = 0;
    J.ctl[CTL_FAULT] = 0;
  }
  if (j >= N) return;
  const unsigned hs = pslot(j, C, slot_div(C));
  D2* const cst = reinterpret_cast<D2*>(const_cast<double*>(J.cst));
  if (constants) {
    const double r = r0[j], d = dr[j];
    const double nd = dens ? dens[j] : 1.0;
    const double w = nd * r * d;                  // eq. macroparticle_weight
    const dd lr = dd_log(r);
    cst[IK_W * S + hs] = d2(w, w / 2.0 - nd * d * d / 8.0);   // and the modified self weight
    cst[IK_R0 * S + hs] = d2(r, 1.0 / r);
    cst[IK_LN * S + hs] = d2(lr.hi, lr.lo);
    const_cast<double*>(J.cst)[2 * IK_DR * S + hs] = d;
  }
  const double r = cst[IK_R0 * S + hs].x;
  for (int s = 0; s < 2; ++s) {
    D2* const st = reinterpret_cast<D2*>(J.st[0]) + (size_t)s * IS_N * S;
    st[IS_RU * S + hs] = d2(r, 0.0);
    st[IS_F * S + hs] = d2(0.0, 0.0);
    J.ord[(size_t)s * S + hs] = j;
  }
}

// rest state of both species of instance blockIdx.y in buffer 0 (control
// words reset), from its constants
__global__ void ions_reset_kernel(const WakeIons* __restrict__ insts) {
  const WakeIons& J = insts[blockIdx.y];
  const int N = J.N, C = J.C;
  const size_t S = (size_t)C * NT;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    J.ctl[CTL_CUR] = 0;
    J.ctl[CTL_BREAK] = -1;
    J.ctl[CTL_NEXT] = 0;
    J.ctl[CTL_FAULT] = 0;
  }
  const unsigned div = slot_div(C);
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < N; j += gridDim.x * blockDim.x) {
    const unsigned hs = pslot(j, C, div);
    const double r = reinterpret_cast<const D2*>(J.cst)[IK_R0 * S + hs].x;
    for (int s = 0; s < 2; ++s) {
      D2* const st = reinterpret_cast<D2*>(J.st[0]) + (size_t)s * IS_N * S;
      st[IS_RU * S + hs] = d2(r, 0.0);
      st[IS_F * S + hs] = d2(0.0, 0.0);
      J.ord[(size_t)s * S + hs] = j;
    }
  }
}

__global__ void ions_get_state_kernel(WakeIons J, int sp, double* __restrict__ out) {
  const int N = J.N, C = J.C;
  const size_t S = (size_t)C * NT;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= N) return;
  const unsigned hs = pslot(j, C, slot_div(C));
  const D2* st = reinterpret_cast<const D2*>(J.st[J.ctl[CTL_CUR] & 1]) + (size_t)sp * IS_N * S;
  const D2 a = st[IS_RU * S + hs], f = st[IS_F * S + hs];
  out[j] = a.x;
  out[(size_t)N + j] = a.y;
  out[(size_t)2 * N + j] = f.x;
  out[(size_t)3 * N + j] = f.y;
}

__global__ void ions_set_state_kernel(WakeIons J, int sp, const double* __restrict__ rho,
                                      const double* __restrict__ u, const double* __restrict__ fr,
                                      const double* __restrict__ fu, int slice) {
  const int N = J.N, C = J.C;
  const size_t S = (size_t)C * NT;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int b = J.ctl[CTL_CUR] & 1;
  if (j < N) {
    const unsigned hs = pslot(j, C, slot_div(C));
    D2* st = reinterpret_cast<D2*>(J.st[b]) + (size_t)sp * IS_N * S;
    st[IS_RU * S + hs] = d2(rho[j], u[j]);
    st[IS_F * S + hs] = d2(fr ? fr[j] : 0.0, fu ? fu[j] : 0.0);
    J.ord[(size_t)sp * S + hs] = j;      // order found again at the next slice
  }
  if (j == 0) {
    J.ctl[CTL_BREAK] = -1;
    J.ctl[CTL_NEXT] = slice;
    J.ctl[CTL_FAULT] = 0;
  }
}

}  // namespace

size_t ions_lds_bytes() { return IonsLds::bytes; }

hipError_t launch_ions_init(const WakeIons& J, const double* r0, const double* dr, const double* dens,
                            bool constants, hipStream_t s) {
  const int blocks = (J.N + 255) / 256;
  hipLaunchKernelGGL(ions_init_kernel, dim3(blocks), dim3(256), 0, s, J, r0, dr, dens, constants ? 1 : 0);
  return hipGetLastError();
}

hipError_t ions_prepare() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&ions_march_kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)IonsLds::bytes);
}

hipError_t launch_ions_march(const WakeIons* d_insts, int n_insts, hipStream_t s) {
  hipLaunchKernelGGL(ions_march_kernel, dim3(n_insts), dim3(NT), IonsLds::bytes, s, d_insts);
  return hipGetLastError();
}

hipError_t launch_ions_reset(const WakeIons* d_insts, int n_insts, hipStream_t s) {
  hipLaunchKernelGGL(ions_reset_kernel, dim3(8, n_insts), dim3(256), 0, s, d_insts);
  return hipGetLastError();
}

hipError_t launch_ions_get_state(const WakeIons& J, int sp, double* out, hipStream_t s) {
  hipLaunchKernelGGL(ions_get_state_kernel, dim3((J.N + 255) / 256), dim3(256), 0, s, J, sp, out);
  return hipGetLastError();
}

hipError_t launch_ions_set_state(const WakeIons& J, int sp, const double* rho, const double* u,
                                 const double* fr, const double* fu, int slice, hipStream_t s) {
  hipLaunchKernelGGL(ions_set_state_kernel, dim3((J.N + 255) / 256), dim3(256), 0, s, J, sp, rho, u, fr,
                     fu, slice);
  return hipGetLastError();
}
