// gfx950 slice marcher of the gridless quasistatic plasma-ring solver.
//
// Model (paper, Sec. "Gridless quasistatic model"): axisymmetric electron
// rings (q=-1, m=1) over immobile ions, marched in xi = -zeta.  Per slice:
// radial order (ring id breaks ties), beam/laser sources, the Gauss/log sums
// for psi and d_rho psi (eqs. dpsi_dr, psi), gamma (eq. motion_4), the
// d_zeta psi sum (eq. dpsi_dzeta with the sign obtained by differentiating
// eq. psi), coefficients A, B, C (eqs. b_coeffs_1-3, ponderomotive term with
// the 1/4 and sign of the physical force), the two-point recursion for
// B_theta^(p) (eq. ai_bi, b_0 = 0, a_N = 0) and the Adams-Bashforth-2 push
// (eqs. motion_1-2).
//
// The recursion x_i = M_i x_{i-1} + s_i (x = (a, b), det M_i = 1) is solved
// in Green's-function form: with the growing mode g (g_0 = (1, 0),
// g_i = M_i g_{i-1}), the decaying mode h (h_N = (0, 1), h_{i-1} = M_i^-1
// h_i) and W = det[g, h] = a-part of g_N,
//   x_i = (h_i E_i - g_i D_i) / W,  E_i = sum_{j<=i} det[g_j, s_j],
//                                    D_i = sum_{j>i}  det[s_j, h_j].
// It solves the same linear system as the paper's shooting (Appendix "Solve
// recursive system") without its exponential loss of digits.
//
// One workgroup owns one instance and marches its slices; thread t owns the
// C = ceil(N / NT) consecutive sorted positions [t*C, t*C + C), stored in
// slots k*NT + t (coalesced).  Two passes over the rings per slice:
//   pass B (forward)  psi, d_rho psi from a double-double prefix of
//                     (w, w ln rho); sources; psibar, gamma, A_i, M_i; the
//                     chunk product G of the M_i and the chunk sum of v_i;
//                     lambda = sum_i G_i^T J s_i with G_i the product up to
//                     ring i and J s = (s_b, -s_a), split as lambda0 +
//                     c lambda1 because s_i is affine in the one unknown
//                     c = -(v of this chunk and every later one).
//   scan              prefix of G (g at the chunk start), suffix of (G^-1, v)
//                     (h at the chunk end; v after the chunk, and its total).
//                     The chunk's sums are then det-sums without another pass:
//                     sum det[g_i, s_i] = g_start . lambda,
//                     sum det[s_i, h_i] = -(G^-1 h_end) . lambda.
//   scan              prefix of the det[g, s] sums, suffix of det[s, h].
//   pass E (backward) s_i again, g and h stepped back by M_i^-1, x_{i-1},
//                     B^(p), outputs, AB2 push, ln rho of the pushed radius.
// If the pushed radii are out of order, runs of positions that must be
// permuted among themselves are found (a run boundary sits where every key
// before is below every key after); short runs are ranked in place, the
// rings of long runs are compacted, sorted and dropped into their freed
// positions.
#include "wake_common.h"
#include "wake_device.h"
#include "wake_cluster.h"
#include "wake_ring.h"
#include "wake_launch.h"

#include <math.h>

#include <algorithm>

__device__ __forceinline__ double uni(double x) {
  const uint64_t v = __double_as_longlong(x);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// A record array kept as planes of 16-B chunks: chunk c of record i sits at
// c * ps + i (ps = slots per plane), so a wave's accesses to one chunk are
// contiguous 16-B lanes.  One uniform base per array.
struct PV {
  GA<D2> g;
  uint32_t ps;
  __device__ __forceinline__ D2 ld(uint32_t c, uint32_t i) const { return g[c * ps + i]; }
  __device__ __forceinline__ void st(uint32_t c, uint32_t i, D2 v) const { g.st(c * ps + i, v); }
  // one double of a chunk (half 0: x, 1: y), an 8-B access
  __device__ __forceinline__ double ldh(uint32_t c, uint32_t i, int half) const {
    return *reinterpret_cast<WAKE_GLOBAL double*>(reinterpret_cast<WAKE_GLOBAL char*>(g.p) +
                                                 (c * ps + i) * 16u + half * 8u);
  }
  __device__ __forceinline__ void sth(uint32_t c, uint32_t i, int half, double v) const {
    *reinterpret_cast<WAKE_GLOBAL double*>(reinterpret_cast<WAKE_GLOBAL char*>(g.p) + (c * ps + i) * 16u +
                                          half * 8u) = v;
  }
  // word i of the plane of 4-B words that starts where chunk c would
  __device__ __forceinline__ int32_t ldi(uint32_t c, uint32_t i) const {
    return reinterpret_cast<WAKE_GLOBAL const int32_t*>(g.p)[4u * c * ps + i];
  }
  __device__ __forceinline__ void sti(uint32_t c, uint32_t i, int32_t v) const {
    reinterpret_cast<WAKE_GLOBAL int32_t*>(g.p)[4u * c * ps + i] = v;
  }
};
__device__ __forceinline__ PV pview(const double* p, uint32_t ps) {
  PV v;
  v.g = uview(reinterpret_cast<const D2*>(p));
  v.ps = __builtin_amdgcn_readfirstlane(ps);
  return v;
}
// sort keys of the ring at slot sl of a state buffer
__device__ __forceinline__ double st_rho(const PV& S, unsigned sl) { return S.ldh(RS_RU, sl, 0); }
__device__ __forceinline__ int32_t st_hs(const PV& S, unsigned sl) { return S.ldi(RS_W, sl); }
// the ring's ion-interval hint (instances without the LDS node table)
__device__ __forceinline__ int32_t st_hint(const PV& S, unsigned sl) { return S.ldi(RS_W, S.ps + sl); }

// ln(rho) of the ring with home slot hs as ln r0 + log1p((rho - r0)/r0): its
// rounding scales with the ring's displacement, not with |ln rho| (the psi
// sums multiply ln rho by the enclosed charge).  r: (r0, 1/r0), l: ln r0.
__device__ __forceinline__ dd ring_log(D2 r, D2 l, double rho) {
  const double l1 = log1p_fast((rho - r.x) * r.y);
  return dd_add_d({l.x, l.y}, l1);
}

template <int NT>
__device__ __forceinline__ int32_t id_of(int32_t hs, int C) {
  return (hs & (NT - 1)) * C + (hs >> __builtin_ctz(NT));
}

// slot of position p (member g = p / (C nt) of a cooperative instance uses
// the single-workgroup layout shifted by g C nt; g = 0 otherwise)
__device__ __forceinline__ unsigned slot_of(int p, int C, int nt) {
  const int P = C * nt, g = p / P, q = p - g * P;
  return (unsigned)(g * P + (q % C) * nt + q / C);
}
// position of slot s (the ring id of home slot s)
__device__ __forceinline__ int pos_of_slot(int s, int C, int nt) {
  const int P = C * nt, g = s / P, r = s - g * P;
  return g * P + (r % nt) * C + r / nt;
}

// Ion psi - psi(0) and d_rho psi at radius r: linear interpolation inside
// the node interval containing r (Sec. "Key algorithmic adjustments"),
// searched from the ring's previous interval h; exact exterior field at and
// beyond the plasma edge.
// Ion fields need: the records R, their count N, the plasma edge Rp and the
// exterior constants (sum w ln r0 as dd, Q as dd).
struct IonView {
  GA<double> R;
  int N;
  double Rp;
  dd T0, Q;
};

// The record of the interval a hint points at (loaded ahead of its use).
__device__ __forceinline__ void ion_load(const IonView& V, int h, double* q) {
  const int j = h < 0 ? 0 : (h > V.N ? V.N : h);
#pragma unroll
  for (int i = 0; i < WAKE_ION_REC; ++i) q[i] = V.R[j * WAKE_ION_REC + i];
}

// q: the record ion_load gave for the same hint h.
__device__ __forceinline__ Lerp ion_fields(const IonView& V, double r, dd lnr, int& h, double* q) {
  if (!(r < V.Rp)) {
    const dd ps = dd_sub(V.T0, dd_mul(V.Q, lnr));
    const dd dp = dd_neg(dd_div_d(V.Q, r));
    return {ps.hi, ps.lo, 0.0, dp.hi, dp.lo, 0.0, 0.0};
  }
  const GA<double>& R = V.R;
  const int N = V.N;
  int j = h < 0 ? 0 : (h > N ? N : h);
  if (!(q[IR_LO] <= r && r < q[IR_HI])) {
    if (q[IR_LO] <= r) {
      int a = j + 1, b, step = 1;     // lo(a) <= r
      for (;;) {
        b = a + step;
        if (b > N) { b = N + 1; break; }
        if (r < R[b * WAKE_ION_REC + IR_LO]) break;
        a = b;
        step <<= 1;
      }
      while (b - a > 1) {
        const int m = (a + b) >> 1;
        if (R[m * WAKE_ION_REC + IR_LO] <= r) a = m; else b = m;
      }
      j = a;
    } else {
      int b = j, a, step = 1;           // lo(b) > r
      for (;;) {
        a = b - step;
        if (a <= 0) { a = 0; break; }
        if (R[a * WAKE_ION_REC + IR_LO] <= r) break;
        b = a;
        step <<= 1;
      }
      while (b - a > 1) {
        const int m = (a + b) >> 1;
        if (R[m * WAKE_ION_REC + IR_LO] <= r) a = m; else b = m;
      }
      j = a;
    }
#pragma unroll
    for (int i = 0; i < WAKE_ION_REC; ++i) q[i] = R[j * WAKE_ION_REC + i];
  }
  h = j;
  const double t = (r - q[IR_LO]) * rcp_nr(q[IR_HI] - q[IR_LO]);
  return {q[IR_PSH], q[IR_PSL], q[IR_DPS], q[IR_DPH], q[IR_DPL], q[IR_DDP], t};
}

// Ion interval of radius r from the interval nodes kept in LDS as floats
// (node j = lower end of record j, j = 0..N): the largest j with
// node_j <= r in float, by a gallop from the guess j then bisection.  The
// record's exact double bounds confirm it when it is used (a radius within
// a float ulp of a node can land one interval off; the exact search in
// ion_fields then corrects it).
__device__ __forceinline__ int ion_find(const float* nodes, int N, double r, int j) {
  const float x = (float)r;
  j = j < 0 ? 0 : (j > N ? N : j);
  int a, b;
  // the common case, at most four nodes up from the guess (the interval of
  // the ring before, in radial order), from one round of independent reads:
  // the gallop's smallest answer took four dependent ones of ~65 cycles, in
  // every lane's slowest order.  Past the last node (nodes[N]) come four
  // that compare false.
  const float n0 = nodes[j], n1 = nodes[j + 1], n2 = nodes[j + 2], n3 = nodes[j + 3], n4 = nodes[j + 4];
  if (n0 <= x) {
    const int c = (n1 <= x ? 1 : 0) + (n2 <= x ? 1 : 0) + (n3 <= x ? 1 : 0) + (n4 <= x ? 1 : 0);
    a = j + c;
    if (c < 4) return a;
    int step = 4;                            // nodes[a] <= x
    for (;;) {
      b = a + step;
      if (b > N) { b = N + 1; break; }
      if (x < nodes[b]) break;
      a = b;
      step <<= 1;
    }
  } else {
    b = j;                                   // nodes[b] > x
    int step = 1;
    for (;;) {
      a = b - step;
      if (a <= 0) { a = 0; break; }
      if (nodes[a] <= x) break;
      b = a;
      step <<= 1;
    }
  }
  while (b - a > 1) {
    const int m = (a + b) >> 1;
    if (nodes[m] <= x) a = m; else b = m;
  }
  return a;
}
// The same with a window [w0, w0 + wn) of the nodes in LDS.  From a guess j
// inside it the search ends at the window's edge at most; from one outside it
// looks only for radii inside.  The exact search in ion_fields starts from
// the record of the interval returned.
__device__ __forceinline__ int ion_find_window(const float* nodes, int w0, int wn, double r, int j) {
  int jr = j - w0;
  if (jr < 0 || jr >= wn) {
    const float x = (float)r;
    if (!(nodes[0] <= x && x < nodes[wn - 1])) return j;
    jr = jr < 0 ? 0 : wn - 1;
  }
  return w0 + ion_find(nodes, wn - 1, r, jr);
}
// ---------------------------------------------------------------------------
// ring-set initialisation: weights, ln r0, ion interval records, state
// ---------------------------------------------------------------------------
// Three kernels over the rings' blocks of NT (in ring order), then one
// over the intervals.  Block b's (w, w ln r0) totals go to tmp[4b..4b+3];
// the serial pass turns them into exclusive offsets, in the order a single
// workgroup marching block by block would have summed them.
template <int NT>
__global__ __launch_bounds__(NT) void init_rings_kernel(WakeInst I, const double* __restrict__ r0,
                                                        const double* __restrict__ dr,
                                                        const double* __restrict__ dens, double* tmp) {
  __shared__ double s_scan[(NT / 64) * 8];
  const int N = I.N;
  const int j = blockIdx.x * NT + threadIdx.x;
  D2* cst = reinterpret_cast<D2*>(const_cast<double*>(I.cst));
  D2* st = reinterpret_cast<D2*>(I.st[0]);
  int32_t* st_w = reinterpret_cast<int32_t*>(I.st[0]);
  const size_t PS = (size_t)I.G * I.C * I.nt;      // slots per plane
  const bool ok = j < N;
  double w = 0.0, wh = 0.0, r = 1.0;
  dd lr = {0.0, 0.0};
  if (ok) {
    r = r0[j];
    const double d = dr[j];
    const double nd = dens ? dens[j] : 1.0;
    w = nd * r * d;                              // eq. macroparticle_weight
    wh = w / 2.0 - nd * d * d / 8.0;             // modified weight
    lr = dd_log(r);
    const unsigned hs = slot_of(j, I.C, I.nt);   // home slot of ring j
    cst[RC_W * PS + hs] = d2(w, wh);
    cst[RC_R0 * PS + hs] = d2(r, 1.0 / r);
    cst[RC_LN * PS + hs] = d2(lr.hi, lr.lo);
    // initial state: position j holds ring j; its interval starts at its node
    st[RS_RU * PS + hs] = d2(r, 0.0);
    st[RS_F * PS + hs] = d2(0.0, 0.0);
    st[RS_LN * PS + hs] = d2(lr.hi, lr.lo);
    st_w[4 * RS_W * PS + hs] = (int32_t)hs;
    st_w[4 * RS_W * PS + PS + hs] = j + 1;
  }
  const dd wl = dd_mul_d(lr, w);
  Pack<4> tot;
  block_prefix<NT, 4>(Pack<4>{{w, 0.0, wl.hi, wl.lo}}, Pack<4>{{0, 0, 0, 0}}, DD2Op(), s_scan, tot);
  if (threadIdx.x == 0)
    for (int i = 0; i < 4; ++i) tmp[4 * blockIdx.x + i] = tot.v[i];
}

// One thread: block totals to exclusive offsets, the totals, record 0, control.
__global__ void init_offsets_kernel(WakeInst I, double* tmp, int n_blocks) {
  if (threadIdx.x != 0) return;
  dd cS = {0.0, 0.0}, cPT = {0.0, 0.0};
  for (int b = 0; b < n_blocks; ++b) {
    const dd tS = {tmp[4 * b], tmp[4 * b + 1]}, tPT = {tmp[4 * b + 2], tmp[4 * b + 3]};
    tmp[4 * b] = cS.hi; tmp[4 * b + 1] = cS.lo; tmp[4 * b + 2] = cPT.hi; tmp[4 * b + 3] = cPT.lo;
    cS = dd_add(cS, tS);
    cPT = dd_add(cPT, tPT);
  }
  double* R = const_cast<double*>(I.ion);
  double* consts = const_cast<double*>(I.tot0);
  R[IR_LO] = 0.0;
  R[IR_PSH] = 0.0; R[IR_PSL] = 0.0; R[IR_DPH] = 0.0; R[IR_DPL] = 0.0;
  consts[0] = cPT.hi; consts[1] = cPT.lo;   // sum_j w_j ln r0_j
  consts[2] = cS.hi; consts[3] = cS.lo;     // total weight Q
  I.ctl[CTL_CUR] = 0;
  I.ctl[CTL_BREAK] = -1;
  I.ctl[CTL_NEXT] = 0;
  I.ctl[CTL_FAULT] = 0;
}

// Node values of the ion rings (node j+1 is ring j) into records j+1.
template <int NT>
__global__ __launch_bounds__(NT) void init_nodes_kernel(WakeInst I, const double* __restrict__ tmp) {
  __shared__ double s_scan[(NT / 64) * 8];
  const int N = I.N;
  const int j = blockIdx.x * NT + threadIdx.x;
  const D2* cst = reinterpret_cast<const D2*>(I.cst);
  const size_t PS = (size_t)I.G * I.C * I.nt;
  const bool ok = j < N;
  double w = 0.0, wh = 0.0, r = 1.0;
  dd lr = {0.0, 0.0};
  if (ok) {
    const unsigned hs = slot_of(j, I.C, I.nt);
    const D2 kw = cst[RC_W * PS + hs], kr = cst[RC_R0 * PS + hs], kl = cst[RC_LN * PS + hs];
    w = kw.x; wh = kw.y; r = kr.x; lr = {kl.x, kl.y};
  }
  const dd wl = dd_mul_d(lr, w);
  Pack<4> tot;
  const Pack<4> pre = block_prefix<NT, 4>(Pack<4>{{w, 0.0, wl.hi, wl.lo}}, Pack<4>{{0, 0, 0, 0}},
                                          DD2Op(), s_scan, tot);
  const dd cS = {tmp[4 * blockIdx.x], tmp[4 * blockIdx.x + 1]};
  const dd cPT = {tmp[4 * blockIdx.x + 2], tmp[4 * blockIdx.x + 3]};
  const dd S = dd_add(cS, {pre.v[0], pre.v[1]});
  const dd PTi = dd_add(dd_add(cPT, {pre.v[2], pre.v[3]}), wl);
  if (ok) {
    // ion ring j (q=+1) at its own radius with self weight w^
    const dd dp = dd_neg(dd_div_d(dd_add_d(S, wh), r));
    const dd ps = dd_neg(dd_sub(dd_mul(dd_add_d(S, w), lr), PTi));
    double* rec = const_cast<double*>(I.ion) + (size_t)(j + 1) * WAKE_ION_REC;
    rec[IR_LO] = r;
    rec[IR_PSH] = ps.hi; rec[IR_PSL] = ps.lo;
    rec[IR_DPH] = dp.hi; rec[IR_DPL] = dp.lo;
  }
}

// Interval ends and steps; the last node is the plasma edge.
__global__ void init_intervals_kernel(WakeInst I) {
  const int N = I.N;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j > N) return;
  double* R = const_cast<double*>(I.ion);
  const dd cPT = {I.tot0[0], I.tot0[1]}, cS = {I.tot0[2], I.tot0[3]};
  double* rec = R + (size_t)j * WAKE_ION_REC;
  double hi, nps_h, nps_l, ndp_h, ndp_l;
  if (j < N) {
    const double* nx = rec + WAKE_ION_REC;
    hi = nx[IR_LO]; nps_h = nx[IR_PSH]; nps_l = nx[IR_PSL]; ndp_h = nx[IR_DPH]; ndp_l = nx[IR_DPL];
  } else {
    const double Rp = I.Rp;
    const dd eps = dd_sub(cPT, dd_mul(cS, dd_log(Rp)));
    const dd edp = dd_neg(dd_div_d(cS, Rp));
    hi = Rp; nps_h = eps.hi; nps_l = eps.lo; ndp_h = edp.hi; ndp_l = edp.lo;
  }
  rec[IR_HI] = hi;
  rec[IR_DPS] = dd_round(dd_sub({nps_h, nps_l}, {rec[IR_PSH], rec[IR_PSL]}));
  rec[IR_DDP] = dd_round(dd_sub({ndp_h, ndp_l}, {rec[IR_DPH], rec[IR_DPL]}));
}

// ---------------------------------------------------------------------------
// ring order
// ---------------------------------------------------------------------------
struct MaxKeyOp {   // (rho, id) maximum
  __device__ __forceinline__ Pack<2> operator()(const Pack<2>& a, const Pack<2>& b) const {
    return key_lt(a.v[0], (int32_t)a.v[1], b.v[0], (int32_t)b.v[1]) ? b : a;
  }
};
struct MinKeyOp {   // (rho, id) minimum
  __device__ __forceinline__ Pack<2> operator()(const Pack<2>& a, const Pack<2>& b) const {
    return key_lt(b.v[0], (int32_t)b.v[1], a.v[0], (int32_t)a.v[1]) ? b : a;
  }
};

// Bitonic sort of n keys (rho, id, slot) in place, over P = next power of two
// slots (the caller pads slots [n, P) with +inf keys).
template <int NT>
__device__ void bitonic_keys(double* kr, int32_t* ki, int32_t* ks, int P) {
  for (int size = 2; size <= P; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = threadIdx.x; i < P; i += NT) {
        const int j = i ^ stride;
        if (j > i) {
          const bool up = (i & size) == 0;
          const bool lt = key_lt(kr[j], ki[j], kr[i], ki[i]);
          if (up ? lt : !lt) {
            const double tr = kr[i]; kr[i] = kr[j]; kr[j] = tr;
            const int32_t ti = ki[i]; ki[i] = ki[j]; ki[j] = ti;
            const int32_t ts = ks[i]; ks[i] = ks[j]; ks[j] = ts;
          }
        }
      }
      __syncthreads();
    }
  }
}

// Fallback order of a cooperative instance, by segments.  A segment
// boundary sits before position p when every key before p is below every
// key from p on; the rings between consecutive boundaries are permuted
// among themselves.  Rings alone in their segment keep their positions; the
// others (M of them) are compacted in position order, sorted together by
// member 0 in LDS, and put back into the positions they left, in order (the
// segments follow each other in key order, so the j-th smallest goes to the
// j-th freed position).  Two exchanges of totals and three fenced ones, in
// place of the bitonic network's one per stage, which remains for M beyond
// the LDS sort (cap bytes at byte offset lo, 16 per key).  Returns the
// barrier count, -1 when a member gave up.
template <int NT>
__device__ __noinline__ int cl_segments(const WAKE_GLOBAL WakeInst* Ig, Cluster cl, int xo, int oko, int lo,
                                        int cap) {
  const WakeInst& I = *(const WakeInst*)Ig;
  double* const s_x = reinterpret_cast<double*>(wake_lds + xo);
  int* const s_ok = reinterpret_cast<int*>(wake_lds + oko);
  constexpr int NW = NT / 64;
  double* const s_scanA = reinterpret_cast<double*>(wake_lds);          // the slice scans' areas
  double* const s_scanB = s_scanA + NW * 16;
  const int tid = threadIdx.x;
  const int N = I.N, C = I.C, P = C * NT;
  const double iC = 1.0 / (double)C, iP = 1.0 / (double)P;
  const int goff = cl.g * P;
  const int Ng = min(P, N - goff);
  const int q0 = tid * C;
  const int cnt = max(0, min(C, Ng - q0));
  double* const L_r = reinterpret_cast<double*>(wake_lds + lo);
  uint64_t* const L_k = reinterpret_cast<uint64_t*>(wake_lds + lo + 8 * P);
  WAKE_GLOBAL int32_t* const perm = gptr(I.perm);
  // this member's keys by position, in the current order
  #pragma unroll 1
  for (int k0 = 0; k0 < cnt; k0 += 8) {
    int src[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) src[j] = k0 + j < cnt ? perm[goff + (k0 + j) * NT + tid] : -1;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (src[j] < 0) continue;
      L_r[q0 + k0 + j] = gptr(I.gk_r)[src[j]];
      L_k[q0 + k0 + j] = ((uint64_t)(uint32_t)gptr(I.gk_i)[src[j]] << 32) | (uint32_t)src[j];
    }
  }
  __syncthreads();
  const Pack<2> k_lo = {{-INFINITY, -2147483648.0}}, k_hi = {{INFINITY, 2147483647.0}};
  // suffix minima inside the chunk, its maximum and minimum
  double sr[16];
  int32_t si[16];
  Pack<2> mx = k_lo, mn = k_hi;
#pragma unroll
  for (int k = 15; k >= 0; --k) {
    if (k < cnt) {
      const Pack<2> x = {{L_r[q0 + k], (double)(int32_t)(L_k[q0 + k] >> 32)}};
      mx = MaxKeyOp()(mx, x);
      mn = MinKeyOp()(mn, x);
    }
    sr[k] = mn.v[0];
    si[k] = (int32_t)mn.v[1];
  }
  Pack<2> tmx, tmn;
  const Pack<2> bmx = block_prefix<NT, 2>(mx, k_lo, MaxKeyOp(), s_scanA, tmx);   // before the chunk
  const Pack<2> bmn = block_suffix<NT, 2>(mn, k_hi, MinKeyOp(), s_scanB, tmn);   // after the chunk
  if (!cl_gather<4, false>(cl, Pack<4>{{tmx.v[0], tmx.v[1], tmn.v[0], tmn.v[1]}}, s_x, s_ok)) return -1;
  Pack<2> gmx, gtot, gmn, gtot2;
  cl_prefix<2, 4>(s_x, 0, cl.g, cl.G, k_lo, MaxKeyOp(), gmx, gtot);    // earlier members
  cl_suffix<2, 4>(s_x, 2, cl.g, cl.G, k_hi, MinKeyOp(), gmn, gtot2);   // later members
  // boundary before position q0 + k: max of every key before it below min
  // of every key from it on; a ring is alone in its segment when there are
  // boundaries before it and after it
  const Pack<2> after = MinKeyOp()(bmn, gmn);
  Pack<2> pm = MaxKeyOp()(gmx, bmx);
  const Pack<2> from0 = MinKeyOp()(Pack<2>{{sr[0], (double)si[0]}}, after);   // every key from q0 on
  bool bnd = key_lt(pm.v[0], (int32_t)pm.v[1], from0.v[0], (int32_t)from0.v[1]);
  uint32_t bad = 0;             // bit k: ring at q0 + k moves
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    if (k < cnt) {
      pm = MaxKeyOp()(pm, Pack<2>{{L_r[q0 + k], (double)(int32_t)(L_k[q0 + k] >> 32)}});
      const Pack<2> m = k + 1 < cnt ? Pack<2>{{sr[k + 1], (double)si[k + 1]}} : after;
      const Pack<2> sm = MinKeyOp()(m, after);
      const bool nb = key_lt(pm.v[0], (int32_t)pm.v[1], sm.v[0], (int32_t)sm.v[1]);
      if (!(bnd && nb)) bad |= 1u << k;
      bnd = nb;
    }
  }
  const double nbad = (double)__builtin_popcount(bad);
  Pack<1> tb;
  const Pack<1> ob = block_prefix<NT, 1>(Pack<1>{{nbad}}, Pack<1>{{0.0}}, SumOp<1>(), s_scanA, tb);
  if (!cl_gather<1, false>(cl, tb, s_x, s_ok)) return -1;
  Pack<1> om, mt;
  cl_prefix<1, 1>(s_x, 0, cl.g, cl.G, Pack<1>{{0.0}}, SumOp<1>(), om, mt);
  const int M = (int)mt.v[0];
  int P2 = 1;
  while (P2 < M) P2 <<= 1;
  if (16 * P2 > cap) return cl_bitonic<NT>(Ig, cl, xo, oko);     // every member takes the same branch
  // compaction in position order: key, slot, and the position it leaves
  WAKE_GLOBAL double* const br = gptr(I.bt_r);
  WAKE_GLOBAL int32_t* const bi = gptr(I.bt_i);
  WAKE_GLOBAL int32_t* const bs = gptr(I.bt_s);
  WAKE_GLOBAL int32_t* const fp = gptr(I.sm_i);
  int j = (int)om.v[0] + (int)ob.v[0];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    if (bad & (1u << k)) {
      br[j] = L_r[q0 + k];
      bi[j] = (int32_t)(L_k[q0 + k] >> 32);
      bs[j] = (int32_t)(uint32_t)L_k[q0 + k];
      fp[j] = goff + q0 + k;
      ++j;
    }
  }
  if (!cl_gather<1>(cl, Pack<1>{{0.0}}, s_x, s_ok)) return -1;
  if (cl.g == 0) {
    double* const K_r = L_r;
    int32_t* const K_i = reinterpret_cast<int32_t*>(K_r + P2);
    int32_t* const K_s = K_i + P2;
    for (int i = tid; i < P2; i += NT) {
      K_r[i] = i < M ? br[i] : INFINITY;
      K_i[i] = i < M ? bi[i] : 0x7fffffff;
      K_s[i] = i < M ? bs[i] : -1;
    }
    __syncthreads();
    bitonic_keys<NT>(K_r, K_i, K_s, P2);
    for (int i = tid; i < M; i += NT) bs[i] = K_s[i];
  }
  if (!cl_gather<1>(cl, Pack<1>{{0.0}}, s_x, s_ok)) return -1;
  // the j-th smallest moving ring to the j-th freed position (this member's)
  const int m0 = (int)om.v[0], m1 = m0 + (int)tb.v[0];
  for (int i = m0 + tid; i < m1; i += NT) perm[cl_slot<NT>(fp[i], C, P, iC, iP)] = bs[i];
  return cl_gather<1>(cl, Pack<1>{{0.0}}, s_x, s_ok) ? cl.round : -1;
}

// Sort the M compacted keys in sk[0]: pieces of WAKE_SORTCAP sorted in LDS,
// then pairwise merges by rank (each key's place in the other run found by
// binary search).  Returns the buffer index holding the result.
template <int NT>
__device__ int sort_keys_global(const WakeInst& I, int M, double* kr, int32_t* ki, int32_t* ks) {
  for (int c0 = 0; c0 < M; c0 += WAKE_SORTCAP) {
    const int len = min(WAKE_SORTCAP, M - c0);
    int P = 1;
    while (P < len) P <<= 1;
    for (int i = threadIdx.x; i < P; i += NT) {
      if (i < len) { kr[i] = I.sk_r[0][c0 + i]; ki[i] = I.sk_i[0][c0 + i]; ks[i] = I.sk_s[0][c0 + i]; }
      else { kr[i] = INFINITY; ki[i] = 0x7fffffff - i; ks[i] = -1; }
    }
    __syncthreads();
    bitonic_keys<NT>(kr, ki, ks, P);
    for (int i = threadIdx.x; i < len; i += NT) {
      I.sk_r[0][c0 + i] = kr[i]; I.sk_i[0][c0 + i] = ki[i]; I.sk_s[0][c0 + i] = ks[i];
    }
    __syncthreads();
  }
  int src = 0;
  for (int run = WAKE_SORTCAP; run < M; run <<= 1) {
    const int dst = 1 - src;
    const double* ar = I.sk_r[src];
    const int32_t* ai = I.sk_i[src];
    for (int e = threadIdx.x; e < M; e += NT) {
      const int base = (e / (2 * run)) * (2 * run);
      const int inA = e - base < run;
      const int ob = inA ? base + run : base;                    // the other run
      const int ol = inA ? min(run, max(0, M - ob)) : run;
      const double r = ar[e];
      const int32_t id = ai[e];
      int lo = 0, hi = ol;                                       // other keys below this key
      while (lo < hi) {
        const int m = (lo + hi) >> 1;
        if (key_lt(ar[ob + m], ai[ob + m], r, id)) lo = m + 1; else hi = m;
      }
      const int own = inA ? e - base : e - base - run;
      const int o = base + own + lo;
      I.sk_r[dst][o] = r; I.sk_i[dst][o] = id; I.sk_s[dst][o] = I.sk_s[src][e];
    }
    __syncthreads();
    src = dst;
  }
  return src;
}

// Runs.  A run boundary sits before position p when every key before p is
// below every key from p on; the rings between consecutive boundaries are
// permuted among themselves.  Runs of one ring stay; runs of up to
// WAKE_SEGMAX rings are ranked by counting; the rings of longer runs are
// compacted, sorted together and placed into their freed positions in order
// (each long run keeps its position range, so the j-th smallest goes to the
// j-th freed position).

// Slot form of position p: (p % C) * NT + p / C, with p / C from a
// reciprocal estimate corrected to the exact quotient.
template <int NT>
__device__ __forceinline__ int pos_index(int p, int C, double iC) {
  int q = (int)((double)p * iC);
  if (q * C > p) --q;
  else if ((q + 1) * C <= p) ++q;
  return (p - q * C) * NT + q;
}

struct MaxIntOp {
  __device__ __forceinline__ Pack<1> operator()(const Pack<1>& a, const Pack<1>& b) const {
    return a.v[0] < b.v[0] ? b : a;
  }
};
struct MinIntOp {
  __device__ __forceinline__ Pack<1> operator()(const Pack<1>& a, const Pack<1>& b) const {
    return b.v[0] < a.v[0] ? b : a;
  }
};

// Order fix-up with the keys in global memory (instances with C > CMAX).
// The keys of the ring at position (t, k) are the current buffer's rho and
// id at slot k*NT + t.  Same runs, ranks and long-run sort as the LDS
// version; prefix maxima, boundaries and run starts go through global
// scratch (sm_r/sm_i, flag, cls); the permutation (slot form) is written to
// the global array perm.
template <int NT>
__device__ __noinline__ void fix_order_big(const WakeInst& I, int buf, double* s_scan,
                                           double* s_scan2, unsigned char* region) {
  const int tid = threadIdx.x;
  const int N = I.N, C = I.C;
  const double iC = 1.0 / (double)C;
  const int p0 = tid * C;
  const int cnt = max(0, min(C, N - p0));
  const PV SB = pview(I.st[buf], (uint32_t)(C * NT));
  const GA<double> PMR = uview(I.sm_r);
  const GA<int32_t> PMI = uview(I.sm_i), FL = uview(I.flag), CL = uview(I.cls), PERM = uview(I.perm);
  // chunk extremes; maximum key before each position of the chunk
  Pack<2> mx = {{-INFINITY, -2147483648.0}}, mn = {{INFINITY, 2147483647.0}};
  #pragma unroll 1
  for (int k = 0; k < cnt; ++k) {
    const unsigned sl = k * NT + tid;
    PMR.st(sl, mx.v[0]);
    PMI.st(sl, (int32_t)mx.v[1]);
    const Pack<2> key = {{st_rho(SB, sl), (double)id_of<NT>(st_hs(SB, sl), C)}};
    mx = MaxKeyOp()(mx, key);
    mn = MinKeyOp()(mn, key);
  }
  Pack<2> before, tb, after, ta;
  block_prefix_suffix<NT, 2, 2, MaxKeyOp, MinKeyOp, false>(
      mx, Pack<2>{{-INFINITY, -2147483648.0}}, MaxKeyOp(), mn, Pack<2>{{INFINITY, 2147483647.0}},
      MinKeyOp(), s_scan, before, tb, after, ta);
  // run boundaries, first and last of the chunk
  Pack<2> sm = after;
  int lb = -1, fb = N;
  #pragma unroll 1
  for (int k = cnt - 1; k >= 0; --k) {
    const unsigned sl = k * NT + tid;
    const Pack<2> key = {{st_rho(SB, sl), (double)id_of<NT>(st_hs(SB, sl), C)}};
    sm = MinKeyOp()(sm, key);
    const Pack<2> pm = MaxKeyOp()(before, Pack<2>{{PMR[sl], (double)PMI[sl]}});
    const bool b = (p0 + k == 0) || key_lt(pm.v[0], (int32_t)pm.v[1], sm.v[0], (int32_t)sm.v[1]);
    FL.st(sl, b ? 1 : 0);
    if (b) {
      if (lb < 0) lb = p0 + k;
      fb = p0 + k;
    }
  }
  Pack<1> ain, at_, ein, et_;
  block_prefix_suffix<NT, 1, 1, MaxIntOp, MinIntOp, false>(
      Pack<1>{{(double)lb}}, Pack<1>{{-1.0}}, MaxIntOp(), Pack<1>{{(double)fb}}, Pack<1>{{(double)N}},
      MinIntOp(), s_scan2, ain, at_, ein, et_);
  // run start of each position
  int a = (int)ain.v[0];
  #pragma unroll 1
  for (int k = 0; k < cnt; ++k) {
    const unsigned sl = k * NT + tid;
    if (FL[sl]) a = p0 + k;
    CL.st(sl, a);
  }
  // classify backward (run end = first boundary after the position); short
  // runs ranked here; long-run positions marked -1
  int e = (int)ein.v[0];
  double nlong = 0.0;
  #pragma unroll 1
  for (int k = cnt - 1; k >= 0; --k) {
    const int p = p0 + k;
    const unsigned sl = k * NT + tid;
    const int ra = CL[sl];
    if (e - ra == 1) {
      PERM.st(sl, (int32_t)sl);
    } else if (e - ra <= WAKE_SEGMAX) {
      const double r = st_rho(SB, sl);
      const int32_t id = id_of<NT>(st_hs(SB, sl), C);
      const int qi = pos_index<NT>(ra, C, iC);
      int qk = qi / NT, qt = qi % NT;
      int rank = 0;
      #pragma unroll 1
      for (int q = ra; q < e; q += 4) {
        unsigned x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {      // past the run end: compare with itself
          x[i] = q + i < e ? (unsigned)(qk * NT + qt) : sl;
          if (++qk == C) { qk = 0; ++qt; }
        }
        double xr[4];
        int32_t xh[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) { xr[i] = st_rho(SB, x[i]); xh[i] = st_hs(SB, x[i]); }
#pragma unroll
        for (int i = 0; i < 4; ++i) rank += key_lt(xr[i], id_of<NT>(xh[i], C), r, id) ? 1 : 0;
      }
      PERM.st((unsigned)pos_index<NT>(ra + rank, C, iC), (int32_t)sl);
    } else {
      CL.st(sl, -1);
      nlong += 1.0;
    }
    if (FL[sl]) e = p;
  }
  Pack<1> tot;
  const Pack<1> j0p = block_prefix<NT, 1>(Pack<1>{{nlong}}, Pack<1>{{0.0}}, SumOp<1>(), s_scan, tot);
  const int M = (int)tot.v[0];
  if (M > 0) {
    // rings of the long runs, compacted in position order; their freed
    // positions (slot form) in free_slot
    double* zr = reinterpret_cast<double*>(region);
    int32_t* zi = reinterpret_cast<int32_t*>(zr + WAKE_SORTCAP);
    int32_t* zs = zi + WAKE_SORTCAP;
    const bool in_lds = M <= WAKE_SORTCAP;
    int j = (int)j0p.v[0];
    #pragma unroll 1
    for (int k = 0; k < cnt; ++k) {
      const unsigned sl = k * NT + tid;
      if (CL[sl] != -1) continue;
      I.free_slot[j] = (int32_t)sl;
      const double r = st_rho(SB, sl);
      const int32_t id = id_of<NT>(st_hs(SB, sl), C);
      if (in_lds) { zr[j] = r; zi[j] = id; zs[j] = (int32_t)sl; }
      else { I.sk_r[0][j] = r; I.sk_i[0][j] = id; I.sk_s[0][j] = (int32_t)sl; }
      ++j;
    }
    __syncthreads();
    if (in_lds) {
      int P = 1;
      while (P < M) P <<= 1;
      for (int i = M + tid; i < P; i += NT) { zr[i] = INFINITY; zi[i] = 0x7fffffff - i; zs[i] = -1; }
      __syncthreads();
      bitonic_keys<NT>(zr, zi, zs, P);
      for (int q = tid; q < M; q += NT) PERM.st((unsigned)I.free_slot[q], zs[q]);
    } else {
      const int b = sort_keys_global<NT>(I, M, zr, zi, zs);
      for (int q = tid; q < M; q += NT) PERM.st((unsigned)I.free_slot[q], I.sk_s[b][q]);
    }
  }
  __syncthreads();
}


// Order fix-up in LDS (C <= CMAX).  The keys of the rings at every position
// are in LDS in slot form (position (t, k) of thread t at index k*NT + t):
// kr (radius), ki (id).  Builds perm[k*NT + t] = slot, in the current buffer,
// of the ring at sorted position (t, k).  Nothing in global memory moves.
// Run boundaries come from register prefix maxima, run extents from a scan
// of the first and last boundary of each chunk; short runs are ranked by
// counting, long runs sorted together.
// (rho, id) order of packed keys: k = id << 16 | slot, so that equal radii
// fall back to the ring id.
__device__ __forceinline__ bool pk_lt(double ra, uint32_t ka, double rb, uint32_t kb) {
  return (ra < rb) | ((ra == rb) & (ka < kb));     // no short-circuit: straight-line selects
}

// One wave puts the positions [b0, b0 + 256) (clipped at N) in (rho, id)
// order: four keys per lane, read through the current order perm, written
// back as the new order of these positions.  MERGE: the two halves of the
// block are each in order.  A block already in order is left alone.
template <int NT, bool MERGE>
__device__ __forceinline__ void sort_block_wave(int b0, int N, int C, double iC, const double* kr,
                                                const uint16_t* ki, uint16_t* perm) {
  const int lane = threadIdx.x & 63;
  double r[4];
  uint32_t k[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int p = b0 + wave_place<MERGE>(j);
    r[j] = INFINITY;
    k[j] = ~0u;
    if (p < N) {
      k[j] = perm[pos_index<NT>(p, C, iC)];
      r[j] = kr[k[j]];
    }
  }
  auto id = [&](uint32_t src) { return ki[src]; };
  if (!wave_sort256<MERGE>(r, k, id)) return;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int p = b0 + 4 * lane + j;
    if (p < N) perm[pos_index<NT>(p, C, iC)] = (uint16_t)k[j];
  }
}

// Whether any of bits lo..hi (inclusive, lo <= hi) of a bit array is set.
__device__ __forceinline__ bool bits_any(const uint64_t* m, int lo, int hi) {
  #pragma unroll 1
  for (int w = lo >> 6; w <= (hi >> 6); ++w) {
    uint64_t x = m[w];
    if (w == (hi >> 6) && (hi & 63) < 63) x &= (2ull << (hi & 63)) - 1ull;
    if (w == (lo >> 6)) x &= ~0ull << (lo & 63);
    if (x) return true;
  }
  return false;
}

// Key at position p through the order perm.
template <int NT>
__device__ __forceinline__ void key_at(int p, int C, double iC, const double* kr, const uint16_t* ki,
                                       const uint16_t* perm, double& r, uint32_t& k) {
  const unsigned src = perm[pos_index<NT>(p, C, iC)];
  r = kr[src];
  k = ((uint32_t)ki[src] << 16) | src;
}

// Order fix-up for nearly sorted keys in LDS: blocks of 256 positions sorted
// by single waves, first at offsets 0, 256, 512, ... and then at 128, 384,
// ... (the second phase's blocks are two sorted halves, merged).  If no ring
// is more than 128 positions from its place in the order,
// the two phases leave the whole sequence sorted (with the keys cut at any
// threshold, the mixed zone left by the first phase lies inside one block
// of the second).  Up to two such rounds; returns whether the order is
// complete (else the caller runs the general fix-up).
//
// dmask: the push's disorder flags, bit t set if thread t's chunk had a pair
// of positions out of order (inside it, or its last position against the
// next chunk's first).  The first round sorts only the blocks of the first
// phase whose chunks flagged disorder (the others are in order), the second
// all of them.  Of the second phase's blocks those over a junction of the
// first phase's left out of order are merged, and the order is checked at
// the second phase's junctions alone: every segment between them is sorted,
// so the sequence is in order when they are.
template <int NT>
__device__ __noinline__ bool fix_order_blocks(const WakeInst& I, const double* kr, const uint16_t* ki,
                                              uint16_t* perm, const uint64_t* dmask) {
  constexpr int NW = NT / 64;
  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63;
  const int N = I.N, C = I.C;
  const double iC = 1.0 / (double)C;
  const int cnt = max(0, min(C, N - tid * C));
  for (int k = 0; k < cnt; ++k) perm[k * NT + tid] = (uint16_t)(k * NT + tid);
  __syncthreads();
  // The callers are compiled knowing which registers this function leaves
  // alone, and keep values there across the call; every slice of the march
  // then pays for the spills that brings, a fix-up or not.  So it claims the
  // scalar registers it does not use.  With this compiler, without the claim and
  // with it: 96 rings 7.6 and 7.25 us per slice, 1000 rings 11.97 and 11.7, 1500
  // 20.1 and 20.05; 7900 rings 80.2 and 81.2, the batch of 512 95.8 and 96.2 ms.
  asm volatile("" ::: "s74", "s75", "s76", "s77", "s78", "s79", "s80", "s81", "s82", "s83", "s84", "s85", "s86",
                      "s87", "s88", "s89", "s90", "s91", "s92", "s93", "s94", "s95", "s96", "s97", "s98", "s99",
                      "s100", "s101");
  // whether the positions before and after junction q are out of order
  auto out = [&](int q) {
    if (q >= N) return false;
    double ra, rb;
    uint32_t ka, kb;
    key_at<NT>(q - 1, C, iC, kr, ki, perm, ra, ka);
    key_at<NT>(q, C, iC, kr, ki, perm, rb, kb);
    return pk_lt(rb, kb, ra, ka);
  };
  #pragma unroll 1
  for (int round = 0; round < 2; ++round) {
    // the first phase's blocks, one per lane
    const int b0 = lane << 8;
    uint64_t bm = __ballot(b0 < N && (round > 0 || bits_any(dmask, b0 / C, min((b0 + 255) / C, NT - 1))));
    int seen = 0;
    #pragma unroll 1
    while (bm) {
      const int b = __builtin_ctzll(bm);
      bm &= bm - 1;
      if (seen++ % NW == wave) sort_block_wave<NT, false>(b * 256, N, C, iC, kr, ki, perm);
    }
    __syncthreads();
    uint64_t jm = __ballot(out(256 * (lane + 1)));     // its junctions, one per lane
    // a merge moves the keys at its junction: the barrier lets every wave read
    // them first, so that all have the same list (7900 rings 80.3 -> 81.2 us per
    // slice, the others unchanged)
    __syncthreads();
    seen = 0;
    #pragma unroll 1
    while (jm) {
      const int b = __builtin_ctzll(jm);
      jm &= jm - 1;
      if (seen++ % NW == wave) sort_block_wave<NT, true>(128 + b * 256, N, C, iC, kr, ki, perm);
    }
    __syncthreads();
    // the same keys in every wave: a uniform answer
    if (!__ballot(out(128 + 256 * lane))) return true;
    __syncthreads();                      // every wave has read the keys before a block moves
  }
  return false;
}

template <int NT, int CMAX>
__device__ __noinline__ void fix_order_lds(const WakeInst& I, double* s_scan, double* s_scan2,
                                           unsigned char* region, const double* kr,
                                           const uint16_t* ki, uint16_t* zf, uint16_t* perm) {
  const int tid = threadIdx.x;
  const int N = I.N, C = I.C;
  const double iC = 1.0 / (double)C;
  const int p0 = tid * C;
  const int cnt = max(0, min(C, N - p0));
  Pack<2> mx = {{-INFINITY, -2147483648.0}}, mn = {{INFINITY, 2147483647.0}};
  double pr[CMAX > 0 ? CMAX : 1];
  int32_t pi[CMAX > 0 ? CMAX : 1];      // maximum key before each position of the chunk
#pragma unroll
  for (int k = 0; k < CMAX; ++k) {
    if (k < cnt) {
      pr[k] = mx.v[0];
      pi[k] = (int32_t)mx.v[1];
      const Pack<2> key = {{kr[k * NT + tid], (double)ki[k * NT + tid]}};
      mx = MaxKeyOp()(mx, key);
      mn = MinKeyOp()(mn, key);
    }
  }
  Pack<2> before, tb, after, ta;
  block_prefix_suffix<NT, 2, 2, MaxKeyOp, MinKeyOp, false>(
      mx, Pack<2>{{-INFINITY, -2147483648.0}}, MaxKeyOp(), mn, Pack<2>{{INFINITY, 2147483647.0}},
      MinKeyOp(), s_scan, before, tb, after, ta);
  // run boundaries of the chunk (bit k: boundary before position p0 + k)
  Pack<2> sm = after;
  unsigned bits = 0;
#pragma unroll
  for (int k = CMAX - 1; k >= 0; --k) {
    if (k < cnt) {
      const Pack<2> key = {{kr[k * NT + tid], (double)ki[k * NT + tid]}};
      sm = MinKeyOp()(sm, key);
      const Pack<2> pm = MaxKeyOp()(before, Pack<2>{{pr[k], (double)pi[k]}});
      const bool b = (p0 + k == 0) || key_lt(pm.v[0], (int32_t)pm.v[1], sm.v[0], (int32_t)sm.v[1]);
      bits |= (unsigned)b << k;
    }
  }
  // last boundary at or before each chunk, first one after it
  const double lb = bits ? (double)(p0 + 31 - __builtin_clz(bits)) : -1.0;
  const double fb = bits ? (double)(p0 + __builtin_ctz(bits)) : (double)N;
  Pack<1> ain, at_, ein, et_;
  block_prefix_suffix<NT, 1, 1, MaxIntOp, MinIntOp, false>(
      Pack<1>{{lb}}, Pack<1>{{-1.0}}, MaxIntOp(), Pack<1>{{fb}}, Pack<1>{{(double)N}}, MinIntOp(),
      s_scan2, ain, at_, ein, et_);
  // classify; rings of short runs placed here
  unsigned lng = 0;
  double nlong = 0.0;
  #pragma unroll 1
  for (int k = 0; k < cnt; ++k) {
    const int p = p0 + k;
    const unsigned own = (unsigned)(k * NT + tid);
    const unsigned below = bits & ((2u << k) - 1u);           // boundaries at or before p
    const unsigned above = bits & ~((2u << k) - 1u);          // boundaries after p
    const int a = below ? p0 + 31 - __builtin_clz(below) : (int)ain.v[0];
    const int e = above ? p0 + __builtin_ctz(above) : (int)ein.v[0];
    if (e - a == 1) { perm[own] = (uint16_t)own; continue; }
    if (e - a <= WAKE_SEGMAX) {
      const double r = kr[own];
      const int32_t id = ki[own];
      int qi = pos_index<NT>(a, C, iC);
      int qk = qi / NT, qt = qi % NT;                          // NT is a power of two
      int rank = 0;
      #pragma unroll 1
      for (int q = a; q < e; q += 4) {
        int x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {       // past the run end: compare with itself
          x[i] = q + i < e ? qk * NT + qt : (int)own;
          if (++qk == C) { qk = 0; ++qt; }
        }
        double xr[4];
        int32_t xi[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) { xr[i] = kr[x[i]]; xi[i] = ki[x[i]]; }
#pragma unroll
        for (int i = 0; i < 4; ++i) rank += key_lt(xr[i], xi[i], r, id) ? 1 : 0;
      }
      perm[pos_index<NT>(a + rank, C, iC)] = (uint16_t)own;
    } else {
      lng |= 1u << k;
      nlong += 1.0;
    }
  }
  Pack<1> tot;
  const Pack<1> j0p = block_prefix<NT, 1>(Pack<1>{{nlong}}, Pack<1>{{0.0}}, SumOp<1>(), s_scan, tot);
  const int M = (int)tot.v[0];
  if (M > 0) {
    // rings of the long runs, compacted in position order; sorted keys in
    // zr/zi/zs (slots), their freed positions in zf (LDS index form)
    double* zr = reinterpret_cast<double*>(region);
    int32_t* zi = reinterpret_cast<int32_t*>(zr + WAKE_SORTCAP);
    int32_t* zs = zi + WAKE_SORTCAP;
    const bool in_lds = M <= WAKE_SORTCAP;
    int j = (int)j0p.v[0];
    #pragma unroll 1
    for (int k = 0; k < cnt; ++k) {
      if (!((lng >> k) & 1u)) continue;
      const int own = k * NT + tid;
      if (in_lds) { zf[j] = (uint16_t)own; zr[j] = kr[own]; zi[j] = ki[own]; zs[j] = own; }
      else { I.free_slot[j] = own; I.sk_r[0][j] = kr[own]; I.sk_i[0][j] = ki[own]; I.sk_s[0][j] = own; }
      ++j;
    }
    __syncthreads();
    if (in_lds) {
      int P = 1;
      while (P < M) P <<= 1;
      for (int i = M + tid; i < P; i += NT) { zr[i] = INFINITY; zi[i] = 0x7fffffff - i; zs[i] = -1; }
      __syncthreads();
      bitonic_keys<NT>(zr, zi, zs, P);
      for (int q = tid; q < M; q += NT) perm[zf[q]] = (uint16_t)zs[q];
    } else {
      const int b = sort_keys_global<NT>(I, M, zr, zi, zs);
      for (int q = tid; q < M; q += NT) perm[I.free_slot[q]] = (uint16_t)I.sk_s[b][q];
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// the slice marcher
// ---------------------------------------------------------------------------
struct BwdMatSumOp {  // (index-order product of inverse transfers, running sum)
  __device__ __forceinline__ Pack<5> operator()(const Pack<5>& lo, const Pack<5>& hi) const {
    Pack<4> m = mat_mul({{lo.v[0], lo.v[1], lo.v[2], lo.v[3]}}, {{hi.v[0], hi.v[1], hi.v[2], hi.v[3]}});
    return {{m.v[0], m.v[1], m.v[2], m.v[3], lo.v[4] + hi.v[4]}};
  }
};
// Cooperative instances: the transfer products and the source det-sums of
// all members from one exchange.  Member m publishes (G_m, V_m), its
// transfer product and v-sum, and four vectors summed
// over its chunks: A = sum Gl^T mu, B = sum Gl^T l1, A' = sum K^T mu,
// B' = sum K^T l1 (Gl: the member's transfers before the chunk; K = adj(G)
// Hl with G the chunk's product and Hl the member's inverse transfers after
// it; l1: the part of the chunk's lambda that multiplies c; mu = lambda0 -
// (v of the chunk and of the member's later chunks) l1).  With gin the
// growing mode entering member m, hin the decaying mode leaving it and Vm
// the v-sum of the members after it, the member's sums of det[g_i, s_i] and
// det[s_i, h_i] are gin.A - Vm gin.B and -hin.A' + Vm hin.B'.  Every member
// forms from the gathered packs (NFT doubles each) its exclusive prefix pg
// and suffix sg of the transfers (inverse transfers from the adjugates of
// the published products, det = 1), their totals, and the det-sums of the
// members before it (e_in) and after it (d_in).  Lane l of a wave takes
// members MPL l .. MPL l + MPL-1 (G <= 64 MPL).  One wave goes forward and
// another backward, each on a SIMD of its own, and they leave their results
// in LDS (every wave doing both took 1.7 us at 40 members, 3.8 at 196).
//
// Forward: out[0..3] = pg, out[4] = e_in, out[5..8] = the total.
template <int NFT, int MPL>
__device__ __forceinline__ void cl_transfer_fwd(const double* s_x, int g, int G, double* out) {
  const int lane = threadIdx.x & 63;
  const FwdMatOp fop;
  auto fwd_of = [&](int m) {
    const double* q = s_x + m * NFT;
    return Pack<4>{{q[0], q[1], q[2], q[3]}};
  };
  Pack<4> bf = mat_ident();
  double bv = 0.0;
#pragma unroll
  for (int j = 0; j < MPL; ++j)
    if (MPL * lane + j < G) {
      bf = fop(bf, fwd_of(MPL * lane + j));
      bv += s_x[(MPL * lane + j) * NFT + 4];
    }
  const Pack<4> inc = wave_prefix_incl(bf, fop);
  const Pack<1> incV = wave_suffix_incl(Pack<1>{{bv}}, SumOp<1>());
  Pack<4> x;                            // the members before this lane's
#pragma unroll
  for (int i = 0; i < 4; ++i) x.v[i] = lane_prev(inc.v[i]);
  double V = lane_next(incV.v[0]);      // v after them
  if (lane == 0) x = mat_ident();
  if (lane == 63) V = 0.0;
  double vm[MPL], etm[MPL];
#pragma unroll
  for (int j = MPL - 1; j >= 0; --j) {
    const int m = MPL * lane + j;
    vm[j] = V;
    if (m < G) V += s_x[m * NFT + 4];
  }
  Pack<4> pg = mat_ident();
#pragma unroll
  for (int j = 0; j < MPL; ++j) {
    const int m = MPL * lane + j;
    etm[j] = 0.0;
    if (m < G) {
      const double* q = s_x + m * NFT;
      const double g0 = x.v[0], g1 = x.v[2];
      etm[j] = (g0 * q[5] + g1 * q[6]) - vm[j] * (g0 * q[7] + g1 * q[8]);
      if (m == g) pg = x;
      x = fop(x, fwd_of(m));
    }
  }
  static_assert(MPL == 1 || MPL == 4, "one or four members per lane");
  double esum = etm[0];
  if constexpr (MPL == 4) esum = (etm[0] + etm[1]) + (etm[2] + etm[3]);
  const Pack<1> eI = wave_prefix_incl(Pack<1>{{esum}}, SumOp<1>());
  double e_own = lane_prev(eI.v[0]);
  if (lane == 0) e_own = 0.0;
  const int jg = g % MPL;
#pragma unroll
  for (int j = 0; j < MPL; ++j)
    if (j < jg) e_own += etm[j];
  if (lane == g / MPL) {
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = pg.v[i];
    out[4] = e_own;
  }
  if (lane == 63) {
#pragma unroll
    for (int i = 0; i < 4; ++i) out[5 + i] = inc.v[i];
  }
}
// Backward: out[0..4] = sg (with the v-sum), out[5] = d_in, out[6..10] = the
// total.
template <int NFT, class BOp, int MPL>
__device__ __forceinline__ void cl_transfer_bwd(const double* s_x, int g, int G, double* out) {
  const int lane = threadIdx.x & 63;
  const Pack<5> I5 = {{1.0, 0.0, 0.0, 1.0, 0.0}};
  const BOp bop;
  auto bwd_of = [&](int m) {
    const double* q = s_x + m * NFT;
    return Pack<5>{{q[3], -q[1], -q[2], q[0], q[4]}};
  };
  Pack<5> bb = I5;
#pragma unroll
  for (int j = MPL - 1; j >= 0; --j)
    if (MPL * lane + j < G) bb = bop(bwd_of(MPL * lane + j), bb);
  const Pack<5> inc = wave_suffix_incl(bb, bop);
  Pack<5> x;                            // the members after this lane's
#pragma unroll
  for (int i = 0; i < 5; ++i) x.v[i] = lane_next(inc.v[i]);
  if (lane == 63) x = I5;
  double dtm[MPL];
  Pack<5> sg = I5;
#pragma unroll
  for (int j = MPL - 1; j >= 0; --j) {
    const int m = MPL * lane + j;
    dtm[j] = 0.0;
    if (m < G) {
      const double* q = s_x + m * NFT;
      const double h0 = x.v[1], h1 = x.v[3];
      dtm[j] = -(h0 * q[9] + h1 * q[10]) + x.v[4] * (h0 * q[11] + h1 * q[12]);
      if (m == g) sg = x;
      x = bop(bwd_of(m), x);
    }
  }
  double dsum = dtm[0];
  if constexpr (MPL == 4) dsum = (dtm[0] + dtm[1]) + (dtm[2] + dtm[3]);
  const Pack<1> dI = wave_suffix_incl(Pack<1>{{dsum}}, SumOp<1>());
  double d_own = lane_next(dI.v[0]);
  if (lane == 63) d_own = 0.0;
  const int jg = g % MPL;
#pragma unroll
  for (int j = 0; j < MPL; ++j)
    if (j > jg) d_own += dtm[j];
  if (lane == g / MPL) {
#pragma unroll
    for (int i = 0; i < 5; ++i) out[i] = sg.v[i];
    out[5] = d_own;
  }
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < 5; ++i) out[6 + i] = inc.v[i];
  }
}

template <int NT>
struct MarchLds {
  static constexpr int NW = NT / 64;
  // rings per thread up to which the keys of every position live in LDS
  static constexpr int CMAX = 16;
  static constexpr int KCAP = NT * CMAX;
  static constexpr size_t region_bytes() {
    const size_t beam = 2 * WAKE_BCAP * sizeof(double);
    const size_t sort = WAKE_SORTCAP * (sizeof(double) + 2 * sizeof(int32_t));
    return beam > sort ? beam : sort;
  }
  // two scan areas, analytic constants, first keys of the chunks
  static constexpr size_t head_bytes() {
    return sizeof(double) * (2 * NW * 16 + 64 + NT) + sizeof(int32_t) * NT;
  }
  // per position (slot form): key radius, key id, slot of the ring
  // (permutation); freed positions of long runs
  static constexpr size_t key_bytes() {
    return (size_t)KCAP * (sizeof(double) + 2 * sizeof(uint16_t)) +
           (size_t)WAKE_SORTCAP * sizeof(uint16_t);
  }
  // ion interval nodes as floats (instances with keys in LDS: N <= KCAP)
  // and four past them
  static constexpr size_t ion_bytes() { return ((size_t)(KCAP + 5) * sizeof(float) + 15) & ~(size_t)15; }
  static constexpr size_t bytes() { return head_bytes() + key_bytes() + region_bytes() + ion_bytes(); }
};
// one workgroup's LDS must fit the 160 KiB of a compute unit
static_assert(MarchLds<256>::bytes() <= 160 * 1024, "LDS layout too large");
static_assert(MarchLds<512>::bytes() <= 160 * 1024, "LDS layout too large");
// the block fix-up checks one junction of 256-position blocks per lane
static_assert(MarchLds<256>::KCAP <= 64 * 256 && MarchLds<512>::KCAP <= 64 * 256, "junctions per lane");
// a cooperative member gathers the packs of every member into its key area
static_assert(MarchLds<256>::key_bytes() >= WAKE_CL_GMAX * 16 * sizeof(double), "pack area");
// field-grid variant: the LDS left beside the layout holds the node records
// of grids up to grid_lds_nodes nodes (else they are read from device memory)
template <int NT>
constexpr int grid_lds_nodes() {
  return (int)((160 * 1024 - MarchLds<NT>::bytes() - 512) / (WAKE_GRID_TAB * sizeof(double)));
}
template <int NT>
constexpr size_t grid_lds_bytes() {
  return (size_t)grid_lds_nodes<NT>() * WAKE_GRID_TAB * sizeof(double);
}

// This slice's analytic source factors (beams: lam += c0 (1 - exp(-rho^2 c1));
// lasers: |a|^2 = c0 exp(-rho^2 c1)) and beam-table entries into LDS.
template <int NT>
__device__ __forceinline__ void stage_analytic(const WakeInst& I, int n, double* s_misc) {
  const int tid = threadIdx.x;
  const double xi = n * I.dxi;
  if (tid < I.n_an) {
    const WAKE_GLOBAL WakeAnalytic& A = gptr(I.an)[tid];
    if (A.kind == 2) {
      const double s2 = A.sigma_r * A.sigma_r;
      const double dl = xi - A.xi_c;
      const double lon = exp(-(dl * dl) / (2.0 * A.sigma_xi * A.sigma_xi));
      s_misc[3 * tid] = 2.0;
      s_misc[3 * tid + 1] = A.q * A.n_peak * lon * s2;
      s_misc[3 * tid + 2] = 1.0 / (2.0 * s2);
    } else {
      const double dl = xi - A.xi_l;
      const double lon = exp(-2.0 * dl * dl / (A.L * A.L));
      s_misc[3 * tid] = 3.0;
      s_misc[3 * tid + 1] = A.a0 * A.a0 * lon;
      s_misc[3 * tid + 2] = 2.0 / (A.w0 * A.w0);
    }
  }
}
template <int NT>
__device__ __forceinline__ void stage_slice(const WakeInst& I, int n, double* s_misc, double* s_br,
                                            double* s_bc) {
  const int tid = threadIdx.x;
  stage_analytic<NT>(I, n, s_misc);
  if (I.nb) {
    const int bt0 = __builtin_amdgcn_readfirstlane(gptr(I.boff)[n]);
    const int bm = __builtin_amdgcn_readfirstlane(gptr(I.boff)[n + 1]) - bt0;
    const WAKE_GLOBAL double* br = gptr(I.br) + bt0;
    const WAKE_GLOBAL double* bc = gptr(I.bcum) + bt0;
    if (bm <= WAKE_BCAP)
      for (int i = tid; i < bm; i += NT) { s_br[i] = br[i]; s_bc[i] = bc[i]; }
  }
}

// The beam-table entries of a slice that one thread stages in LDS, fetched
// into registers ahead of the store (the fetch for slice n+1 is issued when
// pass E of slice n starts, the store follows the pass).
template <int NT>
struct BeamStage {
  static constexpr int BPT = (WAKE_BCAP + NT - 1) / NT;
  double r[BPT], c[BPT];
  int m;                 // entries of the slice; more than WAKE_BCAP: read from global memory
};
template <int NT>
__device__ __forceinline__ void beam_fetch(const WakeInst& I, int n, BeamStage<NT>& b) {
  b.m = 0;
  if (!I.nb) return;
  const int bt0 = __builtin_amdgcn_readfirstlane(gptr(I.boff)[n]);
  b.m = __builtin_amdgcn_readfirstlane(gptr(I.boff)[n + 1]) - bt0;
  if (b.m > WAKE_BCAP) return;
  const WAKE_GLOBAL double* br = gptr(I.br) + bt0;
  const WAKE_GLOBAL double* bc = gptr(I.bcum) + bt0;
#pragma unroll
  for (int q = 0; q < BeamStage<NT>::BPT; ++q) {
    const int i = threadIdx.x + q * NT;
    b.r[q] = 0.0;
    b.c[q] = 0.0;
    if (i < b.m) { b.r[q] = br[i]; b.c[q] = bc[i]; }
  }
}
template <int NT>
__device__ __forceinline__ void beam_store(const BeamStage<NT>& b, double* s_br, double* s_bc) {
  if (b.m > WAKE_BCAP) return;
#pragma unroll
  for (int q = 0; q < BeamStage<NT>::BPT; ++q) {
    const int i = threadIdx.x + q * NT;
    if (i < b.m) { s_br[i] = b.r[q]; s_bc[i] = b.c[q]; }
  }
}

// Per-thread sums of (w, w ln rho) over the rings at this thread's
// positions (ln rho of each ring taken from its slot).  Eight rings at a
// time: their slots and home slots (from the ring ids in LDS when the order
// is there, else from the home-slot words), then (w, w^) and ln rho, so each
// batch costs one round of independent loads (two without the LDS ids).
template <int NT>
__device__ __forceinline__ void chunk_sums(const WakeInst& I, int cur, int cnt, int goff, uint32_t ps,
                                           bool ident, bool lds_perm, const uint16_t* perm,
                                           const uint16_t* ki, dd& sw, dd& swl) {
  const int tid = threadIdx.x;
  const int C = I.C;
  const double iC = 1.0 / (double)C;
  const unsigned smax = ps - 1;
  const PV SC = pview(I.st[cur], ps), KC = pview(I.cst, ps);
  sw = {0.0, 0.0};
  swl = {0.0, 0.0};
  #pragma unroll 1
  for (int k0 = 0; k0 < cnt; k0 += 8) {
    unsigned s[8], hs[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const unsigned sl = (k0 + j) * NT + tid;
      s[j] = 0;
      hs[j] = 0;
      if (k0 + j < cnt) {
        s[j] = ident ? goff + sl : min(lds_perm ? (unsigned)perm[sl] : (unsigned)gptr(I.perm)[goff + sl], smax);
        hs[j] = lds_perm ? (unsigned)pos_index<NT>(ki[s[j]], C, iC) : (unsigned)st_hs(SC, s[j]);
      }
    }
    double w[8];
    D2 l[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      w[j] = k0 + j < cnt ? KC.ldh(RC_W, hs[j], 0) : 0.0;
      l[j] = k0 + j < cnt ? SC.ld(RS_LN, s[j]) : d2(0.0, 0.0);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (k0 + j < cnt) {
        sw = dd_add_d(sw, w[j]);
        swl = dd_add_fast(swl, dd_mul_d(dd{l[j].x, l[j].y}, w[j]));
      }
    }
  }
}

// CL: member `member` of a cooperative instance (I.G workgroups); its
// positions and slots start at goff = member * C * NT, and the slice scans
// and the order fix-up span all members.
// ---------------------------------------------------------------------------
// radial field grid (Fig. 2: fields on an external grid): the ring solve's
// sums evaluated at the uniform nodes r_g = (g + 1/2) dg, g < ng.  A node in
// (rho_{p-1}, rho_p] lies in interval p of the recursion: below it the
// rings before position p, at and above it the rest.
// ---------------------------------------------------------------------------
// Radius of node g: rad[g] for explicit nodes, else (g + 1/2) dg.
__device__ __forceinline__ double grid_node_r(int g, double dg, const WAKE_GLOBAL double* rad) {
  return rad ? rad[g] : ((double)g + 0.5) * dg;
}

// The largest node g with r_g <= x (-1 if none), decided on the node radii
// themselves so that neighbouring intervals split the nodes exactly
// (explicit radii: a binary search; uniform nodes: a guess corrected on the
// radii).
__device__ __forceinline__ int grid_last_below(double x, double dg, double idg, int ng,
                                               const WAKE_GLOBAL double* rad) {
  if (rad) {
    int a = 0, b = ng;                         // nodes at or below x: [0, a)
    while (a < b) {
      const int m = (a + b) >> 1;
      if (rad[m] <= x) a = m + 1; else b = m;
    }
    return a - 1;
  }
  if (!(x >= 0.5 * dg)) return -1;
  const double t = floor(x * idg - 0.5);      // a guess; the node radii decide
  int g = t >= (double)(ng - 1) ? ng - 1 : (int)t;
  if (g < -1) g = -1;
  while (g + 1 < ng && ((double)(g + 1) + 0.5) * dg <= x) ++g;
  while (g >= 0 && ((double)g + 0.5) * dg > x) --g;
  return g;
}

// Per-node hand-over scratch of a slice: 6 chunks of two doubles per node:
// [0] sum of w below, [1] sum of w ln rho below (pass B); [2] (E_z sum at
// and above, a), [3] (b, owner thread) (pass E); [4], [5] the owner's
// partial sums at and above the node of c = w / psibar and c rho (double-
// double; the chi deposit).
constexpr int GS = 6;

// The nodes a slice hands over in pass E: nr real nodes (uniform or explicit
// radii) and, when chi is deposited, one virtual node above the last, at
// r_{nr-1} + (r_{nr-1} - r_{nr-2}) (2 r_0 for a single node), where the last
// node's hat ends.
struct GridNodes {
  const WAKE_GLOBAL double* rad;
  double dg, idg, top;
  int nr, nh;
  __device__ __forceinline__ double r(int g) const { return g < nr ? grid_node_r(g, dg, rad) : top; }
  __device__ __forceinline__ int last_below(double x) const {
    int g = grid_last_below(x, dg, idg, nr, rad);
    if (g == nr - 1 && nh > nr && top <= x) g = nr;
    return g;
  }
};

// psi (eq. psi) and E_r - B_theta = -d_rho psi (eq. dpsi_dr, no ring at r)
// at node g (radius r) of an interval with the sums S, P of weight and
// w ln rho below it.  t0, t1, t2: the node's record (ln r and the immobile
// ions' psi - psi(0) and d_rho psi there, dd pairs, fixed for the solve);
// out: the slice's [4][ng] block.
__device__ __forceinline__ void grid_node_psi(WAKE_GLOBAL double* out, int ng, int g, double r, D2 t0,
                                              D2 t1, D2 t2, dd S, dd P, double psi_axis) {
  const dd pe = dd_add_fast(dd_mul(S, dd{t0.x, t0.y}), dd_neg(P));
  const dd de = dd_div_rcp(S, r, rcp_nr(r));
  out[g] = dd_round(dd_add_fast(pe, dd{t1.x, t1.y})) + psi_axis;
  out[ng + g] = -dd_round(dd_add_fast(de, dd{t2.x, t2.y}));
}

// E_z (eq. dpsi_dzeta: the rings at and above the interval) and
// B_theta = B^(b) + a r + b/r (eq. b_theta_plasma) at node g.
__device__ __forceinline__ void grid_node_b(WAKE_GLOBAL double* out, int ng, int g, double r, double ez,
                                            double a, double b, double bb) {
  const double ir = rcp_nr(r);
  out[2 * ng + g] = ez;
  out[3 * ng + g] = bb + (a * r + b * ir);
}

// chi = n/gamma (reading R20) at the nodes g0, g0 + NT, ... below g1 of a
// slice: a node's full sums D, E of c = w / psibar and c rho at and above it
// are its owner's partial sums plus the owner's later chunks (thr) and, on a
// cooperative instance, the later members (msuf, in LDS); the hats' sums are
// differences of neighbouring nodes' full sums (the virtual node past the
// last included), over the hats' volumes.  all0: the sum of c over every
// ring.  Not inlined: its temporaries stay out of the march's registers.
template <int NT, bool CL>
__device__ __noinline__ void chi_nodes(WAKE_GLOBAL double* gout, int ngB, const WAKE_GLOBAL D2* gscr,
                                       const WAKE_GLOBAL double* thr, const double* msuf, int n_thr,
                                       GridNodes GN, int g0, int g1, dd all0) {
  auto full = [&](int x, dd& d0, dd& d1) {
    const D2 o = gscr[GS * x + 3], p0s = gscr[GS * x + 4], p1s = gscr[GS * x + 5];
    // every node is handed over each slice; the bound keeps a node left
    // unhanded (radii that are not numbers) inside the arrays
    const int ow = (o.y >= 0.0 && o.y < (double)(n_thr)) ? (int)o.y : 0;
    const WAKE_GLOBAL double* t = thr + 4 * (size_t)ow;
    d0 = dd_add({p0s.x, p0s.y}, {t[0], t[1]});
    d1 = dd_add({p1s.x, p1s.y}, {t[2], t[3]});
    if (CL) {
      const double* ms = msuf + 4 * (ow / NT);
      d0 = dd_add(d0, {ms[0], ms[1]});
      d1 = dd_add(d1, {ms[2], ms[3]});
    }
  };
  #pragma unroll 1
  for (int g = g0; g < g1; g += NT) {
    const double rg = GN.r(g), rp = GN.r(g + 1);
    dd D0g, D1g, D0p, D1p;
    full(g, D0g, D1g);
    full(g + 1, D0p, D1p);
    // above the node: sum over [r_g, r_+) of c (r_+ - rho) / (r_+ - r_g)
    dd up = dd_sub(dd_mul_d(dd_sub(D0g, D0p), rp), dd_sub(D1g, D1p));
    up = dd_div_d(up, rp - rg);
    dd lowr;
    double V;
    if (g == 0) {                        // inside the first node: all of it
      lowr = dd_sub(all0, D0g);
      V = 0.5 * rg * rg;
    } else {
      const double rm = GN.r(g - 1);
      dd D0m, D1m;
      full(g - 1, D0m, D1m);
      lowr = dd_sub(dd_sub(D1m, D1g), dd_mul_d(dd_sub(D0m, D0g), rm));
      lowr = dd_div_d(lowr, rg - rm);
      V = (rg - rm) * (rm + 2.0 * rg) / 6.0;
    }
    V += (rp - rg) * (2.0 * rg + rp) / 6.0;
    gout[4 * ngB + g] = dd_round(dd_div_d(dd_add(lowr, up), V));
  }
}

// charge of the analytic beams inside r (staged constants of the slice)
__device__ __forceinline__ double analytic_lam(const double* s_misc, int n_an, double r) {
  double lam = 0.0;
  #pragma unroll 1
  for (int si = 0; si < n_an; ++si)
    if (s_misc[3 * si] == 2.0) lam += s_misc[3 * si + 1] * (-expm1(-r * r * s_misc[3 * si + 2]));
  return lam;
}

template <int NT, bool CL, int GM, bool WIN>
__device__ __forceinline__ void march(const WakeInst& I, int member, const int32_t* queue, unsigned char* smem) {
  // GM: 0 no field grid, 1 field grid, 2 field grid with the chi deposit
  // WIN: cooperative, with a window of the ion nodes in LDS
  constexpr bool GRID = GM > 0;
  constexpr bool CHI = GM > 1;
  constexpr int NW = NT / 64;
  constexpr int CMAX = MarchLds<NT>::CMAX;
  constexpr int KCAP = MarchLds<NT>::KCAP;
  const int tid = threadIdx.x;
  const int N = I.N;
  const int C = I.C;
  const int P = C * NT;                          // positions per member
  const int goff = CL ? member * P : 0;          // this member's first position / slot
  const int Ng = CL ? min(P, N - goff) : N;      // positions of this member
  const int p0 = tid * C;
  const int cnt = max(0, min(C, Ng - p0));   // rings owned by this thread
  const double iC = 1.0 / (double)C, iP = 1.0 / (double)P;
  // ring id of home slot hs
#define WAKE_ID(hs) (CL ? cl_id<NT>((hs), C, P, iP) : id_of<NT>((hs), C))

  double* s_scanA = reinterpret_cast<double*>(smem);      // NW * 16
  double* s_scanB = s_scanA + NW * 16;                     // NW * 16
  double* s_misc = s_scanB + NW * 16;                      // 64
  double* s_fr = s_misc + 64;                              // NT: first pushed key of each chunk
  int32_t* s_fi = reinterpret_cast<int32_t*>(s_fr + NT);  // NT
  double* s_kr = reinterpret_cast<double*>(smem + MarchLds<NT>::head_bytes());
  uint16_t* s_ki = reinterpret_cast<uint16_t*>(s_kr + KCAP);
  uint16_t* s_perm = s_ki + KCAP;
  uint16_t* s_zf = s_perm + KCAP;
  unsigned char* region = smem + MarchLds<NT>::head_bytes() + MarchLds<NT>::key_bytes();
  double* s_br = reinterpret_cast<double*>(region);        // beam radii
  double* s_bc = s_br + WAKE_BCAP;                         // beam cumulative charge
  float* s_ion = reinterpret_cast<float*>(region + MarchLds<NT>::region_bytes());   // ion nodes
  // keys and ring order in LDS (else the order is fixed in global memory)
  const bool lds_keys = !CL && C <= CMAX;
  const uint32_t ps = (uint32_t)(CL ? I.G * P : P);   // slots of the instance
  const unsigned smax = ps - 1;                        // last slot
  const GA<int32_t> gperm = uview(I.perm);
  // slot, in the current buffer, of the ring at this member's position of
  // slot-form index sl
#define WAKE_SLOT(sl) (ident ? (unsigned)(goff + (sl)) \
                             : min(lds_keys ? (unsigned)s_perm[sl] : (unsigned)gperm[goff + (sl)], smax))
  Cluster cl;
  cl.g = member;
  cl.G = CL ? I.G : 1;
  cl.round = 0;
  cl.xd = I.xd;
  cl.xc = I.xc;
  cl.queue = queue;
  if (CL) cl_start(cl);
  double* const s_x = s_kr;                                   // gathered packs (cooperative)
  int* const s_ok = reinterpret_cast<int*>(s_misc + 62);
  uint64_t* const s_dmask = reinterpret_cast<uint64_t*>(s_misc + 32);   // NW words: the push's disorder flags
  uint64_t* const s_bmask = reinterpret_cast<uint64_t*>(s_misc + 40);   // NW words: its breakdown flags
  int32_t* const s_win = reinterpret_cast<int32_t*>(s_misc + 24);       // cooperative: the member's first and last ion interval
  // the same two as byte offsets into the LDS, for the cooperative fix-ups
  const int xo = (int)MarchLds<NT>::head_bytes();
  const int oko = (int)(reinterpret_cast<unsigned char*>(s_ok) - smem);
  // cooperative member-local fix-up rounds in LDS: the key area after the
  // gathered packs (WAKE_CL_GMAX members x 16 doubles)
  const int lo = xo + WAKE_CL_GMAX * 16 * (int)sizeof(double);
  const int lo_cap = (int)MarchLds<NT>::key_bytes() - WAKE_CL_GMAX * 16 * (int)sizeof(double);

  if (__builtin_amdgcn_readfirstlane(I.ctl[CTL_BREAK]) >= 0) return;
  const uint64_t t_start = __builtin_amdgcn_s_memrealtime();
  const int64_t budget = I.budget;
  int cur = __builtin_amdgcn_readfirstlane(I.ctl[CTL_CUR]);
  double rho_mprev = -1.0;   // field grid, cooperative: radius at the previous member's last position
  double rho_mlast = -1.0;   // field grid, cooperative: radius at this member's last position
  __syncthreads();
  // the ring at this thread's k-th position (slot s of the current buffer)
  // is not the one the push wrote there: the chunk's order changed
#define WAKE_MOVED(s, k) ((int)(s) != goff + (k) * NT + tid)
  // injected states may be unsorted
  bool ident = true;
  bool push_keys = false;   // cooperative: the push's first and last keys of the member are in LDS
  bool moved = false;       // a chunk holds rings of another chunk after the fix-up
  if (CL) {
    #pragma unroll 1
    for (int k = 0; k < cnt; ++k) {
      const unsigned sl = goff + k * NT + tid;
      const PV SB = pview(I.st[cur], ps);
      gptr(I.gk_r)[sl] = st_rho(SB, sl);
      gptr(I.gk_i)[sl] = WAKE_ID(st_hs(SB, sl));
    }
    int r = cl_fix<NT>(as_global(I), cl, xo, oko);
    if (r >= 0 && (r & 1)) {      // the block rounds left disorder
      cl.round = r >> 1;
      r = C <= 16 && 16 * P <= lo_cap ? cl_segments<NT>(as_global(I), cl, xo, oko, lo, lo_cap)
                                      : cl_bitonic<NT>(as_global(I), cl, xo, oko);
      if (r >= 0) r <<= 1;
    }
    if (r < 0) {
      if (tid == 0 && member == 0) I.ctl[CTL_FAULT] = 1;
      return;
    }
    cl.round = r >> 1;
    ident = false;
    for (int k = 0; k < cnt; ++k) moved |= WAKE_MOVED(gperm[goff + k * NT + tid], k);
  } else if (lds_keys) {
    #pragma unroll 1
    for (int k = 0; k < cnt; ++k) {
      const unsigned sl = k * NT + tid;
      const PV SB = pview(I.st[cur], ps);
      s_kr[sl] = st_rho(SB, sl);
      s_ki[sl] = (uint16_t)id_of<NT>(st_hs(SB, sl), C);
    }
    __syncthreads();
    fix_order_lds<NT, CMAX>(I, s_scanB, s_scanA, region, s_kr, s_ki, s_zf, s_perm);
    ident = false;
    for (int k = 0; k < cnt; ++k) moved |= WAKE_MOVED(s_perm[k * NT + tid], k);
  } else {
    fix_order_big<NT>(I, cur, s_scanB, s_scanA, region);
    ident = false;
    for (int k = 0; k < cnt; ++k) moved |= WAKE_MOVED(gperm[k * NT + tid], k);
  }
  const dd tot0 = {uni(I.tot0[0]), uni(I.tot0[1])};
  const double dxi = I.dxi;
  IonView IV;
  IV.R = uview(I.ion);
  IV.N = N;
  IV.Rp = I.Rp;
  IV.T0 = tot0;
  IV.Q = {uni(I.tot0[2]), uni(I.tot0[3])};
  const PV KC = pview(I.cst, ps), SCR = pview(I.sc, ps);
  const GA<double> A2 = uview(I.a2), DA2 = uview(I.da2);
  const int n_an = I.n_an;
  const bool has_laser = I.has_laser != 0;
  // ion interval nodes in LDS (float) for the interval search of pass B;
  // read there after the slice-head scan's barriers
  // Cooperative members of more than two rings per thread (WIN) keep a window
  // of them around the member's rings, moved when its rings leave it: the
  // search in device memory, a dependent chain per ring, from each ring's own
  // interval at the previous slice, made the slowest member late.  Eight
  // rings per thread: 20000 rings on 5 members 57.1 -> 54.5 us per slice
  // once the rings moved (39.0 -> 39.6 while they rest), 200000 on 49
  // 55.0 -> 52.8, 40 served requests 191 -> 182 ms; four per thread, 20000
  // rings 33.7 -> 33.0 and 200000 41.3 -> 40.3, three 30.6 -> 30.2 and 37.8 ->
  // 37.6.  With one or two rings
  // per thread that interval comes with the ring, whose record's load need
  // not wait for a search (20000 rings on 40 members 19.2 us per slice, 20.0
  // with the window); a variant of its own, since the window's scalars alone
  // spill registers there.
  const bool lds_ion = CL ? WIN : N <= KCAP;        // the interval nodes in LDS
  const int wn = WIN ? min(N + 1, KCAP + 1) : N + 1;
  int w0 = WIN ? min(max(goff + P / 2 - wn / 2, 0), N + 1 - wn) : 0;
  int hint0 = goff + p0 + 1;           // interval of the thread's first ring (at rest: its node's)
  // field-grid node records in the LDS beyond the layout (read after the
  // slice-head scan's barriers)
  const bool grid_lds = GRID && I.grid_n > 0 && !I.grid_off && I.grid_n <= grid_lds_nodes<NT>();
  D2* const s_gt = reinterpret_cast<D2*>(smem + MarchLds<NT>::bytes());
  if (grid_lds) {
    const WAKE_GLOBAL D2* const t = reinterpret_cast<const WAKE_GLOBAL D2*>(gptr(I.grid_tab));
    for (int i = tid; i < 3 * I.grid_n; i += NT) s_gt[i] = t[i];
  }
  if (lds_ion)
    for (int j = tid; j < wn + 4; j += NT)
      s_ion[j] = j < wn ? (float)IV.R[(w0 + j) * WAKE_ION_REC + IR_LO] : __builtin_nanf("");

  // The per-thread sums of (w, w ln rho), ln rho as the state carries it.
  // The sums in the order the march itself would have left them in (so that
  // a solve split over several launches is bitwise the one-launch solve):
  // the weights always forward (they are summed again only when the chunk's
  // order changed); w ln rho forward in chunks whose order the fix-up
  // changed, backward in the others as the push does.
  dd sw = {0.0, 0.0}, swl = {0.0, 0.0};
  if (moved) {
    chunk_sums<NT>(I, cur, cnt, goff, ps, ident, lds_keys, s_perm, s_ki, sw, swl);
  } else {
    #pragma unroll 1
    for (int k = cnt - 1; k >= 0; --k) {
      const unsigned sl = k * NT + tid;
      const unsigned s = WAKE_SLOT(sl);
      const PV SB = pview(I.st[cur], ps);
      const double w = KC.ldh(RC_W, (unsigned)st_hs(SB, s), 0);
      const D2 l = SB.ld(RS_LN, s);
      swl = dd_add_fast(swl, dd_mul_d(dd{l.x, l.y}, w));
    }
    #pragma unroll 1
    for (int k = 0; k < cnt; ++k) {
      const PV SB = pview(I.st[cur], ps);
      sw = dd_add_d(sw, KC.ldh(RC_W, (unsigned)st_hs(SB, WAKE_SLOT((unsigned)(k * NT + tid))), 0));
    }
  }
  // sums of the thread's own rings in the push's order (what a fix-up that
  // leaves the chunk with its own rings falls back to)
  dd sw_push = sw, swl_push = swl;
  int n = I.first;
  int end = I.first + I.count;
  if (n < end) stage_slice<NT>(I, n, s_misc, s_br, s_bc);
  double bad = 0.0;
  // what the push of slice n-1 left in this workgroup, known after its barriers
  bool any_bad = false, any_dis = false;
  double still = 0.0, had = 0.0;   // cooperative: this member out of order after a round, had one before the meeting
  dd Sm = {0.0, 0.0}, S0b = {0.0, 0.0};   // cooperative: its weight, and before this thread's chunk in it
  bool new_sw = true;          // the chunks' weights changed since the last scan of them
  dd S0 = {0.0, 0.0};          // weight of the chunks before this thread's
  const int aw = __builtin_amdgcn_readfirstlane(((Ng + C - 1) / C + 63) >> 6);   // waves with rings
  int fix_rounds = 0;          // consecutive fix-up rounds at this slice head
  int cl_rounds = 0;           // of which over all members (cooperative)
  int unpushed = cur;          // buffer with the unpushed state of slice n-1

  for (;;) {
    // ---- Gauss/log prefix sum_{k<i} (w_k, w_k ln rho_k); flags of slice n-1 ----
    dd psi_tot;                       // sum of w ln rho
    dd PT0;                           // w ln rho of the chunks before this thread's
    double my_dis = 0.0, bnd = 0.0;   // cooperative: this member's disorder, member boundaries out of order
    if constexpr (CL) {
      // a member whose push came out of order inside its range sorts its
      // blocks before it meets the others: they need not meet again for it
      if (any_dis && n < end) {
        if (tid == 0) atomicAdd(I.cnt + CNT_CL_LOCAL, 1ull);
        const int st = 16 * P <= lo_cap ? cl_fix_local_lds<NT>(as_global(I), member, ident, lo)
                                        : cl_fix_local<NT>(as_global(I), member, ident);
        still = st ? 1.0 : 0.0;
        had = 1.0;
        ident = false;
        bool changed = false;
        if (16 * P <= lo_cap) {
          // the order and the member's first and last keys from the LDS the
          // round worked in (cl_lds_blocks): what it has just written to
          // memory takes a store's and a load's latency, three in a row before
          // the meeting (20000 rings on 5 members 51.2 -> 49.7 us per slice,
          // on 40 members 29.0 -> 28.4)
          const double* const L_r = reinterpret_cast<const double*>(smem + lo);
          const uint64_t* const L_k = reinterpret_cast<const uint64_t*>(smem + lo + 8 * P);
          for (int k = 0; k < cnt; ++k) changed |= WAKE_MOVED((uint32_t)L_k[tid * C + k], k);
          if (tid == 0) {      // (read by this wave only)
            s_fr[0] = L_r[0];
            s_fi[0] = (int32_t)(uint32_t)(L_k[0] >> 32);
            s_misc[48] = L_r[Ng - 1];
            s_misc[49] = (double)(int32_t)(uint32_t)(L_k[Ng - 1] >> 32);
          }
        } else {
          push_keys = false;
          for (int k = 0; k < cnt; ++k) changed |= WAKE_MOVED(gperm[goff + k * NT + tid], k);
        }
        if (changed) chunk_sums<NT>(I, cur, cnt, goff, ps, ident, lds_keys, s_perm, s_ki, sw, swl);
        new_sw = true;
      }
      if (new_sw) {
        Pack<4> t4;
        const Pack<4> pre = block_prefix<NT, 4, DD2FastOp, false>(
            Pack<4>{{sw.hi, sw.lo, swl.hi, swl.lo}}, Pack<4>{{0, 0, 0, 0}}, DD2FastOp(), s_scanA, t4, aw);
        S0b = {pre.v[0], pre.v[1]};
        PT0 = {pre.v[2], pre.v[3]};
        Sm = {t4.v[0], t4.v[1]};
        psi_tot = {t4.v[2], t4.v[3]};
        new_sw = false;
      } else {
        Pack<2> t2;
        const Pack<2> pre = block_prefix<NT, 2, DD1FastOp, false>(Pack<2>{{swl.hi, swl.lo}}, Pack<2>{{0, 0}},
                                                                  DD1FastOp(), s_scanA, t2, aw);
        PT0 = {pre.v[0], pre.v[1]};
        psi_tot = {t2.v[0], t2.v[1]};
      }
      // members' totals, flags (breakdown, still out of order after its own
      // round, whether it had one), their first and last keys in the current
      // order (run boundaries between members) and the time budget
      constexpr int HF = 12;
      Pack<HF> mine = {{Sm.hi, Sm.lo, psi_tot.hi, psi_tot.lo, any_bad ? 1.0 : 0.0, still, 0.0, 0.0, 0.0, 0.0,
                        0.0, had}};
      if (tid < 64) {
        if (push_keys) {       // the push's keys of the first and the last position, kept in LDS
          mine.v[6] = s_fr[0];
          mine.v[7] = (double)s_fi[0];
          mine.v[8] = s_misc[48];
          mine.v[9] = s_misc[49];
        } else {
          const int ql = Ng - 1;
          const unsigned sf = WAKE_SLOT(0u), sL = WAKE_SLOT((unsigned)((ql % C) * NT + ql / C));
          mine.v[6] = gptr(I.gk_r)[sf];
          mine.v[7] = (double)gptr(I.gk_i)[sf];
          mine.v[8] = gptr(I.gk_r)[sL];
          mine.v[9] = (double)gptr(I.gk_i)[sL];
        }
        mine.v[10] = (budget > 0 && n > I.first &&
                      (int64_t)(__builtin_amdgcn_s_memrealtime() - t_start) >= budget) ? 1.0 : 0.0;
      }
      if (!cl_gather<HF, false>(cl, mine, s_x, s_ok)) {
        if (tid == 0 && member == 0) I.ctl[CTL_FAULT] = 1;
        return;
      }
      // one wave per question, the answers through LDS (every wave on all of
      // them took 2.4 us at 40 members, 3.3 at 196)
      const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
      double* const s_res = s_scanB;
      if (wv < 2) {            // w ln rho, w: the members before this one, all of them
        const Pack<2> z = {{0.0, 0.0}};
        Pack<2> pg, tg;
        const int off = wv == 0 ? 2 : 0;
        if (cl.G <= 64) cl_prefix<2, HF, DD1FastOp, 1>(s_x, off, member, cl.G, z, DD1FastOp(), pg, tg);
        else cl_prefix<2, HF, DD1FastOp, 4>(s_x, off, member, cl.G, z, DD1FastOp(), pg, tg);
        if ((tid & 63) == 0) {
          s_res[4 * wv] = pg.v[0]; s_res[4 * wv + 1] = pg.v[1];
          s_res[4 * wv + 2] = tg.v[0]; s_res[4 * wv + 3] = tg.v[1];
        }
      } else if (wv == 2) {    // flags, a member out of time, member boundaries out of order
        bool fb = false, fs = false, ft = false, fh = false, fo = false;
        for (int m = tid & 63; m < cl.G; m += 64) {
          const double* q = s_x + m * HF;
          fb |= q[4] != 0.0;
          fs |= q[5] != 0.0;
          ft |= q[10] != 0.0;
          fh |= q[11] != 0.0;
          fo |= m + 1 < cl.G && key_lt(q[HF + 6], (int32_t)q[HF + 7], q[8], (int32_t)q[9]);
        }
        const int f = (__any(fb) ? 1 : 0) | (__any(fs) ? 2 : 0) | (__any(ft) ? 4 : 0) | (__any(fh) ? 8 : 0) |
                      (__any(fo) ? 16 : 0);
        if ((tid & 63) == 0) s_res[8] = (double)f;
      }
      __syncthreads();
      PT0 = dd_add_fast({s_res[0], s_res[1]}, PT0);
      psi_tot = {s_res[2], s_res[3]};
      S0 = dd_add_fast({s_res[4], s_res[5]}, S0b);
      const int flags = __builtin_amdgcn_readfirstlane((int)s_res[8]);
      if constexpr (GRID) {
        rho_mprev = member > 0 ? s_x[(member - 1) * HF + 8] : -1.0;
        rho_mlast = s_x[member * HF + 8];
      }
      my_dis = still;
      bnd = (flags & 16) ? 1.0 : 0.0;
      any_bad = (flags & 1) != 0;
      any_dis = (flags & 18) != 0;
      if ((flags & 4) && !any_bad) end = n;
      if (fix_rounds == 0 && (flags & 8)) {
        // the members' own round before the meeting
        fix_rounds = 1;
        if (!any_dis && !any_bad && n != end && tid == 0 && member == 0) atomicAdd(I.cnt + CNT_FIXUPS, 1ull);
      }
      __syncthreads();         // the answers are read before a scan writes there again
    }
    if (any_bad) {            // slice n-1 broke down: stop there
      if (tid == 0 && member == 0) { I.ctl[CTL_BREAK] = n - 1; I.ctl[CTL_CUR] = unpushed; I.ctl[CTL_NEXT] = n - 1; }
      return;
    }
    if (n == end) break;
    if (any_dis) {            // pushed radii out of order: new order (then the members' prefix again)
      bool restage = true;    // the general fix-ups use the beam-table area of LDS
      still = 0.0;
      if (tid == 0 && member == 0) atomicAdd(I.cnt + CNT_FIXUPS, 1ull);
      if (CL) {
        // disorder inside members only: up to two member-local block rounds
        // (the first before the meeting; members in order skip them); across
        // member boundaries, or left
        // over, block rounds over all members; after two of these that leave
        // disorder the sort by segments, then the bitonic network
        restage = false;
        if (bnd == 0.0 && fix_rounds < 2 && cl_rounds == 0) {
          if (my_dis == 0.0) {
            ++fix_rounds;
            any_bad = any_dis = false;
            continue;
          }
          if (tid == 0) atomicAdd(I.cnt + CNT_CL_LOCAL, 1ull);
          still = (16 * P <= lo_cap ? cl_fix_local_lds<NT>(as_global(I), member, ident, lo)
                                    : cl_fix_local<NT>(as_global(I), member, ident)) ? 1.0 : 0.0;
        } else {
          int r = -1;
          if (tid == 0 && member == 0)
            atomicAdd(I.cnt + (cl_rounds < 2 ? CNT_CL_ROUNDS
                               : cl_rounds == 2 && C <= 16 && 16 * P <= lo_cap ? CNT_CL_SEGMENTS
                                                                                : CNT_CL_BITONIC), 1ull);
          if (cl_rounds < 2) {
            r = cl_fix_round<NT>(as_global(I), cl, xo, oko, ident, 16 * P <= lo_cap ? lo : -1);
            if (r >= 0) {
              still = (r & 1) ? 1.0 : 0.0;
              r >>= 1;
            }
          } else if (cl_rounds == 2 && C <= 16 && 16 * P <= lo_cap) {
            r = cl_segments<NT>(as_global(I), cl, xo, oko, lo, lo_cap);
          } else {             // exact in any case: the round after it finds the order complete
            r = cl_bitonic<NT>(as_global(I), cl, xo, oko);
          }
          if (r < 0) {
            if (tid == 0 && member == 0) I.ctl[CTL_FAULT] = 1;
            return;
          }
          cl.round = r;
          ++cl_rounds;
        }
        ++fix_rounds;
      } else if (lds_keys) {
        restage = !fix_order_blocks<NT>(I, s_kr, s_ki, s_perm, s_dmask);
        if (restage) {
          if (tid == 0) atomicAdd(I.cnt + CNT_GENERAL, 1ull);
          fix_order_lds<NT, CMAX>(I, s_scanB, s_scanA, region, s_kr, s_ki, s_zf, s_perm);
        }
      } else {
        if (tid == 0) atomicAdd(I.cnt + CNT_GENERAL, 1ull);
        fix_order_big<NT>(I, cur, s_scanB, s_scanA, region);
      }
      ident = false;
      push_keys = false;
      // chunks whose order changed sum again
      bool changed = false;
      for (int k = 0; k < cnt; ++k)
        changed |= WAKE_MOVED(lds_keys ? (int32_t)s_perm[k * NT + tid] : gperm[goff + k * NT + tid], k);
      // (a chunk back to its push order after a later round takes the push's sums again)
      if (changed) {
        chunk_sums<NT>(I, cur, cnt, goff, ps, ident, lds_keys, s_perm, s_ki, sw, swl);
      } else {
        sw = sw_push;
        swl = swl_push;
      }
      if (restage) stage_slice<NT>(I, n, s_misc, s_br, s_bc);
      new_sw = true;
      if (CL) {
        any_bad = any_dis = false;
        continue;
      }
    }
    fix_rounds = 0;
    cl_rounds = 0;
    still = had = 0.0;
    sw_push = sw;
    if constexpr (!CL) {
      // the prefix after any fix-up (its order decides the chunks' sums); the
      // weights' part only when a chunk holds other rings than at the last
      // one, and the flags came with the push: 1000 rings 1.96 -> 1.0 us for
      // this scan, which had carried all six
      if (new_sw) {
        Pack<4> t4;
        const Pack<4> pre = block_prefix<NT, 4, DD2FastOp, false>(
            Pack<4>{{sw.hi, sw.lo, swl.hi, swl.lo}}, Pack<4>{{0, 0, 0, 0}}, DD2FastOp(), s_scanA, t4, aw);
        S0 = {pre.v[0], pre.v[1]};
        PT0 = {pre.v[2], pre.v[3]};
        psi_tot = {t4.v[2], t4.v[3]};
        new_sw = false;
      } else {
        Pack<2> t2;
        const Pack<2> pre = block_prefix<NT, 2, DD1FastOp, false>(Pack<2>{{swl.hi, swl.lo}}, Pack<2>{{0, 0}},
                                                                  DD1FastOp(), s_scanA, t2, aw);
        PT0 = {pre.v[0], pre.v[1]};
        psi_tot = {t2.v[0], t2.v[1]};
      }
    }
    const double psi_axis = dd_round(dd_sub(psi_tot, tot0));
    const bool do_push = n < I.n_xi - 1;
    const bool rec_snap = I.stride > 0 && (n % I.stride) == 0;
    const bool rec_last = n == end - 1;
    const int nb = 1 - cur;
    const PV Sc = pview(I.st[cur], ps), Sn = pview(I.st[nb], ps);
    int bt0 = 0, bm = 0;
    if (I.nb) {
      bt0 = __builtin_amdgcn_readfirstlane(gptr(I.boff)[n]);
      bm = __builtin_amdgcn_readfirstlane(gptr(I.boff)[n + 1]) - bt0;
    }
    const bool staged = bm <= WAKE_BCAP;
    // the slice's table: staged in LDS, or (too long) in device memory; the
    // two are searched by separate code so each takes its own instructions
    const WAKE_GLOBAL double* const gR = gptr(I.br) + bt0;
    const WAKE_GLOBAL double* const gQ = gptr(I.bcum) + bt0;

    // ---- pass B: psi family, sources, local quantities, chunk sums ----
    dd S = S0, PT = PT0;
    Pack<4> G = mat_ident();
    double Vw = 0.0;
    double l0a = 0.0, l0b = 0.0, l1a = 0.0, l1b = 0.0;
    bad = 0.0;
    int blo = 0;
    // loads run ahead: the state of ring k+2 and the constants and ion
    // record of ring k+1 are requested while ring k is computed
    D2 x_ru = d2(1.0, 0.0), x_ln = d2(0.0, 0.0), z_ru = d2(1.0, 0.0), z_ln = d2(0.0, 0.0);
    int32_t x_hs = 0, z_hs = 0;                      // home slots
    int x_hn = 0, z_hn = 0;                          // interval hints (no LDS node table)
    D2 x_wc = d2(0.0, 0.0);                          // (w, w^) of ring k+1
    double x_q[WAKE_ION_REC];
    if (cnt > 0) {
      const unsigned s = WAKE_SLOT(tid);
      x_ru = Sc.ld(RS_RU, s); x_ln = Sc.ld(RS_LN, s); x_hs = st_hs(Sc, s);
      if (!lds_ion) x_hn = st_hint(Sc, s);
    }
    if (cnt > 1) {
      const unsigned s = WAKE_SLOT(NT + tid);
      z_ru = Sc.ld(RS_RU, s); z_ln = Sc.ld(RS_LN, s); z_hs = st_hs(Sc, s);
      if (!lds_ion) z_hn = st_hint(Sc, s);
    }
    // ion interval of the next ring: searched in LDS from the interval of
    // the ring before it (sorted order; the first ring from the interval of
    // the thread's first ring at the previous slice), its records requested
    // one ring ahead; without the LDS table the ring's own interval at the
    // previous slice
    int jn = 0;
    if (cnt > 0) {
      x_wc = KC.ld(RC_W, (unsigned)x_hs);
      jn = !lds_ion ? x_hn : WIN ? ion_find_window(s_ion, w0, wn, x_ru.x, hint0)
                                : ion_find(s_ion, N, x_ru.x, hint0);
      ion_load(IV, jn, x_q);
    }
    // field grid: the interval owning each node hands the node its sums
    // (pass B: weight and w ln rho below it; pass E: the E_z sum and the
    // B^(p) coefficients); every thread then evaluates nodes.  gb_lo: the
    // last node at or below the previous position, gb_next its successor's
    // radius (a ring at or above it owns nodes)
    // this slice's nodes: entries [gofs, gofs + ngB) of a per-slice node
    // set, else the context's nodes (fields of slice n at 4 n grid_n)
    const size_t gofs = !GRID ? 0 : I.grid_off ? (size_t)gptr(I.grid_off)[n] : (size_t)n * (size_t)I.grid_n;
    const int ngB = !GRID ? 0 : I.grid_off ? gptr(I.grid_off)[n + 1] - (int)gofs : I.grid_n;
    const WAKE_GLOBAL double* const grB =
        (GRID && I.grid_rad) ? gptr(I.grid_rad) + (I.grid_off ? gofs : 0) : nullptr;
    const double dgB = I.grid_dr, idgB = 1.0 / dgB;
    WAKE_GLOBAL D2* const gscr = reinterpret_cast<WAKE_GLOBAL D2*>(gptr(I.grid_scr));
    int gb_lo = -1;
    double gb_next = INFINITY;
    if (GRID && ngB > 0 && cnt > 0) {
      double rb = -1.0;
      if (tid > 0) rb = Sc.ld(RS_RU, WAKE_SLOT((unsigned)((C - 1) * NT + tid - 1))).x;
      else if (CL) rb = rho_mprev;
      gb_lo = grid_last_below(rb, dgB, idgB, ngB, grB);
      gb_next = gb_lo + 1 < ngB ? grid_node_r(gb_lo + 1, dgB, grB) : INFINITY;
    }
    #pragma unroll 1
    for (int k = 0; k < cnt; ++k) {
      const unsigned sl = k * NT + tid;
      const double rho = x_ru.x, u = x_ru.y;
      const int32_t hs = x_hs;
      int h = jn;
      const dd lnr = {x_ln.x, x_ln.y};
      const double w = x_wc.x, wh = x_wc.y;
      x_ru = z_ru; x_ln = z_ln; x_hs = z_hs; x_hn = z_hn;
      if (k + 2 < cnt) {
        const unsigned s = WAKE_SLOT(sl + 2 * NT);
        z_ru = Sc.ld(RS_RU, s); z_ln = Sc.ld(RS_LN, s); z_hs = st_hs(Sc, s);
        if (!lds_ion) z_hn = st_hint(Sc, s);
      }
      const double irho = rcp_nr(rho);
      const dd PTi = psi_next(PT, lnr, w);
      const dd Si = dd_add_d(S, w);
      double psi, dpsi;
      psi_family(S, Si, PTi, lnr, rho, irho, wh, ion_fields(IV, rho, lnr, h, x_q), psi, dpsi);
      psi += psi_axis;
      // the next ring's weights and ion record, into the registers just read
      if (k + 1 < cnt) {
        x_wc = KC.ld(RC_W, (unsigned)x_hs);
        jn = !lds_ion ? x_hn : WIN ? ion_find_window(s_ion, w0, wn, x_ru.x, h)
                                  : ion_find(s_ion, N, x_ru.x, h);
        ion_load(IV, jn, x_q);
      }
      if (GRID && rho >= gb_next) {
        // nodes of interval p = (rho_{p-1}, rho_p]: the sums below position p
        const int ghi = grid_last_below(rho, dgB, idgB, ngB, grB);
        #pragma unroll 1
        for (int g = gb_lo + 1; g <= ghi; ++g) {
          gscr[GS * g] = d2(S.hi, S.lo);
          gscr[GS * g + 1] = d2(PT.hi, PT.lo);
        }
        gb_lo = ghi;
        gb_next = gb_lo + 1 < ngB ? grid_node_r(gb_lo + 1, dgB, grB) : INFINITY;
      }
      S = Si;
      PT = PTi;
      // beam charge inside rho (strictly below), analytic beams, lasers
      double lam = 0.0;
      if (bm > 0) {
        if (staged) {
          blo = count_below(s_br, blo, bm, rho, k > 0);
          if (blo > 0) lam = s_bc[blo - 1];
        } else {
          blo = count_below(gR, blo, bm, rho, k > 0);
          if (blo > 0) lam = gQ[blo - 1];
        }
      }
      double aa = 0.0, dda = 0.0;
      #pragma unroll 1
      for (int si = 0; si < n_an; ++si) {
        const double kind = s_misc[3 * si], c0 = s_misc[3 * si + 1], c1 = s_misc[3 * si + 2];
        if (kind == 2.0) {
          lam += c0 * (-expm1(-rho * rho * c1));
        } else {
          const double x = c0 * exp(-rho * rho * c1);
          aa += x;
          dda += -(2.0 * rho * c1) * x;
        }
      }
      const double bb = lam * irho;
      const Local L = local_of(irho, u, w, psi, aa);
      if (!(L.pb > 0.0)) bad = 1.0;
      // s_i with d_zeta psi = (sum of v inside the chunk before the ring + w^
      // share) + c: s_a = s0 - c beta / 2
      const double dz0 = __builtin_fma(wh, L.cu, Vw);
      Vw = __builtin_fma(w, L.cu, Vw);
      double cc, s0;
      ring_source(irho, u, w, L, aa, dpsi, dz0, bb, dda, cc, s0);
      const double hbeta = 0.5 * L.A * u * L.ipb;          // beta = -dB/d(d_zeta psi)
      const double r2 = rho * rho, hAi = 0.5 * L.A * irho, rC = 0.5 * w * cc;
      const double m0 = __builtin_fma(r2, G.v[0], G.v[2]), m1 = __builtin_fma(r2, G.v[1], G.v[3]);
      const double y0 = hAi * m0, y1 = hAi * m1;
      G.v[0] += y0;
      G.v[1] += y1;
      G.v[2] = __builtin_fma(-r2, y0, G.v[2]);
      G.v[3] = __builtin_fma(-r2, y1, G.v[3]);
      l0a = __builtin_fma(-s0, m0, __builtin_fma(G.v[0], rC, l0a));
      l0b = __builtin_fma(-s0, m1, __builtin_fma(G.v[1], rC, l0b));
      l1a = __builtin_fma(hbeta, m0, l1a);
      l1b = __builtin_fma(hbeta, m1, l1b);
      SCR.st(SC_PSI, goff + sl, d2(psi, dpsi));
      if (has_laser) { A2.st(goff + sl, aa); DA2.st(goff + sl, dda); }
      // the ring's interval: its hint at the next slice (the thread's first
      // ring: the next slice's search starts there)
      if (!lds_ion) Sn.sti(RS_W, Sn.ps + goff + sl, h);
      if (k == 0) hint0 = h;
      if (WIN && wn <= N) {     // the member's first and last interval
        if (p0 + k == 0) s_win[0] = h;
        if (p0 + k == Ng - 1) s_win[1] = h;
      }
    }
    if (GRID && ngB > 0 && cnt > 0 && p0 + cnt == Ng && (!CL || member == cl.G - 1)) {
      // nodes beyond the last ring: every ring below them
      #pragma unroll 1
      for (int g = gb_lo + 1; g < ngB; ++g) {
        gscr[GS * g] = d2(S.hi, S.lo);
        gscr[GS * g + 1] = d2(PT.hi, PT.lo);
      }
    }
    // this member's nodes (all of them for a single workgroup)
    int g_begin = 0, g_end = ngB;
    if (GRID && CL && ngB > 0) {
      g_begin = grid_last_below(rho_mprev, dgB, idgB, ngB, grB) + 1;
      if (member < cl.G - 1) g_end = grid_last_below(rho_mlast, dgB, idgB, ngB, grB) + 1;
    }

    // ---- growing mode g (prefix) and decaying mode h (suffix) ----
    Pack<4> gp, gt;
    Pack<5> hx, ht;
    block_prefix_suffix<NT, 4, 5, FwdMatOp, BwdMatSumOp, false>(
        G, mat_ident(), FwdMatOp(), Pack<5>{{G.v[3], -G.v[1], -G.v[2], G.v[0], Vw}},
        Pack<5>{{1.0, 0.0, 0.0, 1.0, 0.0}}, BwdMatSumOp(), s_scanB, gp, gt, hx, ht, aw);
    if (GRID && ngB > 0) {
      // psi, E_r - B_theta and the beam field at this member's nodes (the
      // scans' barriers order the sums written in pass B before these reads)
      const WAKE_GLOBAL D2* const gtab = reinterpret_cast<const WAKE_GLOBAL D2*>(gptr(I.grid_tab)) +
                                         (I.grid_off ? 3 * gofs : 0);
      WAKE_GLOBAL double* const gout = gptr(I.grid) + 5 * gofs;
      #pragma unroll 1
      for (int g = g_begin + tid; g < g_end; g += NT) {
        const double r = grid_node_r(g, dgB, grB);
        D2 t0, t1, t2;
        if (grid_lds) {
          t0 = s_gt[3 * g]; t1 = s_gt[3 * g + 1]; t2 = s_gt[3 * g + 2];
        } else {
          t0 = gtab[3 * g]; t1 = gtab[3 * g + 1]; t2 = gtab[3 * g + 2];
        }
        const D2 sS = gscr[GS * g], sP = gscr[GS * g + 1];
        grid_node_psi(gout, ngB, g, r, t0, t1, t2, dd{sS.x, sS.y}, dd{sP.x, sP.y}, psi_axis);
        double lam = 0.0;
        if (bm > 0) {
          int cb;
          if (staged) {
            cb = count_below(s_br, 0, bm, r, false);
            if (cb > 0) lam = s_bc[cb - 1];
          } else {
            cb = count_below(gR, 0, bm, r, false);
            if (cb > 0) lam = gQ[cb - 1];
          }
        }
        lam += analytic_lam(s_misc, n_an, r);
        gout[3 * ngB + g] = lam * rcp_nr(r);     // B^(b); pass E adds B^(p)
      }
    }
    double e_in = 0.0, d_in = 0.0;       // cooperative: det-sums of the members before / after
    if (CL) {
      // one exchange for the members' transfer products and det-sums: this
      // chunk's parts of the member's A, B, A', B' (Gl, Hl: the member's
      // transfers before the chunk and inverse transfers after it)
      const double vl = Vw + hx.v[4];
      const double mua = l0a - vl * l1a, mub = l0b - vl * l1b;
      const double k0 = G.v[3] * hx.v[0] - G.v[1] * hx.v[2], k1 = G.v[3] * hx.v[1] - G.v[1] * hx.v[3];
      const double k2 = -G.v[2] * hx.v[0] + G.v[0] * hx.v[2], k3 = -G.v[2] * hx.v[1] + G.v[0] * hx.v[3];
      Pack<8> part = {{gp.v[0] * mua + gp.v[2] * mub, gp.v[1] * mua + gp.v[3] * mub,
                       gp.v[0] * l1a + gp.v[2] * l1b, gp.v[1] * l1a + gp.v[3] * l1b,
                       k0 * mua + k2 * mub, k1 * mua + k3 * mub, k0 * l1a + k2 * l1b, k1 * l1a + k3 * l1b}};
      const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
      if (wv < aw) {                     // sums over the wave, then (by the publishing lanes) the waves
        const Pack<8> ws = wave_prefix_incl(part, SumOp<8>());
        if ((tid & 63) == 63) {
#pragma unroll
          for (int i = 0; i < 8; ++i) s_scanA[wv * 8 + i] = ws.v[i];
        }
      }
      auto word = [&](int l) {
        double v = ht.v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v = l == i ? gt.v[i] : v;
        if (l >= 5 && l < 13) {
          v = 0.0;
          for (int w = 0; w < aw; ++w) v += s_scanA[w * 8 + l - 5];
        }
        return v;
      };
      if (!cl_gather_words<13, false>(cl, word, s_x, s_ok)) {
        if (tid == 0 && member == 0) I.ctl[CTL_FAULT] = 1;
        return;
      }
      double* const s_res = s_scanB;
      if (wv == 0) {
        if (cl.G <= 64) cl_transfer_fwd<13, 1>(s_x, member, cl.G, s_res);
        else cl_transfer_fwd<13, 4>(s_x, member, cl.G, s_res);
      } else if (wv == 1) {
        if (cl.G <= 64) cl_transfer_bwd<13, BwdMatSumOp, 1>(s_x, member, cl.G, s_res + 16);
        else cl_transfer_bwd<13, BwdMatSumOp, 4>(s_x, member, cl.G, s_res + 16);
      }
      __syncthreads();
      gp = FwdMatOp()(Pack<4>{{s_res[0], s_res[1], s_res[2], s_res[3]}}, gp);
      e_in = s_res[4];
      gt = Pack<4>{{s_res[5], s_res[6], s_res[7], s_res[8]}};
      hx = BwdMatSumOp()(hx, Pack<5>{{s_res[16], s_res[17], s_res[18], s_res[19], s_res[20]}});
      d_in = s_res[21];
      ht = Pack<5>{{s_res[22], s_res[23], s_res[24], s_res[25], s_res[26]}};
    }
    const double W = gt.v[0];                 // det[g_N, (0,1)]
    const double iW = 1.0 / W;
    const double Vtot = ht.v[4];
    const double Vafter = hx.v[4];
    const double gsa = gp.v[0], gsb = gp.v[2];    // g at the chunk start
    const double hea = hx.v[1], heb = hx.v[3];    // h at the chunk end
    const double c = -(Vw + Vafter);
    const double la = l0a + c * l1a, lb = l0b + c * l1b;
    const double le = gsa * la + gsb * lb;        // sum of det[g_i, s_i] over the chunk
    const double hsa = G.v[3] * hea - G.v[1] * heb;   // h at the chunk start
    const double hsb = -G.v[2] * hea + G.v[0] * heb;
    const double lds = -(hsa * la + hsb * lb);     // sum of det[s_i, h_i] over the chunk
    Pack<1> ep, et, dsf, dt;
    block_prefix_suffix<NT, 1, 1, SumOp<1>, SumOp<1>, false>(
        Pack<1>{{le}}, Pack<1>{{0.0}}, SumOp<1>(), Pack<1>{{lds}}, Pack<1>{{0.0}}, SumOp<1>(),
        s_scanA, ep, et, dsf, dt, aw);
    if (CL) {
      ep.v[0] = e_in + ep.v[0];
      dsf.v[0] = dsf.v[0] + d_in;
    }

    // ---- pass E: B^(p), outputs, push ----
    // the next slice's beam-table entries, fetched now and stored after the pass
    const bool stage_next = do_push && n + 1 < end;
    BeamStage<NT> nbs;
    nbs.m = 0;
    if (stage_next) beam_fetch<NT>(I, n + 1, nbs);
    double ga = G.v[0] * gsa + G.v[1] * gsb;      // g at the chunk end
    double gb = G.v[2] * gsa + G.v[3] * gsb;
    double ha = hea, hb = heb;
    double Vgt = Vafter;
    double E = ep.v[0] + le;
    double D = dsf.v[0];
    double nxt_r = INFINITY, last_r = INFINITY;
    int32_t nxt_i = 0x7fffffff, last_i = 0x7fffffff;
    dd swl2 = {0.0, 0.0};
    double dis_l = 0.0;
    // loads run ahead (the march goes backward): the state of ring k-2 and
    // the constants of ring k-1 are requested while ring k is computed
    D2 y_ru = d2(1.0, 0.0), y_f = d2(0.0, 0.0), y_ps = d2(0.0, 0.0), y_ln = d2(0.0, 0.0);   // ring k-1
    int32_t y_hs = 0;
    D2 v_ru = d2(1.0, 0.0), v_f = d2(0.0, 0.0), v_ps = d2(0.0, 0.0), v_ln = d2(0.0, 0.0);   // ring k-2
    int32_t v_hs = 0;
    int bhi = 0;                // beam-table entries below the ring (pass B's count, met downward)
    D2 c_w = d2(1.0, 0.0);      // ring k-1
    if (cnt > 0) {
      const unsigned sl = (cnt - 1) * NT + tid;
      const unsigned s = WAKE_SLOT(sl);
      y_ru = Sc.ld(RS_RU, s); y_f = Sc.ld(RS_F, s); y_ln = Sc.ld(RS_LN, s);
      y_ps = SCR.ld(SC_PSI, goff + sl);
      y_hs = st_hs(Sc, s);
    }
    if (cnt > 1) {
      const unsigned sl = (cnt - 2) * NT + tid;
      const unsigned s = WAKE_SLOT(sl);
      v_ru = Sc.ld(RS_RU, s); v_f = Sc.ld(RS_F, s); v_ln = Sc.ld(RS_LN, s);
      v_ps = SCR.ld(SC_PSI, goff + sl);
      v_hs = st_hs(Sc, s);
    }
    if (cnt > 0) c_w = KC.ld(RC_W, (unsigned)y_hs);
    // field grid: ge_hi the last node at or below the current ring, ge_top
    // its radius (a previous ring below it means the interval owns nodes).
    // chi (fixed node sets): the nodes also take the sums of c = w / psibar
    // and c rho at and above them within this chunk, and who handed them.
    const bool chi = CHI && ngB > 0 && !I.grid_off && I.grid_chi;
    GridNodes GN;
    GN.rad = grB;
    GN.dg = dgB;
    GN.idg = idgB;
    GN.nr = ngB;
    GN.nh = chi ? ngB + 1 : ngB;
    GN.top = 0.0;
    if (chi) {
      const double rl = grid_node_r(ngB - 1, dgB, grB);
      GN.top = ngB > 1 ? rl + (rl - grid_node_r(ngB - 2, dgB, grB)) : 2.0 * rl;
    }
    const double owner = (double)(member * NT + tid);
    dd cg0 = {0.0, 0.0}, cg1 = {0.0, 0.0};
    int ge_hi = -1;
    double ge_top = -INFINITY, g_lo_r = -1.0;
    if (GRID && ngB > 0 && cnt > 0) {
      if (tid > 0) g_lo_r = Sc.ld(RS_RU, WAKE_SLOT((unsigned)((C - 1) * NT + tid - 1))).x;
      else if (CL) g_lo_r = rho_mprev;
      ge_hi = GN.last_below(y_ru.x);
      if (p0 + cnt == Ng && (!CL || member == cl.G - 1)) {
        // nodes beyond the last ring: interval N (a_N = 0, no ring outside)
        const double a = (ha * E - ga * D) * iW, b = (hb * E - gb * D) * iW;
        #pragma unroll 1
        for (int g = ge_hi + 1; g < GN.nh; ++g) {
          gscr[GS * g + 2] = d2(Vgt, a);
          gscr[GS * g + 3] = d2(b, owner);
          if (CHI) {
            gscr[GS * g + 4] = d2(0.0, 0.0);
            gscr[GS * g + 5] = d2(0.0, 0.0);
          }
        }
      }
      ge_top = ge_hi >= 0 ? GN.r(ge_hi) : -INFINITY;
    }
    #pragma unroll 1
    for (int k = cnt - 1; k >= 0; --k) {
      const unsigned sl = k * NT + tid;
      const double rho = y_ru.x, u = y_ru.y, fr_p = y_f.x, fu_p = y_f.y;
      const int32_t hs = y_hs;
      const double psi = y_ps.x, dpsi = y_ps.y;
      const double w = c_w.x, wh = c_w.y;
      const dd lr0 = {y_ln.x, y_ln.y};
      y_ru = v_ru; y_f = v_f; y_hs = v_hs; y_ps = v_ps; y_ln = v_ln;
      if (k > 1) {
        const unsigned sp = sl - 2 * NT;
        const unsigned s = WAKE_SLOT(sp);
        v_ru = Sc.ld(RS_RU, s); v_f = Sc.ld(RS_F, s); v_ln = Sc.ld(RS_LN, s);
        v_ps = SCR.ld(SC_PSI, goff + sp);
        v_hs = st_hs(Sc, s);
      }
      if (k > 0) c_w = KC.ld(RC_W, (unsigned)y_hs);
      const double a2 = has_laser ? A2[goff + sl] : 0.0, da2 = has_laser ? DA2[goff + sl] : 0.0;
      const double irho = rcp_nr(rho);
      // B^(b) as pass B formed it: the table count, then the analytic beams
      double lam = 0.0;
      if (bm > 0) {
        if (staged) {
          bhi = count_below_down(s_br, bhi, bm, rho, k < cnt - 1);
          if (bhi > 0) lam = s_bc[bhi - 1];
        } else {
          bhi = count_below_down(gR, bhi, bm, rho, k < cnt - 1);
          if (bhi > 0) lam = gQ[bhi - 1];
        }
      }
      #pragma unroll 1
      for (int si = 0; si < n_an; ++si)
        if (s_misc[3 * si] == 2.0) lam += s_misc[3 * si + 1] * (-expm1(-rho * rho * s_misc[3 * si + 2]));
      const double bb = lam * irho;
      const Local L = local_of(irho, u, w, psi, a2);
      const double Vn = __builtin_fma(w, L.cu, Vgt);       // sum of v from this ring on
      const double dz = __builtin_fma(wh, L.cu, -Vn);
      double cc, sa;
      ring_source(irho, u, w, L, a2, dpsi, dz, bb, da2, cc, sa);
      const double r2 = rho * rho, hAi = 0.5 * L.A * irho, rC = 0.5 * w * cc;
      const double mg = __builtin_fma(r2, ga, gb), mh = __builtin_fma(r2, ha, hb);
      D = __builtin_fma(sa, mh, __builtin_fma(-rC, ha, D));    // D_{i-1} (det[s_i, h_i])
      E = __builtin_fma(sa, mg, __builtin_fma(-rC, ga, E));    // E_{i-1} (det[g_i, s_i])
      const double yg = hAi * mg, yh = hAi * mh;               // g, h of interval i-1
      ga -= yg;
      gb = __builtin_fma(r2, yg, gb);
      ha -= yh;
      hb = __builtin_fma(r2, yh, hb);
      // a_{i-1} rho + b_{i-1} / rho from x_{i-1} = (h E - g D) / W, and the
      // ring's own share w^ C / w
      const double bp = irho * __builtin_fma(iW, __builtin_fma(E, mh, -(D * mg)), 0.5 * wh * cc);
      const double bt = bb + bp;
      const double ez = -dz;
      if (!(isfinite(psi) && isfinite(dpsi) && isfinite(ez) && isfinite(bt))) bad = 1.0;
      const int32_t id = WAKE_ID(hs);
      if (rec_snap) {
        WAKE_GLOBAL double* sp = gptr(I.snap) + (size_t)(n / I.stride) * OUT_N * N;
        sp[OUT_PSI * N + id] = psi; sp[OUT_ERBT * N + id] = -dpsi;
        sp[OUT_EZ * N + id] = ez; sp[OUT_BT * N + id] = bt;
        sp[OUT_RHO * N + id] = rho; sp[OUT_UR * N + id] = u;
      }
      if (rec_last) {
        WAKE_GLOBAL double* sp = gptr(I.last);
        sp[OUT_PSI * N + id] = psi; sp[OUT_ERBT * N + id] = -dpsi;
        sp[OUT_EZ * N + id] = ez; sp[OUT_BT * N + id] = bt;
        sp[OUT_RHO * N + id] = rho; sp[OUT_UR * N + id] = u;
      }
      if (do_push) {
        const double f_r = u * L.ipb;
        const double f_u = __builtin_fma(L.ipb, __builtin_fma(L.gm, dpsi, -0.25 * da2), -bt);
        double pr = f_r, pu = f_u;
        if (n > 0) { pr = fr_p; pu = fu_p; }
        double rn = __builtin_fma(dxi, __builtin_fma(1.5, f_r, -0.5 * pr), rho);
        double un = __builtin_fma(dxi, __builtin_fma(1.5, f_u, -0.5 * pu), u);
        double sr = f_r, su = f_u;
        if (rn < 0.0) { rn = -rn; un = -un; sr = -sr; su = -su; }
        if (!(isfinite(rn) && isfinite(un))) bad = 1.0;
        // ln rho moves with the ring: the old value plus log1p of the step
        const dd lr = dd_add_d(lr0, log1p_fast((rn - rho) * irho));
        Sn.st(RS_RU, goff + sl, d2(rn, un));
        Sn.st(RS_F, goff + sl, d2(sr, su));
        Sn.st(RS_LN, goff + sl, d2(lr.hi, lr.lo));
        Sn.sti(RS_W, goff + sl, hs);
        swl2 = dd_add_fast(swl2, dd_mul_d(lr, w));
        if (lds_keys) { s_kr[sl] = rn; s_ki[sl] = (uint16_t)id; }
        if (CL) { gptr(I.gk_r)[goff + sl] = rn; gptr(I.gk_i)[goff + sl] = id; }
        if (!key_lt(rn, id, nxt_r, nxt_i)) dis_l = 1.0;
        if (k == cnt - 1) { last_r = rn; last_i = id; }
        nxt_r = rn;
        nxt_i = id;
      }
      Vgt = Vn;
      if (GRID) {
        if (CHI && chi) {
          const double c = w * L.ipb;
          cg0 = dd_add_d(cg0, c);
          cg1 = dd_add(cg1, two_prod(c, rho));
        }
        const double rlo = k > 0 ? y_ru.x : g_lo_r;
        if (rlo < ge_top) {
          // nodes of interval p = (rho_{p-1}, rho_p]
          const int glo = GN.last_below(rlo) + 1;
          const double a = (ha * E - ga * D) * iW, b = (hb * E - gb * D) * iW;
          #pragma unroll 1
          for (int g = glo; g <= ge_hi; ++g) {
            gscr[GS * g + 2] = d2(Vgt, a);
            gscr[GS * g + 3] = d2(b, owner);
            if (CHI) {
              gscr[GS * g + 4] = d2(cg0.hi, cg0.lo);
              gscr[GS * g + 5] = d2(cg1.hi, cg1.lo);
            }
          }
          ge_hi = glo - 1;
          ge_top = ge_hi >= 0 ? GN.r(ge_hi) : -INFINITY;
        }
      }
    }
    if (tid == 0 && member == 0) { gptr(I.axis)[2 * n] = psi_axis; gptr(I.axis)[2 * n + 1] = Vtot; }
    // order across chunk boundaries: this chunk's first pushed key (+inf if
    // empty) against the previous chunk's last one
    s_fr[tid] = nxt_r;
    s_fi[tid] = nxt_i;
    if (CL && do_push && cnt > 0 && p0 + cnt == Ng) { s_misc[48] = last_r; s_misc[49] = (double)last_i; }
    __syncthreads();          // every wave is done with this slice's table and constants
    if (WIN && wn <= N) {
      // the window follows the member's rings: around them when one end left
      // it (rings spread over more intervals than it holds: around their middle)
      const int j0 = __builtin_amdgcn_readfirstlane(s_win[0]), j1 = __builtin_amdgcn_readfirstlane(s_win[1]);
      const int want = min(max((j0 + j1) / 2 - wn / 2, 0), N + 1 - wn);
      if ((j0 < w0 || j1 >= w0 + wn) && abs(want - w0) > wn / 8) {
        w0 = want;
        for (int j = tid; j < wn; j += NT) s_ion[j] = (float)IV.R[(w0 + j) * WAKE_ION_REC + IR_LO];
      }
    }
    if (stage_next) {
      stage_analytic<NT>(I, n + 1, s_misc);
      beam_store<NT>(nbs, s_br, s_bc);
    }
    {
      // the push's flags, a bit per thread: breakdown, and its chunk out of
      // order inside or against the next chunk's first key
      if (do_push && cnt > 0 && tid + 1 < NT && !key_lt(last_r, last_i, s_fr[tid + 1], s_fi[tid + 1]))
        dis_l = 1.0;
      const uint64_t md = __ballot(dis_l != 0.0), mb = __ballot(bad != 0.0);
      if ((tid & 63) == 0) { s_dmask[tid >> 6] = md; s_bmask[tid >> 6] = mb; }
    }
    // out of time: this slice is the launch's last (one clock read, broadcast;
    // cooperative members decide together at the next slice head)
    if (tid == 0)
      s_misc[63] = !CL && budget > 0 && (int64_t)(__builtin_amdgcn_s_memrealtime() - t_start) >= budget ? 1.0 : 0.0;
    __syncthreads();
    if (s_misc[63] != 0.0) end = n + 1;
    {
      const int lane = tid & 63;
      uint64_t md = 0, mb = 0;
      if (lane < NW) { md = s_dmask[lane]; mb = s_bmask[lane]; }
      any_dis = __ballot(md != 0) != 0;
      any_bad = __ballot(mb != 0) != 0;
    }
    if (GRID && ngB > 0) {
      // E_z and B_theta at this member's nodes (after the barrier above)
      WAKE_GLOBAL double* const gout = gptr(I.grid) + 5 * gofs;
      #pragma unroll 1
      for (int g = g_begin + tid; g < g_end; g += NT) {
        const double r = grid_node_r(g, dgB, grB);
        const D2 e0 = gscr[GS * g + 2], e1 = gscr[GS * g + 3];
        grid_node_b(gout, ngB, g, r, e0.x, e0.y, e1.x, gout[3 * ngB + g]);
      }
      if (CHI && chi) {
        // chi = n/gamma (reading R20): each node's owner adds the sums of
        // the chunks after its own; the hats' sums are differences of the
        // full sums D, E (c and c rho at and above a node) of neighbouring
        // nodes
        Pack<4> tot;
        const Pack<4> later = block_suffix<NT, 4>(Pack<4>{{cg0.hi, cg0.lo, cg1.hi, cg1.lo}},
                                                  Pack<4>{{0.0, 0.0, 0.0, 0.0}}, DD2Op(), s_scanA, tot);
        WAKE_GLOBAL double* const thr = gptr(I.grid_thr);
        #pragma unroll
        for (int i = 0; i < 4; ++i) thr[4 * (size_t)(member * NT + tid) + i] = later.v[i];
        dd all0 = {tot.v[0], tot.v[1]};
        const double* msuf = nullptr;          // sums of the members after each member
        if (CL) {
          // member totals (the fenced form: the nodes' partial sums and the
          // threads' suffixes become visible to every member)
          if (!cl_gather<4, true>(cl, tot, s_x, s_ok)) {
            if (tid == 0 && member == 0) I.ctl[CTL_FAULT] = 1;
            return;
          }
          if (tid == 0) {
            Pack<4> run = {{0.0, 0.0, 0.0, 0.0}};
            for (int m = cl.G - 1; m >= 0; --m) {
              const Pack<4> x = {{s_x[4 * m], s_x[4 * m + 1], s_x[4 * m + 2], s_x[4 * m + 3]}};
              #pragma unroll
              for (int i = 0; i < 4; ++i) s_x[4 * m + i] = run.v[i];
              run = DD2Op()(x, run);
            }
            #pragma unroll
            for (int i = 0; i < 4; ++i) s_x[4 * cl.G + i] = run.v[i];
          }
          __syncthreads();
          all0 = {s_x[4 * cl.G], s_x[4 * cl.G + 1]};
          msuf = s_x;
        } else {
          __syncthreads();
        }
        chi_nodes<NT, CL>(gout, ngB, gscr, thr, msuf, (CL ? cl.G : 1) * NT, GN, g_begin + tid, g_end, all0);
      }
    }
    unpushed = cur;
    if (do_push) {
      // the pushed rings sit at the slots of this slice's positions
      cur = nb;
      ident = true;
      push_keys = CL;
      swl = swl2;
      swl_push = swl2;
    }
    ++n;
  }
  if (tid == 0 && member == 0) {
    I.ctl[CTL_CUR] = cur;
    I.ctl[CTL_NEXT] = end;
    atomicAdd(I.cnt + CNT_SLICES, (unsigned long long)(end - I.first));
    if (CL) atomicAdd(I.cnt + CNT_CL_MEETINGS, (unsigned long long)cl.round);
  }
#undef WAKE_SLOT
#undef WAKE_ID
#undef WAKE_MOVED
}

// the cooperative march as a function of its own (its registers stay out of
// the single-workgroup march, which is inlined into the kernel)
template <int NT, int GM, bool WIN>
__device__ __noinline__ void march_member(const WAKE_GLOBAL WakeInst* I, int member, const int32_t* queue) {
  march<NT, true, GM, WIN>(*(const WakeInst*)I, member, queue, wake_lds);
}

#ifndef WAKE_WAVES_PER_EU
#define WAKE_WAVES_PER_EU 2
#endif
// WAKE_WAVES_PER_EU waves per SIMD (2: up to 256 VGPRs per lane)
template <int NT, int GM>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WAKE_WAVES_PER_EU)))
void wake_march_kernel(const WakeInst* __restrict__ insts, int n_insts, int n_tasks, int32_t* counter) {
  unsigned char* const smem = wake_lds;
  __shared__ int s_idx;
  for (;;) {
    if (threadIdx.x == 0) s_idx = atomicAdd(counter, 1);
    __syncthreads();
    const int idx = __builtin_amdgcn_readfirstlane(s_idx);
    __syncthreads();
    if (idx >= n_tasks) return;   // every workgroup leaves once the queue is empty
    // task idx: member idx - task0 of the last instance with task0 <= idx
    int lo = 0, hi = n_insts;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (__builtin_amdgcn_readfirstlane(insts[mid].task0) <= idx) lo = mid; else hi = mid;
    }
    const WakeInst& I = insts[lo];
    if (I.nt == NT) {
      if (I.G > 1) {
        if (I.C > 2) march_member<NT, GM, true>(as_global(I), idx - I.task0, counter);
        else march_member<NT, GM, false>(as_global(I), idx - I.task0, counter);
      } else {
        march<NT, false, GM, false>(I, 0, counter, smem);
      }
    }
    __syncthreads();
  }
}

__global__ void counter_zero_kernel(int32_t* p) {
  if (threadIdx.x == 0) p[0] = 0;
}

// barrier words of the cooperative instances of a launch start at zero
// and their packs carry no stamp of this launch's rounds
__global__ void cluster_reset_kernel(const WakeInst* __restrict__ insts, int n_insts) {
  for (int i = threadIdx.x; i < n_insts; i += blockDim.x) {
    const int G = insts[i].G;
    if (G <= 1) continue;
    insts[i].xc[0] = 0; insts[i].xc[1] = 0; insts[i].xc[2] = 0;
    for (int k = 0; k < 2 * G; ++k) insts[i].xd[cl_stamp_at(G, k / G, k % G)] = -1.0;
  }
}

// ---------------------------------------------------------------------------
// state transfers by ring id, reset
// ---------------------------------------------------------------------------
__global__ void state_by_id_kernel(WakeInst I, double* rho, double* u, double* fr, double* fu) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= I.N) return;
  const int c = I.ctl[CTL_CUR];
  const unsigned sl = slot_of(p, I.C, I.nt);
  const size_t PS = (size_t)I.G * I.C * I.nt;
  const D2* r = reinterpret_cast<const D2*>(I.st[c]) + sl;
  const int hs = reinterpret_cast<const int32_t*>(I.st[c])[4 * RS_W * PS + sl];
  const int i = pos_of_slot(hs, I.C, I.nt);
  if (rho) rho[i] = r[RS_RU * PS].x;
  if (u) u[i] = r[RS_RU * PS].y;
  if (fr) fr[i] = r[RS_F * PS].x;
  if (fu) fu[i] = r[RS_F * PS].y;
}

// Injected state (by id) at position = id in buffer 0; the marcher orders
// it before its first slice.  Interval hints start at the rings' nodes.
__global__ void state_set_kernel(WakeInst I, const double* rho, const double* u, const double* fr,
                                 const double* fu, int slice) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) { I.ctl[CTL_CUR] = 0; I.ctl[CTL_BREAK] = -1; I.ctl[CTL_NEXT] = slice; I.ctl[CTL_FAULT] = 0; }
  if (i >= I.N) return;
  const unsigned sl = slot_of(i, I.C, I.nt);
  const size_t PS = (size_t)I.G * I.C * I.nt;
  D2* r = reinterpret_cast<D2*>(I.st[0]) + sl;
  const D2* k = reinterpret_cast<const D2*>(I.cst) + sl;
  const dd lr = ring_log(k[RC_R0 * PS], k[RC_LN * PS], rho[i]);
  r[RS_RU * PS] = d2(rho[i], u[i]);
  r[RS_F * PS] = d2(fr ? fr[i] : 0.0, fu ? fu[i] : 0.0);
  r[RS_LN * PS] = d2(lr.hi, lr.lo);
  int32_t* wd = reinterpret_cast<int32_t*>(I.st[0]) + 4 * RS_W * PS;
  wd[sl] = (int32_t)sl;
  wd[PS + sl] = i + 1;
}

// Back to the state at slice 0 (rings at rest at their initial radii);
// one workgroup per instance.
__global__ void state_reset_kernel(const WakeInst* __restrict__ insts, int n_insts) {
  const WakeInst& I = insts[blockIdx.x];
  for (int j = threadIdx.x; j < I.N; j += blockDim.x) {
    const unsigned sl = slot_of(j, I.C, I.nt);
    const size_t PS = (size_t)I.G * I.C * I.nt;
    D2* r = reinterpret_cast<D2*>(I.st[0]) + sl;
    const D2* k = reinterpret_cast<const D2*>(I.cst) + sl;
    r[RS_RU * PS] = d2(k[RC_R0 * PS].x, 0.0);
    r[RS_F * PS] = d2(0.0, 0.0);
    r[RS_LN * PS] = k[RC_LN * PS];
    int32_t* wd = reinterpret_cast<int32_t*>(I.st[0]) + 4 * RS_W * PS;
    wd[sl] = (int32_t)sl;
    wd[PS + sl] = j + 1;
  }
  if (threadIdx.x == 0) { I.ctl[CTL_CUR] = 0; I.ctl[CTL_BREAK] = -1; I.ctl[CTL_NEXT] = 0; I.ctl[CTL_FAULT] = 0; }
}

// Control words of a list of instances into one buffer (4 words each).
__global__ void ctl_gather_kernel(const WakeInst* __restrict__ insts, int n, int32_t* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  for (int w = 0; w < CTL_NWORDS; ++w) out[i * CTL_NWORDS + w] = insts[i].ctl[w];
}

// ---------------------------------------------------------------------------
// host-callable launchers
// ---------------------------------------------------------------------------
struct RowsOut {
  double* q[OUT_N];
};
__global__ void rows_out_kernel(const double* __restrict__ src, size_t n, RowsOut dst) {
  double* const d = dst.q[blockIdx.y];
  if (!d) return;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    d[i] = src[blockIdx.y * n + i];
}
__global__ void axis_out_kernel(const double* __restrict__ axis, size_t n, double* psi, double* ez) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    if (psi) psi[i] = axis[2 * i];
    if (ez) ez[i] = axis[2 * i + 1];
  }
}
static unsigned out_blocks(size_t n) { return (unsigned)std::min<size_t>(std::max<size_t>((n + 255) / 256, 1), 1024); }
hipError_t launch_rows_out(const double* src, size_t n, double* const* dst, int rows, hipStream_t s) {
  RowsOut o = {};
  for (int q = 0; q < rows && q < OUT_N; ++q) o.q[q] = dst[q];
  hipLaunchKernelGGL(rows_out_kernel, dim3(out_blocks(n), rows), dim3(256), 0, s, src, n, o);
  return hipGetLastError();
}
hipError_t launch_axis_out(const double* axis, size_t n, double* psi, double* ez, hipStream_t s) {
  hipLaunchKernelGGL(axis_out_kernel, dim3(out_blocks(n)), dim3(256), 0, s, axis, n, psi, ez);
  return hipGetLastError();
}

hipError_t launch_ctl_gather(const WakeInst* d_insts, int n, int32_t* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(ctl_gather_kernel, dim3((n + 255) / 256), dim3(256), 0, s, d_insts, n, out);
  return hipGetLastError();
}

hipError_t launch_init(const WakeInst& I, const double* r0, const double* dr, const double* dens,
                       hipStream_t s) {
  // block totals / offsets in the fix-up's scratch (4 doubles per block of 256 rings)
  const int nb = (I.N + 255) / 256;
  double* tmp = I.sm_r;
  hipLaunchKernelGGL((init_rings_kernel<256>), dim3(nb), dim3(256), 0, s, I, r0, dr, dens, tmp);
  hipLaunchKernelGGL(init_offsets_kernel, dim3(1), dim3(64), 0, s, I, tmp, nb);
  hipLaunchKernelGGL((init_nodes_kernel<256>), dim3(nb), dim3(256), 0, s, I, (const double*)tmp);
  hipLaunchKernelGGL(init_intervals_kernel, dim3((I.N + 1 + 255) / 256), dim3(256), 0, s, I);
  return hipGetLastError();
}

// Field-grid node table: ln r_g and the immobile ions' psi - psi(0) and
// d_rho psi at r_g (the same interpolation as at the rings), dd pairs.  The
// table is made once per grid, so psi's interpolation is carried out in
// double-double throughout: the weight t = (r - lo)/(hi - lo) from exact
// differences and the step between the nodes' double-double values (at the
// rings the step is rounded to double, which resolves psi to ~1e-16 of the
// step; nodes between rings at rest see psi of order w dr^2 only).
__global__ void grid_init_kernel(WakeInst I, double* tab, int n_entries) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n_entries) return;
  const double r = I.grid_rad ? I.grid_rad[g] : ((double)g + 0.5) * I.grid_dr;
  const dd l = dd_log(r);
  IonView IV;
  IV.R = uview(I.ion);
  IV.N = I.N;
  IV.Rp = I.Rp;
  IV.T0 = {I.tot0[0], I.tot0[1]};
  IV.Q = {I.tot0[2], I.tot0[3]};
  int h = 0;
  double q[WAKE_ION_REC];
  ion_load(IV, h, q);
  const Lerp x = ion_fields(IV, r, l, h, q);
  dd ps = {x.ph, x.pl};
  const dd dp = dd_add_d({x.dh, x.dl}, x.t * x.ds);
  if (r < I.Rp) {
    const dd a = two_sum(r, -q[IR_LO]);            // r - lo, exact
    const dd b = two_sum(q[IR_HI], -q[IR_LO]);     // hi - lo, exact
    dd t = dd_div_d(a, b.hi);
    t = dd_add_d(t, -t.hi * b.lo / b.hi);          // a / (b.hi + b.lo) to second order
    dd nxt;                                         // psi - psi(0) at the upper node
    if (h < I.N) {
      nxt = {I.ion[(size_t)(h + 1) * WAKE_ION_REC + IR_PSH], I.ion[(size_t)(h + 1) * WAKE_ION_REC + IR_PSL]};
    } else {                                        // the plasma edge: exterior value there
      nxt = dd_sub(IV.T0, dd_mul(IV.Q, dd_log(I.Rp)));
    }
    const dd lo_ps = {q[IR_PSH], q[IR_PSL]};
    ps = dd_add(lo_ps, dd_mul(dd_sub(nxt, lo_ps), t));
  }
  double* t = tab + (size_t)WAKE_GRID_TAB * g;
  t[0] = l.hi; t[1] = l.lo;
  t[2] = ps.hi; t[3] = ps.lo;
  t[4] = dp.hi; t[5] = dp.lo;
}

hipError_t launch_grid_init(const WakeInst& I, double* tab, int n_entries, hipStream_t s) {
  if (n_entries <= 0) return hipSuccess;
  hipLaunchKernelGGL(grid_init_kernel, dim3((n_entries + 255) / 256), dim3(256), 0, s, I, tab, n_entries);
  return hipGetLastError();
}

hipError_t launch_reset(const WakeInst* d_insts, int n_insts, hipStream_t s) {
  if (n_insts <= 0) return hipSuccess;
  hipLaunchKernelGGL(state_reset_kernel, dim3(n_insts), dim3(256), 0, s, d_insts, n_insts);
  return hipGetLastError();
}

hipError_t launch_state_by_id(const WakeInst& I, double* rho, double* u, double* fr, double* fu,
                              hipStream_t s) {
  hipLaunchKernelGGL(state_by_id_kernel, dim3((I.N + 255) / 256), dim3(256), 0, s, I, rho, u, fr, fu);
  return hipGetLastError();
}

hipError_t launch_state_set(const WakeInst& I, const double* rho, const double* u, const double* fr,
                            const double* fu, int slice, hipStream_t s) {
  hipLaunchKernelGGL(state_set_kernel, dim3((I.N + 255) / 256), dim3(256), 0, s, I, rho, u, fr, fu,
                     slice);
  return hipGetLastError();
}

#define WAKE_THREADS(X) X(256) X(512)

size_t march_lds_bytes(int nt) {
#define X(a) \
  if (nt == a) return MarchLds<a>::bytes();
  WAKE_THREADS(X)
#undef X
  return 0;
}

hipError_t launch_march(int nt, const WakeInst* d_insts, int n_insts, int n_tasks, int32_t* counter,
                        int grid, int grid_mode, hipStream_t s) {
#define X(a)                                                                                      \
  if (nt == a) {                                                                                  \
    hipLaunchKernelGGL(counter_zero_kernel, dim3(1), dim3(64), 0, s, counter);                     \
    hipLaunchKernelGGL(cluster_reset_kernel, dim3(1), dim3(256), 0, s, d_insts, n_insts);          \
    if (grid_mode == 2)                                                                           \
      hipLaunchKernelGGL((wake_march_kernel<a, 2>), dim3(grid), dim3(a),                          \
                         MarchLds<a>::bytes() + grid_lds_bytes<a>(), s, d_insts, n_insts, n_tasks, \
                         counter);                                                                \
    else if (grid_mode == 1)                                                                      \
      hipLaunchKernelGGL((wake_march_kernel<a, 1>), dim3(grid), dim3(a),                          \
                         MarchLds<a>::bytes() + grid_lds_bytes<a>(), s, d_insts, n_insts, n_tasks, \
                         counter);                                                                \
    else                                                                                          \
      hipLaunchKernelGGL((wake_march_kernel<a, 0>), dim3(grid), dim3(a), MarchLds<a>::bytes(),    \
                         s, d_insts, n_insts, n_tasks, counter);                                  \
    return hipGetLastError();                                                                     \
  }
  WAKE_THREADS(X)
#undef X
  return hipErrorInvalidValue;
}

int march_cmax(int nt) {
#define X(a) \
  if (nt == a) return MarchLds<a>::CMAX;
  WAKE_THREADS(X)
#undef X
  return 0;
}

int march_occupancy(int nt) {
  int nb = 0;
#define X(a)                                                                                      \
  if (nt == a) {                                                                                  \
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, wake_march_kernel<a, 0>, a,         \
                                                     MarchLds<a>::bytes()) != hipSuccess)         \
      return 0;                                                                                   \
    return nb;                                                                                    \
  }
  WAKE_THREADS(X)
#undef X
  return 0;
}

hipError_t march_prepare(int nt) {
#define X(a)                                                                                      \
  if (nt == a) {                                                                                  \
    hipError_t e = hipFuncSetAttribute((const void*)wake_march_kernel<a, 0>,                      \
                                       hipFuncAttributeMaxDynamicSharedMemorySize,                \
                                       (int)MarchLds<a>::bytes());                                \
    if (e != hipSuccess) return e;                                                                \
    e = hipFuncSetAttribute((const void*)wake_march_kernel<a, 1>,                                 \
                            hipFuncAttributeMaxDynamicSharedMemorySize,                           \
                            (int)(MarchLds<a>::bytes() + grid_lds_bytes<a>()));                   \
    if (e != hipSuccess) return e;                                                                \
    return hipFuncSetAttribute((const void*)wake_march_kernel<a, 2>,                              \
                               hipFuncAttributeMaxDynamicSharedMemorySize,                        \
                               (int)(MarchLds<a>::bytes() + grid_lds_bytes<a>()));                \
  }
  WAKE_THREADS(X)
#undef X
  return hipErrorInvalidValue;
}

bool march_threads_ok(int nt) {
#define X(a) \
  if (nt == a) return true;
  WAKE_THREADS(X)
#undef X
  return false;
}
