// Device-side building blocks for the gfx950 ring solver: double-double
// arithmetic, 64-wide wavefront and workgroup scans, and ring-key order.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// The workgroup's dynamic LDS, named once so that code reached through a
// call (not only the kernel itself) addresses it as LDS rather than through
// flat pointers.
extern __shared__ __align__(16) unsigned char wake_lds[];

#define WAKE_GLOBAL __attribute__((address_space(1)))
// A device array's pointer in the global address space (64-bit indexing), so
// that its accesses take global rather than flat instructions (a flat access
// waits for both the memory and the LDS counters).
template <class T>
__device__ __forceinline__ WAKE_GLOBAL T* gptr(T* q) {
  return reinterpret_cast<WAKE_GLOBAL T*>(reinterpret_cast<uint64_t>(q));
}
// An object in device memory handed to a function that is not inlined, typed
// so that the callee reads it with global instructions.
template <class T>
__device__ __forceinline__ const WAKE_GLOBAL T* as_global(const T& x) {
  return (const WAKE_GLOBAL T*)&x;
}

// A per-instance array seen as uniform: its base in scalar registers and in
// the global address space, indexed with 32-bit element offsets (loads and
// stores then take the scalar-base + vector-offset form).
template <class T>
struct GA {
  WAKE_GLOBAL T* p;
  __device__ __forceinline__ T operator[](uint32_t i) const {
    return *reinterpret_cast<WAKE_GLOBAL T*>(reinterpret_cast<WAKE_GLOBAL char*>(p) +
                                            i * (uint32_t)sizeof(T));
  }
  __device__ __forceinline__ void st(uint32_t i, T v) const {
    *reinterpret_cast<WAKE_GLOBAL T*>(reinterpret_cast<WAKE_GLOBAL char*>(p) +
                                     i * (uint32_t)sizeof(T)) = v;
  }
};
template <class T>
__device__ __forceinline__ GA<T> uview(const T* q) {
  const uint64_t v = reinterpret_cast<uint64_t>(q);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  GA<T> g;
  g.p = reinterpret_cast<WAKE_GLOBAL T*>(((uint64_t)hi << 32) | lo);
  return g;
}
// 16-B chunk of a record (two doubles), moved by one 16-B load or store.
typedef double D2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ D2 d2(double x, double y) {
  D2 r;
  r.x = x;
  r.y = y;
  return r;
}
// ---------------------------------------------------------------------------
// double-double (unevaluated sum hi + lo) arithmetic.  Contraction of a
// multiply into an addition is forbidden inside every helper: after
// inlining, `a + b` in two_sum would otherwise fuse with a caller's product
// b = x*y into fma(x, y, a), and the error term would no longer describe the
// rounded sum.  The product error uses an explicit fma.
// ---------------------------------------------------------------------------
struct dd {
  double hi, lo;
};

__device__ __forceinline__ dd dd_make(double a) { return {a, 0.0}; }

__device__ __forceinline__ dd two_sum(double a, double b) {
  _Pragma("clang fp contract(off)")
  double s = a + b;
  double bb = s - a;
  double e = (a - (s - bb)) + (b - bb);
  return {s, e};
}

__device__ __forceinline__ dd fast_two_sum(double a, double b) {
  _Pragma("clang fp contract(off)")
  double s = a + b;
  double e = b - (s - a);
  return {s, e};
}

__device__ __forceinline__ dd two_prod(double a, double b) {
  _Pragma("clang fp contract(off)")
  double p = a * b;
  double e = __builtin_fma(a, b, -p);
  return {p, e};
}

__device__ __forceinline__ dd dd_add(dd a, dd b) {
  _Pragma("clang fp contract(off)")
  dd s = two_sum(a.hi, b.hi);
  dd t = two_sum(a.lo, b.lo);
  s.lo += t.hi;
  s = fast_two_sum(s.hi, s.lo);
  s.lo += t.lo;
  return fast_two_sum(s.hi, s.lo);
}

// Sum with one two_sum of the high parts and the low parts added in
// double: the error stays within a few units of 2^-104 (|a| + |b|), which
// is all the field sums need (they end rounded to double).
__device__ __forceinline__ dd dd_add_fast(dd a, dd b) {
  _Pragma("clang fp contract(off)")
  dd s = two_sum(a.hi, b.hi);
  s.lo += a.lo + b.lo;
  return fast_two_sum(s.hi, s.lo);
}

// 1/x from the hardware reciprocal estimate refined by two Newton steps
// (e = 1 - x r, r += r e): within about an ulp of the rounded quotient,
// without the IEEE division sequence.  x = 0 or +-inf give NaN.
__device__ __forceinline__ double rcp_nr(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = __builtin_fma(-x, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-x, r, 1.0);
  return __builtin_fma(r, e, r);
}

__device__ __forceinline__ dd dd_neg(dd a) { return {-a.hi, -a.lo}; }
__device__ __forceinline__ dd dd_sub(dd a, dd b) { return dd_add(a, dd_neg(b)); }

__device__ __forceinline__ dd dd_add_d(dd a, double b) {
  _Pragma("clang fp contract(off)")
  dd s = two_sum(a.hi, b);
  s.lo += a.lo;
  return fast_two_sum(s.hi, s.lo);
}

__device__ __forceinline__ dd dd_mul_d(dd a, double b) {
  _Pragma("clang fp contract(off)")
  dd p = two_prod(a.hi, b);
  p.lo = __builtin_fma(a.lo, b, p.lo);
  return fast_two_sum(p.hi, p.lo);
}

__device__ __forceinline__ dd dd_div_d(dd a, double b) {
  _Pragma("clang fp contract(off)")
  double q1 = a.hi / b;
  dd r = dd_sub(a, two_prod(q1, b));
  double q2 = r.hi / b;
  return fast_two_sum(q1, q2);
}

__device__ __forceinline__ double dd_round(dd a) {
  _Pragma("clang fp contract(off)") return a.hi + a.lo; }

__device__ __forceinline__ dd dd_mul(dd a, dd b) {
  _Pragma("clang fp contract(off)")
  dd p = two_prod(a.hi, b.hi);
  p.lo = __builtin_fma(a.hi, b.lo, __builtin_fma(a.lo, b.hi, p.lo));
  return fast_two_sum(p.hi, p.lo);
}

// ln(1 + d) for d > -1 in a few dozen operations, to a few ulp:
// 1 + d = m + c exactly (two_sum), m = 2^k f with f in [sqrt(1/2), sqrt(2)),
// ln f = 2 atanh(s) with s = (f - 1) / (f + 1) (|s| < 0.172) summed by its
// Taylor series through s^25 (the next term is below 2^-64 of the sum), and
// ln(1 + d) = k ln 2 + ln f + c / m.  m <= 0 gives NaN.
__device__ __forceinline__ double log1p_fast(double d) {
  _Pragma("clang fp contract(off)")
  if (fabs(d) < 0.00390625) {
    // a slice's step away from the axis: the alternating series through
    // d^7 / 7 (the next term is below 2^-59 of d); half the operations of
    // the atanh form, and no reciprocal
    double p = 1.0 / 7.0;
    p = __builtin_fma(p, d, -1.0 / 6.0);
    p = __builtin_fma(p, d, 1.0 / 5.0);
    p = __builtin_fma(p, d, -1.0 / 4.0);
    p = __builtin_fma(p, d, 1.0 / 3.0);
    p = __builtin_fma(p, d, -0.5);
    return __builtin_fma(d * d, p, d);
  }
  if (fabs(d) < 0.03125) {
    // small steps (the push's common case): 2 atanh(s), s = d / (2 + d),
    // without the range reduction; |s| < 0.016, so the series' first
    // omitted term, 2 s z^5 / 11, is below 1e-19 of the result
    const double s = d * rcp_nr(2.0 + d);
    const double z = s * s;
    double p = 1.0 / 9.0;
    p = __builtin_fma(p, z, 1.0 / 7.0);
    p = __builtin_fma(p, z, 1.0 / 5.0);
    p = __builtin_fma(p, z, 1.0 / 3.0);
    const double two_s = s + s;
    return __builtin_fma(two_s * z, p, two_s);
  }
  const dd mc = two_sum(1.0, d);
  const double m = mc.hi;
  int k = __builtin_amdgcn_frexp_exp(m);
  double f = __builtin_amdgcn_frexp_mant(m);            // [0.5, 1)
  if (f < 0.70710678118654752440) { f = f + f; k -= 1; }
  const double s = (f - 1.0) * rcp_nr(f + 1.0);
  const double z = s * s;
  double p = 1.0 / 25.0;
  p = __builtin_fma(p, z, 1.0 / 23.0);
  p = __builtin_fma(p, z, 1.0 / 21.0);
  p = __builtin_fma(p, z, 1.0 / 19.0);
  p = __builtin_fma(p, z, 1.0 / 17.0);
  p = __builtin_fma(p, z, 1.0 / 15.0);
  p = __builtin_fma(p, z, 1.0 / 13.0);
  p = __builtin_fma(p, z, 1.0 / 11.0);
  p = __builtin_fma(p, z, 1.0 / 9.0);
  p = __builtin_fma(p, z, 1.0 / 7.0);
  p = __builtin_fma(p, z, 1.0 / 5.0);
  p = __builtin_fma(p, z, 1.0 / 3.0);
  const double two_s = s + s;
  const double lf = __builtin_fma(two_s * z, p, two_s);     // 2 s (1 + z p)
  const double LN2_HI = 6.93147180559945286227e-01, LN2_LO = 2.31904681384629955842e-17;
  const double kd = (double)k;
  const double tail = __builtin_fma(kd, LN2_LO, lf + mc.lo * rcp_nr(m));
  const double r = __builtin_fma(kd, LN2_HI, tail);
  return m > 0.0 ? r : __builtin_nan("");
}

// exp(x) to double-double accuracy (|x| < 700): x = k ln2 + t with
// |t| <= ln2/2, Taylor series of e^t in double-double, scaled by 2^k.
__device__ inline dd dd_exp(double x) {
  _Pragma("clang fp contract(off)")
  const dd LN2 = {6.93147180559945286227e-01, 2.31904681384629955842e-17};
  const double kf = rint(x / LN2.hi);
  const dd t = dd_sub(dd_make(x), dd_mul_d(LN2, kf));
  dd term = {1.0, 0.0}, sum = {1.0, 0.0};
  for (int n = 1; n <= 27; ++n) {
    term = dd_div_d(dd_mul(term, t), (double)n);
    sum = dd_add(sum, term);
  }
  const int k = (int)kf;
  return {ldexp(sum.hi, k), ldexp(sum.lo, k)};
}

// ln(r) to double-double accuracy for r > 0: one Newton step on e^y = r
// from the binary64 logarithm.
__device__ inline dd dd_log(double r) {
  _Pragma("clang fp contract(off)")
  const double y = log(r);
  const dd e = dd_exp(y);
  const dd d = dd_sub(dd_make(r), e);
  return two_sum(y, d.hi / e.hi);
}

// ---------------------------------------------------------------------------
// single values moved between lanes of a wave
// ---------------------------------------------------------------------------
// Value of lane (lane ^ lm) of the wave, lm in {1, 2, 4, 8, 16, 32}, by
// register-level moves (DPP within rows of 16 lanes, lane-swap instructions
// across rows and halves) rather than through the LDS crossbar.
__device__ __forceinline__ uint32_t lane_xor(uint32_t x, int lm) {
  const int lane = threadIdx.x & 63;
  switch (lm) {
    case 1: return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true);   // quad_perm 1,0,3,2
    case 2: return __builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, true);   // quad_perm 2,3,0,1
    case 4: {
      const uint32_t up = __builtin_amdgcn_mov_dpp(x, 0x104, 0xF, 0xF, true);   // from lane + 4
      const uint32_t dn = __builtin_amdgcn_mov_dpp(x, 0x114, 0xF, 0xF, true);   // from lane - 4
      return (lane & 4) ? dn : up;
    }
    case 8: return __builtin_amdgcn_mov_dpp(x, 0x128, 0xF, 0xF, true);  // rotate row by 8
    case 16: {
      const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
      return (lane & 16) ? r[0] : r[1];
    }
    default: {
      const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
      return (lane & 32) ? r[0] : r[1];
    }
  }
}
// Value of the next (lane + 1) or previous (lane - 1) lane of the wave (a
// whole-wave DPP shift; the last / first lane reads 0).
__device__ __forceinline__ uint32_t lane_next(uint32_t x) { return __builtin_amdgcn_mov_dpp(x, 0x130, 0xF, 0xF, true); }
__device__ __forceinline__ uint32_t lane_prev(uint32_t x) { return __builtin_amdgcn_mov_dpp(x, 0x138, 0xF, 0xF, true); }
__device__ __forceinline__ double lane_next(double x) {
  const uint64_t v = (uint64_t)__double_as_longlong(x);
  const uint32_t lo = lane_next((uint32_t)v), hi = lane_next((uint32_t)(v >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ double lane_prev(double x) {
  const uint64_t v = (uint64_t)__double_as_longlong(x);
  const uint32_t lo = lane_prev((uint32_t)v), hi = lane_prev((uint32_t)(v >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ double lane_xor(double x, int lm) {
  const uint64_t v = (uint64_t)__double_as_longlong(x);
  const uint32_t lo = lane_xor((uint32_t)v, lm), hi = lane_xor((uint32_t)(v >> 32), lm);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// lane_next and lane_prev of a radius with +inf after the last lane, -inf
// before the first: no lane-edge cases in the compares
__device__ __forceinline__ double lane_next_inf(double x) {
  const uint64_t v = (uint64_t)__double_as_longlong(x);
  const uint32_t lo = lane_next((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0x7ff00000u, (uint32_t)(v >> 32), 0x130, 0xF, 0xF, false);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ double lane_prev_inf(double x) {
  const uint64_t v = (uint64_t)__double_as_longlong(x);
  const uint32_t lo = lane_prev((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0xfff00000u, (uint32_t)(v >> 32), 0x138, 0xF, 0xF, false);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// ---------------------------------------------------------------------------
// 256 rings put in (radius, id) order by one wave: four per lane (lane l:
// positions 4l..4l+3), r the radii, k a word that goes with each; positions
// past the last ring hold +inf and k = ~0
// ---------------------------------------------------------------------------
// The order fix-ups are bound by vector issue (7900 rings on one workgroup:
// 12 of 31 blocks out of order per slice, half of them by more than 32
// positions), so the networks compare radii alone, one instruction where
// (radius, id) took three and two scalar ones on the path to each exchange;
// rings of equal radius, which hardly occur, are put in the order of their
// ids afterwards.  The sort of a block in LDS 2457 -> 1795 instructions, a
// merge 699; 7900 rings once they cross 87.2 -> 80.3 us per slice, 20000 rings
// on 5 members 57 -> 52, on 40 members 32.0 -> 29.0, 4000 rings of two species
// 82.5 -> 78.7.  (Now 7900 rings 81.2, with the barrier before the merges, and
// 4000 of two species 89.1, with their sums exact.)
// Exchanges go by lane masks in scalar registers: left to itself the compiler
// made branches of them, or masks of vector registers.
__device__ __forceinline__ uint64_t lanes_lt(double a, double b) { return __builtin_amdgcn_ballot_w64(a < b); }
__device__ __forceinline__ void wave_take(uint64_t m, double& r, uint32_t& k, double pr, uint32_t pk) {
  const bool t = __builtin_amdgcn_inverse_ballot_w64(m);
  r = t ? pr : r;
  k = t ? pk : k;
}
__device__ __forceinline__ void wave_swap(uint64_t m, double& ra, uint32_t& ka, double& rb, uint32_t& kb) {
  const double r = ra;
  const uint32_t k = ka;
  wave_take(m, ra, ka, rb, kb);
  wave_take(m, rb, kb, r, k);
}
// lanes whose bits of x are all clear
__device__ constexpr uint64_t lanes_clear(int x) {
  uint64_t m = 0;
  for (int l = 0; l < 64; ++l) m |= (uint64_t)((l & x) == 0) << l;
  return m;
}
__device__ __forceinline__ bool wave_ascending(const double* r) {
  const double x = lane_next_inf(r[0]);
  return (lanes_lt(r[1], r[0]) | lanes_lt(r[2], r[1]) | lanes_lt(r[3], r[2]) | lanes_lt(x, r[3])) == 0;
}
// rings of equal radius (r ascending) in the order of id(k); whether any moved
template <class IdOf>
__device__ __forceinline__ bool wave_ties(const double* r, uint32_t* k, IdOf id) {
  const double x = lane_next_inf(r[0]), w = lane_prev_inf(r[3]);
  const bool e0 = (r[0] == r[1]) & (r[1] < INFINITY), e1 = (r[1] == r[2]) & (r[2] < INFINITY),
             e2 = (r[2] == r[3]) & (r[3] < INFINITY), e3 = (r[3] == x) & (x < INFINITY);
  if (!__any(e0 | e1 | e2 | e3)) return false;
  const bool em = (r[0] == w) & (r[0] < INFINITY);
  uint32_t i[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) i[j] = k[j] == ~0u ? ~0u : (uint32_t)id(k[j]);
  bool moved = false;
  // odd-even transposition within the runs of equal radii (at most 256 long)
  #pragma unroll 1
  for (int it = 0; it < 128; ++it) {
    bool m = false;
    auto swap = [&](int a, int b) {
      uint32_t t = i[a]; i[a] = i[b]; i[b] = t;
      t = k[a]; k[a] = k[b]; k[b] = t;
      m = true;
    };
    if (e0 && i[1] < i[0]) swap(0, 1);
    if (e2 && i[3] < i[2]) swap(2, 3);
    if (e1 && i[2] < i[1]) swap(1, 2);
    const uint32_t ni = lane_next(i[0]), nk = lane_next(k[0]), pi = lane_prev(i[3]), pk = lane_prev(k[3]);
    if (e3 && ni < i[3]) { i[3] = ni; k[3] = nk; m = true; }
    if (em && i[0] < pi) { i[0] = pi; k[0] = pk; m = true; }
    if (!__any(m)) break;
    moved = true;
  }
  return moved;
}
__device__ __forceinline__ void lanes_swap(int lm, uint32_t& a, uint32_t& b) {
  const auto v = lm == 16 ? __builtin_amdgcn_permlane16_swap(a, b, false, false)
                          : __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = v[0];
  b = v[1];
}
__device__ __forceinline__ void lanes_swap(int lm, double& ra, uint32_t& ka, double& rb, uint32_t& kb) {
  const uint64_t x = (uint64_t)__double_as_longlong(ra), y = (uint64_t)__double_as_longlong(rb);
  uint32_t xl = (uint32_t)x, xh = (uint32_t)(x >> 32), yl = (uint32_t)y, yh = (uint32_t)(y >> 32);
  lanes_swap(lm, xl, yl);
  lanes_swap(lm, xh, yh);
  lanes_swap(lm, ka, kb);
  ra = __longlong_as_double((long long)(((uint64_t)xh << 32) | xl));
  rb = __longlong_as_double((long long)(((uint64_t)yh << 32) | yl));
}
// compare-exchange stage of a bitonic network at distance d, ascending where
// (position & kk) == 0 (kk = 256: everywhere)
__device__ __forceinline__ void wave_stage(double* r, uint32_t* k, int kk, int d) {
  if (d >= 64) {
    // partner 16 or 32 lanes away: two registers' pairs brought into lanes of
    // their own (the swap exchanges the first's upper rows with the second's
    // lower ones), exchanged there, and taken back
    const uint64_t up = lanes_clear(kk >> 2 & 63);
#pragma unroll
    for (int j = 0; j < 4; j += 2) {
      lanes_swap(d >> 2, r[j], k[j], r[j + 1], k[j + 1]);
      wave_swap(~(lanes_lt(r[j + 1], r[j]) ^ up), r[j], k[j], r[j + 1], k[j + 1]);
      lanes_swap(d >> 2, r[j], k[j], r[j + 1], k[j + 1]);
    }
  } else if (d >= 4) {                // partner in lane ^ (d / 4), same register
    const int lm = d >> 2;
    // the smaller stays where the lane is the lower one of an ascending pair
    // or the upper one of a descending pair (kk >= 8 here: the same for a
    // lane's four positions); equal radii stay
    const uint64_t sm = ~(lanes_clear(lm) ^ lanes_clear(kk >> 2 & 63));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const double pr = lane_xor(r[j], lm);
      const uint32_t pk = lane_xor(k[j], lm);
      wave_take((lanes_lt(pr, r[j]) & sm) | (lanes_lt(r[j], pr) & ~sm), r[j], k[j], pr, pk);
    }
  } else {                            // partner in this lane
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j & d) continue;
      const int jj = j | d;
      const uint64_t up = kk < 4 ? ((j & kk) == 0 ? ~0ull : 0ull) : lanes_clear(kk >> 2 & 63);
      wave_swap(~(lanes_lt(r[jj], r[j]) ^ up), r[j], k[j], r[jj], k[jj]);
    }
  }
}
// Place in the block of a lane's register j when it is loaded: its own
// position; for a merge the second half in reverse, which makes the block
// bitonic.
template <bool MERGE>
__device__ __forceinline__ int wave_place(int j) {
  const int q = 4 * (threadIdx.x & 63) + j;
  return MERGE && q >= 128 ? 383 - q : q;
}
// The block (loaded by wave_place) in order; false if it was already, and
// then nothing may be written back.  Odd-even transposition first: the rings
// of a run of length L reach their places within L phases and never cross a
// run boundary, so blocks with short runs (the common case) are done after a
// few phases.  Order checked every four phases; a block still out of order
// after 32 phases goes through the full bitonic network.  MERGE: the two
// halves are each in order, and the half-cleaning stages of a bitonic merge
// do.
template <bool MERGE, class IdOf>
__device__ __forceinline__ bool wave_sort256(double* r, uint32_t* k, IdOf id) {
  bool moved = true;
  if constexpr (MERGE) {
    // the last radius of the first half against the first of the second
    const uint64_t v = (uint64_t)__double_as_longlong(r[3]);
    const uint64_t x = (uint64_t)__builtin_amdgcn_readlane((uint32_t)(v >> 32), 31) << 32 |
                       (uint32_t)__builtin_amdgcn_readlane((uint32_t)v, 31);
    const uint64_t y = (uint64_t)__builtin_amdgcn_readlane((uint32_t)(v >> 32), 63) << 32 |
                       (uint32_t)__builtin_amdgcn_readlane((uint32_t)v, 63);
    if (lanes_lt(__longlong_as_double((long long)x), __longlong_as_double((long long)y)) != 0) return false;
#pragma unroll
    for (int d = 128; d > 0; d >>= 1) wave_stage(r, k, 256, d);
  } else {
    moved = !wave_ascending(r);
    bool done = !moved;
    #pragma unroll 1
    for (int it = 0; it < 8 && !done; ++it) {
#pragma unroll
      for (int ph = 0; ph < 2; ++ph) {
        // even phase: (0,1) (2,3); odd phase: (1,2) and (3 | next lane's 0)
        wave_swap(lanes_lt(r[1], r[0]), r[0], k[0], r[1], k[1]);
        wave_swap(lanes_lt(r[3], r[2]), r[2], k[2], r[3], k[3]);
        wave_swap(lanes_lt(r[2], r[1]), r[1], k[1], r[2], k[2]);
        const double nr = lane_next_inf(r[0]), pr = lane_prev_inf(r[3]);
        const uint32_t nk = lane_next(k[0]), pk = lane_prev(k[3]);
        wave_take(lanes_lt(nr, r[3]), r[3], k[3], nr, nk);      // the smaller of the pair
        wave_take(lanes_lt(r[0], pr), r[0], k[0], pr, pk);      // the larger
      }
      done = wave_ascending(r);
    }
    if (!done) {
#pragma unroll
      for (int kk = 2; kk <= 256; kk <<= 1) {
#pragma unroll
        for (int d = kk >> 1; d > 0; d >>= 1) wave_stage(r, k, kk, d);
      }
    }
  }
  return wave_ties(r, k, id) || moved;
}

// ---------------------------------------------------------------------------
// packs of doubles moved through cross-lane shuffles and LDS
// ---------------------------------------------------------------------------
template <int NF>
struct Pack {
  double v[NF];
};

// ---------------------------------------------------------------------------
// Wave-level scans on DPP row shifts (lanes of a 16-lane row) and lane reads
// (across rows), then one LDS exchange of the wave totals per workgroup.
// ---------------------------------------------------------------------------
// DPP move of each double of a pack (two 32-bit halves).  CTRL 0x110 + d:
// lane i reads lane i - d of its row; 0x100 + d: lane i + d; 0x138 / 0x130:
// the previous / next lane of the wave.  Lanes with no source read 0.  A
// DPP read from a lane that is switched off reads 0 too, so these moves are
// always evaluated with the whole wave active, never as one operand of ?:
// or && (which evaluates it under a partial mask).
template <int CTRL>
__device__ __forceinline__ double dpp_d(double x) {
  const long long v = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(v >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <int CTRL, int NF>
__device__ __forceinline__ Pack<NF> dpp_pack(const Pack<NF>& p) {
  Pack<NF> r;
#pragma unroll
  for (int i = 0; i < NF; ++i) r.v[i] = dpp_d<CTRL>(p.v[i]);
  return r;
}
// the pack of lane l (l uniform over the wave)
template <int NF>
__device__ __forceinline__ Pack<NF> lane_pack(const Pack<NF>& p, int l) {
  Pack<NF> r;
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    const long long v = __double_as_longlong(p.v[i]);
    const int lo = __builtin_amdgcn_readlane((int)v, l);
    const int hi = __builtin_amdgcn_readlane((int)(v >> 32), l);
    r.v[i] = __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
  }
  return r;
}
template <int NF>
__device__ __forceinline__ Pack<NF> pick(bool c, const Pack<NF>& a, const Pack<NF>& b) {
  Pack<NF> r;
#pragma unroll
  for (int i = 0; i < NF; ++i) r.v[i] = c ? a.v[i] : b.v[i];
  return r;
}

// Inclusive prefix within each 16-lane row over the first M lanes of the
// row (M <= 16), op(earlier, later).
template <int M, int NF, class Op>
__device__ __forceinline__ Pack<NF> row_prefix_incl(Pack<NF> inc, Op op) {
  const int lr = threadIdx.x & 15;
  if (M > 1) { const Pack<NF> o = dpp_pack<0x111>(inc); if (lr >= 1) inc = op(o, inc); }
  if (M > 2) { const Pack<NF> o = dpp_pack<0x112>(inc); if (lr >= 2) inc = op(o, inc); }
  if (M > 4) { const Pack<NF> o = dpp_pack<0x114>(inc); if (lr >= 4) inc = op(o, inc); }
  if (M > 8) { const Pack<NF> o = dpp_pack<0x118>(inc); if (lr >= 8) inc = op(o, inc); }
  return inc;
}
// Inclusive suffix within each row over its first M lanes, op(lower, higher).
template <int M, int NF, class Op>
__device__ __forceinline__ Pack<NF> row_suffix_incl(Pack<NF> inc, Op op) {
  const int lr = threadIdx.x & 15;
  if (M > 1) { const Pack<NF> o = dpp_pack<0x101>(inc); if (lr + 1 < M) inc = op(inc, o); }
  if (M > 2) { const Pack<NF> o = dpp_pack<0x102>(inc); if (lr + 2 < M) inc = op(inc, o); }
  if (M > 4) { const Pack<NF> o = dpp_pack<0x104>(inc); if (lr + 4 < M) inc = op(inc, o); }
  if (M > 8) { const Pack<NF> o = dpp_pack<0x108>(inc); if (lr + 8 < M) inc = op(inc, o); }
  return inc;
}
// Inclusive prefix over the 64 lanes of the wave: within the rows, then each
// odd row takes the row before it (DPP row_bcast:15), then the upper half the
// lower (row_bcast:31).
template <int NF, class Op>
__device__ __forceinline__ Pack<NF> wave_prefix_incl(const Pack<NF>& x, Op op) {
  Pack<NF> inc = row_prefix_incl<16>(x, op);
  const int row = (threadIdx.x & 63) >> 4;
  const Pack<NF> o1 = dpp_pack<0x142>(inc);
  if (row & 1) inc = op(o1, inc);
  const Pack<NF> o2 = dpp_pack<0x143>(inc);
  if (row >= 2) inc = op(o2, inc);
  return inc;
}
// Inclusive suffix over the 64 lanes of the wave (there is no DPP broadcast
// towards lower rows: lane reads).
template <int NF, class Op>
__device__ __forceinline__ Pack<NF> wave_suffix_incl(const Pack<NF>& x, Op op) {
  Pack<NF> inc = row_suffix_incl<16>(x, op);
  const int row = (threadIdx.x & 63) >> 4;
  const Pack<NF> t1 = lane_pack(inc, 16), t3 = lane_pack(inc, 48);
  const Pack<NF> o1 = pick(row < 2, t1, t3);
  if (!(row & 1)) inc = op(inc, o1);
  const Pack<NF> o2 = lane_pack(inc, 32);
  if (row < 2) inc = op(inc, o2);
  return inc;
}
// Combined wave totals, read by every lane from `lds` (aw <= NW packs of NF,
// starting at lds + off, stride S): exclusive prefix for this wave and the
// total.  NW <= 16.
template <int NW, int NF, class Op>
__device__ __forceinline__ void waves_prefix(const double* lds, int off, int S, const Pack<NF>& ident, Op op,
                                             Pack<NF>& pre, Pack<NF>& total, int aw) {
  const int lane = threadIdx.x & 63;
  Pack<NF> a = ident;
  if (lane < aw) {
#pragma unroll
    for (int i = 0; i < NF; ++i) a.v[i] = lds[lane * S + off + i];
  }
  a = row_prefix_incl<NW>(a, op);
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  pre = wv > 0 ? lane_pack(a, wv - 1) : ident;
  total = lane_pack(a, NW - 1);
}
template <int NW, int NF, class Op>
__device__ __forceinline__ void waves_suffix(const double* lds, int off, int S, const Pack<NF>& ident, Op op,
                                             Pack<NF>& suf, Pack<NF>& total, int aw) {
  const int lane = threadIdx.x & 63;
  Pack<NF> a = ident;
  if (lane < aw) {
#pragma unroll
    for (int i = 0; i < NF; ++i) a.v[i] = lds[lane * S + off + i];
  }
  a = row_suffix_incl<NW>(a, op);
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  suf = wv < NW - 1 ? lane_pack(a, wv + 1) : ident;
  total = lane_pack(a, 0);
}

// Workgroup scans.  The elements of waves aw, aw + 1, ... are the identity:
// those waves leave the wave scan out and only take the totals (a scan is
// bound by the SIMDs' issue, so with few rings the idle waves would slow the
// others down).  aw is the same in every thread, 1 <= aw <= NT / 64.

// Exclusive prefix over the workgroup in thread order.  op(earlier, later)
// must be associative; ident must satisfy op(ident, x) == x exactly.
// `lds` holds NT/64 packs.  Every thread also receives the total.  With
// TAIL = false the closing barrier is left out: the caller must not write
// `lds` again before another barrier has been passed by every thread.
template <int NT, int NF, class Op, bool TAIL = true>
__device__ __forceinline__ Pack<NF> block_prefix(const Pack<NF>& x, const Pack<NF>& ident, Op op,
                                                 double* lds, Pack<NF>& total, int aw = NT / 64) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  Pack<NF> ex = ident;
  if (wv < aw) {
    const Pack<NF> inc = wave_prefix_incl(x, op);
    const Pack<NF> sh = dpp_pack<0x138>(inc);       // outside any condition on lanes: every lane active
    ex = pick(lane == 0, ident, sh);
    if (lane == 63) {
#pragma unroll
      for (int i = 0; i < NF; ++i) lds[wv * NF + i] = inc.v[i];
    }
  }
  __syncthreads();
  Pack<NF> pre;
  waves_prefix<NW, NF>(lds, 0, NF, ident, op, pre, total, aw);
  if (TAIL) __syncthreads();
  return op(pre, ex);
}

// Exclusive suffix over the workgroup: result for thread t combines the
// elements of threads t+1 .. NT-1 in thread order, op(lower, higher).
template <int NT, int NF, class Op>
__device__ __forceinline__ Pack<NF> block_suffix(const Pack<NF>& x, const Pack<NF>& ident, Op op,
                                                 double* lds, Pack<NF>& total, int aw = NT / 64) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  Pack<NF> ex = ident;
  if (wv < aw) {
    const Pack<NF> inc = wave_suffix_incl(x, op);
    const Pack<NF> sh = dpp_pack<0x130>(inc);
    ex = pick(lane == 63, ident, sh);
    if (lane == 0) {
#pragma unroll
      for (int i = 0; i < NF; ++i) lds[wv * NF + i] = inc.v[i];
    }
  }
  __syncthreads();
  Pack<NF> suf;
  waves_suffix<NW, NF>(lds, 0, NF, ident, op, suf, total, aw);
  __syncthreads();
  return op(ex, suf);
}

// A prefix (in thread order, opP(earlier, later)) of xp and a suffix
// (opS(lower, higher)) of xs in one pass: one pair of barriers for both.
// `lds` holds NT/64 * (NP + NS) doubles.  TAIL as for block_prefix.
template <int NT, int NP, int NS, class OpP, class OpS, bool TAIL = true>
__device__ __forceinline__ void block_prefix_suffix(const Pack<NP>& xp, const Pack<NP>& idP, OpP opP,
                                                    const Pack<NS>& xs, const Pack<NS>& idS, OpS opS,
                                                    double* lds, Pack<NP>& exP, Pack<NP>& totP,
                                                    Pack<NS>& exS, Pack<NS>& totS, int aw = NT / 64) {
  constexpr int NW = NT / 64;
  constexpr int NF = NP + NS;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  Pack<NP> ep = idP;
  Pack<NS> es = idS;
  if (wv < aw) {
    const Pack<NP> ip = wave_prefix_incl(xp, opP);
    const Pack<NS> is = wave_suffix_incl(xs, opS);
    const Pack<NP> shp = dpp_pack<0x138>(ip);
    const Pack<NS> shs = dpp_pack<0x130>(is);
    ep = pick(lane == 0, idP, shp);
    es = pick(lane == 63, idS, shs);
    if (lane == 63) {
#pragma unroll
      for (int i = 0; i < NP; ++i) lds[wv * NF + i] = ip.v[i];
    }
    if (lane == 0) {
#pragma unroll
      for (int i = 0; i < NS; ++i) lds[wv * NF + NP + i] = is.v[i];
    }
  }
  __syncthreads();
  Pack<NP> pre;
  Pack<NS> suf;
  waves_prefix<NW, NP>(lds, 0, NF, idP, opP, pre, totP, aw);
  waves_suffix<NW, NS>(lds, NP, NF, idS, opS, suf, totS, aw);
  if (TAIL) __syncthreads();
  exP = opP(pre, ep);
  exS = opS(es, suf);
}

// sums of packs (commutative), used with the scans above
template <int NF>
struct SumOp {
  __device__ __forceinline__ Pack<NF> operator()(const Pack<NF>& a, const Pack<NF>& b) const {
    Pack<NF> r;
#pragma unroll
    for (int i = 0; i < NF; ++i) r.v[i] = a.v[i] + b.v[i];
    return r;
  }
};

// pairs of double-doubles: (hi0, lo0, hi1, lo1)
struct DD2Op {
  __device__ __forceinline__ Pack<4> operator()(const Pack<4>& a, const Pack<4>& b) const {
    dd x = dd_add({a.v[0], a.v[1]}, {b.v[0], b.v[1]});
    dd y = dd_add({a.v[2], a.v[3]}, {b.v[2], b.v[3]});
    return {{x.hi, x.lo, y.hi, y.lo}};
  }
};

// one and two double-doubles, with one two_sum each
struct DD1FastOp {
  __device__ __forceinline__ Pack<2> operator()(const Pack<2>& a, const Pack<2>& b) const {
    const dd x = dd_add_fast({a.v[0], a.v[1]}, {b.v[0], b.v[1]});
    return {{x.hi, x.lo}};
  }
};
struct DD2FastOp {
  __device__ __forceinline__ Pack<4> operator()(const Pack<4>& a, const Pack<4>& b) const {
    const dd x = dd_add_fast({a.v[0], a.v[1]}, {b.v[0], b.v[1]});
    const dd y = dd_add_fast({a.v[2], a.v[3]}, {b.v[2], b.v[3]});
    return {{x.hi, x.lo, y.hi, y.lo}};
  }
};

// 2x2 matrices stored (m00, m01, m10, m11).
__device__ __forceinline__ Pack<4> mat_mul(const Pack<4>& a, const Pack<4>& b) {
  return {{a.v[0] * b.v[0] + a.v[1] * b.v[2], a.v[0] * b.v[1] + a.v[1] * b.v[3],
           a.v[2] * b.v[0] + a.v[3] * b.v[2], a.v[2] * b.v[1] + a.v[3] * b.v[3]}};
}

// forward transfer: earlier applied first -> later * earlier
struct FwdMatOp {
  __device__ __forceinline__ Pack<4> operator()(const Pack<4>& earlier, const Pack<4>& later) const {
    return mat_mul(later, earlier);
  }
};

// backward transfer in index order: lower applied last -> lower * higher
struct BwdMatOp {
  __device__ __forceinline__ Pack<4> operator()(const Pack<4>& lower, const Pack<4>& higher) const {
    return mat_mul(lower, higher);
  }
};

__device__ __forceinline__ Pack<4> mat_ident() { return {{1.0, 0.0, 0.0, 1.0}}; }

// ---------------------------------------------------------------------------
// ring order: radius, then ring id
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool key_lt(double ra, int32_t ia, double rb, int32_t ib) {
  return ra < rb || (ra == rb && ia < ib);
}
