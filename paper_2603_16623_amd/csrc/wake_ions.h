// Internal layout of two-species instances (plasma electrons and mobile
// ions), shared by the host runtime and the gfx950 kernels.  Not part of the
// public ABI (include/wake.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wake_common.h"

#define WAKE_IONS_NT 1024      // workgroup threads of the two-species marcher
#define WAKE_IONS_NMAX 8192    // rings per species (the sorted radii of both species sit in LDS)

// All per-ring arrays are planes of 16-B chunks (two doubles), S = 1024 C
// chunks each, so that a wave moves one chunk of 64 consecutive slots as
// contiguous lanes.  Position p's slot is (p % C) * 1024 + p / C; ring id i's
// home slot is the slot of position i, and the constants and the state sit
// there: while rings keep roughly their initial order, their gathers touch
// neighbouring slots (by ring id every lane read a line of its own, one a
// cycle, and that was most of the march's time).
//
// constants by home slot (both species start at the same radii with the
// same weights): (w, w^), (r0, 1/r0), ln r0 (dd), then a plane of 8-B dr
enum { IK_W = 0, IK_R0, IK_LN, IK_DR, IK_DOUBLES = 7 };
// ring state by home slot: (rho, u_r) and the Adams-Bashforth history
enum { IS_RU = 0, IS_F, IS_N };
// per-position work of one species by slot: (w, w^); ln rho (dd); its node
// tables psi (dd), d_rho psi (dd), and (d_zeta psi, B^(p) at the electron
// rings); the fields (psi, d_rho psi) of both species together; (u_r, q u /
// (rho psibar)); (beam field, -); the laser's (|a|^2, gradient), with a laser
// only; for the electrons (A_i, s_a) of the recursion and (d_zeta psi, cc)
enum { IW_W = 0, IW_LN, IW_T0, IW_T1, IW_ZB, IW_F, IW_UC, IW_BB, IW_A2, IW_E, IW_DC, IW_N };

// One two-species instance as the kernels see it.  All pointers are device
// pointers.  Species 0 are the electrons (q = -1, m = 1), species 1 the
// ions (q = +1, m = m_i).  Per species, thread t of the workgroup owns the
// C = ceil(N / 1024) consecutive sorted positions [tC, tC + C).
struct WakeIons {
  int32_t N, n_xi, first, count, stride, C;
  int32_t nb, n_an, has_laser, pad;
  double dxi, m_i;
  WakeAnalytic an[WAKE_MAX_ANALYTIC];
  const int32_t* boff;        // beam table (CSR over slices)
  const double *br, *bcum;
  const double* cst;          // [IK_DOUBLES][S]
  double* st[2];              // two buffers, each [2 species][IS_N][S] chunks
  int32_t* ord;               // [2][S] ring ids in the latest sorted order, by slot
  int32_t* sid;               // [2][S] home slot of the ring at each position, by slot
  int32_t* jx;                // [2][S] rings of the other species below each ring (-1: beyond
                              //        its edge), by slot
  double* work;               // [2 species][IW_N][S] chunks
  double* axis;               // [n_xi][2]: psi(0), E_z(0)
  double* snap[2];            // per species [n_rec][OUT_N][N] by ring id
  double* last[2];            // per species [OUT_N][N]: the last marched slice
  int32_t* ctl;               // [CTL_NWORDS]; CTL_CUR is the state buffer of the next slice
  unsigned long long* cnt;    // [CNT_N]: slices marched, order fix-ups
};

hipError_t launch_ions_init(const WakeIons& J, const double* r0, const double* dr, const double* dens,
                            bool constants, hipStream_t s);
// the marcher's LDS allowance on the current device (before its first launch there)
hipError_t ions_prepare();
hipError_t launch_ions_march(const WakeIons* d_insts, int n_insts, hipStream_t s);
// back to slice 0 with both species at rest, for n records in device memory
// (the records' own fields are read on the device: capturable)
hipError_t launch_ions_reset(const WakeIons* d_insts, int n_insts, hipStream_t s);
// ring state of species sp at the next slice to out [4][N] (rho, u_r, f_rho, f_u)
hipError_t launch_ions_get_state(const WakeIons& J, int sp, double* out, hipStream_t s);
// replace species sp's state (f_rho/f_u may be null: zero) and make `slice` the next slice
hipError_t launch_ions_set_state(const WakeIons& J, int sp, const double* rho, const double* u,
                                 const double* fr, const double* fu, int slice, hipStream_t s);
size_t ions_lds_bytes();
