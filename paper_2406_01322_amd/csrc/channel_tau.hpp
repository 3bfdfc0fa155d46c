// Launchers of the pieced wall-normal solves (channel_tau.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "fft_engine.hpp"

namespace psms {

// nc for which the pieced solves are built (the lengths of the channel step)
bool tau_pieces_nc(int nc);

// The implicit wall-normal solves of psms_wall_solve for nl lines, right-hand
// sides given: omega (Dirichlet, beta_ns + k^2), w (psi, then w, with w' = 0 at
// both walls), phi (Neumann, beta_a + k^2, then beta_b + k^2).  [nc+1][nl] each.
struct WallTauArgs {
  const cpx<double>* g_om;
  const cpx<double>* g_w;
  const cpx<double>* g_phi;
  cpx<double>* om;
  cpx<double>* w;
  cpx<double>* phi;
  const double* kx;
  const double* ky;
  long long nl;
  double beta_ns, beta_a, beta_b;
};
hipError_t launch_wall_tau(const WallTauArgs& a, int nc, hipStream_t st);

// The channel step from the transformed products to the new state: explicit
// terms, Adams-Bashforth with the history, right-hand sides, solves of every
// line and of the mean flow, and D w, D phi of the new state.  Arrays [nc+1][nl].
struct ChanTauArgs {
  const cpx<double>* terms;   // [6] (4 in single phase) A, B, P, Q, a, c of launch_dct_chterms, n <= kz read
  long long nzl;              // (nc + 1) nl
  int kz;
  cpx<double>* om;            // state (in/out)
  cpx<double>* w;
  cpx<double>* phi;
  cpx<double>* hist;          // [3] H_omega, H_w, S_phi of the previous step (in/out)
  cpx<double>* mean;          // [nc+1][2] U, V (in/out)
  cpx<double>* hmean;         // [nc+1][2] (in/out)
  cpx<double>* dw;            // D w, D phi of the new state
  cpx<double>* dphi;
  const double* kx;
  const double* ky;
  const double* wh;           // homogeneous w solutions and their sums (launch_tau_hom)
  const double* mh;
  long long nl;
  double re, beta, dt, forcing, inv_pe, e_coef, g_phi_scale, a_fac, b_fac;
  int ab1, fs, sp;            // fs: bit 0 / 1 the top / bottom wall is free-slip
};
hipError_t launch_chan_tau(const ChanTauArgs& a, int nc, hipStream_t st);

// D w and (narr = 2) D phi of a state, bit for bit as launch_chan_tau leaves them
hipError_t launch_tau_deriv(const cpx<double>* w, const cpx<double>* phi, cpx<double>* dw, cpx<double>* dphi, int narr,
                            int nc, long long nl, hipStream_t st);

// wh [nc+1][nl] and mh [2][nl] for w between no-slip walls: psi = 1 at both walls
// for the even parity, +-1 for the odd, beta + k^2; mh[p][l] = sum_{n = p mod 2} n^2 wh_n
hipError_t launch_tau_hom(double beta, const double* kx, const double* ky, int nc, long long nl, double* wh,
                          double* mh, hipStream_t st);

}  // namespace psms
