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

}  // namespace psms
