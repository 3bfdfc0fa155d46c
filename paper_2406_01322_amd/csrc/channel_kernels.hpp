// Launchers of the wall-normal (Chebyshev) kernels.  Lines are stored
// position-major: coefficient / point n of line l at n * nlines + l.
#pragma once

#include <hip/hip_runtime.h>

#include "fft_engine.hpp"

namespace psms {

bool supported_nc(int nc);

template <typename T>
hipError_t launch_dct(int nc, const cpx<T>* in, cpx<T>* out, long long nlines, int dir, hipStream_t st);
// nfield fields fstride elements apart in one launch; tw: exp(-2 pi i m / (2 nc)),
// m < 2 nc, or NULL (computed in the kernel)
template <typename T>
hipError_t launch_dct_fields(int nc, const cpx<T>* in, cpx<T>* out, long long nlines, long long fstride, int nfield,
                             const cpx<T>* tw, int dir, hipStream_t st);
// The forward transform of the channel step's products: in [8 or 6][j][line] T_xx T_yy
// T_zz T_xy T_xz T_yz (a, c); out [nterm][n][line] FP64, n <= kz only, the
// nterm = 6 (4 in single phase) arrays A, B, P, Q (a, c) of channel_tau.hip
template <typename T>
hipError_t launch_dct_chterms(int nc, const cpx<T>* in, cpx<double>* out, long long nlines, long long fstride, int nterm,
                              const double* kx, const double* ky, const cpx<T>* tw, int kz, hipStream_t st);
// The inverse transform of the channel step's fields u, v, w, phi, i ky phi, D phi
// (nfield = 6, or 3: u, v, w; [nfield][n][line] out, fstride apart), each value formed from the FP64
// state as it is loaded (u, v by continuity and the definition of omega_z;
// the mean line, l = 0, carries U, V from mean [n][2]).
struct ChanFieldSrc {
  const cpx<double>* om;
  const cpx<double>* w;
  const cpx<double>* phi;
  const cpx<double>* dw;
  const cpx<double>* dphi;
  const cpx<double>* mean;
  const double* kx;
  const double* ky;
  long long nlines;
};
template <typename T>
hipError_t launch_dct_chfields(int nc, const ChanFieldSrc& fs, cpx<T>* out, long long fstride, int nfield,
                               const cpx<T>* tw, hipStream_t st);
hipError_t launch_chebd(const cpx<double>* a, cpx<double>* d, int nc, long long nlines, hipStream_t st);
hipError_t launch_helm(const cpx<double>* g, cpx<double>* f, double* xw, int nc, long long nlines,
                       const double* beta_line, double beta_add, const double* kx, const double* ky, int neumann,
                       const cpx<double>* bcv, cpx<double> top_c, cpx<double> bot_c, hipStream_t st);
// independent tau problems (D^2 - (beta_add + kx^2 + ky^2)) f = g of one launch;
// kx = NULL means k^2 = 0, g = NULL a zero right-hand side; xw: (nc+1) nlines
// doubles of scratch per problem
constexpr int kHelmBatchMax = 4;
struct HelmProblem {
  const cpx<double>* g;
  cpx<double>* f;
  double* xw;
  long long nlines;
  double beta_add;
  const double* kx;
  const double* ky;
  int neumann;   // Neumann conditions at both walls, else Dirichlet
  cpx<double> top_c, bot_c;
};
struct HelmBatch {
  HelmProblem p[kHelmBatchMax];
  int np;
};
hipError_t launch_helm_batch(const HelmBatch& b, int nc, hipStream_t st);
hipError_t launch_influence(cpx<double>* wp, const cpx<double>* wt, const cpx<double>* wb, int nc, long long nlines,
                            const double* kx, const double* ky, hipStream_t st);
// u, v from omega and w (continuity and eq. omegadef; zero where kx = ky = 0)
hipError_t launch_cheb_uv(const cpx<double>* om, const cpx<double>* w, cpx<double>* u, cpx<double>* v, int nc,
                          long long nlines, const double* kx, const double* ky, hipStream_t st);

}  // namespace psms
