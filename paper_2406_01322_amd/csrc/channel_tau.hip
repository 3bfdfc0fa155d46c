// Wall-normal Chebyshev-tau solves in pieces (Sec. 2.2 items iv and v; the rows
// are in tau_rows.hpp).
//
// The chain of one line and parity (n = par + 2 i, i = 0..m) is cut into PC
// pieces of LEN terms.  A wavefront holds one piece of 64 lines (lane = line, so
// that each term's load is 1 KB of consecutive lines and a piece's indices n are
// uniform: the rows' constants come through scalar loads), a workgroup all
// pieces of a chain, which pass their maps to each other through LDS.  Every
// sweep of the elimination is a composition of maps, so a chain takes PC short
// serial sweeps side by side instead of one long one:
//   downward, X_i = -A_i / (B_i + C_i X_{i+1}), Y_i = (R_i - C_i Y_{i+1}) /
//     (B_i + C_i X_{i+1}): with X = x / d and Y = y / d, (x, d, y) <- (-A d,
//     B d + C x, R d - C y) is linear.  Each piece forms its map without a
//     division, composes those of the pieces above its own, and then runs its
//     own terms with the X and Y that come in (rows are diagonally dominant: no
//     pivoting, as in the serial elimination);
//   upward, a_i = P_i a_0 + Q_i: affine maps, with the sums of P_i, Q_i and n^2
//     P_i, n^2 Q_i for the boundary rows and for w' at the walls.
// The solution stays in registers, so two chained problems (psi then w, xi then
// phi) read their right-hand side once and write only the last solution.
#include <hip/hip_runtime.h>

#include "channel_tau.hpp"
#include "tau_rows.hpp"

namespace psms {

namespace {

// One wavefront's place: piece pc of the chain of parity par, lane's line.  sh
// holds NV values for every wavefront and lane.
template <int NC_, int PC_, int NV_>
struct TauWave {
  static constexpr int NC = NC_, PC = PC_, NV = NV_, NW = PC_;
  static constexpr int LEN = (NC / 2 + 1 + PC - 1) / PC;
  static constexpr int THREADS = 64 * NW;
  double* sh;
  int pc, ln, par, i0, m;
  __device__ __forceinline__ TauWave(double* s, int parity) : sh(s) {
    pc = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    ln = int(threadIdx.x & 63);
    par = parity;
    i0 = pc * LEN;
    m = (NC - par) / 2;
  }
  __device__ __forceinline__ int n(int k) const { return par + 2 * (i0 + k); }
  __device__ __forceinline__ bool in(int k) const { return i0 + k <= m; }   // uniform
  __device__ __forceinline__ void put(int v, double x) const { sh[(v * NW + pc) * 64 + ln] = x; }
  __device__ __forceinline__ double get(int v, int piece) const { return sh[(v * NW + piece) * 64 + ln]; }
};

template <int NR>
struct TauSums {
  double p1, pn;            // sum P_i, sum n^2 P_i over the chain
  double q1[NR], qn[NR];    // the same of Q_i
  double pin, qin[NR];      // P and Q that come into the piece
};

// Elimination of (D^2 - be) f = g for NR real right-hand sides.  On entry r[k][c]
// holds the piece's g (zero for n > NC - 2 and past the chain); on return X[k]
// and r[k] = Y hold the maps a_i = X_i a_{i-1} + Y_i, and S the chain's sums.
template <int NR, class W>
__device__ __forceinline__ void tau_reduce(const W& t, double be, double (&r)[W::LEN][NR], double (&X)[W::LEN],
                                           TauSums<NR>& S) {
  constexpr int LEN = W::LEN, PC = W::PC, NC = W::NC;
  static_assert(W::NV >= 3 + 3 * NR && W::NV >= 4 + 2 * NR, "LDS values");
  // the neighbouring pieces' g
  double gp[NR], gn[NR];
#pragma unroll
  for (int c = 0; c < NR; ++c) {
    t.put(c, r[0][c]);
    t.put(NR + c, r[LEN - 1][c]);
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < NR; ++c) {
    gp[c] = t.pc > 0 ? t.get(NR + c, t.pc - 1) : 0.0;
    gn[c] = t.pc + 1 < PC ? t.get(c, t.pc + 1) : 0.0;
  }
  __syncthreads();
  // right-hand sides R and the piece's map (x, d, y) -> (xx x + xd d, dx x + dd d, al y + u x + v d)
  double xx = 1.0, xd = 0.0, dx = 0.0, dd = 1.0, al = 1.0, u[NR], v[NR];
#pragma unroll
  for (int c = 0; c < NR; ++c) u[c] = v[c] = 0.0;
#pragma unroll
  for (int k = LEN - 1; k >= 0; --k) {
    const int n = t.n(k);
    if (t.in(k) && t.i0 + k >= 1) {
      const double cm2 = (n == 2) ? 2.0 : 1.0;
      const double en = (n <= NC - 2) ? 1.0 : 0.0, en2 = (n + 2 <= NC - 2) ? 1.0 : 0.0;
      const double q1 = kTauQ.q[0][n], q2 = kTauQ.q[1][n], q3 = kTauQ.q[2][n];
      const double A = cm2 * be * q1, B = -(1.0 + en * be * q2), C = en2 * be * q3;
#pragma unroll
      for (int c = 0; c < NR; ++c) {
        const double g0 = r[k][c], gm = k > 0 ? r[k > 0 ? k - 1 : 0][c] : gp[c];
        const double R = -cm2 * gm * q1 + g0 * q2 - gn[c] * q3;   // g = 0 past NC - 2: e_n, e_{n+2} are in g
        gn[c] = g0;
        r[k][c] = R;
        u[c] = R * dx - C * u[c];
        v[c] = R * dd - C * v[c];
      }
      const double ndx = B * dx + C * xx, ndd = B * dd + C * xd;
      xx = -A * dx;
      xd = -A * dd;
      dx = ndx;
      dd = ndd;
      al = -C * al;
      if (LEN > 9 && k % 8 == 0 && k > 0) {   // keep the map's entries in range: divide by 2^exponent(dd)
        const int ex = -__builtin_amdgcn_frexp_exp(dd);
        xx = ldexp(xx, ex); xd = ldexp(xd, ex); dx = ldexp(dx, ex); dd = ldexp(dd, ex); al = ldexp(al, ex);
#pragma unroll
        for (int c = 0; c < NR; ++c) {
          u[c] = ldexp(u[c], ex);
          v[c] = ldexp(v[c], ex);
        }
      }
    }
  }
  {
    const double inv = 1.0 / dd;
    t.put(0, xx * inv);
    t.put(1, xd * inv);
    t.put(2, dx * inv);
    t.put(3, al * inv);
#pragma unroll
    for (int c = 0; c < NR; ++c) {
      t.put(4 + c, u[c] * inv);
      t.put(4 + NR + c, v[c] * inv);
    }
  }
  __syncthreads();
  double Xn, Yn[NR];
  {
    double x = 0.0, d = 1.0, y[NR];   // above the chain: X = Y = 0
#pragma unroll
    for (int c = 0; c < NR; ++c) y[c] = 0.0;
#pragma unroll 1
    for (int j = PC - 1; j > t.pc; --j) {
      const double a = t.get(3, j);
#pragma unroll
      for (int c = 0; c < NR; ++c) y[c] = a * y[c] + t.get(4 + c, j) * x + t.get(4 + NR + c, j) * d;
      const double nx = t.get(0, j) * x + t.get(1, j) * d;
      d = t.get(2, j) * x + d;
      x = nx;
    }
    const double inv = 1.0 / d;
    Xn = x * inv;
#pragma unroll
    for (int c = 0; c < NR; ++c) Yn[c] = y[c] * inv;
  }
  // the piece's own X and Y
#pragma unroll
  for (int k = LEN - 1; k >= 0; --k) {
    const int n = t.n(k);
    if (t.in(k) && t.i0 + k >= 1) {
      const double cm2 = (n == 2) ? 2.0 : 1.0;
      const double en = (n <= NC - 2) ? 1.0 : 0.0, en2 = (n + 2 <= NC - 2) ? 1.0 : 0.0;
      const double A = cm2 * be * kTauQ.q[0][n], B = -(1.0 + en * be * kTauQ.q[1][n]), C = en2 * be * kTauQ.q[2][n];
      const double den = 1.0 / (B + C * Xn);
      Xn = -A * den;
      X[k] = Xn;
#pragma unroll
      for (int c = 0; c < NR; ++c) {
        Yn[c] = (r[k][c] - C * Yn[c]) * den;
        r[k][c] = Yn[c];
      }
    } else {                         // i = 0 (P_0 = 1, Q_0 = 0) or past the chain
      X[k] = 1.0;
#pragma unroll
      for (int c = 0; c < NR; ++c) r[k][c] = 0.0;
    }
  }
  __syncthreads();                   // the maps have been read
  // upward: the piece's P, Q and its parts of the sums for P_in = 1, Q_in = 0
  double pl = 1.0, bq[NR], s1p = 0.0, snp = 0.0, s1q[NR], snq[NR];
#pragma unroll
  for (int c = 0; c < NR; ++c) bq[c] = s1q[c] = snq[c] = 0.0;
#pragma unroll
  for (int k = 0; k < LEN; ++k) {
    if (t.in(k)) {
      const double dn = double(t.n(k)), n2 = dn * dn;
      pl = X[k] * pl;
      s1p += pl;
      snp += n2 * pl;
#pragma unroll
      for (int c = 0; c < NR; ++c) {
        bq[c] = X[k] * bq[c] + r[k][c];
        s1q[c] += bq[c];
        snq[c] += n2 * bq[c];
      }
    }
  }
  t.put(0, pl);
  t.put(1, s1p);
  t.put(2, snp);
#pragma unroll
  for (int c = 0; c < NR; ++c) {
    t.put(3 + c, bq[c]);
    t.put(3 + NR + c, s1q[c]);
    t.put(3 + 2 * NR + c, snq[c]);
  }
  __syncthreads();
  double p = 1.0, q[NR];
  S.p1 = S.pn = 0.0;
#pragma unroll
  for (int c = 0; c < NR; ++c) q[c] = S.q1[c] = S.qn[c] = 0.0;
#pragma unroll 1
  for (int j = 0; j < PC; ++j) {
    if (j == t.pc) {
      S.pin = p;
#pragma unroll
      for (int c = 0; c < NR; ++c) S.qin[c] = q[c];
    }
    const double s1 = t.get(1, j), sn = t.get(2, j), l = t.get(0, j);
    S.p1 += p * s1;
    S.pn += p * sn;
#pragma unroll
    for (int c = 0; c < NR; ++c) {
      S.q1[c] += s1 * q[c] + t.get(3 + NR + c, j);
      S.qn[c] += sn * q[c] + t.get(3 + 2 * NR + c, j);
      q[c] = l * q[c] + t.get(3 + c, j);
    }
    p *= l;
  }
  __syncthreads();
}

// the piece's coefficients a_i = P_i a0 + Q_i into r
template <int NR, class W>
__device__ __forceinline__ void tau_values(const W& t, double (&r)[W::LEN][NR], const double (&X)[W::LEN],
                                           const TauSums<NR>& S, const double (&a0)[NR]) {
  double p = S.pin, q[NR];
#pragma unroll
  for (int c = 0; c < NR; ++c) q[c] = S.qin[c];
#pragma unroll
  for (int k = 0; k < W::LEN; ++k) {
    p = X[k] * p;
#pragma unroll
    for (int c = 0; c < NR; ++c) {
      q[c] = X[k] * q[c] + r[k][c];
      r[k][c] = p * a0[c] + q[c];
    }
  }
}

// a solution as the next problem's right-hand side: nothing past n = NC - 2
template <int NR, class W>
__device__ __forceinline__ void tau_as_rhs(const W& t, double (&r)[W::LEN][NR]) {
#pragma unroll
  for (int k = 0; k < W::LEN; ++k)
    if (!t.in(k) || t.n(k) > W::NC - 2)
#pragma unroll
      for (int c = 0; c < NR; ++c) r[k][c] = 0.0;
}

// right-hand side entries of the piece (complex into r[k][0..1])
template <int NR, class W>
__device__ __forceinline__ void tau_load(const W& t, const cpx<double>* __restrict__ g, long long nl, long long l,
                                         double (&r)[W::LEN][NR]) {
#pragma unroll
  for (int k = 0; k < W::LEN; ++k) {
    cpx<double> x = {0.0, 0.0};
    if (t.in(k) && t.n(k) <= W::NC - 2) x = g[(long long)t.n(k) * nl + l];
    r[k][0] = x.re;
    r[k][1] = x.im;
  }
}

template <int NR, class W>
__device__ __forceinline__ void tau_store(const W& t, cpx<double>* __restrict__ f, long long nl, long long l,
                                          const double (&r)[W::LEN][NR]) {
#pragma unroll
  for (int k = 0; k < W::LEN; ++k)
    if (t.in(k)) f[(long long)t.n(k) * nl + l] = cpx<double>{r[k][0], r[k][1]};
}

// ---------------------------------------------------------------------------
// psms_wall_solve: blockIdx.y = 0 w, 1 omega, 2 phi; blockIdx.z the parity.  The
// homogeneous w solution (psi = 1 at both walls for the even parity, +-1 for the
// odd) is a third, real right-hand side of the w chains: w'(+1) = +-w'(-1) splits
// by parity, so each parity's correction makes its own sum n^2 w_n vanish.
// Measured at 7310 lines x 129: 55 us (90 MB read and written; bound by the chains'
// latency at one workgroup of 8 wavefronts per compute unit, 188 VGPRs), where one
// lane per chain took three launches of 55 us and 174 us for the influence sums.
// Held to 128 VGPRs it spills 200 bytes a lane.
// ---------------------------------------------------------------------------
template <int NC>
__global__ void __launch_bounds__(512) k_wall_tau(WallTauArgs a) {
  using W = TauWave<NC, 8, 12>;
  __shared__ double sh[W::NV * W::NW * 64];
  const W t(sh, int(blockIdx.z));
  const long long l = (long long)blockIdx.x * 64 + t.ln;
  const bool valid = l < a.nl;
  const long long lc = valid ? l : 0;   // lanes past the last line read line 0 and store nothing
  const double kx = a.kx[lc], ky = a.ky[lc], k2 = kx * kx + ky * ky;
  double X[W::LEN];
  if (blockIdx.y == 0) {
    double r[W::LEN][3];
    tau_load(t, a.g_w, a.nl, lc, r);
#pragma unroll
    for (int k = 0; k < W::LEN; ++k) r[k][2] = 0.0;
    TauSums<3> S;
    tau_reduce(t, a.beta_ns + k2, r, X, S);
    double a0[3] = {-S.q1[0] / S.p1, -S.q1[1] / S.p1, (1.0 - S.q1[2]) / S.p1};
    tau_values(t, r, X, S, a0);
    tau_as_rhs(t, r);
    tau_reduce(t, k2, r, X, S);
    double sn[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      a0[c] = -S.q1[c] / S.p1;
      sn[c] = a0[c] * S.pn + S.qn[c];   // sum n^2 w_n
    }
    tau_values(t, r, X, S, a0);
    const bool mean = kx == 0.0 && ky == 0.0;   // no wall-normal velocity there
    const double c0 = -sn[0] / sn[2], c1 = -sn[1] / sn[2];
#pragma unroll
    for (int k = 0; k < W::LEN; ++k) {
      r[k][0] = mean ? 0.0 : r[k][0] + c0 * r[k][2];
      r[k][1] = mean ? 0.0 : r[k][1] + c1 * r[k][2];
    }
    if (valid) tau_store(t, a.w, a.nl, l, r);
    return;
  }
  double r[W::LEN][2];
  TauSums<2> S;
  if (blockIdx.y == 1) {
    tau_load(t, a.g_om, a.nl, lc, r);
    tau_reduce(t, a.beta_ns + k2, r, X, S);
    const double a0[2] = {-S.q1[0] / S.p1, -S.q1[1] / S.p1};
    tau_values(t, r, X, S, a0);
    if (valid) tau_store(t, a.om, a.nl, l, r);
    return;
  }
  tau_load(t, a.g_phi, a.nl, lc, r);
  for (int s = 0; s < 2; ++s) {   // xi, then phi: no flux through the walls
    tau_reduce(t, (s ? a.beta_b : a.beta_a) + k2, r, X, S);
    const double a0[2] = {-S.qn[0] / S.pn, -S.qn[1] / S.pn};
    tau_values(t, r, X, S, a0);
    if (s == 0) tau_as_rhs(t, r);
  }
  if (valid) tau_store(t, a.phi, a.nl, l, r);
}

#define PSMS_FOR_EACH_TAU_NC(X) X(4) X(6) X(8) X(12) X(16) X(24) X(32) X(48) X(64) X(96) X(128) X(256)

}  // namespace

bool tau_pieces_nc(int nc) {
  switch (nc) {
#define PSMS_CASE(NC) case NC:
    PSMS_FOR_EACH_TAU_NC(PSMS_CASE)
#undef PSMS_CASE
    return true;
    default:
      return false;
  }
}

hipError_t launch_wall_tau(const WallTauArgs& a, int nc, hipStream_t st) {
  if (a.nl < 1) return a.nl == 0 ? hipSuccess : hipErrorInvalidValue;
  const dim3 grid(unsigned((a.nl + 63) / 64), 3, 2);
  switch (nc) {
#define PSMS_CASE(NC) \
  case NC: k_wall_tau<NC><<<grid, 512, 0, st>>>(a); return hipGetLastError();
    PSMS_FOR_EACH_TAU_NC(PSMS_CASE)
#undef PSMS_CASE
  }
  return hipErrorInvalidValue;
}

}  // namespace psms
