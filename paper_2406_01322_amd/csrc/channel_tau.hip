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

// Pieces of a chain: 8, and one up to nc = 16 (9 terms, what a piece has at nc = 128).
// Pieces of one or two terms leave wavefronts with nothing to do, which costs little
// while a launch is a few workgroups and everything once it fills the chip (five wall
// solves of 60000 lines, 8 pieces and one: nc = 4 509 and 122 us, nc = 16 617 and 178; a
// 256 x 128 x 17 channel step 93 and 84), and one piece has the smaller error (omega at
// nc = 16, beta 3e6: 5.3e-14 and 3.6e-14).  Two or four pieces for nc = 24 to 48 are faster
// as well (60000 lines, nc = 24: 670 and 289), but their error is larger (1.3e-14 and 2.6e-14).
constexpr int tau_pieces(int nc) { return nc <= 16 ? 1 : 8; }
constexpr int tau_len(int nc) { return (nc / 2 + 1 + tau_pieces(nc) - 1) / tau_pieces(nc); }

// The rows (tau_rows.hpp) of chain length NC at every piece's slots, by parity:
// c_{n-2} q1, e_n q2, e_{n+2} q3, zero for n < 2 and past the chain (there e_n q2 is 1:
// a row of the others' size, since they are scaled by beta).  There the map
// is X = Y = 0 whatever comes in, which is right above the chain and unread below
// it, so the sweeps need no branch.  A wavefront reads LEN consecutive entries of
// each at uniform addresses: a few wide scalar loads that are waited for once (a
// scalar load for every term, waited for one by one, took a third of the kernel).
template <int NC>
struct TauTab {
  static constexpr int SLOTS = tau_pieces(NC) * tau_len(NC);
  double a[2][SLOTS], b[2][SLOTS], c[2][SLOTS];
};
template <int NC>
constexpr TauTab<NC> make_tau_tab() {
  TauTab<NC> t{};
  const TauQ q = make_tau_q();
  for (int p = 0; p < 2; ++p)
    for (int i = 1; i < TauTab<NC>::SLOTS; ++i) {
      const int n = p + 2 * i;
      if (n > NC) {
        t.b[p][i] = 1.0;
        continue;
      }
      t.a[p][i] = (n == 2 ? 2.0 : 1.0) * q.q[0][n];
      t.b[p][i] = n <= NC - 2 ? q.q[1][n] : 0.0;
      t.c[p][i] = n + 2 <= NC - 2 ? q.q[2][n] : 0.0;
    }
  return t;
}
template <int NC>
__constant__ const TauTab<NC> kTauTab = make_tau_tab<NC>();

// One wavefront's place: piece pc of the chain of parity par, lane's line.  sh
// holds NV values for every wavefront and lane.  With BOTH, a workgroup holds the
// chains of both parities (for boundary rows that couple them), else the one of
// blockIdx.z.
template <int NC_, int NV_, bool BOTH_ = false>
struct TauWave {
  static constexpr int NC = NC_, PC = tau_pieces(NC_), NV = NV_;
  static constexpr bool BOTH = BOTH_;
  static constexpr int NW = BOTH ? 2 * PC : PC;
  static constexpr int LEN = tau_len(NC);
  double* sh;
  int pc, ln, par, i0, m;
  __device__ __forceinline__ TauWave(double* s) : sh(s) {
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    pc = wave % PC;
    ln = int(threadIdx.x & 63);
    par = BOTH ? wave / PC : int(blockIdx.z);
    i0 = pc * LEN;
    m = (NC - par) / 2;
  }
  __device__ __forceinline__ int n(int k) const { return par + 2 * (i0 + k); }
  __device__ __forceinline__ bool in(int k) const { return i0 + k <= m; }   // uniform
  // n of slot k as a double, opaque to the compiler: each sweep counts in steps of
  // 2 from its own start instead of holding every n in registers
  __device__ __forceinline__ double dn(int k) const {
    int v = par + 2 * (i0 + k);
    asm volatile("" : "+s"(v));
    return double(v);
  }
  __device__ __forceinline__ double& at(int v, int parity, int piece) const {
    return sh[(v * NW + (BOTH ? parity * PC : 0) + piece) * 64 + ln];
  }
  __device__ __forceinline__ void put(int v, double x) const { at(v, par, pc) = x; }
  __device__ __forceinline__ double get(int v, int piece) const { return at(v, par, piece); }
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
  constexpr int LEN = W::LEN, PC = W::PC;
  static_assert(W::NV >= 3 + 3 * NR && W::NV >= 4 + 2 * NR, "LDS values");
  double ra[LEN], rb[LEN], rc[LEN];
  {
    const double *pa = &kTauTab<W::NC>.a[t.par][t.i0], *pb = &kTauTab<W::NC>.b[t.par][t.i0],
                 *pt = &kTauTab<W::NC>.c[t.par][t.i0];
#pragma unroll
    for (int k = 0; k < LEN; ++k) {
      ra[k] = pa[k];
      rb[k] = pb[k];
      rc[k] = pt[k];
    }
  }
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
  // right-hand sides R and the piece's map (x, d, y) -> (xx x + xd d, dx x + dd d, al y + u x + v d).
  // The rows are taken times sc, a power of two near 1 / (1 + be), which leaves the
  // map's entries over dd as they are and keeps a piece's product in range for any be
  const double sc = ldexp(1.0, -__builtin_amdgcn_frexp_exp(1.0 + be)), bes = be * sc;
  double xx = 1.0, xd = 0.0, dx = 0.0, dd = 1.0, al = 1.0, u[NR], v[NR];   // u, v before their factor sc
#pragma unroll
  for (int c = 0; c < NR; ++c) u[c] = v[c] = 0.0;
#pragma unroll
  for (int k = LEN - 1; k >= 0; --k) {
    const double A = bes * ra[k], B = -(sc + bes * rb[k]), C = bes * rc[k];
#pragma unroll
    for (int c = 0; c < NR; ++c) {
      const double g0 = r[k][c], gm = k > 0 ? r[k > 0 ? k - 1 : 0][c] : gp[c];
      const double R = -ra[k] * gm + rb[k] * g0 - rc[k] * gn[c];
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
  }
  {
    const double inv = 1.0 / dd, invs = inv * sc;
    t.put(0, xx * inv);
    t.put(1, xd * inv);
    t.put(2, dx * inv);
    t.put(3, al * inv);
#pragma unroll
    for (int c = 0; c < NR; ++c) {
      t.put(4 + c, u[c] * invs);
      t.put(4 + NR + c, v[c] * invs);
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
  // the piece's own X and Y.  The rows' coefficients are formed again: kept from
  // the first sweep they would take 6 registers a term.
  asm volatile("" : "+v"(be));
#pragma unroll
  for (int k = LEN - 1; k >= 0; --k) {
    const double C = be * rc[k], den = 1.0 / (C * Xn - (1.0 + be * rb[k]));
    Xn = -(be * ra[k]) * den;
    X[k] = Xn;
#pragma unroll
    for (int c = 0; c < NR; ++c) {
      Yn[c] = (r[k][c] - C * Yn[c]) * den;
      r[k][c] = Yn[c];
    }
  }
  if (t.i0 == 0) X[0] = 1.0;         // i = 0: P_0 = 1, Q_0 = 0
  __syncthreads();                   // the maps have been read
  // upward: the piece's P, Q and its parts of the sums for P_in = 1, Q_in = 0
  double pl = 1.0, bq[NR], s1p = 0.0, snp = 0.0, s1q[NR], snq[NR];
#pragma unroll
  for (int c = 0; c < NR; ++c) bq[c] = s1q[c] = snq[c] = 0.0;
  double n = t.dn(0);
#pragma unroll
  for (int k = 0; k < LEN; ++k, n += 2.0) {
    const double n2 = n * n;
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

// f at n + UP of the piece's indices (complex, into x[k][0..1]; zero past nmax and
// past the chain).  A load under a branch is waited for at the branch's end, so
// every slot loads, the ones that are zero row UP of the chain.
template <int UP, int NR, class W>
__device__ __forceinline__ void tau_load(const W& t, const cpx<double>* __restrict__ f, long long stride, unsigned l,
                                         int nmax, double (&x)[W::LEN][NR]) {
#pragma unroll
  for (int k = 0; k < W::LEN; ++k) {
    const bool ok = t.in(k) && t.n(k) + UP <= nmax;   // uniform
    const cpx<double> v = (f + (long long)(ok ? t.n(k) + UP : UP) * stride)[l];
    x[k][0] = ok ? v.re : 0.0;
    x[k][1] = ok ? v.im : 0.0;
  }
}

template <int NR, class W>
__device__ __forceinline__ void tau_store(const W& t, cpx<double>* __restrict__ f, long long nl, long long l,
                                          const double (&r)[W::LEN][NR]) {
#pragma unroll
  for (int k = 0; k < W::LEN; ++k)
    if (t.in(k)) (f + (long long)t.n(k) * nl)[l] = cpx<double>{r[k][0], r[k][1]};
}

// ---------------------------------------------------------------------------
// psms_wall_solve: blockIdx.y = 0 w, 1 omega, 2 phi; blockIdx.z the parity.  The
// homogeneous w solution (psi = 1 at both walls for the even parity, +-1 for the
// odd) is a third, real right-hand side of the w chains: w'(+1) = +-w'(-1) splits
// by parity, so each parity's correction makes its own sum n^2 w_n vanish.
// Measured at 7310 lines x 129: 47 us (90 MB read and written; bound by the chains'
// latency at one workgroup of 8 wavefronts, two a SIMD, per compute unit), where one
// lane per chain took three launches of 55 us and 174 us for the influence sums.
// ---------------------------------------------------------------------------
template <int NC>
__global__ void __launch_bounds__(64 * tau_pieces(NC)) k_wall_tau(WallTauArgs a) {
  using W = TauWave<NC, 12>;
  __shared__ double sh[W::NV * W::NW * 64];
  const W t(sh);
  const long long l = (long long)blockIdx.x * 64 + t.ln;
  const bool valid = l < a.nl;
  const long long lc = valid ? l : 0;   // lanes past the last line read line 0 and store nothing
  const double kx = a.kx[lc], ky = a.ky[lc], k2 = kx * kx + ky * ky;
  double X[W::LEN];
  if (blockIdx.y == 0) {
    double r[W::LEN][3], a0[3], sn[3];
    tau_load<0>(t, a.g_w, a.nl, unsigned(lc), NC - 2, r);
#pragma unroll
    for (int k = 0; k < W::LEN; ++k) r[k][2] = 0.0;
    TauSums<3> S;
#pragma unroll 1
    for (int s = 0; s < 2; ++s) {   // psi, then w
      tau_reduce(t, s ? k2 : a.beta_ns + k2, r, X, S);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        a0[c] = ((c == 2 && s == 0 ? 1.0 : 0.0) - S.q1[c]) / S.p1;
        sn[c] = a0[c] * S.pn + S.qn[c];   // sum n^2 a_n
      }
      tau_values(t, r, X, S, a0);
      if (s == 0) tau_as_rhs(t, r);
    }
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
  // omega (Dirichlet, one problem) or xi, then phi (no flux through the walls)
  const bool phi = blockIdx.y == 2;
  double r[W::LEN][2];
  TauSums<2> S;
  tau_load<0>(t, phi ? a.g_phi : a.g_om, a.nl, unsigned(lc), NC - 2, r);
#pragma unroll 1
  for (int s = phi ? 0 : 1; s < 2; ++s) {
    tau_reduce(t, (phi ? (s ? a.beta_b : a.beta_a) : a.beta_ns) + k2, r, X, S);
    const double p = phi ? S.pn : S.p1;
    const double a0[2] = {-(phi ? S.qn[0] : S.q1[0]) / p, -(phi ? S.qn[1] : S.q1[1]) / p};
    tau_values(t, r, X, S, a0);
    if (s == 0) tau_as_rhs(t, r);
  }
  if (valid) tau_store(t, phi ? a.phi : a.om, a.nl, l, r);
}

// ---------------------------------------------------------------------------
// The channel step's wall-normal half: explicit terms, Adams-Bashforth, the
// right-hand sides, the solves, and the derivatives the next step starts from.
// blockIdx.y = 0 w, 1 omega, 2 phi (two-phase), last the mean lines U, V.
//
// With S = div T the explicit terms of a line need only four combinations of the
// six products, formed where the forward Chebyshev transform loads them:
//   A = (ky^2 - kx^2) T_xy + kx ky (T_xx - T_yy),  B = i kx T_yz - i ky T_xz,
//   P = i kx T_xz + i ky T_yz,  Q = kx^2 T_xx + 2 kx ky T_xy + ky^2 T_yy - k^2 T_zz:
//   H_omega = (curl S)_z = A + D B,   H_w = lap_h S_z - D div_h S = D Q - (D^2 + k^2) P.
// The mean line (kx = ky = 0, where all four vanish) carries T_xz in B and T_yz in Q,
// for S_x = D T_xz and S_y = D T_yz.  D and D^2 are suffix sums along a parity
// chain, so they split over the pieces like the elimination: each lane sums its
// terms, the pieces' totals go through LDS, and the lane repeats its sums from
// what comes in.  A parity's chain reads B, Q of the other parity and A, P of its
// own, so every array is read once.
//
// Bytes per step at 256 x 128 x 129: 309 MB counted, 189 read (state and history, phi
// twice, six term arrays up to n = kz, wh) and 121 written (state, history, D w, D
// phi), 60 us at the rate of a copy, where separate derivative, assembly and solve
// passes moved 900 MB.  Measured there: 94 us, where the derivative, assembly and solve
// launches took 211 us; 256 x 256 x 257 single phase 264 us, where they took 935 us.
// It is bound by the latency of its chains of FP64 operations, scans and barriers
// (a workgroup takes 20 to 30 us and a compute unit holds one, two wavefronts a SIMD,
// 188 VGPRs): held to 128 VGPRs it spills and takes 30% longer, 16 pieces of 5 terms take
// 6% longer, and unrolled scans over the pieces change nothing.  The chains of nc = 256
// have 17 terms a piece: 256 VGPRs and 80 more in scratch.
// With different walls (BOTH) the workgroup's 1024 threads hold it to 128 VGPRs: 23, 61
// and 433 are spilled at nc = 96, 128 and 256.  It takes 31 us at 128 x 96 x 65, 71 at
// 128 x 96 x 129 and 191 at 96 x 64 x 257, where the former launches took 120, 259 and 433.
// ---------------------------------------------------------------------------

// (D f)_n = s_n sum_{j >= n, j = n mod 2} 2 (j + 1) f_{j+1} (s_0 = 1/2): the piece's
// total from x = f_{n+1}, put at values v, v + 1
template <class W>
__device__ __forceinline__ void d_put(const W& t, int v, const double (&x)[W::LEN][2]) {
  double a = 0.0, b = 0.0, n1 = t.dn(0) + 1.0;
#pragma unroll
  for (int k = 0; k < W::LEN; ++k, n1 += 2.0) {
    a += n1 * x[k][0];                         // x = 0 past the chain
    b += n1 * x[k][1];
  }
  t.put(v, 2.0 * a);
  t.put(v + 1, 2.0 * b);
}
// sum of values v, v + 1 over the pieces above
template <class W>
__device__ __forceinline__ void d_carry(const W& t, int v, double (&c)[2]) {
  c[0] = c[1] = 0.0;
#pragma unroll 1
  for (int j = W::PC - 1; j > t.pc; --j) {
    c[0] += t.get(v, j);
    c[1] += t.get(v + 1, j);
  }
}
// (D^2 f)_n = s_n sum_{j >= n} 2 (j + 1) b_{j+1}, b_{j+1} = sum_{p > j} 2 p f_p: the
// piece's totals of both sums (the second for nothing coming into the first) at v .. v + 3
template <class W>
__device__ __forceinline__ void d2_put(const W& t, int v, const double (&f)[W::LEN][2]) {
  double a[2] = {0.0, 0.0}, b[2] = {0.0, 0.0}, tn = 2.0 * t.dn(W::LEN - 1);
#pragma unroll
  for (int k = W::LEN - 1; k >= 0; --k, tn -= 4.0) {   // past the chain: f = 0 and nothing has come in
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      b[c] += (tn + 2.0) * a[c];
      a[c] += tn * f[k][c];
    }
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    t.put(v + c, a[c]);
    t.put(v + 2 + c, b[c]);
  }
}
// both sums over the pieces above: a into the first, b into the second
template <class W>
__device__ __forceinline__ void d2_carry(const W& t, int v, double (&a)[2], double (&b)[2]) {
  a[0] = a[1] = b[0] = b[1] = 0.0;
#pragma unroll 1
  for (int j = W::PC - 1; j > t.pc; --j) {
    int cnt = t.m + 1 - j * W::LEN;               // terms of piece j
    cnt = cnt < 0 ? 0 : cnt > W::LEN ? W::LEN : cnt;
    // sum of 2 (n + 1) over them
    const double wt = 2.0 * double(cnt * (t.par + 1) + cnt * (2 * j * W::LEN + cnt - 1));
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      b[c] += t.get(v + 2 + c, j) + wt * a[c];
      a[c] += t.get(v + c, j);
    }
  }
}

// D of the piece's solution r into out (indices n - 1; out_nc = 0).  The sums are
// explicit fused multiply-adds: the step and k_tau_deriv have to give the same bits,
// and which products the compiler fuses by itself depends on the kernel around them.
template <class W>
__device__ __forceinline__ void d_store(const W& t, cpx<double>* __restrict__ out, long long nl, unsigned l, bool valid,
                                        const double (&r)[W::LEN][2]) {
  double a[2] = {0.0, 0.0}, c[2], n = t.dn(0);
#pragma unroll
  for (int k = 0; k < W::LEN; ++k, n += 2.0) {   // r = 0 past the chain
    a[0] = __builtin_fma(n, r[k][0], a[0]);
    a[1] = __builtin_fma(n, r[k][1], a[1]);
  }
  t.put(0, 2.0 * a[0]);
  t.put(1, 2.0 * a[1]);
  __syncthreads();
  d_carry(t, 0, c);
  if (!valid) return;
  double tn = 2.0 * t.dn(W::LEN - 1);
#pragma unroll
  for (int k = W::LEN - 1; k >= 0; --k, tn -= 4.0) {
    c[0] = __builtin_fma(tn, r[k][0], c[0]);
    c[1] = __builtin_fma(tn, r[k][1], c[1]);
    if (t.in(k) && t.n(k) >= 1) {
      const double s = t.n(k) == 1 ? 0.5 : 1.0;
      (out + (long long)(t.n(k) - 1) * nl)[l] = cpx<double>{s * c[0], s * c[1]};
    }
  }
  if (t.par == 1 && t.pc == 0) out[(long long)W::NC * nl + l] = cpx<double>{0.0, 0.0};
}

// first coefficient of the solution for zero boundary values: bit 0 / 1 of bc
// makes the top / bottom wall Neumann.  The same condition at both walls splits
// by parity; different ones couple the parities (BOTH).
template <class W>
__device__ __forceinline__ void chan_a0(const W& t, int bc, const TauSums<2>& S, double (&a0)[2]) {
  if (bc == 0 || bc == 3) {
    const double p = bc ? S.pn : S.p1;
#pragma unroll
    for (int c = 0; c < 2; ++c) a0[c] = -(bc ? S.qn[c] : S.q1[c]) / p;
    return;
  }
  if constexpr (W::BOTH) {
    if (t.pc == 0) {
      t.put(0, S.p1);
      t.put(1, S.pn);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        t.put(2 + c, S.q1[c]);
        t.put(4 + c, S.qn[c]);
      }
    }
    __syncthreads();
    // rows f(+1) or f'(+1) (1 or n^2) and f(-1) or f'(-1) ((-1)^n or -(-1)^n n^2)
    const int tp = bc & 1, bp = bc >> 1;
    const double t0 = t.at(tp, 0, 0), t1 = t.at(tp, 1, 0);
    const double e = bp ? -1.0 : 1.0;
    const double b0 = e * t.at(bp, 0, 0), b1 = -e * t.at(bp, 1, 0);
    const double det = t0 * b1 - t1 * b0;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const double rt = -(t.at(2 + 2 * tp + c, 0, 0) + t.at(2 + 2 * tp + c, 1, 0));
      const double rb = -e * (t.at(2 + 2 * bp + c, 0, 0) - t.at(2 + 2 * bp + c, 1, 0));
      a0[c] = t.par == 0 ? (rt * b1 - t1 * rb) / det : (t0 * rb - b0 * rt) / det;
    }
    __syncthreads();
  }
}

// The four equations run the same code, so that a compute unit's workgroups share
// it in the instruction cache: with H = D x + hd D^2 f + hf f (- a),
//   w      x = Q,    f = P,                       hd = -1, hf = -k^2
//   omega  x = B,    f = A,                       hd = 0,  hf = 1
//   phi    x = 0,    f = c / Pe - (1 + s Ch^2) / Pe phi, hd = 1, hf = -k^2, - a
//   U, V   x = T_xz, T_yz of the mean line, f = 0
// then the right-hand side from the state and one or two solves.
template <int NC, bool BOTH>
__global__ void __launch_bounds__((BOTH ? 128 : 64) * tau_pieces(NC)) k_chan_tau(ChanTauArgs a) {
  using W = TauWave<NC, 9, BOTH>;
  constexpr int LEN = W::LEN;
  __shared__ double sh[W::NV * W::NW * 64];
  const W t(sh);
  const int y = int(blockIdx.y);
  const int eq = a.sp && y == 2 ? 3 : y;     // 0 w, 1 omega, 2 phi, 3 the mean lines
  if (eq == 3 && blockIdx.x) return;
  // the equation's arrays: explicit terms (x, f), history, state, its stride and line
  const long long nt = a.nl;                 // line stride of the terms
  const long long ns = eq == 3 ? 2 : nt;     // of the state and the history
  const long long l = eq == 3 ? t.ln : (long long)blockIdx.x * 64 + t.ln;
  const bool valid = l < ns;
  const unsigned lc = valid ? unsigned(l) : 0u;   // lanes past the last line read line 0 and store nothing
  const unsigned lt = eq == 3 ? 0u : lc;
  cpx<double>* __restrict__ state = eq == 0 ? a.w : eq == 1 ? a.om : eq == 2 ? a.phi : a.mean;
  cpx<double>* __restrict__ hist = eq == 3 ? a.hmean : a.hist + (eq == 0 ? 1 : eq == 1 ? 0 : 2) * a.nzl;
  const double kx = eq == 3 ? 0.0 : a.kx[lc], ky = eq == 3 ? 0.0 : a.ky[lc], k2 = kx * kx + ky * ky;
  double x[LEN][2], c[2], e[2], b[2];
  {
    double f[LEN][2];
    if (eq == 2) {
      tau_load<0>(t, a.terms + 5 * a.nzl, nt, lc, a.kz, f);
      tau_load<0>(t, state, ns, lc, NC, x);
#pragma unroll
      for (int k = 0; k < LEN; ++k)
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          f[k][d] = a.inv_pe * f[k][d] - a.e_coef * x[k][d];
          x[k][d] = 0.0;
        }
    } else {
      // the mean lines: T_xz, T_yz of line 0 in the arrays B, Q
      const cpx<double>* up = a.terms + (eq == 0 || (eq == 3 && lc == 1) ? 3 : 1) * a.nzl;
      tau_load<1>(t, up, nt, lt, a.kz, x);
      tau_load<0>(t, a.terms + (eq == 0 ? 2 : 0) * a.nzl, nt, lt, a.kz, f);
    }
    // H into x
    d_put(t, 0, x);
    d2_put(t, 2, f);
    __syncthreads();
    d_carry(t, 0, c);
    d2_carry(t, 2, e, b);
    __syncthreads();
    {
      const double hd = eq == 0 ? -1.0 : eq == 2 ? 1.0 : 0.0;
      // omega and w vanish on the mean line
      const double live = eq < 2 && lc == 0 ? 0.0 : 1.0;
      const double hf = eq == 1 ? live : -k2;
      double tn = 2.0 * t.dn(LEN - 1);
#pragma unroll
      for (int k = LEN - 1; k >= 0; --k, tn -= 4.0) {
        const double s = k == 0 && t.n(0) == 0 ? 0.5 * live : live;
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          c[d] += (tn + 2.0) * x[k][d];
          b[d] += (tn + 2.0) * e[d];
          e[d] += tn * f[k][d];
          x[k][d] = s * (c[d] + hd * b[d]) + hf * f[k][d];
        }
      }
    }
  }
  if (eq == 2) {
    double adv[LEN][2];
    tau_load<0>(t, a.terms + 4 * a.nzl, nt, lc, a.kz, adv);
#pragma unroll
    for (int k = 0; k < LEN; ++k)
#pragma unroll
      for (int d = 0; d < 2; ++d) x[k][d] -= adv[k][d];
  }
  // Adams-Bashforth with the history: x <- E
  {
    double hp[LEN][2];
    tau_load<0>(t, hist, ns, lc, NC, hp);
#pragma unroll
    for (int k = 0; k < LEN; ++k) {
      if (valid && t.in(k)) (hist + (long long)t.n(k) * ns)[lc] = cpx<double>{x[k][0], x[k][1]};
#pragma unroll
      for (int d = 0; d < 2; ++d) x[k][d] = a.ab1 ? x[k][d] : 1.5 * x[k][d] - 0.5 * hp[k][d];
    }
  }
  double st[LEN][2];
  tau_load<0>(t, state, ns, lc, NC, st);
  if (eq == 2) {
#pragma unroll
    for (int k = 0; k < LEN; ++k)
#pragma unroll
      for (int d = 0; d < 2; ++d) st[k][d] = a.g_phi_scale * (st[k][d] + a.dt * x[k][d]);
  } else {
    if (eq == 3 && lc == 0 && t.i0 == 0 && t.par == 0) x[0][0] += a.forcing;   // -dP/dx on T_0
    // g = -(D^2 - k^2 + beta) f - 2 Re E, f the state or, for w, psi = (D^2 - k^2) w
#pragma unroll 1
    for (int pass = eq == 0 ? 0 : 1; pass < 2; ++pass) {
      d2_put(t, 0, st);
      __syncthreads();
      d2_carry(t, 0, e, b);
      __syncthreads();
      const double r2 = pass ? -2.0 * a.re : 0.0, sg = pass ? -1.0 : 1.0, bt = pass ? a.beta : 0.0;
      double tn = 2.0 * t.dn(LEN - 1);
#pragma unroll
      for (int k = LEN - 1; k >= 0; --k, tn -= 4.0) {
        const double s = k == 0 && t.n(0) == 0 ? 0.5 : 1.0;
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          b[d] += (tn + 2.0) * e[d];
          e[d] += tn * st[k][d];
          const double lap = s * b[d] - k2 * st[k][d];
          st[k][d] = t.in(k) ? sg * (lap + bt * st[k][d]) + r2 * x[k][d] : 0.0;
        }
      }
    }
  }
  tau_as_rhs(t, st);
  // the solves: one (omega, mean) or two (psi, w; xi, phi)
  double X[LEN], a0[2];
  TauSums<2> S;
  const int nsolve = eq == 0 || eq == 2 ? 2 : 1;
  const int bc = eq == 2 ? 3 : eq == 0 ? 0 : a.fs;
#pragma unroll 1
  for (int s = 0; s < nsolve; ++s) {
    const double be = eq == 2 ? (s ? a.b_fac : a.a_fac) : eq == 0 && s ? 0.0 : a.beta;
    tau_reduce(t, be + k2, st, X, S);
    chan_a0(t, bc, S, a0);
    tau_values(t, st, X, S, a0);
    if (s + 1 < nsolve) tau_as_rhs(t, st);
  }
  if (eq == 0) {
    // w' = 0 at the no-slip walls: c wh (wh: psi = 1 at both walls for the even
    // parity, +-1 for the odd; sn = sum n^2 w_n, w'(+-1) = sum of +-sn over the parities)
    const double sn[2] = {a0[0] * S.pn + S.qn[0], a0[1] * S.pn + S.qn[1]};
    double cw[2] = {0.0, 0.0};
    if (a.fs == 0) {
      const double r = -1.0 / a.mh[(long long)t.par * nt + lc];
      cw[0] = r * sn[0];
      cw[1] = r * sn[1];
    }
    if constexpr (BOTH) {                         // one no-slip wall: its condition couples the parities
      if (t.pc == 0) {
        t.put(0, sn[0]);
        t.put(1, sn[1]);
      }
      __syncthreads();
      const double m0 = a.mh[lc], m1 = a.mh[nt + lc];
      // the homogeneous solution with psi = 1 at that wall alone is (wh_even +- wh_odd) / 2
      const double sg = a.fs == 1 ? -1.0 : 1.0;   // bit 0: the top wall is free-slip
      const double r = -1.0 / (m0 + m1);
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        const double v = r * (t.at(d, 0, 0) + sg * t.at(d, 1, 0));
        cw[d] = t.par == 0 ? v : sg * v;
      }
      __syncthreads();
    }
    if (a.fs != 3) {
#pragma unroll
      for (int k = 0; k < LEN; ++k) {
        const double h = (a.wh + (long long)(t.in(k) ? t.n(k) : 0) * nt)[lc];
#pragma unroll
        for (int d = 0; d < 2; ++d) st[k][d] += t.in(k) ? cw[d] * h : 0.0;
      }
    }
    if (lc == 0)
#pragma unroll
      for (int k = 0; k < LEN; ++k) st[k][0] = st[k][1] = 0.0;
  }
  if (valid) tau_store(t, state, ns, lc, st);
  if (eq == 0 || eq == 2) d_store(t, eq == 0 ? a.dw : a.dphi, nt, lc, valid, st);
}

// D w (blockIdx.y = 0) and D phi of a state that no step has left: the arithmetic
// of the step's own derivatives, so that a run continued from a saved state
// takes the same bits as the run that saved it.
template <int NC>
__global__ void __launch_bounds__(64 * tau_pieces(NC)) k_tau_deriv(const cpx<double>* __restrict__ w, const cpx<double>* __restrict__ phi,
                                                   cpx<double>* __restrict__ dw, cpx<double>* __restrict__ dphi,
                                                   long long nl) {
  using W = TauWave<NC, 2>;
  __shared__ double sh[W::NV * W::NW * 64];
  const W t(sh);
  const long long l = (long long)blockIdx.x * 64 + t.ln;
  const bool valid = l < nl;
  const unsigned lc = valid ? unsigned(l) : 0u;
  double r[W::LEN][2];
  tau_load<0>(t, blockIdx.y ? phi : w, nl, lc, NC, r);
  d_store(t, blockIdx.y ? dphi : dw, nl, lc, valid, r);
}

// The homogeneous w solutions of a context (beta + k^2 is fixed): psi with value 1
// at both walls (even parity) or +-1 (odd), w from it, zero at the walls: wh
// [nc+1][nl], and mh[parity][nl] = sum n^2 wh_n.
template <int NC>
__global__ void __launch_bounds__(64 * tau_pieces(NC)) k_tau_hom(double beta, const double* __restrict__ kx,
                                                 const double* __restrict__ ky, long long nl, double* __restrict__ wh,
                                                 double* __restrict__ mh) {
  using W = TauWave<NC, 6>;
  __shared__ double sh[W::NV * W::NW * 64];
  const W t(sh);
  const long long l = (long long)blockIdx.x * 64 + t.ln;
  const bool valid = l < nl;
  const long long lc = valid ? l : 0;
  const double k2 = kx[lc] * kx[lc] + ky[lc] * ky[lc];
  double X[W::LEN], r[W::LEN][1], a0[1];
  TauSums<1> S;
#pragma unroll
  for (int k = 0; k < W::LEN; ++k) r[k][0] = 0.0;
  tau_reduce(t, beta + k2, r, X, S);
  a0[0] = (1.0 - S.q1[0]) / S.p1;
  tau_values(t, r, X, S, a0);
  tau_as_rhs(t, r);
  tau_reduce(t, k2, r, X, S);
  a0[0] = -S.q1[0] / S.p1;
  tau_values(t, r, X, S, a0);
  if (!valid) return;
#pragma unroll
  for (int k = 0; k < W::LEN; ++k)
    if (t.in(k)) wh[(long long)t.n(k) * nl + l] = r[k][0];
  if (t.pc == 0) mh[(long long)t.par * nl + l] = a0[0] * S.pn + S.qn[0];
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

hipError_t launch_chan_tau(const ChanTauArgs& a, int nc, hipStream_t st) {
  if (a.nl < 1) return hipErrorInvalidValue;
  const bool both = a.fs == 1 || a.fs == 2;
  const dim3 grid(unsigned((a.nl + 63) / 64), a.sp ? 3 : 4, both ? 1 : 2);
  switch (nc) {
#define PSMS_CASE(NC) \
  case NC: \
    if (both) k_chan_tau<NC, true><<<grid, 128 * tau_pieces(NC), 0, st>>>(a); \
    else k_chan_tau<NC, false><<<grid, 64 * tau_pieces(NC), 0, st>>>(a); \
    return hipGetLastError();
    PSMS_FOR_EACH_TAU_NC(PSMS_CASE)
#undef PSMS_CASE
  }
  return hipErrorInvalidValue;
}

hipError_t launch_tau_deriv(const cpx<double>* w, const cpx<double>* phi, cpx<double>* dw, cpx<double>* dphi, int narr,
                            int nc, long long nl, hipStream_t st) {
  if (nl < 1 || narr < 1 || narr > 2) return hipErrorInvalidValue;
  const dim3 grid(unsigned((nl + 63) / 64), unsigned(narr), 2);
  switch (nc) {
#define PSMS_CASE(NC) case NC: k_tau_deriv<NC><<<grid, 64 * tau_pieces(NC), 0, st>>>(w, phi, dw, dphi, nl); return hipGetLastError();
    PSMS_FOR_EACH_TAU_NC(PSMS_CASE)
#undef PSMS_CASE
  }
  return hipErrorInvalidValue;
}

hipError_t launch_tau_hom(double beta, const double* kx, const double* ky, int nc, long long nl, double* wh,
                          double* mh, hipStream_t st) {
  if (nl < 1) return hipErrorInvalidValue;
  const dim3 grid(unsigned((nl + 63) / 64), 1, 2);
  switch (nc) {
#define PSMS_CASE(NC) \
  case NC: k_tau_hom<NC><<<grid, 64 * tau_pieces(NC), 0, st>>>(beta, kx, ky, nl, wh, mh); return hipGetLastError();
    PSMS_FOR_EACH_TAU_NC(PSMS_CASE)
#undef PSMS_CASE
  }
  return hipErrorInvalidValue;
}

hipError_t launch_wall_tau(const WallTauArgs& a, int nc, hipStream_t st) {
  if (a.nl < 1) return a.nl == 0 ? hipSuccess : hipErrorInvalidValue;
  const dim3 grid(unsigned((a.nl + 63) / 64), 3, 2);
  switch (nc) {
#define PSMS_CASE(NC) \
  case NC: k_wall_tau<NC><<<grid, 64 * tau_pieces(NC), 0, st>>>(a); return hipGetLastError();
    PSMS_FOR_EACH_TAU_NC(PSMS_CASE)
#undef PSMS_CASE
  }
  return hipErrorInvalidValue;
}

}  // namespace psms
