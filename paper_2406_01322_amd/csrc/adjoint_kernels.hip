// Discrete adjoint of the periodic-box step (FP64).
//
// The step maps (x^n, h^n) to x^{n+1} = A x^n + B (alpha S^n + beta h^n),
// h^{n+1} = S^n with S^n = R(x^n; We) the projected nonlinear terms.  Its
// transpose, given lam = dJ/dx^{n+1} and mu = dJ/dh^{n+1}, is
//   Sbar = alpha B lam + mu,  mu^n = beta B lam,
//   lam^n = A lam + (dR/dx)^T Sbar,  dJ/dWe += (dR/dWe)^T Sbar,
// under the half-spectrum inner product sum_k w_k Re(conj(a_k) b_k)
// (w = 1 at kx = 0, 2 otherwise), for which per-mode real factors are
// self-adjoint, (i k)^T = -i k, and the transforms are transposes of each
// other up to n^3.  R in the divergence form of the forward kernels:
//   S_i = P sum_j i k_j F(T_ij), T_ij = -u_i u_j + c (|g|^2 d_ij - g_i g_j),
//   S_phi = -F(u.g) - (k^2/Pe) F(phi^3) + E k^2 phi_hat, g = grad phi.
// Kernels (one adjoint step = z_in, y-inverse, x, y-forward, z_out):
//   k_zadj_in   per mode: Sbar, mu^n, A lam + E k^2 Sbar_phi, and the spectral
//               cotangents of the 8 transformed products, z-inverted;
//   k_xadj      per row pair: the physical forward fields (x-inverse of the
//               forward step's y-inverse output), the transposed products and
//               the We term, x-forward of the 7 field cotangents;
//   k_zadj_out  per line: z-forward of the 7 cotangents, added into lam^n.
#include <hip/hip_runtime.h>

#include "adjoint_kernels.hpp"
#include "fft_engine.hpp"

namespace psms {

// -------------------------------------------------------------------------
template <int N>
__global__ void __launch_bounds__(256) k_zadj_in(cpx<double>* __restrict__ lam, cpx<double>* __restrict__ mu,
                                                 cpx<double>* __restrict__ gout, const cpx<double>* __restrict__ tw_g,
                                                 AdjCoef ac) {
  using P = Plan<N>;
  using G = Tile<P>;
  constexpr int E = G::E, L = G::L, LP = L + 1, K = G::K, C = G::C, H = G::H;
  constexpr int Q = C * H;
  constexpr long long M = (long long)C * Q;
  constexpr int RI = first_radix<P, 1>(), RO = last_radix<P, 1>();
  __shared__ cpx<double> tw[N];
  __shared__ cpx<double> lds[2][N * LP];
  const int tid = threadIdx.x;
  const int line = tid % L, t = tid / L;
  for (int i = tid; i < N; i += blockDim.x) tw[i] = tw_g[i];
  const int q = blockIdx.x * L + line;
  const bool valid = q < Q;
  const int iy = valid ? q / H : 0, ix = valid ? q % H : 0;
  const double kx = double(ix), ky = double(iy <= K ? iy : iy - C);
  const IdxPosMajor idx{LP, line};
  int par = 0;

  cpx<double> sb[4][E];  // projected Sbar_u (3) and Sbar_phi at the owned modes
  double kz[E];
  bool inb[E];
#pragma unroll
  for (int b = 0; b < E / RI; ++b)
#pragma unroll
    for (int r = 0; r < RI; ++r) {
      const int e = b * RI + r;
      const int p = slot_pos<P, RI>(t, b, r);
      const int s = band_slot(p, C, N);
      inb[e] = valid && s >= 0;
      kz[e] = double(signed_k(p, N));
#pragma unroll
      for (int c = 0; c < 4; ++c) sb[c][e] = cpx<double>{0.0, 0.0};
      if (inb[e]) {
        const long long id = (long long)s * Q + q;
        const double k2 = kx * kx + ky * ky + kz[e] * kz[e];
        const double a = 0.5 * ac.dt * ac.nu * k2;
        const double Au = (1.0 - a) / (1.0 + a), Bu = ac.dt / (1.0 + a);
        const double Bp = ac.dt / (1.0 + ac.dt * ac.ch2_pe * (k2 * k2 + ac.s * k2));
        const double Ap = Bp / ac.dt;
        cpx<double> S[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const double A = (c < 3) ? Au : Ap, B = (c < 3) ? Bu : Bp;
          const cpx<double> l = lam[c * M + id], m = mu[c * M + id];
          S[c] = cpx<double>{ac.alpha * B * l.re + m.re, ac.alpha * B * l.im + m.im};
          mu[c * M + id] = cpx<double>{ac.beta * B * l.re, ac.beta * B * l.im};
          lam[c * M + id] = cpx<double>{A * l.re, A * l.im};
        }
        if (k2 == 0.0) {
          S[0] = S[1] = S[2] = S[3] = cpx<double>{0.0, 0.0};
        } else {
          const double ir = 1.0 / k2, kze = kz[e];
          const cpx<double> kd = {kx * S[0].re + ky * S[1].re + kze * S[2].re,
                                  kx * S[0].im + ky * S[1].im + kze * S[2].im};
          S[0].re -= kx * kd.re * ir; S[0].im -= kx * kd.im * ir;
          S[1].re -= ky * kd.re * ir; S[1].im -= ky * kd.im * ir;
          S[2].re -= kze * kd.re * ir; S[2].im -= kze * kd.im * ir;
          // direct dependence of S_phi on phi_hat
          const cpx<double> lp = lam[3 * M + id];
          lam[3 * M + id] = cpx<double>{lp.re + ac.e_coef * k2 * S[3].re, lp.im + ac.e_coef * k2 * S[3].im};
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) sb[c][e] = S[c];
      }
    }
  __syncthreads();

  // cotangents of F(T_xx), F(T_yy), F(T_zz), F(T_xy), F(T_xz), F(T_yz), F(a), F(c);
  // the field index is a compile-time constant in each body
  static_for<0, 8>([&](auto fc) {
    constexpr int f = decltype(fc)::value;
    cpx<double> v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      // -i k s  ->  (k s.im, -k s.re)
      const double kze = kz[e];
      cpx<double> x;
      if constexpr (f == 0) x = {kx * sb[0][e].im, -kx * sb[0][e].re};
      else if constexpr (f == 1) x = {ky * sb[1][e].im, -ky * sb[1][e].re};
      else if constexpr (f == 2) x = {kze * sb[2][e].im, -kze * sb[2][e].re};
      else if constexpr (f == 3) x = {ky * sb[0][e].im + kx * sb[1][e].im, -ky * sb[0][e].re - kx * sb[1][e].re};
      else if constexpr (f == 4) x = {kze * sb[0][e].im + kx * sb[2][e].im, -kze * sb[0][e].re - kx * sb[2][e].re};
      else if constexpr (f == 5) x = {kze * sb[1][e].im + ky * sb[2][e].im, -kze * sb[1][e].re - ky * sb[2][e].re};
      else if constexpr (f == 6) x = {-sb[3][e].re, -sb[3][e].im};
      else {
        const double k2 = kx * kx + ky * ky + kze * kze;
        x = {-k2 * ac.inv_pe * sb[3][e].re, -k2 * ac.inv_pe * sb[3][e].im};
      }
      v[e] = x;
    }
    fft_line<double, P, 1>(v, lds[0], lds[1], par, t, idx, tw);
    cpx<double>* dst = gout + (long long)f * N * Q;
    if (valid) {
#pragma unroll
      for (int b = 0; b < E / RO; ++b)
#pragma unroll
        for (int r = 0; r < RO; ++r) dst[(long long)slot_pos<P, RO>(t, b, r) * Q + q] = v[b * RO + r];
    }
  });
}

// -------------------------------------------------------------------------
// x stage of the adjoint.  yf: the forward step's y-inverse output
// [6][N][N][H] (u v w phi dy_phi dz_phi), yb: the product cotangents after
// the y-inverse [8][N][N][H]; out: [7][N][N][H] x-forward of the cotangents
// of u v w phi gx gy gz.  part[blockIdx.x]: this block's share of
// sum_x sum_f Tbar_f dT_f/dc (the We term before the factor -c/(We n^3)).
// A wavefront per field, as in the forward step's x stage: wavefront w of a workgroup
// inverts forward field w and cotangent w of the same LW row pairs (8 has no forward
// field) and leaves the physical values in LDS; after the barrier the first seven
// form and transform one field's cotangent each, and the last sums the We term.  In
// registers, one thread's 22 transforms and 12 fields left one wavefront a SIMD: 158
// us at 128^3 against 114 us (worth 46 us of memory traffic: the rest is LDS exchanges and
// reads at two workgroups a CU).
template <int N>
struct AdjTile {
  using P = Plan<N>;
  static constexpr int E = P::E, TT = N / E, LW = 64 / TT, K = (N - 1) / 3, H = K + 1;
  static constexpr bool SWZ = N % 16 == 0;
  static constexpr int LP = SWZ ? kRowStrideSwz<N> : kRowStride<N>;
  static constexpr int RS = LW * LP > 64 * E ? LW * LP : 64 * E;   // a field's LDS region
  static_assert(TT <= 64 && 64 % TT == 0, "a wavefront holds whole lines");
  static constexpr int blocks() { return int(((long long)N * N / 2 + LW - 1) / LW); }
};
template <int N>
__global__ void __launch_bounds__(512) k_xadj(const cpx<double>* __restrict__ yf, const cpx<double>* __restrict__ yb,
                                              cpx<double>* __restrict__ out, const cpx<double>* __restrict__ tw_g,
                                              double csig, double* __restrict__ part) {
  using P = Plan<N>;
  using A = AdjTile<N>;
  constexpr int E = A::E, TT = A::TT, LW = A::LW, K = A::K, H = A::H, RS = A::RS;
  constexpr int RI = first_radix<P, 1>(), RO = last_radix<P, -1>();
  static_assert(last_radix<P, 1>() == first_radix<P, -1>(), "mirrored radix order");
  constexpr long long ROWS = (long long)N * N, FS = ROWS * H;
  __shared__ cpx<double> twf[tw_size<P, -1>()];
  __shared__ cpx<double> twi[tw_size<P, 1>()];
  __shared__ cpx<double> lds[15][RS];   // u v w gx gy gz phi, then the 8 cotangents
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t = lane % TT, line = lane / TT;
  const long long r0 = ((long long)xcd_tile(blockIdx.x, gridDim.x) * LW + line) * 2;
  const bool valid = r0 < ROWS;   // ROWS is even: both rows exist
  using Idx = std::conditional_t<A::SWZ, IdxLineSwz<N, TT>, IdxLineMajor<N, TT>>;
  const Idx idx{line * A::LP};
  const bool dx = wv == 3;        // gx = i kx phi
  const cpx<double>* sf = yf + (wv < 3 ? wv : wv == 4 ? 4 : wv == 5 ? 5 : 3) * FS + (valid ? r0 : 0) * H;
  const cpx<double>* sb = yb + wv * FS + (valid ? r0 : 0) * H;
  cpx<double> v[2][E];
  // the packed complex line row0 + i row1 of both fields in Hermitian-extended order
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int p = slot_pos<P, RI>(t, e / RI, e % RI);
    const int k = (p <= N / 2) ? p : N - p;
    const bool in = valid && k <= K;
    const cpx<double> zero = {0.0, 0.0};
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const cpx<double>* src = g ? sb : sf;
      cpx<double> a = in ? src[k] : zero, b = in ? src[H + k] : zero;
      if (g == 0 && dx) {
        const double kk = double(k);
        a = cpx<double>{-kk * a.im, kk * a.re};
        b = cpx<double>{-kk * b.im, kk * b.re};
      }
      if (k == 0) {
        a.im = 0.0;
        b.im = 0.0;
      }
      v[g][e] = (p <= N / 2) ? cpx<double>{a.re - b.im, a.im + b.re} : cpx<double>{a.re + b.im, b.re - a.im};
    }
  }
  build_twiddles<double, P, -1>(twf, [&](int m) { return tw_g[m]; }, tid, int(blockDim.x));
  build_twiddles<double, P, 1>(twi, [&](int m) { return tw_g[m]; }, tid, int(blockDim.x));
  __syncthreads();
  int par = 0;
  if (wv < 7) {
    fft_lines<double, P, 1, 2>(v, lds[wv], 7 * RS, 0, par, t, idx, twi);
    wave_lds_sync();   // the exchange's reads, before the values over them
#pragma unroll
    for (int e = 0; e < E; ++e) lds[wv][e * 64 + lane] = v[0][e];
  } else {
    fft_lines<double, P, 1, 1>(v + 1, lds[14], 0, 0, par, t, idx, twi);
    wave_lds_sync();
  }
#pragma unroll
  for (int e = 0; e < E; ++e) lds[7 + wv][e * 64 + lane] = v[1][e];
  __syncthreads();
  const double c2 = 2.0 * csig;
  auto at = [&](int f, int e) { return lds[f][e * 64 + lane]; };
  // component-wise products of the two rows
  auto mul = [](cpx<double> a, cpx<double> b) { return cpx<double>{a.re * b.re, a.im * b.im}; };
  static_for<0, 7>([&](auto fc) {
    constexpr int F = decltype(fc)::value;
    if (wv == F) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        auto f = [&](int i) { return at(i, e); };
        auto x = [&](int i) { return at(7 + i, e); };
        cpx<double> r;
        if constexpr (F < 3) {
          // u: -2 u x0 - v x3 - w x4 + gx x6; v: -2 v x1 - u x3 - w x5 + gy x6; w: ..
          constexpr int i1 = F == 0 ? 1 : 0, c1 = F == 2 ? 4 : 3, i2 = F == 2 ? 1 : 2, d1 = F == 0 ? 4 : 5;
          const cpx<double> a = mul(f(F), x(F)), b = mul(f(i1), x(c1)), c = mul(f(i2), x(d1)), d = mul(f(3 + F), x(6));
          r = cpx<double>{-2.0 * a.re - b.re - c.re + d.re, -2.0 * a.im - b.im - c.im + d.im};
        } else if constexpr (F == 6) {
          const cpx<double> ph = f(6), a = mul(mul(ph, ph), x(7));
          r = cpx<double>{3.0 * a.re, 3.0 * a.im};
        } else {
          // gx: 2c gx (x1 + x2) - c gy x3 - c gz x4 + u x6; gy: 2c gy (x0 + x2) - c gx x3 - c gz x5 + v x6; gz: ..
          constexpr int g = F - 3, n1 = g == 0 ? 1 : 0, n2 = g == 2 ? 1 : 2;
          constexpr int i1 = g == 0 ? 4 : 3, c1 = g == 2 ? 4 : 3, i2 = g == 2 ? 4 : 5, d1 = g == 0 ? 4 : 5;
          const cpx<double> a = mul(f(F), cadd(x(n1), x(n2))), b = mul(f(i1), x(c1)), c = mul(f(i2), x(d1)),
                            d = mul(f(g), x(6));
          r = cpx<double>{c2 * a.re - csig * (b.re + c.re) + d.re, c2 * a.im - csig * (b.im + c.im) + d.im};
        }
        v[0][e] = r;
      }
    }
  });
  if (wv == 7) {
    double dwe = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const cpx<double> gx = at(3, e), gy = at(4, e), gz = at(5, e);
      const cpx<double> xx = mul(gx, gx), yy = mul(gy, gy), zz = mul(gz, gz);
      const cpx<double> s0 = mul(at(7, e), cadd(yy, zz)), s1 = mul(at(8, e), cadd(xx, zz)), s2 = mul(at(9, e), cadd(xx, yy));
      const cpx<double> s3 = mul(at(10, e), mul(gx, gy)), s4 = mul(at(11, e), mul(gx, gz)), s5 = mul(at(12, e), mul(gy, gz));
      const cpx<double> d = csub(cadd(cadd(s0, s1), s2), cadd(cadd(s3, s4), s5));
      dwe += d.re + d.im;
    }
    if (!valid) dwe = 0.0;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) dwe += __shfl_xor(dwe, d);   // fixed order: deterministic
    if (lane == 0) part[blockIdx.x] = dwe;
  }
  __syncthreads();
  if (wv == 7) return;
  cpx<double>* buf = lds[wv];
  fft_lines<double, P, -1, 1>(v, buf, 0, 0, par, t, idx, twf);
  wave_lds_sync();
  // natural order, then the retained kx of both rows
#pragma unroll
  for (int e = 0; e < E; ++e) buf[idx(slot_pos<P, RO>(t, e / RO, e % RO))] = v[0][e];
  wave_lds_sync();
  cpx<double>* dst = out + (wv < 3 ? wv : wv == 6 ? 3 : wv + 1) * FS + r0 * H;
  for (int k = t; valid && k < H; k += TT) {
    const cpx<double> zk = buf[idx(k)], zm = buf[idx((N - k) % N)];
    dst[k] = cpx<double>{0.5 * (zk.re + zm.re), 0.5 * (zk.im - zm.im)};
    dst[H + k] = cpx<double>{0.5 * (zk.im + zm.im), 0.5 * (zm.re - zk.re)};
  }
}

// -------------------------------------------------------------------------
// z-forward of the 7 field cotangents [7][N][C][H] and accumulation into lam:
// lam_u += F(ubar), lam_phi += F(phibar) - sum_j i k_j F(gbar_j).
template <int N>
__global__ void __launch_bounds__(256) k_zadj_out(const cpx<double>* __restrict__ zin, cpx<double>* __restrict__ lam,
                                                  const cpx<double>* __restrict__ tw_g, double inv_n3) {
  using P = Plan<N>;
  using G = Tile<P>;
  constexpr int E = G::E, L = G::L, LP = L + 1, K = G::K, C = G::C, H = G::H;
  constexpr int Q = C * H;
  constexpr long long M = (long long)C * Q;
  constexpr int RF = first_radix<P, -1>(), RL = last_radix<P, -1>();
  __shared__ cpx<double> tw[N];
  __shared__ cpx<double> lds[2][N * LP];
  const int tid = threadIdx.x;
  const int line = tid % L, t = tid / L;
  for (int i = tid; i < N; i += blockDim.x) tw[i] = tw_g[i];
  const int q = blockIdx.x * L + line;
  const bool valid = q < Q;
  const int iy = valid ? q / H : 0, ix = valid ? q % H : 0;
  const double kx = double(ix), ky = double(iy <= K ? iy : iy - C);
  const IdxPosMajor idx{LP, line};
  int par = 0;
  cpx<double> acc[4][E];
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int e = 0; e < E; ++e) acc[c][e] = cpx<double>{0.0, 0.0};
  __syncthreads();
#pragma unroll 1
  for (int f = 0; f < 7; ++f) {
    cpx<double> v[E];
    const cpx<double>* src = zin + (long long)f * N * Q;
#pragma unroll
    for (int b = 0; b < E / RF; ++b)
#pragma unroll
      for (int r = 0; r < RF; ++r)
        v[b * RF + r] = valid ? src[(long long)slot_pos<P, RF>(t, b, r) * Q + q] : cpx<double>{0.0, 0.0};
    fft_line<double, P, -1>(v, lds[0], lds[1], par, t, idx, tw);
#pragma unroll
    for (int b = 0; b < E / RL; ++b)
#pragma unroll
      for (int r = 0; r < RL; ++r) {
        const int e = b * RL + r;
        const cpx<double> w = {v[e].re * inv_n3, v[e].im * inv_n3};
        const double kz = double(signed_k(slot_pos<P, RL>(t, b, r), N));
        if (f == 0) acc[0][e] = cadd(acc[0][e], w);
        else if (f == 1) acc[1][e] = cadd(acc[1][e], w);
        else if (f == 2) acc[2][e] = cadd(acc[2][e], w);
        else if (f == 3) acc[3][e] = cadd(acc[3][e], w);
        else {
          const double k = (f == 4) ? kx : (f == 5) ? ky : kz;   // -i k w
          acc[3][e].re += k * w.im;
          acc[3][e].im -= k * w.re;
        }
      }
  }
  if (valid) {
#pragma unroll
    for (int b = 0; b < E / RL; ++b)
#pragma unroll
      for (int r = 0; r < RL; ++r) {
        const int e = b * RL + r;
        const int s = band_slot(slot_pos<P, RL>(t, b, r), C, N);
        if (s >= 0) {
          const long long id = (long long)s * Q + q;
#pragma unroll
          for (int c = 0; c < 4; ++c) lam[c * M + id] = cadd(lam[c * M + id], acc[c][e]);
        }
      }
  }
}

// Terminal cotangent of J = V (<|grad phi|^2> + 1/2 <|u|^2>):
// lam_u = V u_hat, lam_phi = 2 V k^2 phi_hat, mu = 0 (compact band, per mode).
__global__ void k_adj_terminal(const cpx<double>* __restrict__ st, cpx<double>* __restrict__ lam,
                               cpx<double>* __restrict__ mu, int K, int C, int H, long long M, double vol) {
  for (long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x; id < M;
       id += (long long)gridDim.x * blockDim.x) {
    const int ix = int(id % H);
    const int iy = int((id / H) % C);
    const int iz = int(id / ((long long)H * C));
    const double kx = ix, ky = (iy <= K) ? iy : iy - C, kz = (iz <= K) ? iz : iz - C;
    const double k2 = kx * kx + ky * ky + kz * kz;
    for (int c = 0; c < 3; ++c) {
      const cpx<double> a = st[c * M + id];
      lam[c * M + id] = cpx<double>{vol * a.re, vol * a.im};
    }
    const cpx<double> p = st[3 * M + id];
    lam[3 * M + id] = cpx<double>{2.0 * vol * k2 * p.re, 2.0 * vol * k2 * p.im};
    for (int c = 0; c < 4; ++c) mu[c * M + id] = cpx<double>{0.0, 0.0};
  }
}

// acc[0] += scale * sum(part[0..n-1]) in a fixed order (one block).
__global__ void k_adj_sum(const double* __restrict__ part, int n, double scale, double* __restrict__ acc) {
  __shared__ double red[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) s += part[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int k = blockDim.x / 2; k > 0; k >>= 1) {
    if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) acc[0] += scale * red[0];
}

// -------------------------------------------------------------------------
#define PSMS_FOR_EACH_N(X) X(8) X(12) X(16) X(24) X(32) X(48) X(64) X(96) X(128) X(192) X(256)

namespace {
template <int N>
hipError_t adj_n(int stage, cpx<double>* lam, cpx<double>* mu, const cpx<double>* a, const cpx<double>* b,
                 cpx<double>* out, const cpx<double>* tw, const AdjCoef& ac, double csig, double* part,
                 hipStream_t st) {
  using P = Plan<N>;
  using G = Tile<P>;
  const int Q = G::C * G::H;
  const unsigned threads = unsigned(G::L * G::TT);
  if (stage == 0) {
    k_zadj_in<N><<<unsigned((Q + G::L - 1) / G::L), threads, 0, st>>>(lam, mu, out, tw, ac);
  } else if (stage == 1) {
    k_xadj<N><<<unsigned(AdjTile<N>::blocks()), 512, 0, st>>>(a, b, out, tw, csig, part);
  } else {
    k_zadj_out<N><<<unsigned((Q + G::L - 1) / G::L), threads, 0, st>>>(a, lam, tw, ac.inv_n3);
  }
  return hipGetLastError();
}
}  // namespace

int adj_xblocks(int n) {
  switch (n) {
#define PSMS_CASE(NN) \
  case NN: return AdjTile<NN>::blocks();
    PSMS_FOR_EACH_N(PSMS_CASE)
#undef PSMS_CASE
  }
  return 0;
}

hipError_t launch_adj_stage(int n, int stage, cpx<double>* lam, cpx<double>* mu, const cpx<double>* a,
                            const cpx<double>* b, cpx<double>* out, const cpx<double>* tw, const AdjCoef& ac,
                            double csig, double* part, hipStream_t st) {
  switch (n) {
#define PSMS_CASE(NN) case NN: return adj_n<NN>(stage, lam, mu, a, b, out, tw, ac, csig, part, st);
    PSMS_FOR_EACH_N(PSMS_CASE)
#undef PSMS_CASE
  }
  return hipErrorInvalidValue;
}

hipError_t launch_adj_terminal(const cpx<double>* state, cpx<double>* lam, cpx<double>* mu, int K, int C, int H,
                               long long M, double vol, hipStream_t st) {
  long long b = (M + 255) / 256;
  if (b > 65536) b = 65536;
  k_adj_terminal<<<unsigned(b), 256, 0, st>>>(state, lam, mu, K, C, H, M, vol);
  return hipGetLastError();
}

hipError_t launch_adj_sum(const double* part, int n, double scale, double* acc, hipStream_t st) {
  k_adj_sum<<<1, 256, 0, st>>>(part, n, scale, acc);
  return hipGetLastError();
}

}  // namespace psms
