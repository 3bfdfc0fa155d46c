// Wall-normal (Chebyshev) kernels of the channel: Sec. 2.2 and Sec. 3.2.
//
//  * k_dct: the Chebyshev transform as a DCT-I obtained from the FFT of the
//    2 nc-point even extension of each line (Sec. 3.2.1), applied to the real
//    and imaginary parts at once; k_dct_half the same through one nc-point
//    FFT.  Lines are (kx, ky) pairs, stored position-major ([n][line]), so the
//    lanes of a wavefront read consecutive lines and no transpose is needed.
//    Both read through a source: an array, or the channel step's fields formed
//    from the state as they are loaded.
//  * k_cheb_seg: derivative in coefficient space, the backward recurrence
//    c_{n-1} b_{n-1} = b_{n+1} + 2 n a_n summed piecewise along each parity chain.
//  * k_helm: the Chebyshev-tau Helmholtz problem (D^2 - beta) f = g with two
//    Dirichlet or Neumann boundary rows, in FP64.  Rewriting the tau rows with
//    the integration recurrence turns each parity (even / odd n) into a
//    tridiagonal system plus one boundary row; it is solved by one downward
//    elimination sweep and two upward sweeps, one thread per (line, parity)
//    (the banded wall-normal solves of Sec. 3.2.2).  The solves of the channel
//    step and of psms_wall_solve are in channel_tau.hip.
//  * k_influence: the influence-matrix combination that enforces w' = 0 at the
//    walls; k_cheb_uv: u, v from continuity and eq. omegadef.
#include <hip/hip_runtime.h>

#include "channel_kernels.hpp"
#include "fft_engine.hpp"
#include "tau_rows.hpp"

namespace psms {

namespace {

// The transforms' plans: radix 8 for lines of 128 and 256, half the threads and one
// exchange (with its barrier) fewer (256 x 256 x 257 in FP64: products 206 -> 185 us,
// fields 140 -> 128; five steps of 256 x 128 x 129 in MIXED 1433 -> 1424 us).  The
// 512-point extension (FP32, nc = 256) still runs radix 4 and 2 on 8 lines; 8 x 8 x 8 on
// 8 lines measured 200 against 246 us for ten transforms of 14706 lines and is not built.
template <int N>
struct DctPlanSel {
  using type = Plan<N>;
};
template <> struct DctPlanSel<128> { using type = PlanT<128, 8, 8, 8, 2>; };
template <> struct DctPlanSel<256> { using type = PlanT<256, 8, 8, 8, 4>; };
template <int N>
using DctPlan = typename DctPlanSel<N>::type;

// 16 lines per workgroup (8 for the 512-point extension, nc = 256): the lanes
// of a position read 16 consecutive lines (128 bytes in FP32), and the LDS
// tile stays within 160 KB in FP64.
template <class P>
struct CTile {
  static constexpr int N = P::N;
  static constexpr int E = P::E;
  static constexpr int TT = N / E;
  static constexpr int L = (16 * TT <= 1024) ? 16 : 1024 / TT;
  static_assert(L * TT <= 1024, "workgroup size");
  static_assert(2 * N * (L + 1) * 16 + N * 16 <= 160 * 1024, "LDS tile");
};

}  // namespace

// Where the DCT kernels read their input: an array [field][n][line] (ArraySrc), the
// channel step's fields formed from the FP64 state as they are loaded
// (ChanFieldSrc: u, v by continuity and the definition of omega_z, w, phi, i ky phi,
// D phi), or its combinations of the products (ChanTermSrc).  The last two serve
// two transforms that share inputs to one workgroup: pair Q reads Raw values at a
// point (all rows of a thread are loaded before the first is used) and forms both
// inputs from them.  field(q, side): the transform of a pair's side.
template <typename T>
struct ArraySrc {
  static constexpr int kPairs = 1, kSides = 1;
  const cpx<T>* in;
  long long fstride;
  struct Line {};
  using Raw = cpx<T>;
  __device__ __forceinline__ Line at(long long) const { return {}; }
  __device__ __forceinline__ static int field(int q, int) { return q; }
  template <int Q>
  __device__ __forceinline__ Raw load(long long id) const {
    return in[(long long)blockIdx.y * fstride + id];
  }
  template <int Q>
  __device__ __forceinline__ void form(const Raw& r, const Line&, bool, int, long long, cpx<T>& a, cpx<T>&) const {
    a = r;
  }
};
template <typename T>
struct ChanFieldSrcT {
  static constexpr int kPairs = 3, kSides = 2;
  ChanFieldSrc s;
  struct Line {
    double kx, ky, ik2;
  };
  struct Raw {
    cpx<double> x[2];
  };
  __device__ __forceinline__ Line at(long long l) const {
    const double kx = s.kx[l], ky = s.ky[l];
    return Line{kx, ky, 1.0 / (kx * kx + ky * ky)};
  }
  // (u, v), (w, D phi), (phi, i ky phi)
  __device__ __forceinline__ static int field(int q, int side) {
    return q == 0 ? side : q == 1 ? 2 + 3 * side : 3 + side;
  }
  template <int Q>
  __device__ __forceinline__ Raw load(long long id) const {
    if constexpr (Q == 0) return Raw{{s.om[id], s.dw[id]}};
    else if constexpr (Q == 1) return Raw{{s.w[id], s.dphi[id]}};
    else return Raw{{s.phi[id], cpx<double>{0.0, 0.0}}};
  }
  template <int Q>
  __device__ __forceinline__ void form(const Raw& r, const Line& k, bool mean, int j, long long id, cpx<T>& a,
                                       cpx<T>& b) const {
    cpx<double> x, y;
    if constexpr (Q == 0) {
      const cpx<double> o = r.x[0], d = r.x[1];
      const cpx<double> p = {k.kx * d.re + k.ky * o.re, k.kx * d.im + k.ky * o.im};
      const cpx<double> q = {k.ky * d.re - k.kx * o.re, k.ky * d.im - k.kx * o.im};
      x = cpx<double>{k.ik2 * (-1.0 * p.im), k.ik2 * (1.0 * p.re)};   // i p / k^2
      y = cpx<double>{k.ik2 * (-1.0 * q.im), k.ik2 * (1.0 * q.re)};
      if (mean) {                                                     // the mean line carries U, V
        x = s.mean[2 * j];
        y = s.mean[2 * j + 1];
      }
    } else if constexpr (Q == 1) {
      x = r.x[0];
      y = r.x[1];
    } else {
      x = r.x[0];
      y = cpx<double>{-k.ky * x.im, k.ky * x.re};
    }
    a = cpx<T>{T(x.re), T(x.im)};
    b = cpx<T>{T(y.re), T(y.im)};
  }
};

// The combinations of the transformed products that the wall-normal right-hand
// sides need, formed in FP64 from the y-forward output [8][j][line] and rounded
// once to the transform's precision: four transforms and FP64 arrays in place of
// six.
template <typename T>
struct ChanTermSrcT {
  static constexpr int kPairs = 3, kSides = 2;
  const cpx<T>* t;   // T_xx T_yy T_zz T_xy T_xz T_yz (a, c), fstride apart
  long long fstride;
  const double* kxl;
  const double* kyl;
  struct Line {
    double kx, ky;
  };
  struct Raw {
    cpx<T> x[4];
  };
  __device__ __forceinline__ Line at(long long l) const { return Line{kxl[l], kyl[l]}; }
  // (A, Q), (B, P), (a, c)
  __device__ __forceinline__ static int field(int q, int side) {
    return q == 0 ? 3 * side : q == 1 ? 1 + side : 4 + side;
  }
  template <int Q>
  __device__ __forceinline__ Raw load(long long id) const {
    const cpx<T> z = {T(0), T(0)};
    if constexpr (Q == 0) return Raw{{t[id], t[fstride + id], t[2 * fstride + id], t[3 * fstride + id]}};
    else return Raw{{t[(2 + 2 * Q) * fstride + id], t[(3 + 2 * Q) * fstride + id], z, z}};
  }
  template <int Q>
  __device__ __forceinline__ void form(const Raw& r, const Line& k, bool mean, int j, long long id, cpx<T>& a,
                                       cpx<T>& b) const {
    if constexpr (Q == 2) {
      a = r.x[0];
      b = r.x[1];
      return;
    }
    auto up = [](cpx<T> v) { return cpx<double>{double(v.re), double(v.im)}; };
    const double kx = k.kx, ky = k.ky;
    cpx<double> x, y;
    if constexpr (Q == 0) {
      // (ky^2 - kx^2) T_xy + kx ky (T_xx - T_yy); kx^2 T_xx + 2 kx ky T_xy + ky^2 T_yy - k^2 T_zz
      const cpx<double> xx = up(r.x[0]), yy = up(r.x[1]), zz = up(r.x[2]), xy = up(r.x[3]);
      const double ca = ky * ky - kx * kx, cb = kx * ky;
      x = cpx<double>{ca * xy.re + cb * (xx.re - yy.re), ca * xy.im + cb * (xx.im - yy.im)};
      const double da = kx * kx, db = 2.0 * kx * ky, dc = ky * ky, dd = da + dc;
      y = cpx<double>{da * xx.re + db * xy.re + dc * yy.re - dd * zz.re, da * xx.im + db * xy.im + dc * yy.im - dd * zz.im};
    } else {
      // i kx T_yz - i ky T_xz, i kx T_xz + i ky T_yz
      const cpx<double> xz = up(r.x[0]), yz = up(r.x[1]);
      x = cpx<double>{-(kx * yz.im - ky * xz.im), kx * yz.re - ky * xz.re};
      y = cpx<double>{-(kx * xz.im + ky * yz.im), kx * xz.re + ky * yz.re};
    }
    a = cpx<T>{T(x.re), T(x.im)};
    b = cpx<T>{T(y.re), T(y.im)};
    if (mean) {   // the mean line: T_xz in the second array, T_yz in the fourth
      a = Q == 0 ? cpx<T>{T(0), T(0)} : r.x[0];
      b = Q == 0 ? t[5 * fstride + id] : cpx<T>{T(0), T(0)};
    }
  }
};

// f(integral_constant<int, q>) for the run-time pair q (uniform in a workgroup)
template <class Src, class F>
__device__ __forceinline__ void with_pair(int q, F&& f) {
  if constexpr (Src::kPairs == 1) f(std::integral_constant<int, 0>{});
  else if (q == 0) f(std::integral_constant<int, 0>{});
  else if (q == 1) f(std::integral_constant<int, 1>{});
  else f(std::integral_constant<int, 2>{});
}

// The workgroup's lines staged through LDS: each input is read once (a transform's
// positions need x_j twice), and a pair's inputs for both its sides.  The step's
// transforms are bound by these reads and their writes: at 256 x 256 x 257 in FP64
// the products' took 350 us and the fields' 211 with a workgroup a field reading
// each input twice, 185 and 128 now (0.52 and 0.24 GB); at 256 x 128 x 129 in FP32
// 54 and 48 us, now 32 and 32.
// put(j, a, b) with the sides' inputs a[0], b[0] at j = 0 .. NC, a thread's rows
// being t, t + TT, ..; PAIRED: j = 0 .. NC / 2, and a[1], b[1] at NC - j.
template <typename T, class Src, int NC, int TT, bool PAIRED, class Put>
__device__ __forceinline__ void dct_stage(const Src& src, int q, int t, long long l, long long nlines, bool mean,
                                          Put&& put) {
  constexpr int NJ = PAIRED ? NC / 2 : NC;         // rows 0 .. NJ
  constexpr int NR = NJ / TT;                      // whole rounds; then the rows past them
  static_assert(NR * TT <= NJ && (NR + 1) * TT > NJ, "rows");
  const typename Src::Line k = src.at(l);
  with_pair<Src>(q, [&](auto qi) {
    constexpr int Q = decltype(qi)::value;
    typename Src::Raw ra[NR + 1], rb[PAIRED ? NR + 1 : 1];
    const bool more = t <= NJ - NR * TT;
#pragma unroll
    for (int i = 0; i <= NR; ++i) {
      const int j = t + ((i < NR || more) ? i * TT : 0);
      ra[i] = src.template load<Q>((long long)j * nlines + l);
      if constexpr (PAIRED) rb[i] = src.template load<Q>((long long)(NC - j) * nlines + l);
    }
#pragma unroll
    for (int i = 0; i <= NR; ++i) {
      if (i == NR && !more) break;
      const int j = t + i * TT;
      cpx<T> a[2] = {}, b[2] = {};   // at j and NC - j
      src.template form<Q>(ra[i], k, mean, j, (long long)j * nlines + l, a[0], b[0]);
      if constexpr (PAIRED) src.template form<Q>(rb[i], k, mean, NC - j, (long long)(NC - j) * nlines + l, a[1], b[1]);
      put(j, a, b);
    }
  });
}

// dir = +1: values at the CGL points -> Chebyshev coefficients,
//   a_n = G_n / (nc cbar_n),  G = FFT of the even extension of f;
// dir = -1: coefficients -> values, f_j = FFT of the even extension of b with
//   b_0 = a_0, b_nc = a_nc, b_n = a_n / 2.
// out64 (forward only, if not NULL): the coefficients n <= kz are written in
// FP64 instead (the products' Chebyshev truncation; its reader takes the others
// as zero), so the step needs no separate promotion pass.
// both: a workgroup transforms both sides of a pair, one after the other; else
// each side has a workgroup (blockIdx.y = 2 pair + side).
template <typename T, int N, class Src>
__global__ void __launch_bounds__(CTile<DctPlan<N>>::L * CTile<DctPlan<N>>::TT)
k_dct(Src src, cpx<T>* __restrict__ out, long long nlines, int nfield, int both, int dir, long long fstride,
      const cpx<T>* __restrict__ tw_g, cpx<double>* __restrict__ out64, int kz) {
  using P = DctPlan<N>;
  using G = CTile<P>;
  constexpr int E = G::E, L = G::L, LP = L + 1, TT = G::TT, NC = N / 2;
  constexpr int RI = first_radix<P, -1>(), RO = last_radix<P, -1>();
  __shared__ cpx<T> tw[N];
  __shared__ cpx<T> lds[2][N * LP];
  const int tid = threadIdx.x;
  const int line = tid % L, t = tid / L;
  const int q = (Src::kSides == 1 || both) ? blockIdx.y : blockIdx.y / 2;
  const int side0 = (Src::kSides == 1 || both) ? 0 : blockIdx.y % 2, side1 = (Src::kSides == 2 && both) ? 1 : side0;
  if (src.field(q, side0) >= nfield) return;
  if (tw_g) {
    for (int i = tid; i < N; i += blockDim.x) tw[i] = tw_g[i];
  } else {
    for (int i = tid; i < N; i += blockDim.x) {
      double s, c;
      sincospi(-2.0 * double(i) / double(N), &s, &c);
      tw[i] = cpx<T>{T(c), T(s)};
    }
  }
  const long long l = (long long)xcd_tile(blockIdx.x, gridDim.x) * L + line;
  const bool valid = l < nlines;
  const IdxPosMajor idx{LP, line};
  dct_stage<T, Src, NC, TT, false>(src, q, t, valid ? l : nlines - 1, nlines, l == 0, [&](int j, cpx<T>* a, cpx<T>* b) {
    if (dir < 0 && j != 0 && j != NC) {
      a[0] = cpx<T>{T(0.5) * a[0].re, T(0.5) * a[0].im};
      b[0] = cpx<T>{T(0.5) * b[0].re, T(0.5) * b[0].im};
    }
    if (side0 == 0) lds[0][idx(j)] = a[0];
    if (Src::kSides == 2 && side1 == 1) lds[1][idx(j)] = b[0];
  });
  __syncthreads();
  // the even extension at the positions the FFT starts from
  cpx<T> v[Src::kSides][E];
#pragma unroll
  for (int h = 0; h < Src::kSides; ++h)
    if (h >= side0 && h <= side1) {
#pragma unroll
      for (int b = 0; b < E / RI; ++b)
#pragma unroll
        for (int r = 0; r < RI; ++r) {
          const int p = slot_pos<P, RI>(t, b, r);
          v[h][b * RI + r] = lds[h][idx((p <= NC) ? p : N - p)];
        }
    }
#pragma unroll
  for (int h = 0; h < Src::kSides; ++h) {
    if (h < side0 || h > side1 || src.field(q, h) >= nfield) continue;
    __syncthreads();   // the staged lines (the previous transform's exchanges) have been read
    int par = 0;
    fft_line<T, P, -1>(v[h], lds[0], lds[1], par, t, idx, tw);
    if (valid) {
      const long long fo = (long long)src.field(q, h) * fstride;
#pragma unroll
      for (int b = 0; b < E / RO; ++b)
#pragma unroll
        for (int r = 0; r < RO; ++r) {
          const int p = slot_pos<P, RO>(t, b, r);
          if (p <= NC) {
            cpx<T> x = v[h][b * RO + r];
            if (dir > 0) {
              const T sc = T(1.0 / (double(NC) * ((p == 0 || p == NC) ? 2.0 : 1.0)));
              x.re *= sc;
              x.im *= sc;
            }
            if (!out64)
              out[fo + (long long)p * nlines + l] = x;
            else if (p <= kz)
              out64[fo + (long long)p * nlines + l] = cpx<double>{double(x.re), double(x.im)};
          }
        }
    }
  }
}

// The same transform through one FFT of nc points instead of 2 nc (the
// half-length route to the DCT-I; Sec. 3.2.1 names it as the next step).  With
// the end points halved, C_k = sum_j w_j x_j cos(pi j k / nc) (w_0 = w_nc = 1/2)
// is obtained from Z = FFT_nc(y),
//   y_0 = (x_0 + x_nc) / 2,  y_j = (x_j + x_{nc-j}) / 2 - sin(pi j / nc) (x_j - x_{nc-j}):
// the even part of y carries the cosines of even order and the odd part, with
// the sine, the differences of neighbouring odd orders, so
//   C_{2k} = (Z_k + Z_{nc-k}) / 2,
//   C_{2k+1} = C_{2k-1} + (i / 2) (Z_k - Z_{nc-k}),  C_1 = sum_j w_j x_j cos(pi j / nc)
// (complex x: the real and imaginary parts go through the one FFT together).
// The odd orders are running sums over k, formed in FP64: each thread of a
// line sums a contiguous run of k, and the runs' totals give every thread its
// starting value.  The lower half sums up from C_1, the upper half down from C_{nc-1} =
// sum_j (-1)^j w_j x_j cos(pi j / nc): a rounding error of an increment stays in all orders
// after it, and derivatives weigh the highest orders most (relative L2 error of the
// upper half of a smooth line's coefficients, one sum from C_1 and two: nc = 128 8.3e-16
// and 3.7e-16, nc = 256 1.3e-15 and 5.7e-16; the time is the same).  dir = +1: x = f, a_n = 2 C_n / (nc cbar_n); dir = -1:
// x = cbar a, f_j = C_j.  tw_g: exp(-i pi m / nc), m < 2 nc (or NULL).
template <typename T, int NC, class Src>
__global__ void __launch_bounds__(CTile<DctPlan<NC>>::L * CTile<DctPlan<NC>>::TT)
k_dct_half(Src src, cpx<T>* __restrict__ out, long long nlines, int nfield, int both, int dir, long long fstride,
           const cpx<T>* __restrict__ tw_g, cpx<double>* __restrict__ out64, int kz) {
  using P = DctPlan<NC>;
  using G = CTile<P>;
  constexpr int E = G::E, L = G::L, LP = L + 1, TT = G::TT;
  constexpr int RI = first_radix<P, -1>(), RO = last_radix<P, -1>();
  constexpr int NK = NC / 2 - 1;                 // increments of the odd orders, k = 1 .. NC/2 - 1
  constexpr int CS = (NK + TT - 1) / TT;         // a thread's run of k
  static_assert(2 * NC * LP * int(sizeof(cpx<T>)) + 3 * NC * int(sizeof(cpx<T>)) <= 160 * 1024, "LDS");
  constexpr int TW = (64 / L < TT) ? 64 / L : TT, NW = TT / TW;   // threads of a line in a wavefront, wavefronts
  static_assert(64 % L == 0 && TT % TW == 0, "lane = line + L (t mod TW)");
  static_assert(NW * L * 3 * 16 <= NC * LP * int(sizeof(cpx<T>)), "partial sums fit one exchange buffer");
  static_assert(NW % 2 == 0 && TW % 2 == 0, "halves of the odd orders by wavefront, rows of one parity by thread");
  __shared__ cpx<T> tw2[2 * NC];                 // exp(-i pi m / NC)
  __shared__ cpx<T> tw[NC];                      // exp(-2 pi i m / NC)
  __shared__ cpx<T> lds[2][NC * LP];
  const int tid = threadIdx.x;
  const int line = tid % L, t = tid / L;
  const int q = (Src::kSides == 1 || both) ? blockIdx.y : blockIdx.y / 2;
  const int side0 = (Src::kSides == 1 || both) ? 0 : blockIdx.y % 2, side1 = (Src::kSides == 2 && both) ? 1 : side0;
  if (src.field(q, side0) >= nfield) return;
  for (int i = tid; i < 2 * NC; i += blockDim.x) {
    cpx<T> w;
    if (tw_g) {
      w = tw_g[i];
    } else {
      double s, c;
      sincospi(-double(i) / double(NC), &s, &c);
      w = cpx<T>{T(c), T(s)};
    }
    tw2[i] = w;
    if (!(i & 1)) tw[i >> 1] = w;
  }
  const long long l = (long long)xcd_tile(blockIdx.x, gridDim.x) * L + line;
  const bool valid = l < nlines;
  const IdxPosMajor idx{LP, line};
  __syncthreads();
  // y of each side, and this thread's share of its C_1 (rows j of t's parity)
  double c1r[Src::kSides] = {}, c1i[Src::kSides] = {};
  dct_stage<T, Src, NC, TT, true>(src, q, t, valid ? l : nlines - 1, nlines, l == 0, [&](int j, cpx<T>* a, cpx<T>* b) {
    const T cj = tw2[j].re, sj = -tw2[j].im;   // cos, sin (pi j / NC)
#pragma unroll
    for (int h = 0; h < Src::kSides; ++h) {
      if (h < side0 || h > side1) continue;
      cpx<T> xa = h ? b[0] : a[0], xb = h ? b[1] : a[1];   // x_j, x_{NC-j}
      if (dir < 0 && j == 0) {                 // x = cbar a: the end points doubled
        xa = cpx<T>{T(2) * xa.re, T(2) * xa.im};
        xb = cpx<T>{T(2) * xb.re, T(2) * xb.im};
      }
      const cpx<T> sm = {T(0.5) * (xa.re + xb.re), T(0.5) * (xa.im + xb.im)};
      const cpx<T> df = {xa.re - xb.re, xa.im - xb.im};
      if (j == 0) {
        lds[h][idx(0)] = sm;
        c1r[h] += 0.5 * double(xa.re) - 0.5 * double(xb.re);   // w_0 x_0 cos 0 + w_NC x_NC cos pi
        c1i[h] += 0.5 * double(xa.im) - 0.5 * double(xb.im);
      } else {
        lds[h][idx(j)] = cpx<T>{sm.re - sj * df.re, sm.im - sj * df.im};
        if (j != NC / 2) {
          lds[h][idx(NC - j)] = cpx<T>{sm.re + sj * df.re, sm.im + sj * df.im};
          c1r[h] += double(cj) * (double(xa.re) - double(xb.re));
          c1i[h] += double(cj) * (double(xa.im) - double(xb.im));
        }
      }
    }
  });
  __syncthreads();
  cpx<T> v[Src::kSides][E];
#pragma unroll
  for (int h = 0; h < Src::kSides; ++h)
    if (h >= side0 && h <= side1) {
#pragma unroll
      for (int b = 0; b < E / RI; ++b)
#pragma unroll
        for (int r = 0; r < RI; ++r) v[h][b * RI + r] = lds[h][idx(slot_pos<P, RI>(t, b, r))];
    }
#pragma unroll
  for (int h = 0; h < Src::kSides; ++h) {
    if (h < side0 || h > side1 || src.field(q, h) >= nfield) continue;
    __syncthreads();   // the staged lines (the previous transform's Z and sums) have been read
    int par = 0;
    fft_line<T, P, -1>(v[h], lds[0], lds[1], par, t, idx, tw);
    // Z in natural order in lds[0]
    __syncthreads();
#pragma unroll
    for (int b = 0; b < E / RO; ++b)
#pragma unroll
      for (int r = 0; r < RO; ++r) lds[0][idx(slot_pos<P, RO>(t, b, r))] = v[h][b * RO + r];
    // sums over the TW threads of a line in this wavefront by shuffles, and the
    // wavefronts' totals through lds[1]: C_1, C_{NC-1} (the threads' shares with the
    // sign of their rows) and the runs
    cpx<double>* ps = reinterpret_cast<cpx<double>*>(lds[1]);     // [3][TT / TW][L]
    const int tw_i = t % TW, w = t / TW;
    const bool up = w >= NW / 2;                                  // uniform: this wavefront sums down from C_{NC-1}
    cpx<double> c1 = {c1r[h], c1i[h]};
#pragma unroll
    for (int d = 2; d < TW; d <<= 1) c1 = cadd(c1, cpx<double>{__shfl_xor(c1.re, L * d), __shfl_xor(c1.im, L * d)});
    const cpx<double> c1o = {__shfl_xor(c1.re, L), __shfl_xor(c1.im, L)};   // the other parity's
    if (tw_i == 0) {
      ps[w * L + line] = cadd(c1, c1o);
      ps[(NW + w) * L + line] = csub(c1, c1o);
    }
    __syncthreads();
    // this thread's run of increments (i/2)(Z_k - Z_{NC-k}), k in [k0, k1)
    const int k0 = 1 + t * CS, k1 = (k0 + CS <= NK + 1) ? k0 + CS : NK + 1;
    auto incr = [&](int k) {
      const cpx<T> a = lds[0][idx(k)], c = lds[0][idx(NC - k)];
      return cpx<double>{-0.5 * (double(a.im) - double(c.im)), 0.5 * (double(a.re) - double(c.re))};
    };
    cpx<double> run = {0.0, 0.0};
#pragma unroll 2
    for (int k = k0; k < k1; ++k) run = cadd(run, incr(k));
    // the runs of this wavefront from its end of the sum up to this thread's
    const int lane = tid & 63, from = up ? TW - 1 - tw_i : tw_i, step = up ? L : -L;
    auto before_by = [&](cpx<double> v, int d) {
      return cpx<double>{__shfl(v.re, lane + d * step), __shfl(v.im, lane + d * step)};
    };
    cpx<double> upto = run;
#pragma unroll
    for (int d = 1; d < TW; d <<= 1) {
      const cpx<double> o = before_by(upto, d);
      if (from >= d) upto = cadd(upto, o);
    }
    if (from == TW - 1) ps[(2 * NW + w) * L + line] = upto;
    cpx<double> before = before_by(upto, 1);
    if (from == 0) before = cpx<double>{0.0, 0.0};
    __syncthreads();
    if (!valid) continue;
    const long long fo = (long long)src.field(q, h) * fstride;
    auto put = [&](int n, double re, double im) {
      if (dir > 0) {
        const double sc = 2.0 / (double(NC) * ((n == 0 || n == NC) ? 2.0 : 1.0));
        re *= sc;
        im *= sc;
      }
      if (!out64)
        out[fo + (long long)n * nlines + l] = cpx<T>{T(re), T(im)};
      else if (n <= kz)
        out64[fo + (long long)n * nlines + l] = cpx<double>{re, im};
    };
    // even orders
#pragma unroll 1
    for (int k = t; k <= NC / 2; k += TT) {
      const cpx<T> a = lds[0][idx(k)], c = lds[0][idx((NC - k) % NC)];
      put(2 * k, 0.5 * (double(a.re) + double(c.re)), 0.5 * (double(a.im) + double(c.im)));
    }
    // odd orders: C_1 plus the runs before this thread's, or C_{NC-1} less those after
    // it, then its own run
    cpx<double> c = {0.0, 0.0}, r = before;
#pragma unroll 4
    for (int u = 0; u < NW; ++u) c = cadd(c, ps[((up ? NW : 0) + u) * L + line]);
#pragma unroll 4
    for (int u = 0; u < NW / 2; ++u)
      if (up ? NW - 1 - u > w : u < w) r = cadd(r, ps[(2 * NW + (up ? NW - 1 - u : u)) * L + line]);
    if (!up) {
      c = cadd(c, r);
      if (t == 0) put(1, c.re, c.im);
#pragma unroll 1
      for (int k = k0; k < k1; ++k) {
        c = cadd(c, incr(k));
        put(2 * k + 1, c.re, c.im);
      }
    } else {
      c = csub(c, r);
#pragma unroll 1
      for (int k = k1 - 1; k >= k0; --k) {
        put(2 * k + 1, c.re, c.im);
        c = csub(c, incr(k));
      }
    }
  }
}

// Coefficients of d/dz: b_nc = 0, c_{m} b_{m} = b_{m+2} + 2 (m+1) a_{m+1} for
// m = nc-1 .. 0 (c_0 = 2, else 1).  The recurrence links m to m+2 only, so the
// outputs of each parity form a chain, and along a chain they are suffix sums:
//   c_m b_m = sum_{j >= m, j = m mod 2} 2 (j+1) a_{j+1}.
// A chain of cnt terms (m = top, top-2, ..) is cut into PC pieces (8, or 16
// for the longest chains) of at most LEN terms; each lane sums its piece, and
// the pieces' totals are combined by a scan across the lanes.  A wavefront
// holds the chains of one parity of 64 / PC consecutive lines: lane =
// (64 / PC) piece + line, so that for one term the lanes of a piece read
// consecutive lines (128 or 64 contiguous bytes), and each lane issues its
// piece's loads at once.  (One lane per chain would leave a 256 x 129 line set
// with fewer wavefronts than SIMDs, each waiting on one load per term.)
namespace {

// exclusive scan over the PC pieces of a chain (lanes 64 / PC apart), piece
// `pc` of this lane
template <int PC>
__device__ __forceinline__ cpx<double> piece_carry(cpx<double> tot, int pc) {
  constexpr int LPW = 64 / PC;
  auto up = [](cpx<double> v, int d) { return cpx<double>{__shfl_up(v.re, LPW * d), __shfl_up(v.im, LPW * d)}; };
  cpx<double> inc = tot;
#pragma unroll
  for (int d = 1; d < PC; d <<= 1) {
    const cpx<double> o = up(inc, d);
    if (pc >= d) inc = cadd(inc, o);
  }
  const cpx<double> ex = up(inc, 1);
  return pc == 0 ? cpx<double>{0.0, 0.0} : ex;
}

template <int LEN, int PC>
__global__ void __launch_bounds__(256) k_cheb_seg(const cpx<double>* __restrict__ a, cpx<double>* __restrict__ out,
                                                  int nc, long long nlines) {
  constexpr int LPW = 64 / PC;   // lines per wavefront
  const int lane = threadIdx.x & 63;
  const int pc = lane / LPW;
  const long long groups = (nlines + LPW - 1) / LPW;
  const long long wave = ((long long)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (wave >= 2 * groups) return;   // whole wavefronts
  const int q = int(wave / groups);
  const long long l = (wave % groups) * LPW + (lane % LPW);
  const bool valid = l < nlines;
  const int top = ((nc - q) & 1) ? nc - 1 : nc;   // largest m <= nc of parity q
  const int cnt = top / 2 + 1;                     // terms m = top, top - 2, .., q
  const int i0 = pc * LEN;
  cpx<double> x[LEN];
#pragma unroll
  for (int k = 0; k < LEN; ++k) {
    const int m = top - 2 * (i0 + k);
    x[k] = cpx<double>{0.0, 0.0};
    if (valid && i0 + k < cnt && m + 1 <= nc) {
      const cpx<double> v = a[(long long)(m + 1) * nlines + l];
      x[k] = cpx<double>{2.0 * (m + 1) * v.re, 2.0 * (m + 1) * v.im};
    }
  }
#pragma unroll
  for (int k = 1; k < LEN; ++k) x[k] = cadd(x[k - 1], x[k]);
  const cpx<double> c = piece_carry<PC>(x[LEN - 1], pc);
#pragma unroll
  for (int k = 0; k < LEN; ++k) {
    const int m = top - 2 * (i0 + k);
    if (valid && i0 + k < cnt) {
      const double s = (m == 0) ? 0.5 : 1.0;
      const cpx<double> bm = cadd(c, x[k]);
      out[(long long)m * nlines + l] = cpx<double>{s * bm.re, s * bm.im};
    }
  }
}

// u = i (kx D w + ky omega) / k^2, v = i (ky D w - kx omega) / k^2 (0 where k = 0),
// D w by the pieced recurrence of k_cheb_seg in the same pass: w and omega are
// read once and u, v written (7310 lines x 129: 12.0 us; the derivative and the
// combination as two passes 20.4).
template <int LEN, int PC>
__global__ void __launch_bounds__(256) k_cheb_uv(const cpx<double>* __restrict__ om, const cpx<double>* __restrict__ w,
                                                 int nc, long long nlines, const double* __restrict__ kxl,
                                                 const double* __restrict__ kyl, cpx<double>* __restrict__ u,
                                                 cpx<double>* __restrict__ v) {
  constexpr int LPW = 64 / PC;   // lines per wavefront
  const int lane = threadIdx.x & 63;
  const int pc = lane / LPW;
  const long long groups = (nlines + LPW - 1) / LPW;
  const long long wave = ((long long)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (wave >= 2 * groups) return;   // whole wavefronts
  const int q = int(wave / groups);
  const long long l = (wave % groups) * LPW + (lane % LPW);
  const bool valid = l < nlines;
  const double kx = valid ? kxl[l] : 0.0, ky = valid ? kyl[l] : 0.0, k2 = kx * kx + ky * ky;
  const double ik = k2 != 0.0 ? 1.0 / k2 : 0.0;
  const int top = ((nc - q) & 1) ? nc - 1 : nc;
  const int cnt = top / 2 + 1;
  const int i0 = pc * LEN;
  cpx<double> x[LEN], o[LEN];
#pragma unroll
  for (int k = 0; k < LEN; ++k) {
    const int m = top - 2 * (i0 + k);
    x[k] = o[k] = cpx<double>{0.0, 0.0};
    if (valid && i0 + k < cnt) {
      if (m + 1 <= nc) {
        const cpx<double> a = w[(long long)(m + 1) * nlines + l];
        x[k] = cpx<double>{2.0 * (m + 1) * a.re, 2.0 * (m + 1) * a.im};
      }
      o[k] = om[(long long)m * nlines + l];
    }
  }
#pragma unroll
  for (int k = 1; k < LEN; ++k) x[k] = cadd(x[k - 1], x[k]);
  const cpx<double> c = piece_carry<PC>(x[LEN - 1], pc);
#pragma unroll
  for (int k = 0; k < LEN; ++k) {
    const int m = top - 2 * (i0 + k);
    if (valid && i0 + k < cnt) {
      const double s = (m == 0) ? 0.5 : 1.0;
      const cpx<double> d = {s * (c.re + x[k].re), s * (c.im + x[k].im)};
      const cpx<double> su = {kx * d.re + ky * o[k].re, kx * d.im + ky * o[k].im};
      const cpx<double> sv = {ky * d.re - kx * o[k].re, ky * d.im - kx * o[k].im};
      const bool mean = k2 == 0.0;   // left to the mean flow
      u[(long long)m * nlines + l] = mean ? cpx<double>{0.0, 0.0} : cpx<double>{-su.im * ik, su.re * ik};
      v[(long long)m * nlines + l] = mean ? cpx<double>{0.0, 0.0} : cpx<double>{-sv.im * ik, sv.re * ik};
    }
  }
}
}  // namespace

// Chebyshev-tau Helmholtz solve (D^2 - beta) f = g, one thread per (line,
// parity): the rows of tau_rows.hpp, a tridiagonal chain per parity, and one
// boundary row per parity, of f (Dirichlet) or f' (Neumann) at the walls.
// beta = beta_line[l] (if given) + beta_add + (kx_l^2 + ky_l^2 if kx given).
// Boundary values: bcv[2l], bcv[2l+1] (top z=+1, bottom z=-1; if given)
// plus the constants top_c, bot_c.  g may be NULL (zero).  xw: nc+1 doubles
// per line of scratch.

// downward sweep of parity p: a_i = X_i a_{i-1} + Y_i for the indices
// n = p + 2 i, i = m..1 (X in xw, Y in f).  TAB: nc <= kTauQMax, the rows' constants
// from the table; else by division.
template <bool TAB>
__device__ __forceinline__ void helm_down(const cpx<double>* __restrict__ g, cpx<double>* __restrict__ f,
                                          double* __restrict__ xw, int nc, long long nlines, double be, int p,
                                          long long l) {
  const int m = (nc - p) / 2;
  auto G = [&](int n) -> cpx<double> {
    if (!g || n > nc - 2 || n < 0) return cpx<double>{0.0, 0.0};
    return g[(long long)n * nlines + l];
  };
  double Xn = 0.0;
  cpx<double> Yn = {0.0, 0.0};
  cpx<double> gm = G(p + 2 * m - 2), g0 = G(p + 2 * m), g2 = G(p + 2 * m + 2);
#pragma unroll 4
  for (int i = m; i >= 1; --i) {
    const int n = p + 2 * i;
    const double cm2 = (n - 2 == 0) ? 2.0 : 1.0;
    const double en = (n <= nc - 2) ? 1.0 : 0.0;
    const double en2 = (n + 2 <= nc - 2) ? 1.0 : 0.0;
    const double dn = double(n);
    const double q1 = TAB ? kTauQ.q[0][n] : 1.0 / (4.0 * dn * (dn - 1.0));
    const double q2 = TAB ? kTauQ.q[1][n] : 1.0 / (2.0 * (dn * dn - 1.0));
    const double q3 = TAB ? kTauQ.q[2][n] : 1.0 / (4.0 * dn * (dn + 1.0));
    const double A = cm2 * be * q1;
    const double B = -(1.0 + en * be * q2);
    const double C = en2 * be * q3;
    const cpx<double> R = {-cm2 * gm.re * q1 + en * g0.re * q2 - en2 * g2.re * q3,
                           -cm2 * gm.im * q1 + en * g0.im * q2 - en2 * g2.im * q3};
    const double den = 1.0 / (B + C * Xn);
    const double X = -A * den;
    const cpx<double> Y = {(R.re - C * Yn.re) * den, (R.im - C * Yn.im) * den};
    xw[(long long)n * nlines + l] = X;
    f[(long long)n * nlines + l] = Y;
    Xn = X;
    Yn = Y;
    g2 = g0;
    g0 = gm;
    gm = G(n - 4);
  }
}

// upward sweep 1 of parity p: a_i = P_i a_p + Q_i; the boundary row's sums over the
// chain (weights 1, Dirichlet, or n^2, Neumann)
__device__ __forceinline__ void helm_up1(const cpx<double>* __restrict__ f, const double* __restrict__ xw, int nc,
                                         long long nlines, int p, long long l, bool neu, double& SP,
                                         cpx<double>& SQ) {
  const int m = (nc - p) / 2;
  double P = 1.0;
  cpx<double> Qv = {0.0, 0.0};
  SP = 0.0;
  SQ = cpx<double>{0.0, 0.0};
#pragma unroll 4
  for (int i = 0; i <= m; ++i) {
    const int n = p + 2 * i;
    if (i > 0) {
      const double X = xw[(long long)n * nlines + l];
      const cpx<double> Y = f[(long long)n * nlines + l];
      P = X * P;
      Qv = cpx<double>{X * Qv.re + Y.re, X * Qv.im + Y.im};
    }
    const double w = neu ? double(n) * double(n) : 1.0;
    SP += w * P;
    SQ.re += w * Qv.re;
    SQ.im += w * Qv.im;
  }
}

// upward sweep 2 of parity p from its first coefficient a
__device__ __forceinline__ void helm_up2(cpx<double>* __restrict__ f, const double* __restrict__ xw, int nc,
                                         long long nlines, int p, long long l, cpx<double> a) {
  const int m = (nc - p) / 2;
  f[(long long)p * nlines + l] = a;
#pragma unroll 4
  for (int i = 1; i <= m; ++i) {
    const int n = p + 2 * i;
    const double X = xw[(long long)n * nlines + l];
    const cpx<double> Y = f[(long long)n * nlines + l];
    a = cpx<double>{X * a.re + Y.re, X * a.im + Y.im};
    f[(long long)n * nlines + l] = a;
  }
}

template <bool TAB>
__device__ __forceinline__ void helm_line(const cpx<double>* __restrict__ g, cpx<double>* __restrict__ f,
                                          double* __restrict__ xw, int nc, long long nlines,
                                          const double* __restrict__ beta_line, double beta_add,
                                          const double* __restrict__ kx, const double* __restrict__ ky, bool neu,
                                          const cpx<double>* __restrict__ bcv, cpx<double> top, cpx<double> bot,
                                          long long id) {
  const long long l = id % nlines;
  const int p = int(id / nlines);             // parity
  double be = beta_add;
  if (beta_line) be += beta_line[l];
  if (kx) be += kx[l] * kx[l] + ky[l] * ky[l];
  if (bcv) {
    top = cadd(top, bcv[2 * l]);
    bot = cadd(bot, bcv[2 * l + 1]);
  }
  // the rows (top +- bottom)/2 restricted to this parity: sum_i w_i a_i = s
  const bool plus = (p == 0) != neu;          // Dirichlet even, Neumann odd: (top + bottom) / 2
  const cpx<double> s = plus ? cpx<double>{0.5 * (top.re + bot.re), 0.5 * (top.im + bot.im)}
                             : cpx<double>{0.5 * (top.re - bot.re), 0.5 * (top.im - bot.im)};
  helm_down<TAB>(g, f, xw, nc, nlines, be, p, l);
  double SP;
  cpx<double> SQ;
  helm_up1(f, xw, nc, nlines, p, l, neu, SP, SQ);
  helm_up2(f, xw, nc, nlines, p, l, cpx<double>{(s.re - SQ.re) / SP, (s.im - SQ.im) / SP});
}

template <bool TAB>
__global__ void k_helm(const cpx<double>* __restrict__ g, cpx<double>* __restrict__ f, double* __restrict__ xw,
                       int nc, long long nlines, const double* __restrict__ beta_line, double beta_add,
                       const double* __restrict__ kx, const double* __restrict__ ky, int neumann,
                       const cpx<double>* __restrict__ bcv, cpx<double> top_c, cpx<double> bot_c) {
  const long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= 2 * nlines) return;
  helm_line<TAB>(g, f, xw, nc, nlines, beta_line, beta_add, kx, ky, neumann != 0, bcv, top_c, bot_c, id);
}

// Several independent problems in one launch (blockIdx.y selects the problem):
// each thread's elimination is a sequential chain, so more chains per launch
// hide more of their memory latency.
template <bool TAB>
__global__ void k_helm_batch(HelmBatch b, int nc) {
  const HelmProblem& P = b.p[blockIdx.y];
  const long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= 2 * P.nlines) return;
  helm_line<TAB>(P.g, P.f, P.xw, nc, P.nlines, nullptr, P.beta_add, P.kx, P.ky, P.neumann != 0, nullptr, P.top_c,
                 P.bot_c, id);
}

// w = w_p + c_t w_t + c_b w_b with (c_t, c_b) making w'(+1) = w'(-1) = 0;
// w = 0 where kx = ky = 0.  Written over w_p.
__global__ void k_influence(cpx<double>* __restrict__ wp, const cpx<double>* __restrict__ wt,
                            const cpx<double>* __restrict__ wb, int nc, long long nlines,
                            const double* __restrict__ kx, const double* __restrict__ ky) {
  const long long l = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (l >= nlines) return;
  const bool mean = (kx[l] == 0.0 && ky[l] == 0.0);
  cpx<double> dpt = {0, 0}, dpb = {0, 0};
  double dtt = 0, dtb = 0, dbt = 0, dbb = 0;
#pragma unroll 4
  for (int n = 0; n <= nc; ++n) {
    const double w2 = double(n) * double(n);
    const double sg = (n & 1) ? w2 : -w2;  // (-1)^(n+1) n^2
    const long long o = (long long)n * nlines + l;
    const cpx<double> a = wp[o];
    dpt.re += w2 * a.re; dpt.im += w2 * a.im;
    dpb.re += sg * a.re; dpb.im += sg * a.im;
    dtt += w2 * wt[o].re; dtb += sg * wt[o].re;
    dbt += w2 * wb[o].re; dbb += sg * wb[o].re;
  }
  // [dtt dbt; dtb dbb] (c_t, c_b) = -(dpt, dpb)
  const double det = dtt * dbb - dbt * dtb;
  const cpx<double> ct = {(-dpt.re * dbb + dbt * dpb.re) / det, (-dpt.im * dbb + dbt * dpb.im) / det};
  const cpx<double> cb = {(-dtt * dpb.re + dtb * dpt.re) / det, (-dtt * dpb.im + dtb * dpt.im) / det};
#pragma unroll 4
  for (int n = 0; n <= nc; ++n) {
    const long long o = (long long)n * nlines + l;
    cpx<double> w = {0.0, 0.0};
    if (!mean) {
      const cpx<double> a = wp[o];
      const double t = wt[o].re, b = wb[o].re;
      w = cpx<double>{a.re + ct.re * t + cb.re * b, a.im + ct.im * t + cb.im * b};
    }
    wp[o] = w;
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
#define PSMS_FOR_EACH_2NC(X) X(8) X(12) X(16) X(24) X(32) X(48) X(64) X(96) X(128) X(192) X(256) X(512)

bool supported_nc(int nc) {
  switch (2 * nc) {
#define PSMS_CASE(NN) case NN:
    PSMS_FOR_EACH_2NC(PSMS_CASE)
#undef PSMS_CASE
    return true;
    default:
      return false;
  }
}

namespace {
// Both sides of a pair in one workgroup where that still leaves every CU one: it
// reads the pair's inputs once (two steps of the 256 x 256 x 257 channel: 2593
// against 2742 us with a workgroup a side; 32 x 24 x 33, ten steps: 550 against 512).
template <class Src>
dim3 dct_grid(long long tiles, int nfield, int& both) {
  const int pairs = Src::kSides == 1 ? nfield : (nfield + 1) / 2;
  both = Src::kSides == 2 && tiles * pairs >= 256;
  return dim3(unsigned(tiles), unsigned(Src::kSides == 1 || both ? pairs : 2 * pairs));
}
template <typename T, int N, class Src>
hipError_t dct_n(const Src& in, cpx<T>* out, long long nlines, int dir, long long fstride, int nfield,
                 const cpx<T>* tw, cpx<double>* out64, int kz, hipStream_t st) {
  // Long FP64 lines take the nc-point route: half the exchange traffic (14706
  // lines, nc = 96, 128, 256: 15.8, 19.8, 44.5 us against 19.1, 23.1, 49.0).
  // Short ones keep the even extension, with its three barriers fewer, in channels of
  // any size (us a step, extension against nc-point: 64 x 64 x 49 51 / 55, 256 x 128 x
  // 49 162 / 171, 128 x 96 x 65 100 / 104, 256 x 128 x 65 219 / 223); alone it loses
  // from 44000 lines of nc = 64 on (100000 lines 45 against 40 us).  FP32
  // lines keep it too: its transform is cheap against the nc-point route's FP64
  // sums (256 x 128 x 129 step: 1.45 ms against 1.55 for five), and every order
  // is formed by itself.
  int both = 0;
  if constexpr (N >= 192 && sizeof(T) == 8) {   // nc = N / 2 >= 96
    using G = CTile<DctPlan<N / 2>>;
    const dim3 grid = dct_grid<Src>((nlines + G::L - 1) / G::L, nfield, both);
    k_dct_half<T, N / 2, Src><<<grid, unsigned(G::L * G::TT), 0, st>>>(in, out, nlines, nfield, both, dir, fstride, tw,
                                                                       out64, kz);
  } else {
    using G = CTile<DctPlan<N>>;
    const dim3 grid = dct_grid<Src>((nlines + G::L - 1) / G::L, nfield, both);
    k_dct<T, N, Src><<<grid, unsigned(G::L * G::TT), 0, st>>>(in, out, nlines, nfield, both, dir, fstride, tw, out64,
                                                              kz);
  }
  return hipGetLastError();
}
unsigned blocks(long long n, int bs) {
  long long b = (n + bs - 1) / bs;
  return unsigned(b < 1 ? 1 : b);
}
}  // namespace

template <typename T>
hipError_t launch_dct(int nc, const cpx<T>* in, cpx<T>* out, long long nlines, int dir, hipStream_t st) {
  return launch_dct_fields<T>(nc, in, out, nlines, 0, 1, nullptr, dir, st);
}

template <typename T>
hipError_t launch_dct_fields(int nc, const cpx<T>* in, cpx<T>* out, long long nlines, long long fstride, int nfield,
                             const cpx<T>* tw, int dir, hipStream_t st) {
  if (nfield < 1 || nlines == 0) return hipSuccess;
  const ArraySrc<T> src{in, fstride};
  switch (2 * nc) {
#define PSMS_CASE(NN) case NN: return dct_n<T, NN>(src, out, nlines, dir, fstride, nfield, tw, nullptr, 0, st);
    PSMS_FOR_EACH_2NC(PSMS_CASE)
#undef PSMS_CASE
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_dct_chfields(int nc, const ChanFieldSrc& fs, cpx<T>* out, long long fstride, int nfield,
                               const cpx<T>* tw, hipStream_t st) {
  if (fs.nlines == 0) return hipSuccess;
  ChanFieldSrcT<T> src{fs};
  if (nfield == 3) src.s.dphi = fs.w;   // the pair's other side, not transformed: no reads of its own
  switch (2 * nc) {
#define PSMS_CASE(NN) case NN: return dct_n<T, NN>(src, out, fs.nlines, -1, fstride, nfield, tw, nullptr, 0, st);
    PSMS_FOR_EACH_2NC(PSMS_CASE)
#undef PSMS_CASE
  }
  return hipErrorInvalidValue;
}
template hipError_t launch_dct_chfields<float>(int, const ChanFieldSrc&, cpx<float>*, long long, int,
                                               const cpx<float>*, hipStream_t);
template hipError_t launch_dct_chfields<double>(int, const ChanFieldSrc&, cpx<double>*, long long, int,
                                                const cpx<double>*, hipStream_t);

template <typename T>
hipError_t launch_dct_chterms(int nc, const cpx<T>* in, cpx<double>* out, long long nlines, long long fstride, int nterm,
                              const double* kx, const double* ky, const cpx<T>* tw, int kz, hipStream_t st) {
  if (nlines == 0) return hipSuccess;
  const ChanTermSrcT<T> src{in, fstride, kx, ky};
  switch (2 * nc) {
#define PSMS_CASE(NN) case NN: return dct_n<T, NN>(src, (cpx<T>*)nullptr, nlines, +1, fstride, nterm, tw, out, kz, st);
    PSMS_FOR_EACH_2NC(PSMS_CASE)
#undef PSMS_CASE
  }
  return hipErrorInvalidValue;
}
template hipError_t launch_dct_chterms<float>(int, const cpx<float>*, cpx<double>*, long long, long long, int,
                                              const double*, const double*, const cpx<float>*, int, hipStream_t);
template hipError_t launch_dct_chterms<double>(int, const cpx<double>*, cpx<double>*, long long, long long, int,
                                               const double*, const double*, const cpx<double>*, int, hipStream_t);

hipError_t launch_chebd(const cpx<double>* a, cpx<double>* d, int nc, long long nlines, hipStream_t st) {
  if (nlines < 0 || nc < 1) return hipErrorInvalidValue;
  if (nlines == 0) return hipSuccess;
  // 8 pieces per chain (8 lines a wavefront) up to 9 terms a piece, else 16
  // pieces (4 lines a wavefront), which keeps the longest chains (nc = 256) at
  // 9 terms a piece and off the register limit
  const int need = (nc / 2 + 1 + 7) / 8;
  const int pcs = need <= 9 ? 8 : 16;
  const dim3 grid(blocks(2 * ((nlines + 64 / pcs - 1) / (64 / pcs)) * 64, 256));
#define PSMS_SEG(LEN, PCS) \
  if (pcs == PCS && (nc / 2 + PCS) / PCS <= LEN) { \
    k_cheb_seg<LEN, PCS><<<grid, 256, 0, st>>>(a, d, nc, nlines); \
    return hipGetLastError(); \
  }
  PSMS_SEG(1, 8) PSMS_SEG(2, 8) PSMS_SEG(3, 8) PSMS_SEG(5, 8) PSMS_SEG(9, 8) PSMS_SEG(9, 16)
#undef PSMS_SEG
  return hipErrorInvalidValue;   // nc > 287
}

hipError_t launch_helm(const cpx<double>* g, cpx<double>* f, double* xw, int nc, long long nlines,
                       const double* beta_line, double beta_add, const double* kx, const double* ky, int neumann,
                       const cpx<double>* bcv, cpx<double> top_c, cpx<double> bot_c, hipStream_t st) {
  const unsigned nb = blocks(2 * nlines, 64);
  if (nc <= kTauQMax)
    k_helm<true><<<nb, 64, 0, st>>>(g, f, xw, nc, nlines, beta_line, beta_add, kx, ky, neumann, bcv, top_c, bot_c);
  else
    k_helm<false><<<nb, 64, 0, st>>>(g, f, xw, nc, nlines, beta_line, beta_add, kx, ky, neumann, bcv, top_c, bot_c);
  return hipGetLastError();
}

hipError_t launch_helm_batch(const HelmBatch& b, int nc, hipStream_t st) {
  if (b.np < 0 || b.np > kHelmBatchMax) return hipErrorInvalidValue;
  long long most = 0;
  for (int i = 0; i < b.np; ++i) {
    if (b.p[i].nlines < 0) return hipErrorInvalidValue;
    most = most > b.p[i].nlines ? most : b.p[i].nlines;
  }
  if (b.np == 0 || most == 0) return hipSuccess;
  const dim3 grid(blocks(2 * most, 64), unsigned(b.np));
  if (nc <= kTauQMax) k_helm_batch<true><<<grid, 64, 0, st>>>(b, nc);
  else k_helm_batch<false><<<grid, 64, 0, st>>>(b, nc);
  return hipGetLastError();
}

hipError_t launch_influence(cpx<double>* wp, const cpx<double>* wt, const cpx<double>* wb, int nc, long long nlines,
                            const double* kx, const double* ky, hipStream_t st) {
  k_influence<<<blocks(nlines, 64), 64, 0, st>>>(wp, wt, wb, nc, nlines, kx, ky);
  return hipGetLastError();
}

hipError_t launch_cheb_uv(const cpx<double>* om, const cpx<double>* w, cpx<double>* u, cpx<double>* v, int nc,
                          long long nlines, const double* kx, const double* ky, hipStream_t st) {
  if (nlines < 0 || nc < 1) return hipErrorInvalidValue;
  if (nlines == 0) return hipSuccess;
  const int need = (nc / 2 + 1 + 7) / 8;
  const int pcs = need <= 9 ? 8 : 16;   // as in launch_chebd
  const dim3 grid(blocks(2 * ((nlines + 64 / pcs - 1) / (64 / pcs)) * 64, 256));
#define PSMS_SEG(LEN, PCS) \
  if (pcs == PCS && (nc / 2 + PCS) / PCS <= LEN) { \
    k_cheb_uv<LEN, PCS><<<grid, 256, 0, st>>>(om, w, nc, nlines, kx, ky, u, v); \
    return hipGetLastError(); \
  }
  PSMS_SEG(1, 8) PSMS_SEG(2, 8) PSMS_SEG(3, 8) PSMS_SEG(5, 8) PSMS_SEG(9, 8) PSMS_SEG(9, 16)
#undef PSMS_SEG
  return hipErrorInvalidValue;   // nc > 287
}

template hipError_t launch_dct<double>(int, const cpx<double>*, cpx<double>*, long long, int, hipStream_t);
template hipError_t launch_dct_fields<double>(int, const cpx<double>*, cpx<double>*, long long, long long, int,
                                              const cpx<double>*, int, hipStream_t);
template hipError_t launch_dct_fields<float>(int, const cpx<float>*, cpx<float>*, long long, long long, int,
                                             const cpx<float>*, int, hipStream_t);
template hipError_t launch_dct<float>(int, const cpx<float>*, cpx<float>*, long long, int, hipStream_t);

}  // namespace psms
