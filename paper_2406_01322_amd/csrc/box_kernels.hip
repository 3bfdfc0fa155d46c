// HIP kernels of the periodic-box Navier-Stokes + Cahn-Hilliard step (gfx950).
//
// The step of Sec. 2.2 (steps ii-v) is executed as four kernels per time step,
// all on the caller's stream:
//   k_ystep<+1>  y-inverse of u, v, w, phi, d_z phi, plus i k_y phi
//   k_xfield     x-inverse (7 fields), the pointwise products (Sec. 3.2.2,
//                Hadamard products) and the x-forward of the 8 products
//                (k_xstep: FP64 rows of 256)
//   k_ystep<-1>  y-forward with 2/3 truncation
//   k_zstep      z-forward, spectral RHS assembly, Leray projection, CN/AB2
//                (NS) and IE/AB2 (CH) updates, then the z-inverse of the new
//                state for the next step (k_zfield: few lines).
// Spectral data is stored only inside the retained band |k_i| <= K =
// floor((N-1)/3), so the transforms never read or write discarded modes.
//
// Layouts (complex values interleaved re, im):
//   state, history : [4][C kz][C ky][H kx] double   (C = 2K+1, H = K+1)
//   G (z-inverse)  : [5][N z][C ky][H kx]           (u, v, w, phi, d_z phi)
//   Y (y-inverse)  : [6][N z][N y][H kx]            (u, v, w, phi, d_y phi, d_z phi)
//   X (x-forward)  : [8][N z][N y][H kx]            (T_xx T_yy T_zz T_xy T_xz T_yz, a, c)
//   W (y-forward)  : [8][N z][C ky][H kx]
//
// Every kernel is instantiated per transform length N (compile time) so that
// all index arithmetic folds to constants.  The step kernels read their
// pointers and coefficients from a device table of boxes (BoxDev) indexed by
// blockIdx.z, so one launch advances every box of a given size.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "box_kernels.hpp"
#include "fft_engine.hpp"

// The build compiles this file twice, side by side: with PSMS_PART = 64 the FP64
// instantiations and everything that is not a template, with PSMS_PART = 32 the
// FP32 instantiations.
#ifndef PSMS_PART
#error "compile with -DPSMS_PART=64 and -DPSMS_PART=32"
#endif

namespace psms {

template <typename T>
__device__ __forceinline__ cpx<T> to_cpx(cpx<double> v) { return {T(v.re), T(v.im)}; }


// ---------------------------------------------------------------------------
// batched transforms along a strided axis (y or z): L lines per workgroup,
// lanes line-fastest, LDS element (pos, line) at pos * (L+1) + line.
// S = -1 forward (output band of n_out slots), S = +1 inverse (input band of
// n_in slots, zero-padded).  Output field f reads input field (fmap >> 4f)&15;
// bit f of dmask multiplies by i k along the axis.
// ---------------------------------------------------------------------------
template <typename T, class P, int S, int V>
__device__ __forceinline__ void lines_body(const cpx<T>* __restrict__ src, cpx<T>* __restrict__ dst,
                                           const cpx<T>* __restrict__ tw_g, const LineArgs& a, bool deriv) {
  using G = Tile<P, V>;
  constexpr int N = P::N;
  constexpr bool SWZ = N >= 256;   // see the LDS index functors
  constexpr int E = G::E, L = G::L, LP = SWZ ? L : L + 1;
  constexpr int RI = first_radix<P, S>(), RO = last_radix<P, S>();
  __shared__ cpx<T> tw[N];
  __shared__ cpx<T> lds[2][N * LP];
  const int tid = threadIdx.x;
  const int line = tid % L, t = tid / L;
  for (int i = tid; i < N; i += blockDim.x) tw[i] = tw_g[i];
  const long long gl = (long long)xcd_tile(blockIdx.x, gridDim.x) * L + line;
  const bool valid = gl < a.nlines;
  const long long o = valid ? gl / a.inner : 0, i = valid ? gl % a.inner : 0;

  cpx<T> v[E];
#pragma unroll
  for (int b = 0; b < E / RI; ++b) {
#pragma unroll
    for (int r = 0; r < RI; ++r) {
      const int p = slot_pos<P, RI>(t, b, r);
      const int s = band_slot(p, a.n_in, N);
      cpx<T> x = {T(0), T(0)};
      if (valid && s >= 0) {
        x = ld_global(src + (o * a.n_in + s) * a.inner + i);
        if (S > 0 && deriv) {
          const T k = T(signed_k(p, N));
          x = cpx<T>{-k * x.im, k * x.re};
        }
      }
      v[b * RI + r] = x;
    }
  }
  __syncthreads();
  int par = 0;
  if constexpr (SWZ)
    fft_line<T, P, S>(v, lds[0], lds[1], par, t, IdxPosSwz{LP, line}, tw);
  else
    fft_line<T, P, S>(v, lds[0], lds[1], par, t, IdxPosMajor{LP, line}, tw);
  const T sc = T(a.scale);
#pragma unroll
  for (int b = 0; b < E / RO; ++b) {
#pragma unroll
    for (int r = 0; r < RO; ++r) {
      const int p = slot_pos<P, RO>(t, b, r);
      const int s = band_slot(p, a.n_out, N);
      if (valid && s >= 0) {
        cpx<T> x = v[b * RO + r];
        if (S < 0 && deriv) {
          const T k = T(signed_k(p, N));
          x = cpx<T>{-k * x.im, k * x.re};
        }
        st_global(dst + (o * a.n_out + s) * a.inner + i, cpx<T>{sc * x.re, sc * x.im});
      }
    }
  }
}

template <typename T, int N, int S>
__global__ void __launch_bounds__(256) k_lines(const cpx<T>* __restrict__ in, cpx<T>* __restrict__ out,
                                               const cpx<T>* __restrict__ tw_g, LineArgs a) {
  const int fo = blockIdx.y;
  lines_body<T, Plan<N>, S, 2>(in + (long long)((a.fmap >> (4 * fo)) & 15) * a.in_fstride,
                         out + (long long)fo * a.out_fstride, tw_g, a, (a.dmask >> fo) & 1);
}

// y stages of the step for box box0 + blockIdx.z.
//   S = +1: G [5][N][C][H] (bufb) -> Y [6][N][N][H] (bufa); output 4 is i ky phi.
//   S = -1: X [8][N][N][H] (bufb) -> W [8][N][C][H] (bufa), truncated to the band.
template <typename T, int N, int S, int V>
__global__ void __launch_bounds__(64 << V) k_ystep(const BoxDev* __restrict__ boxes, int box0,
                                                   const cpx<T>* __restrict__ tw_g) {
  using P = Plan<N>;
  using G = Tile<P, V>;
  const BoxDev& bx = boxes[box0 + blockIdx.z];
  const int fo = blockIdx.y;
  LineArgs a;
  a.inner = G::H;
  a.nlines = (long long)N * G::H;
  a.scale = 1.0;
  const long long nq = (long long)N * G::C * G::H, nnh = (long long)N * N * G::H;
  if (S > 0) {
    a.n_in = G::C;
    a.n_out = N;
    const int fin = (fo <= 3) ? fo : fo - 1;
    lines_body<T, P, S, V>(static_cast<const cpx<T>*>(bx.bufb) + fin * nq,
                           static_cast<cpx<T>*>(bx.bufa) + fo * nnh,
                           tw_g, a, fo == 4);
  } else {
    a.n_in = N;
    a.n_out = G::C;
    lines_body<T, P, S, V>(static_cast<const cpx<T>*>(bx.bufb) + fo * nnh,
                           static_cast<cpx<T>*>(bx.bufa) + fo * nq,
                           tw_g, a, false);
  }
}

// ---------------------------------------------------------------------------
// real transforms along x (contiguous rows), two rows packed per complex FFT
// (z = a + i b).  L row pairs per workgroup, lanes position-fastest, LDS
// element (pos, pair) at pair * (N+1) + pos.
// ---------------------------------------------------------------------------
template <typename T, int N>
__global__ void __launch_bounds__(256) k_rows_fwd(const T* __restrict__ in, cpx<T>* __restrict__ out,
                                                  const cpx<T>* __restrict__ tw_g, RowArgs a) {
  using P = Plan<N>;
  using G = Tile<P>;
  constexpr int E = G::E, TT = G::TT, L = G::L, LP = kRowStride<N>;
  constexpr int RI = first_radix<P, -1>(), RO = last_radix<P, -1>();
  __shared__ cpx<T> tw[tw_size<P, -1>()];
  __shared__ cpx<T> lds[2][L * LP];
  const int tid = threadIdx.x;
  const int t = tid % TT, line = tid / TT;
  build_twiddles<T, P, -1>(tw, [&](int m) { return tw_g[m]; }, tid, int(blockDim.x));
  const T* src = in + (long long)blockIdx.y * a.in_fstride;
  cpx<T>* dst = out + (long long)blockIdx.y * a.out_fstride;
  const long long r0 = ((long long)blockIdx.x * L + line) * 2;
  const bool v0 = r0 < a.nrows, v1 = r0 + 1 < a.nrows;
  cpx<T> v[E];
#pragma unroll
  for (int b = 0; b < E / RI; ++b)
#pragma unroll
    for (int r = 0; r < RI; ++r) {
      const int p = slot_pos<P, RI>(t, b, r);
      v[b * RI + r] = cpx<T>{v0 ? src[r0 * N + p] : T(0), v1 ? src[(r0 + 1) * N + p] : T(0)};
    }
  __syncthreads();
  int par = 0;
  const IdxLineMajor<N, TT> idx{line * LP};
  fft_line<T, P, -1>(v, lds[0], lds[1], par, t, idx, tw);
  cpx<T>* Lb = par ? lds[1] : lds[0];
#pragma unroll
  for (int b = 0; b < E / RO; ++b)
#pragma unroll
    for (int r = 0; r < RO; ++r) Lb[idx(slot_pos<P, RO>(t, b, r))] = v[b * RO + r];
  wave_lds_sync();  // the line's threads are one wavefront's lanes
  const T h = T(0.5) * T(a.scale);
  for (int k = t; k < a.n_out; k += TT) {
    const cpx<T> zk = Lb[idx(k)];
    const cpx<T> zm = Lb[idx((N - k) % N)];
    if (v0) dst[r0 * a.n_out + k] = cpx<T>{h * (zk.re + zm.re), h * (zk.im - zm.im)};
    if (v1) dst[(r0 + 1) * a.n_out + k] = cpx<T>{h * (zk.im + zm.im), h * (zm.re - zk.re)};
  }
}

template <typename T, int N>
__global__ void __launch_bounds__(256) k_rows_inv(const cpx<T>* __restrict__ in, T* __restrict__ out,
                                                  const cpx<T>* __restrict__ tw_g, RowArgs a) {
  using P = Plan<N>;
  using G = Tile<P>;
  constexpr int E = G::E, TT = G::TT, L = G::L, LP = kRowStride<N>;
  constexpr int RI = first_radix<P, 1>(), RO = last_radix<P, 1>();
  __shared__ cpx<T> tw[tw_size<P, 1>()];
  __shared__ cpx<T> lds[2][L * LP];
  const int tid = threadIdx.x;
  const int t = tid % TT, line = tid / TT;
  build_twiddles<T, P, 1>(tw, [&](int m) { return tw_g[m]; }, tid, int(blockDim.x));
  const cpx<T>* src = in + (long long)blockIdx.y * a.in_fstride;
  T* dst = out + (long long)blockIdx.y * a.out_fstride;
  const long long r0 = ((long long)blockIdx.x * L + line) * 2;
  const bool v0 = r0 < a.nrows, v1 = r0 + 1 < a.nrows;
  cpx<T> v[E];
#pragma unroll
  for (int b = 0; b < E / RI; ++b)
#pragma unroll
    for (int r = 0; r < RI; ++r) {
      const int p = slot_pos<P, RI>(t, b, r);
      const int k = (p <= N / 2) ? p : N - p;
      cpx<T> A = {T(0), T(0)}, B = {T(0), T(0)};
      if (k < a.n_in) {
        if (v0) A = src[r0 * a.n_in + k];
        if (v1) B = src[(r0 + 1) * a.n_in + k];
        if (k == 0 || 2 * k == N) {  // entries that are real for a real signal
          A.im = T(0);
          B.im = T(0);
        }
      }
      v[b * RI + r] = (p <= N / 2) ? cpx<T>{A.re - B.im, A.im + B.re}   // A + i B
                                   : cpx<T>{A.re + B.im, B.re - A.im};  // conj(A) + i conj(B)
    }
  __syncthreads();
  int par = 0;
  fft_line<T, P, 1>(v, lds[0], lds[1], par, t, IdxLineMajor<N, TT>{line * LP}, tw);
  const T sc = T(a.scale);
#pragma unroll
  for (int b = 0; b < E / RO; ++b)
#pragma unroll
    for (int r = 0; r < RO; ++r) {
      const int p = slot_pos<P, RO>(t, b, r);
      if (v0) dst[r0 * N + p] = sc * v[b * RO + r].re;
      if (v1) dst[(r0 + 1) * N + p] = sc * v[b * RO + r].im;
    }
}

// ---------------------------------------------------------------------------
// fused x stage of the step.  Each row pair (rows 2l, 2l+1 of the N^2 rows
// z N + y) is one complex line.  The 7 physical fields stay in registers at
// the positions the inverse leaves them, which are the positions the forward
// transform starts from, so the products need no data exchange.
// ---------------------------------------------------------------------------
// Staging of the x stage's inputs through LDS by direct global->LDS copies.
// A wavefront transforms LPW = 64 / TT consecutive row pairs, i.e. 2 LPW
// consecutive rows of H retained complex values each: one contiguous run of
// BYTES bytes per field, copied in 16-byte pieces (lane l of copy i moves
// piece 64 i + l to byte 16 (64 i + l) of the staging area).
template <typename T, int N, int TT, int H>
struct XStage {
  static_assert(TT <= 64 && 64 % TT == 0, "a wavefront holds whole lines");
  static constexpr int LPW = 64 / TT;
  static constexpr int BYTES = LPW * 2 * H * int(sizeof(cpx<T>));
  static_assert(BYTES % 16 == 0, "16-byte pieces");
  static constexpr int PIECES = BYTES / 16;
  static constexpr int NI = (PIECES + 63) / 64;
};
// Copy the pieces of one field that lie within `left` bytes of src.  dst is
// the wavefront's staging area (wave-uniform); each active lane's 16 bytes
// land at dst + 1024 i + 16 lane.
template <class XS>
__device__ __forceinline__ void xstage_copy(const char* src, char* dst, int lane, long long left) {
#pragma unroll
  for (int i = 0; i < XS::NI; ++i) {
    const int j = i * 64 + lane;
    if (j < XS::PIECES && (long long)(j + 1) * 16 <= left)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + 16 * j),
                                       (__attribute__((address_space(3))) void*)(dst + 1024 * i), 16, 0, 0);
  }
}
// the copies issued by this wavefront have landed in LDS (vmcnt = 0)
__device__ __forceinline__ void xstage_wait() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0), expcnt and lgkmcnt unconstrained
  __builtin_amdgcn_wave_barrier();
  asm volatile("" ::: "memory");
}
// this wavefront's reads of the staging area have completed (lgkmcnt = 0), so
// the next copies may overwrite it
__device__ __forceinline__ void xstage_release() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
  __builtin_amdgcn_wave_barrier();
  asm volatile("" ::: "memory");
}

// Product F of the x stage (divergence form, eqs. NSE, kort, CHE) at slot e,
// component c (0: row 2l, 1: row 2l + 1) of the 7 physical fields u, v, w,
// phi, dx phi, dy phi, dz phi.
template <int F, typename T, int E>
__device__ __forceinline__ T xproduct(const cpx<T> (&ph)[7][E], int e, int c, T cs) {
  const T u = c ? ph[0][e].im : ph[0][e].re;
  const T vv = c ? ph[1][e].im : ph[1][e].re;
  const T w = c ? ph[2][e].im : ph[2][e].re;
  const T p3 = c ? ph[3][e].im : ph[3][e].re;
  const T gx = c ? ph[4][e].im : ph[4][e].re;
  const T gy = c ? ph[5][e].im : ph[5][e].re;
  const T gz = c ? ph[6][e].im : ph[6][e].re;
  if constexpr (F == 0) return -u * u + cs * (gy * gy + gz * gz);      // T_xx
  else if constexpr (F == 1) return -vv * vv + cs * (gx * gx + gz * gz);  // T_yy
  else if constexpr (F == 2) return -w * w + cs * (gx * gx + gy * gy);    // T_zz
  else if constexpr (F == 3) return -u * vv - cs * gx * gy;               // T_xy
  else if constexpr (F == 4) return -u * w - cs * gx * gz;                // T_xz
  else if constexpr (F == 5) return -vv * w - cs * gy * gz;               // T_yz
  else if constexpr (F == 6) return u * gx + vv * gy + w * gz;            // u . grad phi
  else return p3 * p3 * p3;                                               // phi^3
}

// the same in single phase: -u_i u_j of the 3 fields u, v, w
template <int F, typename T, int E>
__device__ __forceinline__ T xproduct(const cpx<T> (&ph)[3][E], int e, int c, T) {
  constexpr int i = F < 3 ? F : F == 5 ? 1 : 0, j = F < 3 ? F : F == 3 ? 1 : 2;
  const T a = c ? ph[i][e].im : ph[i][e].re, b = c ? ph[j][e].im : ph[j][e].re;
  return -a * b;
}

// order in which the x stage forms and transforms the products
template <bool SP>
constexpr int xstep_fwd_order(int f) {
  constexpr int two_phase[8] = {7, 6, 0, 1, 2, 3, 4, 5};
  return SP ? f : two_phase[f];
}

// CH: the same stage on rows of any count (the plane channel's x stage:
// xrows = (nc + 1) ny rows of the y-inverse, kx = kxs k for x periods other
// than 2 pi); the box passes xrows = N^2 and kxs = 1 implicitly.  SP: single
// phase, 3 fields in and 6 products out; bound by memory: 255 us at 256 x 256 x
// 257 in FP64, where x-inverse, products and x-forward as passes of their own,
// with the physical fields stored between them, took 760 us.
template <typename T, int N, int V, bool CH = false, bool SP = false>
__global__ void __launch_bounds__(64 << V) __attribute__((amdgpu_waves_per_eu(1)))
k_xstep(const BoxDev* __restrict__ boxes, int box0, const cpx<T>* __restrict__ tw_g, long long xrows, double kxs) {
  using P = Plan<N>;
  using G = Tile<P, V>;
  const BoxDev& bx = boxes[box0 + blockIdx.z];
  const cpx<T>* __restrict__ yin = static_cast<const cpx<T>*>(bx.bufa);
  cpx<T>* __restrict__ xout = static_cast<cpx<T>*>(bx.bufb);
  const double csig_d = bx.csig;
  constexpr int E = G::E, TT = G::TT, L = G::L, LP = kRowStride<N>, K = G::K, H = G::H;
  constexpr int NV = SP ? 3 : 7, NPR = SP ? 6 : 8;   // fields, products
  constexpr int NFF = 2;                             // products per forward group
  constexpr int RI = first_radix<P, 1>();   // inverse starts with R[NST-1]
  constexpr int RP = last_radix<P, 1>();    // inverse ends / forward starts with R[0]
  constexpr int RO = last_radix<P, -1>();   // forward ends with R[NST-1]
  const long long ROWS = CH ? xrows : (long long)N * N;
  __shared__ cpx<T> twf[tw_size<P, -1>()];
  __shared__ cpx<T> twi[tw_size<P, 1>()];
  __shared__ cpx<T> lds[NFF][L * LP];
  __shared__ __attribute__((aligned(16))) char xstage_lds[(64 << V) / 64 * 2 * XStage<T, N, TT, H>::BYTES];
  const int tid = threadIdx.x;
  const int t = tid % TT, line = tid / TT;
  build_twiddles<T, P, -1>(twf, [&](int m) { return tw_g[m]; }, tid, int(blockDim.x));
  build_twiddles<T, P, 1>(twi, [&](int m) { return tw_g[m]; }, tid, int(blockDim.x));
  const long long r0 = ((long long)xcd_tile(blockIdx.x, gridDim.x) * L + line) * 2;
  const bool valid = r0 < ROWS;  // ROWS is even: both rows exist
  const IdxLineMajor<N, TT> idx{line * LP};
  int par = 0;
  __syncthreads();

  // x-inverse of u v w phi dx_phi dy_phi dz_phi, two fields at a time; each of
  // the pair exchanges through its own buffer lds[g] (wavefront-local)
  cpx<T> ph[NV][E];
  // the packed complex line z = row0 + i row1 in Hermitian-extended FFT order
  auto pack_slot = [&](int vf, int e, cpx<T> A, cpx<T> B, cpx<T>& z) {
    const int p = slot_pos<P, RI>(t, e / RI, e % RI);
    const int k = (p <= N / 2) ? p : N - p;
    if (vf == 4) {
      const T kx = CH ? T(double(k) * kxs) : T(k);
      A = cpx<T>{-kx * A.im, kx * A.re};
      B = cpx<T>{-kx * B.im, kx * B.re};
    }
    if (k == 0) {
      A.im = T(0);
      B.im = T(0);
    }
    z = (p <= N / 2) ? cpx<T>{A.re - B.im, A.im + B.re} : cpx<T>{A.re + B.im, B.re - A.im};
  };
  constexpr int FS = L * LP;  // buffer of the second transform of a pair
  // Direct-to-LDS staging: the rows of one field that a wavefront transforms
  // are one contiguous run of XS::BYTES bytes, copied by a few 16-byte
  // global_load_lds instructions into the wavefront's staging area while the
  // previous pair is transformed (no registers held in flight).
  using XS = XStage<T, N, TT, H>;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  char* stg = xstage_lds + wv * 2 * XS::BYTES;
  // first row of the wavefront (uniform across it)
  const int wrow0 = __builtin_amdgcn_readfirstlane(int(r0) - 2 * ((tid & 63) / TT));
  auto dma_pair = [&](int vf0) {
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const int vf = vf0 + g;
      if (vf >= NV) continue;
      const int fin = (vf <= 3) ? vf : vf - 1;
      const char* src = reinterpret_cast<const char*>(yin + (long long)fin * ROWS * H + (long long)wrow0 * H);
      const long long left = (ROWS - wrow0) * H * (long long)sizeof(cpx<T>);   // bytes of the field from here
      xstage_copy<XS>(src, stg + g * XS::BYTES, lane, left);
    }
  };
  dma_pair(0);
#pragma unroll
  for (int vf = 0; vf < NV; vf += 2) {
    const int nf = (vf + 1 < NV) ? 2 : 1;
    cpx<T> v[2][E];
    xstage_wait();
#pragma unroll
    for (int g = 0; g < 2; ++g)
      if (g < nf) {
        const cpx<T>* sg = reinterpret_cast<const cpx<T>*>(stg + g * XS::BYTES) + ((tid & 63) / TT) * 2 * H;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int p = slot_pos<P, RI>(t, e / RI, e % RI);
          const int k = (p <= N / 2) ? p : N - p;
          cpx<T> A = {T(0), T(0)}, B = {T(0), T(0)};
          if (valid && k <= K) {
            A = sg[k];
            B = sg[H + k];
          }
          pack_slot(vf + g, e, A, B, v[g][e]);
        }
      }
    xstage_release();
    if (vf + 2 < NV) dma_pair(vf + 2);
    if (nf == 2) {
      fft_lines<T, P, 1, 2>(v, lds[0], FS, 0, par, t, idx, twi);
    } else {
      fft_lines<T, P, 1, 1>(v, lds[0], FS, 0, par, t, idx, twi);
    }
#pragma unroll
    for (int g = 0; g < 2; ++g)
      if (g < nf)
#pragma unroll
        for (int e = 0; e < E; ++e) ph[vf + g][e] = v[g][e];
  }

  // products and x-forward, NFF fields at a time in the order phi^3, u . grad
  // phi, T_xx .. T_yz (phi is then dead after the first group); the field
  // indices are compile-time constants, so the products are straight-line code
  const T cs = T(csig_d);
  const T h = T(0.5);
  static_assert(RP == first_radix<P, -1>(), "mirrored radix order");
  static_for<0, NPR / NFF>([&](auto gi) {
    constexpr int f0 = decltype(gi)::value * NFF;
    cpx<T> v[NFF][E];
    static_for<0, NFF>([&](auto gc) {
      constexpr int g = decltype(gc)::value;
      constexpr int F = xstep_fwd_order<SP>(f0 + g);
#pragma unroll
      for (int e = 0; e < E; ++e) v[g][e] = cpx<T>{xproduct<F>(ph, e, 0, cs), xproduct<F>(ph, e, 1, cs)};
    });
    fft_lines<T, P, -1, NFF>(v, lds[0], FS, 0, par, t, idx, twf);
    // natural order through the group's buffers, then the retained kx of both rows
#pragma unroll
    for (int g = 0; g < NFF; ++g)
#pragma unroll
      for (int b = 0; b < E / RO; ++b)
#pragma unroll
        for (int r = 0; r < RO; ++r) lds[g][idx(slot_pos<P, RO>(t, b, r))] = v[g][b * RO + r];
    wave_lds_sync();  // the line's threads are one wavefront's lanes
    static_for<0, NFF>([&](auto gc) {
      constexpr int g = decltype(gc)::value;
      cpx<T>* dst = xout + (long long)xstep_fwd_order<SP>(f0 + g) * ROWS * H;
      for (int k = t; valid && k < H; k += TT) {
        const cpx<T> zk = lds[g][idx(k)];
        const cpx<T> zm = lds[g][idx((N - k) % N)];
        st_global(dst + r0 * H + k, cpx<T>{h * (zk.re + zm.re), h * (zk.im - zm.im)});
        st_global(dst + (r0 + 1) * H + k, cpx<T>{h * (zk.im + zm.im), h * (zm.re - zk.re)});
      }
    });
  });
}

// ---------------------------------------------------------------------------
// The x stage with a wavefront per field: the wavefronts of a workgroup hold the
// same LW row pairs, wavefront f inverts field f, leaves its physical values in
// LDS, forms product f from those of the others and transforms it forward.  One
// chain of two transforms in a thread where k_xstep has 15, and registers for 4
// to 8 wavefronts a SIMD.  Small grids are bound by that chain (32^3 FP64 box:
// 16.4 -> 6.3 us; step 37.8 -> 29.0 us).  Large ones are bound by LDS traffic and
// memory together: the fields' exchange adds to the former, and larger radices,
// for which the registers are there now, take more away (N = 128: two
// exchanges a transform, not three; N = 256 in FP32: one).  Each product takes its own
// wavefront's field from registers (22 LDS reads a point, not 28).  The stage with
// k_xstep and now, us: FP64 64^3 17.2 -> 9.8, 96^3 64.7 -> 25.4, 128^3 51.8 -> 47.8,
// 192^3 349 -> 201; FP32 32^3 13.0 -> 5.2, 64^3 13.7 -> 7.9, 96^3 32.4 -> 17.2, 128^3
// 28.8 -> 28.9, 192^3 148 -> 114, 256^3 199 -> 189 (96 and 192 with their radix-6 plans
// here, radix 3 and 2 there).  128^3 in FP32 is no faster and large sweeps of 32^3
// boxes in FP32 up to 2% slower (128 boxes 177 -> 180 us a step; radix 8 x 4 would take
// 170 there, but 0.7 us more than the 18.0 of a single box).  With radix 4 throughout, the
// larger FP32 grids lost: steps of 128^3 81.4 -> 82.8, 256^3 758 -> 850.  Workgroups that
// walk over tiles, with or
// without the next tile's loads in flight, were 2 to 15% slower.
// ---------------------------------------------------------------------------
template <typename T, int N>
struct XPlanSel {
  using type = Plan<N>;
};
template <typename T> struct XPlanSel<T, 64> { using type = PlanT<64, 8, 8, 8>; };
template <typename T> struct XPlanSel<T, 128> { using type = PlanT<128, 8, 8, 8, 2>; };
template <> struct XPlanSel<float, 256> { using type = PlanT<256, 16, 16, 16>; };
template <typename T, int N>
using XPlan = typename XPlanSel<T, N>::type;
// FP64 rows of 256 keep the fields in registers (k_xstep): 1174 us a step against
// 1233 on the single-phase 256 x 256 x 257 channel, 1266 against 1276 on the 256^3 box.
// (The two-phase channel alone would gain: 256 x 128 x 129 434 against 424.)
template <typename T, int N>
constexpr bool kXfield = !(sizeof(T) == 8 && N == 256);
template <typename T, int N, bool CH = false, bool SP = false>
__global__ void __launch_bounds__(SP ? 384 : 512)
k_xfield(const BoxDev* __restrict__ boxes, int box0, const cpx<T>* __restrict__ tw_g, long long xrows, double kxs) {
  using P = XPlan<T, N>;
  const BoxDev& bx = boxes[box0 + blockIdx.z];
  const cpx<T>* __restrict__ yin = static_cast<const cpx<T>*>(bx.bufa);
  cpx<T>* __restrict__ xout = static_cast<cpx<T>*>(bx.bufb);
  constexpr int E = P::E, TT = N / E, LW = 64 / TT, K = (N - 1) / 3, H = K + 1;
  static_assert(TT <= 64 && 64 % TT == 0, "a wavefront holds whole lines");
  constexpr bool SWZ = P::E == 16;   // the padded rows would leave one workgroup on a CU
  constexpr int LP = SWZ ? kRowStrideSwz<N> : kRowStride<N>;
  constexpr int RS = LW * LP > 64 * E ? LW * LP : 64 * E;   // a wavefront's LDS region
  constexpr int NV = SP ? 3 : 7, NPR = SP ? 6 : 8;
  constexpr int RI = first_radix<P, 1>(), RO = last_radix<P, -1>();
  static_assert(last_radix<P, 1>() == first_radix<P, -1>(), "mirrored radix order");
  const long long ROWS = CH ? xrows : (long long)N * N;
  __shared__ cpx<T> twf[tw_size<P, -1>()];
  __shared__ cpx<T> twi[tw_size<P, 1>()];
  __shared__ cpx<T> lds[NPR][RS];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t = lane % TT, line = lane / TT;
  const long long r0 = ((long long)xcd_tile(blockIdx.x, gridDim.x) * LW + line) * 2;
  const bool valid = r0 < ROWS;   // ROWS is even: both rows exist
  using Idx = std::conditional_t<SWZ, IdxLineSwz<N, TT>, IdxLineMajor<N, TT>>;
  const Idx idx{line * LP};
  cpx<T>* buf = lds[wv];
  int par = 0;
  cpx<T> a[E], b[E];
  if (wv < NV) {
    const cpx<T>* src = yin + (long long)(wv <= 3 ? wv : wv - 1) * ROWS * H + (valid ? r0 : 0) * H;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int p = slot_pos<P, RI>(t, e / RI, e % RI);
      const int k = (p <= N / 2) ? p : N - p;
      const bool in = valid && k <= K;
      a[e] = in ? ld_global(src + k) : cpx<T>{T(0), T(0)};
      b[e] = in ? ld_global(src + H + k) : cpx<T>{T(0), T(0)};
    }
  }
  build_twiddles<T, P, -1>(twf, [&](int m) { return tw_g[m]; }, tid, int(blockDim.x));
  build_twiddles<T, P, 1>(twi, [&](int m) { return tw_g[m]; }, tid, int(blockDim.x));
  __syncthreads();
  cpx<T> v[1][E];
  if (wv < NV) {
    const bool dx = wv == 4;   // i kx times phi
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int p = slot_pos<P, RI>(t, e / RI, e % RI);
      const int k = (p <= N / 2) ? p : N - p;
      cpx<T> A = a[e], B = b[e];
      if (dx) {
        const T kx = CH ? T(double(k) * kxs) : T(k);
        A = cpx<T>{-kx * A.im, kx * A.re};
        B = cpx<T>{-kx * B.im, kx * B.re};
      }
      if (k == 0) {
        A.im = T(0);
        B.im = T(0);
      }
      v[0][e] = (p <= N / 2) ? cpx<T>{A.re - B.im, A.im + B.re} : cpx<T>{A.re + B.im, B.re - A.im};
    }
    fft_lines<T, P, 1, 1>(v, buf, 0, 0, par, t, idx, twi);
    wave_lds_sync();   // the exchange's reads, before the values over them
#pragma unroll
    for (int e = 0; e < E; ++e) buf[e * 64 + lane] = v[0][e];
  }
  __syncthreads();
  const T cs = T(bx.csig);
  static_for<0, NPR>([&](auto fc) {
    constexpr int F = decltype(fc)::value;
    if (wv == F) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        cpx<T> ph[NV][1];
#pragma unroll
        for (int g = 0; g < NV; ++g) ph[g][0] = g == F ? v[0][e] : lds[g][e * 64 + lane];   // its own is at hand
        v[0][e] = cpx<T>{xproduct<F>(ph, 0, 0, cs), xproduct<F>(ph, 0, 1, cs)};
      }
    }
  });
  __syncthreads();
  fft_lines<T, P, -1, 1>(v, buf, 0, 0, par, t, idx, twf);
  wave_lds_sync();
  // natural order, then the retained kx of both rows
#pragma unroll
  for (int e = 0; e < E; ++e) buf[idx(slot_pos<P, RO>(t, e / RO, e % RO))] = v[0][e];
  wave_lds_sync();
  const T h = T(0.5);
  cpx<T>* dst = xout + (long long)wv * ROWS * H + r0 * H;
  for (int k = t; valid && k < H; k += TT) {
    const cpx<T> zk = buf[idx(k)], zm = buf[idx((N - k) % N)];
    st_global(dst + k, cpx<T>{h * (zk.re + zm.re), h * (zk.im - zm.im)});
    st_global(dst + H + k, cpx<T>{h * (zk.im + zm.im), h * (zm.re - zk.re)});
  }
}

// ---------------------------------------------------------------------------
// The spectral update of one mode, shared by the two z kernels: a box gives the same
// bits whichever runs it, so every product that is added to is an explicit fma.
// ---------------------------------------------------------------------------
// s += i k w
__device__ __forceinline__ void add_ik(cpx<double>& s, double k, cpx<double> w) {
  s.re = __builtin_fma(-k, w.im, s.re);
  s.im = __builtin_fma(k, w.re, s.im);
}
// product f's contribution (x: its transform at the mode) to S = (Sx, Sy, Sz, Sp); in
// the order f = 0 .. 7
template <int f>
__device__ __forceinline__ void add_product(cpx<double> (&S)[4], cpx<double> x, double kx, double ky, double kz,
                                            double k2, const StepCoef& sc) {
  const cpx<double> w = {x.re * sc.inv_n3, x.im * sc.inv_n3};
  if constexpr (f == 0) add_ik(S[0], kx, w);                 // d_x T_xx
  else if constexpr (f == 1) add_ik(S[1], ky, w);            // d_y T_yy
  else if constexpr (f == 2) add_ik(S[2], kz, w);            // d_z T_zz
  else if constexpr (f == 3) {                               // T_xy
    add_ik(S[0], ky, w);
    add_ik(S[1], kx, w);
  } else if constexpr (f == 4) {                             // T_xz
    add_ik(S[0], kz, w);
    add_ik(S[2], kx, w);
  } else if constexpr (f == 5) {                             // T_yz
    add_ik(S[1], kz, w);
    add_ik(S[2], ky, w);
  } else if constexpr (f == 6) {                             // -u.grad(phi)
    S[3].re = __builtin_fma(-sc.inv_n3, x.re, S[3].re);
    S[3].im = __builtin_fma(-sc.inv_n3, x.im, S[3].im);
  } else {                                                   // lap(phi^3) / Pe
    const double c = k2 * sc.inv_pe;
    S[3].re = __builtin_fma(-c, w.re, S[3].re);
    S[3].im = __builtin_fma(-c, w.im, S[3].im);
  }
}
// projection, history and the implicit steps of the mode at `id` of the arrays state
// and hist (M entries a component): S -> the terms kept in hist, u -> the new state.
// old_state(c), old_hist(c): the values before (old_hist not called for ab1).
template <class State, class Hist>
__device__ __forceinline__ void mode_update(cpx<double> (&S)[4], cpx<double> (&u)[4], const State& old_state,
                                            const Hist& old_hist, cpx<double>* state, cpx<double>* hist, long long M,
                                            long long id, double kx, double ky, double kz, double k2,
                                            const StepCoef& sc, cpx<double>* sphi0) {
  auto fma = [](double a, double b, double c) { return __builtin_fma(a, b, c); };
  const double ec = sc.e_coef * k2;
  const cpx<double> ph = old_state(3);
  S[3].re = fma(ec, ph.re, S[3].re);
  S[3].im = fma(ec, ph.im, S[3].im);
  if (k2 == 0.0) {
    if (sphi0) st_global(sphi0, S[3]);   // the mean of S_phi, a divergence: rounding level
#pragma unroll
    for (int c = 0; c < 4; ++c) S[c] = cpx<double>{0.0, 0.0};
  } else {  // Leray projection
    const double ir = 1.0 / k2;
    const double kdr = fma(kz, S[2].re, fma(ky, S[1].re, kx * S[0].re));
    const double kdi = fma(kz, S[2].im, fma(ky, S[1].im, kx * S[0].im));
    const double k[3] = {kx, ky, kz};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      S[c].re = fma(-(k[c] * kdr), ir, S[c].re);
      S[c].im = fma(-(k[c] * kdi), ir, S[c].im);
    }
  }
  cpx<double> ex[4] = {S[0], S[1], S[2], S[3]};
  if (!sc.ab1) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const cpx<double> hp = old_hist(c);
      ex[c] = cpx<double>{fma(1.5, S[c].re, -0.5 * hp.re), fma(1.5, S[c].im, -0.5 * hp.im)};
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) st_global(hist + c * M + id, S[c]);
  const double a = 0.5 * sc.dt * sc.nu * k2;
  const double ia = 1.0 / (1.0 + a), b = 1.0 - a;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const cpx<double> o = old_state(c);
    u[c] = cpx<double>{fma(sc.dt, ex[c].re, b * o.re) * ia, fma(sc.dt, ex[c].im, b * o.im) * ia};
    st_global(state + c * M + id, u[c]);
  }
  const double den = 1.0 / fma(sc.dt * sc.ch2_pe, fma(k2, k2, sc.s * k2), 1.0);
  u[3] = cpx<double>{fma(sc.dt, ex[3].re, ph.re) * den, fma(sc.dt, ex[3].im, ph.im) * den};
  st_global(state + 3 * M + id, u[3]);
}
// kx^2 + ky^2 + kz^2 of integers: exact in any order
__device__ __forceinline__ double k_sq(double kx, double ky, double kz) { return kx * kx + ky * ky + kz * kz; }

// ---------------------------------------------------------------------------
// fused z stage: z-forward of the 8 products, RHS, projection, update, and the
// z-inverse of the new state.  One line per retained (ky, kx) pair q; each
// thread keeps the modes its forward transform leaves in registers, which are
// the inputs its inverse transform starts from.
// do_update = 0 only loads the state and performs the z-inverse (prologue).
// ---------------------------------------------------------------------------
template <typename T, int N, int V>
__global__ void __launch_bounds__(64 << V) k_zstep(const BoxDev* __restrict__ boxes, int box0,
                                                   const cpx<T>* __restrict__ tw_g, int do_update) {
  using P = Plan<N>;
  using G = Tile<P, V>;
  const BoxDev& bx = boxes[box0 + blockIdx.z];
  const cpx<T>* __restrict__ rhs = static_cast<const cpx<T>*>(bx.bufa);
  cpx<double>* __restrict__ state = bx.state;
  cpx<double>* __restrict__ hist = bx.hist;
  cpx<T>* __restrict__ gout = static_cast<cpx<T>*>(bx.bufb);
  const StepCoef sc = bx.sc;
  constexpr int E = G::E, L = G::L, LP = L, K = G::K, C = G::C, H = G::H;   // swizzled tile
  constexpr int Q = C * H;
  constexpr long long M = (long long)C * Q;
  constexpr int RF = first_radix<P, -1>();   // forward starts with R[0]
  constexpr int RL = last_radix<P, -1>();    // forward ends / inverse starts with R[NST-1]
  static_assert(RL == first_radix<P, 1>(), "mirrored radix order");
  __shared__ cpx<T> tw[N];
  // two lines per exchange (one per field of a pair), each with its two
  // ping-pong buffers: line f, parity par at lds[2 f + par]
  __shared__ cpx<T> lds[4][N * LP];
  const int tid = threadIdx.x;
  const int line = tid % L, t = tid / L;
  for (int i = tid; i < N; i += blockDim.x) tw[i] = tw_g[i];
  const int q = xcd_tile(blockIdx.x, gridDim.x) * L + line;
  const bool valid = q < Q;
  const int iy = valid ? q / H : 0, ix = valid ? q % H : 0;
  const double kx = double(ix);
  const double ky = double(iy <= K ? iy : iy - C);
  const IdxPosSwz idx{LP, line};
  int par = 0;

  // band membership and wavenumber of the slots the forward leaves in registers
  bool inb[E];
  int slot[E];
  double kz[E];
#pragma unroll
  for (int b = 0; b < E / RL; ++b)
#pragma unroll
    for (int r = 0; r < RL; ++r) {
      const int p = slot_pos<P, RL>(t, b, r);
      const int s = band_slot(p, C, N);
      inb[b * RL + r] = valid && s >= 0;
      slot[b * RL + r] = s;
      kz[b * RL + r] = double(signed_k(p, N));
    }

  cpx<double> acc[4][E];
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int e = 0; e < E; ++e) acc[c][e] = cpx<double>{0.0, 0.0};

  __syncthreads();
  if (do_update) {
    // the forward transforms two products at a time (one barrier per exchange
    // for both), the next pair's loads in flight while a pair is transformed
    cpx<T> nx[2][E];
    auto load_pair = [&](int f0) {
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const cpx<T>* src = rhs + (long long)(f0 + g) * N * Q;
#pragma unroll
        for (int b = 0; b < E / RF; ++b)
#pragma unroll
          for (int r = 0; r < RF; ++r)
            nx[g][b * RF + r] = valid ? ld_global(src + (long long)slot_pos<P, RF>(t, b, r) * Q + q) : cpx<T>{T(0), T(0)};
      }
    };
    load_pair(0);
    // product f's contribution to the accumulators; f is a compile-time
    // constant in each call, so the accumulation is straight-line code
    auto accumulate = [&](auto fc, const cpx<T>* v) {
      constexpr int f = decltype(fc)::value;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        if (inb[e]) {
          cpx<double> S[4] = {acc[0][e], acc[1][e], acc[2][e], acc[3][e]};
          add_product<f>(S, cpx<double>{double(v[e].re), double(v[e].im)}, kx, ky, kz[e], k_sq(kx, ky, kz[e]), sc);
#pragma unroll
          for (int c = 0; c < 4; ++c) acc[c][e] = S[c];
        }
      }
    };
    static_for<0, 4>([&](auto pc) {
      constexpr int f0 = decltype(pc)::value * 2;
      cpx<T> v[2][E];
#pragma unroll
      for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int e = 0; e < E; ++e) v[g][e] = nx[g][e];
      if constexpr (f0 + 2 < 8) load_pair(f0 + 2);
      fft_lines<T, P, -1, 2>(v, lds[0], 2 * N * LP, N * LP, par, t, idx, tw);
      accumulate(std::integral_constant<int, f0>(), v[0]);
      accumulate(std::integral_constant<int, f0 + 1>(), v[1]);
    });
    // spectral update of the owned modes (FP64)
#pragma unroll
    for (int e = 0; e < E; ++e) {
      if (inb[e]) {
        const long long id = (long long)slot[e] * Q + q;
        cpx<double> S[4] = {acc[0][e], acc[1][e], acc[2][e], acc[3][e]}, u[4];
        mode_update(
            S, u, [&](int c) { return ld_global(state + c * M + id); }, [&](int c) { return ld_global(hist + c * M + id); },
            state, hist, M, id, kx, ky, kz[e], k_sq(kx, ky, kz[e]), sc, bx.sphi0);
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c][e] = u[c];
      }
    }
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      if (inb[e]) {
        const long long id = (long long)slot[e] * Q + q;
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c][e] = ld_global(state + c * M + id);
      }
    }
  }

  // z-inverse of u, v, w, phi and i kz phi, two fields at a time
  auto inv_fields = [&](auto gc, auto nc) {
    constexpr int g0 = decltype(gc)::value, nf = decltype(nc)::value;
    cpx<T> v[nf][E];
#pragma unroll
    for (int g = 0; g < nf; ++g)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        cpx<double> x = {0.0, 0.0};
        if (inb[e]) {
          if (g0 + g < 4) x = acc[g0 + g][e];
          else x = cpx<double>{-kz[e] * acc[3][e].im, kz[e] * acc[3][e].re};
        }
        v[g][e] = to_cpx<T>(x);
      }
    fft_lines<T, P, 1, nf>(v, lds[0], 2 * N * LP, N * LP, par, t, idx, tw);
    if (valid) {
#pragma unroll
      for (int g = 0; g < nf; ++g) {
        cpx<T>* dst = gout + (long long)(g0 + g) * N * Q;
#pragma unroll
        for (int b = 0; b < E / RF; ++b)
#pragma unroll
          for (int r = 0; r < RF; ++r) st_global(dst + (long long)slot_pos<P, RF>(t, b, r) * Q + q, v[g][b * RF + r]);
      }
    }
  };
  using std::integral_constant;
  inv_fields(integral_constant<int, 0>(), integral_constant<int, 2>());
  inv_fields(integral_constant<int, 2>(), integral_constant<int, 2>());
  inv_fields(integral_constant<int, 4>(), integral_constant<int, 1>());
}

// ---------------------------------------------------------------------------
// The z stage with a group of threads per field: group f transforms product f of
// L lines forward and leaves the band's modes in LDS; the modes are then updated one
// to a thread; group f < 5 inverts the new state's field f.  One line set of a small
// grid leaves k_zstep with a few workgroups (8 at 32^3), each a chain of 13 transforms
// and, per thread, E modes' updates: 15 us at 32^3, where this takes 6.5.  Steps with
// k_zstep and with it, us: FP64 32^3 28.0 -> 19.4, 48^3 37.6 -> 24.6, 64^3 41.0 -> 34.1,
// 96^3 75.3 -> 71.2; FP32 32^3 25.3 -> 18.0, 64^3 33.2 -> 28.0, 96^3 58.6 -> 50.3.
// ---------------------------------------------------------------------------
// lines of a workgroup: 64-byte rows
template <typename T>
constexpr int kZlines = 64 / int(sizeof(cpx<T>));
// The most lines (over all boxes) of a launch for which it runs.  Beyond, the chip is
// full and its barriers and LDS passes cost more than they save: FP64 16 and 32 boxes of
// 32^3 (3696, 7392 lines) 51 and 80 us against 55 and 78, 4 and 16 of 48^3 (1984, 7936)
// 48 and 116 against 60 and 107, 4 of 64^3 (3784) 72 against 69; FP32 4 of 64^3 54
// against 52, 1 and 4 of 96^3 (2016, 8064) 50 and 130 against 59 and 115.
template <typename T, int N>
constexpr int kZfieldMost = N > 96 ? 0 : N >= (sizeof(T) == 8 ? 48 : 64) ? 2048 : 4096;
template <typename T, int N>
constexpr int kZthreads = 8 * (N / Plan<N>::E) * kZlines<T>;
template <typename T, int N>
__global__ void __launch_bounds__((kZthreads<T, N>))
k_zfield(const BoxDev* __restrict__ boxes, int box0, const cpx<T>* __restrict__ tw_g, int do_update) {
  using P = Plan<N>;
  const BoxDev& bx = boxes[box0 + blockIdx.z];
  const cpx<T>* __restrict__ rhs = static_cast<const cpx<T>*>(bx.bufa);
  cpx<double>* __restrict__ state = bx.state;
  cpx<double>* __restrict__ hist = bx.hist;
  cpx<T>* __restrict__ gout = static_cast<cpx<T>*>(bx.bufb);
  const StepCoef sc = bx.sc;
  constexpr int E = P::E, TT = N / E, L = kZlines<T>, K = (N - 1) / 3, C = 2 * K + 1, H = K + 1;
  constexpr int Q = C * H, THREADS = kZthreads<T, N>;
  constexpr long long M = (long long)C * Q;
  constexpr int RF = first_radix<P, -1>(), RL = last_radix<P, -1>();
  static_assert(RL == first_radix<P, 1>(), "mirrored radix order");
  static_assert(C * L <= THREADS && THREADS <= 1024, "a mode per thread");
  __shared__ cpx<T> tw[N];
  __shared__ cpx<T> lds[2][8][N * L];
  const int tid = threadIdx.x;
  const int line = tid % L, t = tid / L % TT, f = tid / (L * TT);
  const int q = xcd_tile(blockIdx.x, gridDim.x) * L + line;
  const bool valid = q < Q;
  cpx<T> v[1][E];
  if (do_update) {
    const cpx<T>* src = rhs + (long long)f * N * Q + (valid ? q : 0);
#pragma unroll
    for (int b = 0; b < E / RF; ++b)
#pragma unroll
      for (int r = 0; r < RF; ++r) v[0][b * RF + r] = ld_global(src + (long long)slot_pos<P, RF>(t, b, r) * Q);
  }
  // the mode that this thread updates
  const int slot = tid / L;
  const bool mode = valid && slot < C;
  const long long id = (long long)(mode ? slot : 0) * Q + (mode ? q : 0);
  cpx<double> u[4], hp[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    u[c] = ld_global(state + c * M + id);
    hp[c] = cpx<double>{0.0, 0.0};
    if (do_update && !sc.ab1) hp[c] = ld_global(hist + c * M + id);
  }
  for (int i = tid; i < N; i += THREADS) tw[i] = tw_g[i];
  const IdxPosSwz idx{L, line};
  int par = 0;
  __syncthreads();
  const int iy = valid ? q / H : 0, ix = valid ? q % H : 0;
  const double kx = double(ix), ky = double(iy <= K ? iy : iy - C), kz = double(slot <= K ? slot : slot - C);
  if (do_update) {
    fft_lines<T, P, -1, 1>(v, lds[0][f], 0, 8 * N * L, par, t, idx, tw);
    __syncthreads();   // the exchanges' reads, before the modes over them
#pragma unroll
    for (int b = 0; b < E / RL; ++b)
#pragma unroll
      for (int r = 0; r < RL; ++r) {
        const int s = band_slot(slot_pos<P, RL>(t, b, r), C, N);
        if (s >= 0) lds[0][f][s * L + line] = v[0][b * RL + r];
      }
    __syncthreads();
  }
  if (mode) {
    if (do_update) {
      cpx<double> S[4] = {};
      const double k2 = k_sq(kx, ky, kz);
      static_for<0, 8>([&](auto fc) {
        constexpr int g = decltype(fc)::value;
        const cpx<T> x = lds[0][g][slot * L + line];
        add_product<g>(S, cpx<double>{double(x.re), double(x.im)}, kx, ky, kz, k2, sc);
      });
      cpx<double> un[4];
      mode_update(
          S, un, [&](int c) { return u[c]; }, [&](int c) { return hp[c]; }, state, hist, M, id, kx, ky, kz, k2, sc,
          bx.sphi0);
#pragma unroll
      for (int c = 0; c < 4; ++c) u[c] = un[c];
    }
    const cpx<double> kp = {-kz * u[3].im, kz * u[3].re};
#pragma unroll
    for (int c = 0; c < 5; ++c) lds[1][c][slot * L + line] = to_cpx<T>(c < 4 ? u[c] : kp);
  }
  __syncthreads();
  // z-inverse of u, v, w, phi and i kz phi (groups 5 .. 7 only keep the barriers)
#pragma unroll
  for (int b = 0; b < E / RL; ++b)
#pragma unroll
    for (int r = 0; r < RL; ++r) {
      const int s = band_slot(slot_pos<P, RL>(t, b, r), C, N);
      v[0][b * RL + r] = (valid && f < 5 && s >= 0) ? lds[1][f][s * L + line] : cpx<T>{T(0), T(0)};
    }
  __syncthreads();
  par = 0;
  fft_lines<T, P, 1, 1>(v, lds[0][f], 0, 8 * N * L, par, t, idx, tw);
  if (valid && f < 5) {
    cpx<T>* dst = gout + (long long)f * N * Q + q;
#pragma unroll
    for (int b = 0; b < E / RF; ++b)
#pragma unroll
      for (int r = 0; r < RF; ++r) st_global(dst + (long long)slot_pos<P, RF>(t, b, r) * Q, v[0][b * RF + r]);
  }
}

// ---------------------------------------------------------------------------
// small per-mode kernels
// ---------------------------------------------------------------------------

// compact band [nf][C][C][H] -> full half spectra out.p[f] [n][n][n/2+1].  One
// plane kz of one field per blockIdx.y, z, kExpandPer entries a thread in 32-bit
// index arithmetic.  HBM-bound (128^3: 20 MB read, 68 MB written): 4 fields
// take 13.1 us (6.7 TB/s), where 64-bit divisions by run-time sizes took 49 us in two launches.
constexpr int kExpandPer = 4;
template <typename T>
__global__ void __launch_bounds__(256) k_expand(const cpx<T>* __restrict__ cmp, SpecOut<T> out, BoxGeom g) {
  const int n = g.n, nh = n / 2 + 1, kzp = int(blockIdx.y), f = int(blockIdx.z);
  const int sz = band_slot(kzp, g.C, n);
  const cpx<T>* src = cmp + f * g.M + (long long)sz * g.C * g.H;
  cpx<T>* dst = out.p[f] + (long long)kzp * n * nh;
#pragma unroll
  for (int k = 0; k < kExpandPer; ++k) {
    const unsigned id = (blockIdx.x * kExpandPer + k) * 256u + threadIdx.x;
    if (id >= unsigned(n * nh)) break;
    const int kyp = int(id / unsigned(nh)), kxp = int(id % unsigned(nh));
    const int sy = band_slot(kyp, g.C, n);
    cpx<T> v = {T(0), T(0)};
    if (sz >= 0 && sy >= 0 && kxp < g.H) v = ld_global(src + sy * g.H + kxp);
    st_global(dst + id, v);
  }
}

template <typename T>
__global__ void k_compact(const cpx<T>* __restrict__ full, cpx<T>* __restrict__ cmp, BoxGeom g, int nf) {
  const int n = g.n, nh = n / 2 + 1;
  const long long tot = g.M * nf;
  for (long long id = blockIdx.x * (long long)blockDim.x + threadIdx.x; id < tot;
       id += (long long)gridDim.x * blockDim.x) {
    const long long f = id / g.M, r = id % g.M;
    const int ix = int(r % g.H);
    const int iy = int((r / g.H) % g.C);
    const int iz = int(r / ((long long)g.H * g.C));
    const int py = full_pos(iy, g.C, n), pz = full_pos(iz, g.C, n);
    cmp[id] = full[f * (long long)n * n * nh + ((long long)pz * n + py) * nh + ix];
  }
}

// a compact FP64 band converted to precision T (n entries)
template <typename T>
__global__ void k_band_to(const cpx<double>* __restrict__ a, cpx<T>* __restrict__ out, long long n) {
  for (long long id = blockIdx.x * (long long)blockDim.x + threadIdx.x; id < n;
       id += (long long)gridDim.x * blockDim.x) {
    const cpx<double> v = a[id];
    out[id] = cpx<T>{T(v.re), T(v.im)};
  }
}

// f <- f^3 over n values
template <typename T>
__global__ void k_cube(T* __restrict__ f, long long n) {
  for (long long id = blockIdx.x * (long long)blockDim.x + threadIdx.x; id < n;
       id += (long long)gridDim.x * blockDim.x) {
    const T a = f[id];
    f[id] = a * a * a;
  }
}

// The pressure that the projection removes, from the compact spectra of the six
// products T_ij (order xx, yy, zz, xy, xz, yz; [6][M], precision T): with
// S_i = i k_j T_ij and lap p = div S, p_hat = k_i k_j T_ij / k^2 (FP64; k = 0 -> 0).
template <typename T>
__global__ void k_pressure_band(const cpx<T>* __restrict__ t6, BoxGeom g, cpx<double>* __restrict__ p) {
  for (long long id = blockIdx.x * (long long)blockDim.x + threadIdx.x; id < g.M;
       id += (long long)gridDim.x * blockDim.x) {
    const int ix = int(id % g.H);
    const int iy = int((id / g.H) % g.C);
    const int iz = int(id / ((long long)g.H * g.C));
    const double kx = ix, ky = (iy <= g.K) ? iy : iy - g.C, kz = (iz <= g.K) ? iz : iz - g.C;
    const double k2 = kx * kx + ky * ky + kz * kz;
    const double w[6] = {kx * kx, ky * ky, kz * kz, 2.0 * kx * ky, 2.0 * kx * kz, 2.0 * ky * kz};
    double re = 0.0, im = 0.0;
#pragma unroll
    for (int f = 0; f < 6; ++f) {
      const cpx<T> a = t6[f * g.M + id];
      re += w[f] * double(a.re);
      im += w[f] * double(a.im);
    }
    p[id] = (k2 == 0.0) ? cpx<double>{0.0, 0.0} : cpx<double>{re / k2, im / k2};
  }
}

#if PSMS_PART == 64
// Leray projection of the compact velocity [3][M] in place (k = 0 -> 0).
__global__ void k_project(cpx<double>* __restrict__ u, BoxGeom g) {
  for (long long id = blockIdx.x * (long long)blockDim.x + threadIdx.x; id < g.M;
       id += (long long)gridDim.x * blockDim.x) {
    const int ix = int(id % g.H);
    const int iy = int((id / g.H) % g.C);
    const int iz = int(id / ((long long)g.H * g.C));
    const double kx = ix, ky = (iy <= g.K) ? iy : iy - g.C, kz = (iz <= g.K) ? iz : iz - g.C;
    const double k2 = kx * kx + ky * ky + kz * kz;
    cpx<double> a = u[id], b = u[g.M + id], c = u[2 * g.M + id];
    if (k2 == 0.0) {
      a = b = c = cpx<double>{0.0, 0.0};
    } else {
      const double ir = 1.0 / k2;
      const double dre = kx * a.re + ky * b.re + kz * c.re, dim = kx * a.im + ky * b.im + kz * c.im;
      a.re -= kx * dre * ir; a.im -= kx * dim * ir;
      b.re -= ky * dre * ir; b.im -= ky * dim * ir;
      c.re -= kz * dre * ir; c.im -= kz * dim * ir;
    }
    u[id] = a;
    u[g.M + id] = b;
    u[2 * g.M + id] = c;
  }
}

#endif

// Full half spectra [nf][n][n][n/2+1]: optional 2/3 mask and i k_axis factor,
// scale (index arithmetic as k_expand).
template <typename T>
__global__ void __launch_bounds__(256) k_spec_finish(const cpx<T>* __restrict__ in, cpx<T>* __restrict__ out,
                                                     BoxGeom g, int dealias, int axis, double scale) {
  const int n = g.n, nh = n / 2 + 1, kzp = int(blockIdx.y);
  const long long plane = ((long long)blockIdx.z * n + kzp) * n * nh;
#pragma unroll
  for (int k = 0; k < kExpandPer; ++k) {
    const unsigned id = (blockIdx.x * kExpandPer + k) * 256u + threadIdx.x;
    if (id >= unsigned(n * nh)) break;
    const int kyp = int(id / unsigned(nh)), kxp = int(id % unsigned(nh));
    cpx<T> v = in[plane + id];
    if (dealias && (kxp > g.K || band_slot(kyp, g.C, n) < 0 || band_slot(kzp, g.C, n) < 0)) v = cpx<T>{T(0), T(0)};
    if (axis >= 0) {
      const int kk = (axis == 0) ? kxp : signed_k(axis == 1 ? kyp : kzp, n);
      v = cpx<T>{-T(kk) * v.im, T(kk) * v.re};
    }
    out[plane + id] = cpx<T>{T(scale) * v.re, T(scale) * v.im};
  }
}

#if PSMS_PART == 64
// Helmholtz (lap - lambda_f) f = g per mode: f = -g / (k^2 + lambda_f).
__global__ void k_helmholtz_box(const cpx<double>* __restrict__ rhs, cpx<double>* __restrict__ out, BoxGeom g,
                                int nf, double lam) {
  const int n = g.n, nh = n / 2 + 1;
  const long long per = (long long)n * n * nh;
  const long long tot = per * nf;
  for (long long id = blockIdx.x * (long long)blockDim.x + threadIdx.x; id < tot;
       id += (long long)gridDim.x * blockDim.x) {
    const long long r = id % per;
    const int kxp = int(r % nh);
    const int ky = signed_k(int((r / nh) % n), n);
    const int kz = signed_k(int(r / ((long long)nh * n)), n);
    const double den = double(kxp) * kxp + double(ky) * ky + double(kz) * kz + lam;
    const cpx<double> v = rhs[id];
    out[id] = (den != 0.0) ? cpx<double>{-v.re / den, -v.im / den} : cpx<double>{0.0, 0.0};
  }
}

// Index maps of the compact band as used by every kernel: for slot (f=0) id,
// writes kz, ky, kx and the offset into the full half spectrum.
__global__ void k_index_maps(int* __restrict__ out, BoxGeom g) {
  const int n = g.n, nh = n / 2 + 1;
  for (long long id = blockIdx.x * (long long)blockDim.x + threadIdx.x; id < g.M;
       id += (long long)gridDim.x * blockDim.x) {
    const int ix = int(id % g.H);
    const int iy = int((id / g.H) % g.C);
    const int iz = int(id / ((long long)g.H * g.C));
    const int py = full_pos(iy, g.C, n), pz = full_pos(iz, g.C, n);
    out[4 * id + 0] = signed_k(pz, n);
    out[4 * id + 1] = signed_k(py, n);
    out[4 * id + 2] = ix;
    out[4 * id + 3] = int(((long long)pz * n + py) * nh + ix);
  }
}

// CFL number dt max_x sum_i |u_i| / dx (dx = 2 pi / n): block maxima of
// scale sum_i |u_i| over the n points of the three physical components, then
// k_max_final.
__global__ void k_cfl_partial(const double* __restrict__ u, const double* __restrict__ v, const double* __restrict__ w,
                              long long n, double scale, double* __restrict__ part) {
  __shared__ double sh[256];
  double m = 0.0;
  for (long long id = blockIdx.x * (long long)blockDim.x + threadIdx.x; id < n; id += (long long)gridDim.x * blockDim.x)
    m = fmax(m, scale * fabs(u[id]) + scale * fabs(v[id]) + scale * fabs(w[id]));
  const int t = threadIdx.x;
  sh[t] = m;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (t < s) sh[t] = fmax(sh[t], sh[t + s]);
    __syncthreads();
  }
  if (t == 0) part[blockIdx.x] = sh[0];
}

__global__ void k_max_final(const double* __restrict__ part, int nb, double* __restrict__ out) {
  __shared__ double sh[256];
  double m = 0.0;
  for (int i = threadIdx.x; i < nb; i += blockDim.x) m = fmax(m, part[i]);
  const int t = threadIdx.x;
  sh[t] = m;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (t < s) sh[t] = fmax(sh[t], sh[t + s]);
    __syncthreads();
  }
  if (t == 0) out[0] = sh[0];
}

// Diagnostics over the compact state, two-pass deterministic reduction.
// part[b] = {ke, grad2, max_div, nonfinite}
__global__ void k_diag_partial(const cpx<double>* __restrict__ st, BoxGeom g, double* __restrict__ part) {
  __shared__ double sh[4][256];
  double ke = 0.0, gr = 0.0, md = 0.0, nf = 0.0;
  for (long long id = blockIdx.x * (long long)blockDim.x + threadIdx.x; id < g.M;
       id += (long long)gridDim.x * blockDim.x) {
    const int ix = int(id % g.H);
    const int iy = int((id / g.H) % g.C);
    const int iz = int(id / ((long long)g.H * g.C));
    const double kx = ix, ky = (iy <= g.K) ? iy : iy - g.C, kz = (iz <= g.K) ? iz : iz - g.C;
    const double w = (ix == 0) ? 1.0 : 2.0;
    const cpx<double> a = st[id], b = st[g.M + id], c = st[2 * g.M + id], p = st[3 * g.M + id];
    const double e = a.re * a.re + a.im * a.im + b.re * b.re + b.im * b.im + c.re * c.re + c.im * c.im;
    ke += 0.5 * w * e;
    gr += w * (kx * kx + ky * ky + kz * kz) * (p.re * p.re + p.im * p.im);
    const double dre = kx * a.re + ky * b.re + kz * c.re, dim = kx * a.im + ky * b.im + kz * c.im;
    const double d = sqrt(dre * dre + dim * dim);
    md = fmax(md, d);
    const double s = e + p.re * p.re + p.im * p.im;
    if (!isfinite(s)) nf += 1.0;
  }
  const int t = threadIdx.x;
  sh[0][t] = ke; sh[1][t] = gr; sh[2][t] = md; sh[3][t] = nf;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (t < s) {
      sh[0][t] += sh[0][t + s];
      sh[1][t] += sh[1][t + s];
      sh[2][t] = fmax(sh[2][t], sh[2][t + s]);
      sh[3][t] += sh[3][t + s];
    }
    __syncthreads();
  }
  if (t == 0) {
    part[4 * blockIdx.x + 0] = sh[0][0];
    part[4 * blockIdx.x + 1] = sh[1][0];
    part[4 * blockIdx.x + 2] = sh[2][0];
    part[4 * blockIdx.x + 3] = sh[3][0];
  }
}

__global__ void k_diag_final(const double* __restrict__ part, int nb, const cpx<double>* __restrict__ st, BoxGeom g,
                             double* __restrict__ out) {
  __shared__ double sh[4][256];
  const int t = threadIdx.x;
  double a = 0.0, b = 0.0, c = 0.0, d = 0.0;
  for (int i = t; i < nb; i += blockDim.x) {
    a += part[4 * i];
    b += part[4 * i + 1];
    c = fmax(c, part[4 * i + 2]);
    d += part[4 * i + 3];
  }
  sh[0][t] = a; sh[1][t] = b; sh[2][t] = c; sh[3][t] = d;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (t < s) {
      sh[0][t] += sh[0][t + s];
      sh[1][t] += sh[1][t + s];
      sh[2][t] = fmax(sh[2][t], sh[2][t + s]);
      sh[3][t] += sh[3][t + s];
    }
    __syncthreads();
  }
  if (t == 0) {
    out[0] = st[3 * g.M].re;  // mean phi = phi_hat(0)
    out[1] = sh[0][0];
    out[2] = sh[1][0];
    out[3] = sh[2][0];
    out[4] = sh[3][0];
  }
}

#endif

// ---------------------------------------------------------------------------
// host-side launchers (dispatch on the transform length)
// ---------------------------------------------------------------------------
#define PSMS_FOR_EACH_N(X) X(8) X(12) X(16) X(24) X(32) X(48) X(64) X(96) X(128) X(192) X(256)

#if PSMS_PART == 64
bool supported_n(int n) {
  switch (n) {
#define PSMS_CASE(NN) case NN:
    PSMS_FOR_EACH_N(PSMS_CASE)
#undef PSMS_CASE
    return true;
    default:
      return false;
  }
}

#endif

namespace {

template <typename T, int N>
hipError_t lines_n(int dir, const cpx<T>* in, cpx<T>* out, const cpx<T>* tw, const LineArgs& a, int nfield,
                   hipStream_t st) {
  using P = Plan<N>;
  using G = Tile<P>;
  const dim3 grid(unsigned((a.nlines + G::L - 1) / G::L), unsigned(nfield));
  const dim3 block(unsigned(G::L * G::TT));
  if (dir < 0) k_lines<T, N, -1><<<grid, block, 0, st>>>(in, out, tw, a);
  else k_lines<T, N, 1><<<grid, block, 0, st>>>(in, out, tw, a);
  return hipGetLastError();
}

template <typename T, int N>
hipError_t rows_n(int dir, const void* in, void* out, const cpx<T>* tw, const RowArgs& a, int nfield,
                  hipStream_t st) {
  using P = Plan<N>;
  using G = Tile<P>;
  const long long pairs = (a.nrows + 1) / 2;
  const dim3 grid(unsigned((pairs + G::L - 1) / G::L), unsigned(nfield));
  const dim3 block(unsigned(G::L * G::TT));
  if (dir < 0)
    k_rows_fwd<T, N><<<grid, block, 0, st>>>(static_cast<const T*>(in), static_cast<cpx<T>*>(out), tw, a);
  else
    k_rows_inv<T, N><<<grid, block, 0, st>>>(static_cast<const cpx<T>*>(in), static_cast<T*>(out), tw, a);
  return hipGetLastError();
}

// The y stages' largest variant: 512 threads in FP32 (twice the lines per
// workgroup, so each position's row segment is 128 bytes, a whole cache line;
// measured faster), 256 in FP64 (measured slower at 512).
template <typename T, int V>
constexpr int kYVariant = (V == 2 && sizeof(T) == 4) ? 3 : V;

template <typename T, int N, int V>
hipError_t step_nv(int stage, const BoxDev* boxes, int box0, int nbox, const cpx<T>* tw, int do_update,
                   hipStream_t st) {
  using P = Plan<N>;
  using G = Tile<P, V>;
  const unsigned threads = unsigned(G::L * G::TT);
  switch (stage) {
    case 0: {  // y-inverse, 6 output fields
      using GY = Tile<P, kYVariant<T, V>>;
      const dim3 grid(unsigned(((long long)N * GY::H + GY::L - 1) / GY::L), 6, unsigned(nbox));
      k_ystep<T, N, 1, kYVariant<T, V>><<<grid, unsigned(GY::L * GY::TT), 0, st>>>(boxes, box0, tw);
      break;
    }
    case 1: {  // x stage with products
      const long long pairs = (long long)N * N / 2;
      if constexpr (kXfield<T, N>) {   // the same workgroups in every variant
        constexpr int LW = 64 / (N / XPlan<T, N>::E);
        k_xfield<T, N><<<dim3(unsigned((pairs + LW - 1) / LW), 1, unsigned(nbox)), 512, 0, st>>>(boxes, box0, tw, 0, 1.0);
      } else {
        const dim3 grid(unsigned((pairs + G::L - 1) / G::L), 1, unsigned(nbox));
        k_xstep<T, N, V><<<grid, threads, 0, st>>>(boxes, box0, tw, 0, 1.0);
      }
      break;
    }
    case 2: {  // y-forward, 8 fields
      using GY = Tile<P, kYVariant<T, V>>;
      const dim3 grid(unsigned(((long long)N * GY::H + GY::L - 1) / GY::L), 8, unsigned(nbox));
      k_ystep<T, N, -1, kYVariant<T, V>><<<grid, unsigned(GY::L * GY::TT), 0, st>>>(boxes, box0, tw);
      break;
    }
    default: {  // z stage with the update
      const int Q = G::C * G::H;
      if constexpr (kZfieldMost<T, N> > 0) {
        if ((long long)Q * nbox <= kZfieldMost<T, N>) {   // the same workgroups in every variant
          constexpr int L = kZlines<T>;
          k_zfield<T, N><<<dim3(unsigned((Q + L - 1) / L), 1, unsigned(nbox)), kZthreads<T, N>, 0, st>>>(boxes, box0, tw,
                                                                                                       do_update);
          break;
        }
      }
      const dim3 grid(unsigned((Q + G::L - 1) / G::L), 1, unsigned(nbox));
      k_zstep<T, N, V><<<grid, threads, 0, st>>>(boxes, box0, tw, do_update);
      break;
    }
  }
  return hipGetLastError();
}

template <typename T, int N>
hipError_t step_n(int stage, int variant, const BoxDev* boxes, int box0, int nbox, const cpx<T>* tw, int do_update,
                  hipStream_t st) {
  switch (variant) {
    case 0: return step_nv<T, N, 0>(stage, boxes, box0, nbox, tw, do_update, st);
    case 1: return step_nv<T, N, 1>(stage, boxes, box0, nbox, tw, do_update, st);
    default: return step_nv<T, N, 2>(stage, boxes, box0, nbox, tw, do_update, st);
  }
}

}  // namespace

template <typename T, int N>
hipError_t xstage_rows_n(const BoxDev* dev, const cpx<T>* tw, long long rows, double kxs, bool sp, hipStream_t st) {
  const long long pairs = rows / 2;
  if constexpr (kXfield<T, N>) {
    constexpr int LW = 64 / (N / XPlan<T, N>::E);
    const dim3 grid(unsigned((pairs + LW - 1) / LW), 1, 1);
    if (sp) k_xfield<T, N, true, true><<<grid, 384, 0, st>>>(dev, 0, tw, rows, kxs);
    else k_xfield<T, N, true><<<grid, 512, 0, st>>>(dev, 0, tw, rows, kxs);
  } else {
    using G = Tile<Plan<N>, 2>;
    const dim3 grid(unsigned((pairs + G::L - 1) / G::L), 1, 1);
    if (sp) k_xstep<T, N, 2, true, true><<<grid, unsigned(G::L * G::TT), 0, st>>>(dev, 0, tw, rows, kxs);
    else k_xstep<T, N, 2, true><<<grid, unsigned(G::L * G::TT), 0, st>>>(dev, 0, tw, rows, kxs);
  }
  return hipGetLastError();
}

template <typename T>
hipError_t launch_xstage_rows(int n, const BoxDev* dev, const cpx<T>* tw, long long rows, double kxs, bool sp,
                              hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  if (rows % 2) return hipErrorInvalidValue;   // rows are transformed in pairs
  switch (n) {
#define PSMS_CASE(NN) case NN: return xstage_rows_n<T, NN>(dev, tw, rows, kxs, sp, st);
    PSMS_FOR_EACH_N(PSMS_CASE)
#undef PSMS_CASE
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_lines(int n, int dir, const cpx<T>* in, cpx<T>* out, const cpx<T>* tw, const LineArgs& a,
                        int nfield, hipStream_t st) {
  switch (n) {
#define PSMS_CASE(NN) case NN: return lines_n<T, NN>(dir, in, out, tw, a, nfield, st);
    PSMS_FOR_EACH_N(PSMS_CASE)
#undef PSMS_CASE
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_rows(int n, int dir, const void* in, void* out, const cpx<T>* tw, const RowArgs& a, int nfield,
                       hipStream_t st) {
  switch (n) {
#define PSMS_CASE(NN) case NN: return rows_n<T, NN>(dir, in, out, tw, a, nfield, st);
    PSMS_FOR_EACH_N(PSMS_CASE)
#undef PSMS_CASE
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_step_stage(int n, int stage, int variant, const BoxDev* boxes, int box0, int nbox,
                             const cpx<T>* tw, int do_update, hipStream_t st) {
  if (nbox < 1) return hipSuccess;
  switch (n) {
#define PSMS_CASE(NN) case NN: return step_n<T, NN>(stage, variant, boxes, box0, nbox, tw, do_update, st);
    PSMS_FOR_EACH_N(PSMS_CASE)
#undef PSMS_CASE
  }
  return hipErrorInvalidValue;
}

static unsigned grid_for(long long tot) {
  long long b = (tot + 255) / 256;
  if (b > 65536) b = 65536;
  if (b < 1) b = 1;
  return unsigned(b);
}

template <typename T>
hipError_t launch_expand(const cpx<T>* cmp, const SpecOut<T>& out, const BoxGeom& g, int nf, hipStream_t st) {
  if (nf < 1 || nf > kSpecOutMax) return hipErrorInvalidValue;
  const unsigned per = unsigned(g.n) * unsigned(g.n / 2 + 1), chunk = 256u * kExpandPer;
  k_expand<T><<<dim3((per + chunk - 1) / chunk, unsigned(g.n), unsigned(nf)), 256, 0, st>>>(cmp, out, g);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_compact(const cpx<T>* full, cpx<T>* cmp, const BoxGeom& g, int nf, hipStream_t st) {
  k_compact<T><<<grid_for(g.M * nf), 256, 0, st>>>(full, cmp, g, nf);
  return hipGetLastError();
}
#if PSMS_PART == 64
hipError_t launch_project(cpx<double>* u, const BoxGeom& g, hipStream_t st) {
  k_project<<<grid_for(g.M), 256, 0, st>>>(u, g);
  return hipGetLastError();
}
#endif

template <typename T>
hipError_t launch_band_to(const cpx<double>* a, cpx<T>* out, long long n, hipStream_t st) {
  k_band_to<T><<<grid_for(n), 256, 0, st>>>(a, out, n);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_cube(T* f, long long n, hipStream_t st) {
  k_cube<T><<<grid_for(n), 256, 0, st>>>(f, n);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_pressure_band(const cpx<T>* t6, const BoxGeom& g, cpx<double>* p, hipStream_t st) {
  k_pressure_band<T><<<grid_for(g.M), 256, 0, st>>>(t6, g, p);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_spec_finish(const cpx<T>* in, cpx<T>* out, const BoxGeom& g, int nf, int dealias, int axis,
                              double scale, hipStream_t st) {
  if (nf < 1) return hipErrorInvalidValue;
  const unsigned per = unsigned(g.n) * unsigned(g.n / 2 + 1), chunk = 256u * kExpandPer;
  k_spec_finish<T><<<dim3((per + chunk - 1) / chunk, unsigned(g.n), unsigned(nf)), 256, 0, st>>>(in, out, g, dealias,
                                                                                              axis, scale);
  return hipGetLastError();
}
#if PSMS_PART == 64
hipError_t launch_helmholtz_box(const cpx<double>* rhs, cpx<double>* out, const BoxGeom& g, double lam,
                                hipStream_t st) {
  const long long tot = (long long)g.n * g.n * (g.n / 2 + 1);
  k_helmholtz_box<<<grid_for(tot), 256, 0, st>>>(rhs, out, g, 1, lam);
  return hipGetLastError();
}
hipError_t launch_index_maps(int* out, const BoxGeom& g, hipStream_t st) {
  k_index_maps<<<grid_for(g.M), 256, 0, st>>>(out, g);
  return hipGetLastError();
}
hipError_t launch_cfl(const double* u, const double* v, const double* w, long long n, double scale, double* part,
                      int max_blocks, double* out, hipStream_t st) {
  long long b = (n + 255) / 256;
  if (b > max_blocks) b = max_blocks;
  if (b < 1) b = 1;
  k_cfl_partial<<<unsigned(b), 256, 0, st>>>(u, v, w, n, scale, part);
  k_max_final<<<1, 256, 0, st>>>(part, int(b), out);
  return hipGetLastError();
}

hipError_t launch_diag(const cpx<double>* state, const BoxGeom& g, double* part, int max_blocks, double* out,
                       hipStream_t st) {
  long long nb = (g.M + 255) / 256;
  if (nb > max_blocks) nb = max_blocks;
  k_diag_partial<<<unsigned(nb), 256, 0, st>>>(state, g, part);
  k_diag_final<<<1, 256, 0, st>>>(part, int(nb), state, g, out);
  return hipGetLastError();
}

#endif

#if PSMS_PART == 64
using PartT = double;
template hipError_t launch_expand<double>(const cpx<double>*, const SpecOut<double>&, const BoxGeom&, int,
                                          hipStream_t);
template hipError_t launch_compact<double>(const cpx<double>*, cpx<double>*, const BoxGeom&, int, hipStream_t);
#else
using PartT = float;
template hipError_t launch_band_to<float>(const cpx<double>*, cpx<float>*, long long, hipStream_t);
#endif
template hipError_t launch_xstage_rows<PartT>(int, const BoxDev*, const cpx<PartT>*, long long, double, bool,
                                              hipStream_t);
template hipError_t launch_cube<PartT>(PartT*, long long, hipStream_t);
template hipError_t launch_pressure_band<PartT>(const cpx<PartT>*, const BoxGeom&, cpx<double>*, hipStream_t);
template hipError_t launch_lines<PartT>(int, int, const cpx<PartT>*, cpx<PartT>*, const cpx<PartT>*, const LineArgs&,
                                        int, hipStream_t);
template hipError_t launch_rows<PartT>(int, int, const void*, void*, const cpx<PartT>*, const RowArgs&, int,
                                       hipStream_t);
template hipError_t launch_step_stage<PartT>(int, int, int, const BoxDev*, int, int, const cpx<PartT>*, int,
                                             hipStream_t);
template hipError_t launch_spec_finish<PartT>(const cpx<PartT>*, cpx<PartT>*, const BoxGeom&, int, int, int, double,
                                              hipStream_t);

}  // namespace psms
