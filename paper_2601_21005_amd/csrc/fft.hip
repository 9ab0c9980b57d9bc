// 3D FFT passes for H|psi> and the split-operator steps (Sec. 2.2: FFT pairs
// switch between the position representation, where V is diagonal, and the
// momentum representation, where T is diagonal).
//
// Passes over a batch of vectors (x fastest), the first and the last with a
// whole xy plane per workgroup:
//   plane   x and y transform of one xy plane of one vector, with fused
//           epilogues on the inverse pass (V psi, Chebyshev update, Poisson
//           outputs);
//   pencil  TX neighbouring columns along z (coalesced rows of TX complex):
//           forward z -> k-space multiplier -> inverse z;
//   xlines, ypencil  x lines and y columns in two passes, where a plane does
//           not fit in LDS or spills registers (160^2, and 112^2 in FP64).
// Small batches carry the projector gather in the same launches.
#include "fft_reg.h"
#include "kb_gather.h"

namespace sgw {

constexpr int NT_FFT = 256;

struct PassArgs {
  const void *src = nullptr;
  void *dst = nullptr;
  int64_t ld_src = 0, ld_dst = 0, ld_x = 0;
  const void *tw0 = nullptr;                   // twiddles of the pass's axis (x and y are equal)
  const void *k2x = nullptr, *k2y = nullptr, *k2z = nullptr;
  int nx = 0, ny = 0, nz = 0;
  int mode = 0;          // PlaneMode (inverse passes) / 0 forward
  int inverse = 0;       // y pencils
  int mul = 0;           // MulMode (z pencils)
  int rev = 0;           // 1: vectors in descending order of blockIdx.y
  double tau = 0, ecut = 0, invN = 0;
  int64_t N = 0;
  EpiArgs e;
};

// ----------------------------------------------------------------- epilogue
template <typename R, int MODE>
__device__ __forceinline__ void epilogue(const PassArgs &a, int64_t v, int64_t r,
                                         cplx<R> val) {
  using C = cplx<R>;
  switch (MODE) {
    case PLANE_FWD:
    case PLANE_INV_STORE:
      static_cast<C *>(a.dst)[v * a.ld_dst + r] = val;
      break;
    case PLANE_INV_HPSI: {
      const C x = static_cast<const C *>(a.e.x)[v * a.ld_x + r];
      const R V = static_cast<const R *>(a.e.vloc)[r];
      val.x += V * x.x;
      val.y += V * x.y;
      static_cast<C *>(a.dst)[v * a.ld_dst + r] = val;
    } break;
    case PLANE_INV_CHEB: {
      // x = v_n:  w = (H x - c x)/R ; v_{n+1} = s2 w - v_{n-1} (no v_{n-1}
      // on the first step).  The projector part of H x is added to v_{n+1}
      // afterwards, so v_{n-1} and v_n are complete here; on odd n the pair
      // b_{n-1} v_{n-1} + b_n v_n goes into acc.
      const int64_t o = v * a.ld_x + r;
      const C x = static_cast<const C *>(a.e.x)[o];
      const R V = static_cast<const R *>(a.e.vloc)[r];
      const R c = (R)a.e.c, iR = (R)a.e.invR, s2 = (R)a.e.scale2;
      C *vold = static_cast<C *>(a.e.vold);
      C *vout = a.e.vout ? static_cast<C *>(a.e.vout) : vold;
      C *acc = static_cast<C *>(a.e.acc);
      C p;
      p.x = p.y = 0;
      if (!a.e.first) p = vold[o];
      C nv;
      nv.x = s2 * ((val.x + (V - c) * x.x) * iR) - p.x;
      nv.y = s2 * ((val.y + (V - c) * x.y) * iR) - p.y;
      vout[o] = nv;
      if (a.e.acc_mode) {
        R b0r = (R)a.e.cprev_re, b0i = (R)a.e.cprev_im, b1r = (R)a.e.coef_re, b1i = (R)a.e.coef_im;
        if (a.e.coef_dev) {
          const int k = a.e.term_dev[0];
          b0r = (R)a.e.coef_dev[2 * k - 2];
          b0i = (R)a.e.coef_dev[2 * k - 1];
          b1r = (R)a.e.coef_dev[2 * k];
          b1i = (R)a.e.coef_dev[2 * k + 1];
        }
        C sm;
        sm.x = sm.y = 0;
        if (a.e.acc_mode == 2) sm = acc[o];
        sm.x += b0r * p.x - b0i * p.y;
        sm.y += b0r * p.y + b0i * p.x;
        sm.x += b1r * x.x - b1i * x.y;
        sm.y += b1r * x.y + b1i * x.x;
        acc[o] = sm;
      }
    } break;
    case PLANE_INV_POISSON: {
      const int64_t o = v * a.N + r;
      const R V = static_cast<const R *>(a.e.vloc)[r];
      static_cast<R *>(a.e.r0)[o] = V + val.x - static_cast<const R *>(a.e.vh0)[o];
      static_cast<R *>(a.e.r1)[o] = val.y;
    } break;
    case PLANE_INV_SPLIT: {
      const int64_t o = v * a.N + r;
      if (a.e.r0) static_cast<R *>(a.e.r0)[o] = val.x;
      if (a.e.r1) static_cast<R *>(a.e.r1)[o] = val.y;
    } break;
  }
}

// ----------------------------------------------------------------- plane
// One xy plane of one vector per workgroup, the points in registers
// throughout: two stages of the x transform, two of the y transform, an
// exchange through LDS between them, and rows of x from and to memory, in
// whole cache lines, where a pass reads and writes most.  The passes are bound
// by HBM (16, 24 and 40 B per point); what has to be avoided is a second pass
// and too few bytes in flight.  Real and imaginary parts are exchanged one
// after the other, through half the LDS, so a plane of 128^2 in FP32 (75 KB,
// 62 registers) stays twice on a CU.  Forward pass of 800 MB: 128^2 285 us
// (5.7 TB/s) where x lines and y pencils took 272 + 265, 96^2 283 from 303 +
// 265, 80^2 286 from 372, FP64 64^2 301 from 282 + 270, FP64 128^2 321 from
// 267 + 250; 32^2 to 64^2 as before (282 us).  The planes that would not fit
// (FP64 160^2) or that spill registers in every pass (FP32 160^2, FP64 112^2:
// 391 and 401 us against 304 + 263 and 297 + 255) keep the two passes; of those
// used, FP32 112^2 with the H psi epilogue spills four registers and FP64 128^2
// with the Chebyshev epilogue six.
template <typename R, int N, int MODE = PLANE_FWD> struct PlaneShape {
  static constexpr bool D = sizeof(R) == 8;
  static constexpr int T = N == 128 ? 1024 : N == 112 ? 448 : N == 96 ? 768 : N == 80 ? 448
                         : N == 64 ? 512 : N == 56 ? 448 : N == 48 ? 192 : N == 40 ? 320
                         : N == 32 ? 256 : N == 24 ? 192 : N == 16 ? 128 : 64;
  // waves per SIMD to fit the registers for: two workgroups per CU
  static constexpr int WPE = !D && N == 128 && MODE != PLANE_INV_CHEB && MODE != PLANE_INV_SPLIT ? 8
                           : !D && N == 112 && MODE != PLANE_INV_CHEB ? 4 : 1;
  // odd pitch: lanes on successive lines fall on distinct banks; at 128 and
  // 64 also wide enough that the runs of R1 points of neighbouring lines do
  static constexpr int P = N == 128 ? 145 : N == 64 ? 73 : N + 1;
  // FP32 inverse transforms of 96 and more take y before x, at one exchange
  // more: the order in which x lines and y pencils round.  The TDH's response
  // field, a small difference of orbitals, amplifies another rounding to some
  // 2e-5 of itself (96^3), so results recorded with that order stay what they
  // are (x before y: H psi on 24 vectors of 96^3 300 us against 304, 112^3 498
  // against 506, 128^3 669 against 672, as accurate)
  static constexpr bool YFIRST = !D && N >= 96;
  static constexpr size_t lds = (size_t)N * P * sizeof(R) + N * sizeof(cplx<R>);
  static constexpr bool fits = lds <= 160 * 1024 && !(D && N == 112) && !(!D && N == 160);
};

// plane z of vector v; s: N P values, tw: N
template <typename R, int N, int MODE>
__device__ __forceinline__ void plane_pass(const PassArgs &a, int z, int64_t v, R *s,
                                           cplx<R> *tw) {
  constexpr bool INV = MODE != PLANE_FWD;
  using C = cplx<R>;
  using Sh = PlaneShape<R, N, MODE>;
  constexpr int R1 = Radix<N>::R1, R2 = Radix<N>::R2, P = Sh::P, T = Sh::T;
  constexpr bool YF = INV && Sh::YFIRST;
  const int tid = threadIdx.x;
  const int64_t plane = (int64_t)z * (N * N);
  const C *src = static_cast<const C *>(a.src) + v * a.ld_src + plane;
  Stage<C, R1, N * R2, T> s1;
  Stage<C, R2, N * R1, T> s2;
  s1.each(tid, [&](int q, int b) {
#pragma unroll
    for (int i = 0; i < R1; ++i)
      s1.v[q][i] = src[YF ? (b / N + i * R2) * N + b % N : (b / R2) * N + b % R2 + i * R2];
  });
  for (int i = tid; i < N; i += T) tw[i] = static_cast<const C *>(a.tw0)[i];
  if (INV) s1.map(tid, [](C z, int, int) { return cconj(z); });
  // where the values of a stage sit in the exchange: x butterflies
  // b = (line fast, j), or (j fast, line) as loaded; y butterflies (x fast, j);
  // first-stage inputs and outputs, second-stage inputs (= outputs)
  auto x1 = [](int b, int i) { return (b % N) * P + b / N + i * R2; };
  auto x1o = [](int b, int i) { return (b % N) * P + (b / N) * R1 + i; };
  auto x1l = [](int b, int i) { return (b / R2) * P + (b % R2) * R1 + i; };
  auto x2 = [](int b, int i) { return (b % N) * P + b / N + i * R1; };
  auto y1 = [](int b, int i) { return (b / N + i * R2) * P + b % N; };
  auto y1o = [](int b, int i) { return ((b / N) * R1 + i) * P + b % N; };
  auto y2 = [](int b, int i) { return (b / N + i * R1) * P + b % N; };
  auto j_of = [](int b) { return b / N; };
  s1.template run<N, 1>(tid, tw, j_of);
  if constexpr (YF) {
    exchange<true, C>(s, tid, s1, s2, true, y1o, y2);
    s2.template run<N, R1>(tid, tw, j_of);
    exchange<true, C>(s, tid, s2, s1, true, y2, x1);
    s1.template run<N, 1>(tid, tw, j_of);
    exchange<true, C>(s, tid, s1, s2, true, x1o, x2);
    s2.template run<N, R1>(tid, tw, j_of);
    exchange<true, C>(s, tid, s2, s2, false, x2, y2);   // rows again, for whole cache lines
  } else {
    exchange<true, C>(s, tid, s1, s2, true, x1l, x2);
    s2.template run<N, R1>(tid, tw, j_of);
    exchange<true, C>(s, tid, s2, s1, true, x2, y1);
    s1.template run<N, 1>(tid, tw, j_of);
    exchange<true, C>(s, tid, s1, s2, false, y1o, y2);
    s2.template run<N, R1>(tid, tw, j_of);
  }
  constexpr int STEP = R1 * N;           // butterfly b's output i is at point b + i STEP
  if (INV) s2.map(tid, [](C z, int, int) { return cconj(z); });
  // epilogue operands are loaded CH points at a time before their stores (the
  // stores would otherwise order every later load); 10 at once hold 132
  // registers (80^2 filter terms of 24 vectors 255 us against 240 with 5, and
  // 250 with the points in LDS)
  constexpr int CH = R2 % 4 == 0 ? 4 : R2 % 5 == 0 ? 5 : R2;
  if constexpr (MODE == PLANE_INV_CHEB) {
    const C *xp = static_cast<const C *>(a.e.x) + v * a.ld_x + plane;
    C *vp = static_cast<C *>(a.e.vold) + v * a.ld_x + plane;
    C *wp = (a.e.vout ? static_cast<C *>(a.e.vout) : static_cast<C *>(a.e.vold)) + v * a.ld_x + plane;
    C *ap = static_cast<C *>(a.e.acc) + v * a.ld_x + plane;
    const R *Vp = static_cast<const R *>(a.e.vloc) + plane;
    const bool first = a.e.first != 0;
    const int am = a.e.acc_mode;
    const R c = (R)a.e.c, iR = (R)a.e.invR, s2c = (R)a.e.scale2;
    R b0r = (R)a.e.cprev_re, b0i = (R)a.e.cprev_im, b1r = (R)a.e.coef_re, b1i = (R)a.e.coef_im;
    if (am && a.e.coef_dev) {
      const int k = a.e.term_dev[0];
      b0r = (R)a.e.coef_dev[2 * k - 2];
      b0i = (R)a.e.coef_dev[2 * k - 1];
      b1r = (R)a.e.coef_dev[2 * k];
      b1i = (R)a.e.coef_dev[2 * k + 1];
    }
    s2.each(tid, [&](int q, int b) {
      const int e0 = b;
#pragma unroll
      for (int h = 0; h < R2 / CH; ++h) {
        C xs[CH], ps[CH], ss[CH];
        R Vs[CH];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
          const int e = e0 + (h * CH + i) * STEP;
          xs[i] = xp[e];
          Vs[i] = Vp[e];
          ps[i].x = ps[i].y = 0;
          ss[i].x = ss[i].y = 0;
          if (!first) ps[i] = vp[e];
          if (am == 2) ss[i] = ap[e];
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) {
          const int e = e0 + (h * CH + i) * STEP;
          const C val = s2.v[q][h * CH + i], x = xs[i], pv = ps[i];
          // w = (H x - c x)/R; v_{n+1} = s2 w - v_{n-1}; on odd n
          // acc (+)= b_{n-1} v_{n-1} + b_n v_n.  The projector part of H x is
          // added to v_{n+1} afterwards, so v_{n-1} and v_n are complete here.
          C nv;
          nv.x = s2c * ((val.x + (Vs[i] - c) * x.x) * iR) - pv.x;
          nv.y = s2c * ((val.y + (Vs[i] - c) * x.y) * iR) - pv.y;
          wp[e] = nv;
          if (am) {
            C sm = ss[i];
            sm.x += b0r * pv.x - b0i * pv.y;
            sm.y += b0r * pv.y + b0i * pv.x;
            sm.x += b1r * x.x - b1i * x.y;
            sm.y += b1r * x.y + b1i * x.x;
            ap[e] = sm;
          }
        }
      }
    });
  } else if constexpr (MODE == PLANE_INV_HPSI) {
    // H psi = (T psi) + V psi
    const C *xp = static_cast<const C *>(a.e.x) + v * a.ld_x + plane;
    const R *Vp = static_cast<const R *>(a.e.vloc) + plane;
    C *dp = static_cast<C *>(a.dst) + v * a.ld_dst + plane;
    s2.each(tid, [&](int q, int b) {
      const int e0 = b;
      constexpr int CX = R2 % 4 == 0 ? 4 : R2;
#pragma unroll
      for (int h = 0; h < R2 / CX; ++h) {
        C xs[CX];
        R Vs[CX];
#pragma unroll
        for (int i = 0; i < CX; ++i) {
          xs[i] = xp[e0 + (h * CX + i) * STEP];
          Vs[i] = Vp[e0 + (h * CX + i) * STEP];
        }
#pragma unroll
        for (int i = 0; i < CX; ++i) {
          C val = s2.v[q][h * CX + i];
          val.x += Vs[i] * xs[i].x;
          val.y += Vs[i] * xs[i].y;
          dp[e0 + (h * CX + i) * STEP] = val;
        }
      }
    });
  } else {
    s2.each(tid, [&](int q, int b) {
      const int e0 = b;
#pragma unroll
      for (int i = 0; i < R2; ++i) epilogue<R, MODE>(a, v, plane + e0 + i * STEP, s2.v[q][i]);
    });
  }
}

// vector of a workgroup in the passes' order
__device__ __forceinline__ int64_t vec_of(const PassArgs &a, int i, int nvec) {
  return a.rev ? nvec - 1 - i : i;
}

template <typename R, int N, int MODE>
__global__ __launch_bounds__((PlaneShape<R, N>::T), (PlaneShape<R, N, MODE>::WPE)) void k_plane(PassArgs a) {
  using Sh = PlaneShape<R, N, MODE>;
  __shared__ R s[N * Sh::P];
  __shared__ cplx<R> tw[N];
  plane_pass<R, N, MODE>(a, blockIdx.x, vec_of(a, blockIdx.y, gridDim.y), s, tw);
}

// The forward pass of a small batch with the projector gather of the same
// vectors beside it, in the first workgroups (their waves past the gather's
// four end at once).  A launch costs about as much as either does on one or a
// few vectors, and neither fills the device.  H psi with the gather and the
// reduction (k_pencil_reduce) in launches of their own and beside the passes:
// 40^3 1 vector 29.2 -> 22.2 us, 8 vectors 38.8 -> 30.7, 48 vectors 78 -> 69;
// 64^3 1 vector 40.5 -> 32.7, 16 vectors 82.6 -> 75.0; 96^3 8 vectors 125 ->
// 117.  Registers are the larger of the two parts', which the planes of a
// large batch would pay for in waves: kb_rides ends at 1024 gather workgroups,
// from where (64^3, 32 vectors: 135 us either way) nothing is gained.
template <int N>
__global__ __launch_bounds__((PlaneShape<float, N>::T), (PlaneShape<float, N>::WPE)) void
k_plane_gather(PassArgs a, KbGather<float> g, int nvec) {
  using Sh = PlaneShape<float, N>;
  __shared__ __align__(16) float s[N * Sh::P > RIDE_LDS ? N * Sh::P : RIDE_LDS];
  __shared__ float2 tw[N];
  const int ng = g.gx * g.gy, b = blockIdx.x;
  if (b < ng) {
    if (threadIdx.x < NTK)
      gather_tile<OpF32, RIDE_NVB, RIDE_MT, N % 16 == 0 ? 4 : 3>(g, b % g.gx, b / g.gx, g.gy, s);
    return;
  }
  plane_pass<float, N, PLANE_FWD>(a, (b - ng) % a.nz, vec_of(a, (b - ng) / a.nz, nvec), s, tw);
}

// ----------------------------------------------------------------- xlines
template <typename R, int NX, int NL, int MODE>
__global__ __launch_bounds__(NT_FFT) void k_xlines(PassArgs a) {
  constexpr bool INV = MODE != PLANE_FWD;
  using C = cplx<R>;
  constexpr int P = NX + 1;
  constexpr int E = NX * NL;
  __shared__ C s[NL * P];
  __shared__ C twx[NX];
  const int tid = threadIdx.x;
  const int64_t v = a.rev ? gridDim.y - 1 - blockIdx.y : blockIdx.y;
  const int64_t nlines = (int64_t)a.ny * a.nz;
  const int64_t l0 = (int64_t)blockIdx.x * NL;
  for (int i = tid; i < NX; i += NT_FFT) twx[i] = static_cast<const C *>(a.tw0)[i];
  const C *src = static_cast<const C *>(a.src) + v * a.ld_src;
#pragma unroll
  for (int q = 0; q < (E + NT_FFT - 1) / NT_FFT; ++q) {
    const int e = tid + q * NT_FFT;
    if ((E % NT_FFT == 0 || e < E) && l0 + e / NX < nlines) {
      C val = src[l0 * NX + e];
      if (INV) val = cconj(val);
      s[(e / NX) * P + (e % NX)] = val;
    }
  }
  __syncthreads();
  lds_fft<C, NX, NL, P, 1, true, NT_FFT>(s, twx, tid);
#pragma unroll
  for (int q = 0; q < (E + NT_FFT - 1) / NT_FFT; ++q) {
    const int e = tid + q * NT_FFT;
    if ((E % NT_FFT == 0 || e < E) && l0 + e / NX < nlines) {
      C val = s[(e / NX) * P + (e % NX)];
      if (INV) val = cconj(val);
      epilogue<R, MODE>(a, v, l0 * NX + e, val);
    }
  }
}

// ----------------------------------------------------------------- pencil
template <typename C, typename R> __device__ __forceinline__ C cmake_r(R re, R im) {
  C c; c.x = re; c.y = im; return c;
}

template <typename R>
__device__ __forceinline__ cplx<R> kmul(const PassArgs &a, int ix, int iy, int iz) {
  using C = cplx<R>;
  const R k2 = static_cast<const R *>(a.k2x)[ix] + static_cast<const R *>(a.k2y)[iy] +
               static_cast<const R *>(a.k2z)[iz];
  C m;
  m.y = 0;
  if (a.mul == MUL_COUL) {
    m.x = k2 > (R)0 ? (R)(4.0 * M_PI) / k2 * (R)a.invN : (R)0;
  } else {
    R T = (R)0.5 * k2;
    if (a.ecut > 0 && T > (R)a.ecut) T = (R)a.ecut;
    if (a.mul == MUL_KIN) {
      m.x = T * (R)a.invN;
    } else {  // MUL_PROP: exp(-i T tau) / N
      R sn, cs;
      if constexpr (sizeof(R) == 4) sincosf(T * (R)a.tau, &sn, &cs);
      else sincos(T * (R)a.tau, &sn, &cs);
      m.x = cs * (R)a.invN;
      m.y = -sn * (R)a.invN;
    }
  }
  return m;
}

// y lines of grids whose planes do not fit: columns x0..x0+TX-1 of one xy
// plane, in LDS.
template <typename R, int NLEN, int TX>
__global__ __launch_bounds__(NT_FFT) void k_ypencil(PassArgs a) {
  using C = cplx<R>;
  constexpr int P = TX + 1;
  constexpr int E = NLEN * TX;
  __shared__ C s[NLEN * P];
  __shared__ C tw[NLEN];
  const int tid = threadIdx.x;
  const int nxb = a.nx / TX;
  const int xb = blockIdx.x % nxb;
  const int z = blockIdx.x / nxb;
  const int64_t v = a.rev ? gridDim.y - 1 - blockIdx.y : blockIdx.y;
  const int64_t stride = a.nx;
  C *data = static_cast<C *>(a.dst) + v * a.ld_dst + xb * TX + (int64_t)z * a.nx * a.ny;
  for (int i = tid; i < NLEN; i += NT_FFT) tw[i] = static_cast<const C *>(a.tw0)[i];
#pragma unroll
  for (int q = 0; q < (E + NT_FFT - 1) / NT_FFT; ++q) {
    const int e = tid + q * NT_FFT;
    if (E % NT_FFT == 0 || e < E) {
      C val = data[(e / TX) * stride + (e % TX)];
      if (a.inverse) val = cconj(val);
      s[(e / TX) * P + (e % TX)] = val;
    }
  }
  __syncthreads();
  lds_fft<C, NLEN, TX, 1, P, true, NT_FFT>(s, tw, tid);
#pragma unroll
  for (int q = 0; q < (E + NT_FFT - 1) / NT_FFT; ++q) {
    const int e = tid + q * NT_FFT;
    if (E % NT_FFT == 0 || e < E) {
      C val = s[(e / TX) * P + (e % TX)];
      if (a.inverse) val = cconj(val);
      data[(e / TX) * stride + (e % TX)] = val;
    }
  }
}

// z lines of TX neighbouring columns x0..x0+TX-1: forward transform, k-space
// multiplier, inverse transform, with the points in registers.  The forward
// transform's last stage (radix R2) leaves thread (c, k) the points k + i R1,
// the very ones that a radix-R2 FIRST stage of the inverse needs: where that
// order of the inverse's stages is the usual one (R1 = R2), and in FP64, the
// multiplier and the turn to the inverse need no exchange and the pass has
// two; in FP32 the others take a third one and keep the usual order, whose
// last bits the TDH's response field (a small difference of orbitals)
// amplifies.  (Stages that start and end in LDS take seven.)  Bound by HBM;
// rows of TX complex (256 B and more) matter most.  Forward + inverse of 800
// MB: 40^3 501 -> 237 us, 56^3 652 -> 354, 48^3 404 -> 340, 128^3 394 -> 340,
// FP64 40^3 451 -> 316, FP64 160^3 684 -> 545; 64^3 and 32^3 as before.
template <typename R, int N, int TX> struct PencilShape {
  static constexpr int R1 = Radix<N>::R1, R2 = Radix<N>::R2;
  static constexpr bool D = sizeof(R) == 8;
  // threads for the smaller count of butterflies of a stage, or the larger
  // where that measured faster (FP64 80^3: 455 -> 332 us, FP32 48^3: 386 -> 340)
  static constexpr int LO = R1 < R2 ? R1 : R2, HI = R1 < R2 ? R2 : R1;
  static constexpr int T = (TX * ((D && N <= 80) || N == 48 || N == 24 ? HI : LO) + 63) / 64 * 64;
  static constexpr int P = TX + 1;
  static constexpr bool SPLIT = D && N > 64;
  static constexpr bool TURN = D || R1 == R2;
  // FP32 lines of 96 points round a twiddle product the other way round (see
  // butterfly), at every width: without it the TDH's response field at 96^3
  // moves by 2e-5 to 6e-5 of itself, as accurate and no faster; results
  // recorded with it stay what they are
  static constexpr bool ALT = !D && N == 96;
};

// columns block bx of vector v; s: N P complex (N P values where SPLIT), tw: N
template <typename R, int N, int TX>
__device__ __forceinline__ void pencil_pass(const PassArgs &a, int bx, int64_t v, R *s,
                                            cplx<R> *tw) {
  using C = cplx<R>;
  using Sh = PencilShape<R, N, TX>;
  constexpr int R1 = Radix<N>::R1, R2 = Radix<N>::R2, P = Sh::P, T = Sh::T;
  const int tid = threadIdx.x;
  const int nxb = a.nx / TX;
  const int x0 = (bx % nxb) * TX, y = bx / nxb;
  const int64_t stride = (int64_t)a.nx * a.ny;
  const int64_t base = x0 + (int64_t)y * a.nx;
  // in place on dst, or from src (ld_src) into dst when src is given
  C *data = static_cast<C *>(a.dst) + v * a.ld_dst + base;
  const C *in = a.src ? static_cast<const C *>(a.src) + v * a.ld_src + base : data;
  Stage<C, R1, TX * R2, T> s1;
  Stage<C, R2, TX * R1, T> s2;
  auto col_of = [](int b) { return b / TX; };
  s1.each(tid, [&](int q, int b) {
#pragma unroll
    for (int i = 0; i < R1; ++i) s1.v[q][i] = in[(b / TX + i * R2) * stride + b % TX];
  });
  for (int i = tid; i < N; i += T) tw[i] = static_cast<const C *>(a.tw0)[i];
  s1.template run<N, 1>(tid, tw, col_of);
  exchange<Sh::SPLIT, C>(
      s, tid, s1, s2, true, [](int b, int i) { return ((b / TX) * R1 + i) * P + b % TX; },
      [](int b, int i) { return (b / TX + i * R1) * P + b % TX; });
  s2.template run<N, R1, Sh::ALT>(tid, tw, col_of);
  s2.map(tid, [&](C z, int b, int i) {
    const C m = kmul<R>(a, x0 + b % TX, y, b / TX + i * R1);
    return cmake_r<C>(fma(m.x, z.x, -(m.y * z.y)), -fma(m.y, z.x, m.x * z.y));   // conj(m z)
  });
  if constexpr (Sh::TURN) {
    s2.template run<N, 1>(tid, tw, [](int) { return 0; });
    exchange<Sh::SPLIT, C>(
        s, tid, s2, s1, false, [](int b, int i) { return ((b / TX) * R2 + i) * P + b % TX; },
        [](int b, int i) { return (b / TX + i * R2) * P + b % TX; });
    s1.template run<N, R2>(tid, tw, col_of);
    s1.each(tid, [&](int q, int b) {
#pragma unroll
      for (int i = 0; i < R1; ++i) data[(b / TX + i * R2) * stride + b % TX] = cconj(s1.v[q][i]);
    });
  } else {
    exchange<Sh::SPLIT, C>(
        s, tid, s2, s1, true, [](int b, int i) { return (b / TX + i * R1) * P + b % TX; },
        [](int b, int i) { return (b / TX + i * R2) * P + b % TX; });
    s1.template run<N, 1>(tid, tw, col_of);
    exchange<Sh::SPLIT, C>(
        s, tid, s1, s2, false, [](int b, int i) { return ((b / TX) * R1 + i) * P + b % TX; },
        [](int b, int i) { return (b / TX + i * R1) * P + b % TX; });
    s2.template run<N, R1, Sh::ALT>(tid, tw, col_of);
    s2.each(tid, [&](int q, int b) {
#pragma unroll
      for (int i = 0; i < R2; ++i) data[(b / TX + i * R1) * stride + b % TX] = cconj(s2.v[q][i]);
    });
  }
}

template <typename R, int N, int TX>
__global__ __launch_bounds__((PencilShape<R, N, TX>::T)) void k_pencil(PassArgs a) {
  using Sh = PencilShape<R, N, TX>;
  __shared__ __align__(16) R s[N * Sh::P * (Sh::SPLIT ? 1 : 2)];   // complex unless SPLIT
  __shared__ cplx<R> tw[N];
  pencil_pass<R, N, TX>(a, blockIdx.x, vec_of(a, blockIdx.y, gridDim.y), s, tw);
}

// the z pass with the reduction of the gather's partial sums beside it, as in
// k_plane_gather (workgroups of four waves and more)
template <int N, int TX>
__global__ __launch_bounds__((PencilShape<float, N, TX>::T)) void k_pencil_reduce(
    PassArgs a, KbReduce<float> r, int nvec) {
  using Sh = PencilShape<float, N, TX>;
  constexpr int E = N * Sh::P * (Sh::SPLIT ? 1 : 2);
  __shared__ __align__(16) float s[E > 4 * NTK ? E : 4 * NTK];
  __shared__ float2 tw[N];
  const int nr = r.gx * r.nproj, b = blockIdx.x;
  if (b < nr) {
    if (threadIdx.x < NTK)
      reduce_projector<float>(r, b % r.gx, b / r.gx, reinterpret_cast<double2 *>(s));
    return;
  }
  const int npen = a.nx / TX * a.ny;
  pencil_pass<float, N, TX>(a, (b - nr) % npen, vec_of(a, (b - nr) / npen, nvec), s, tw);
}

// ----------------------------------------------------------------- dispatch
template <int N> constexpr int pencil_tx() { return N % 16 == 0 ? 16 : N % 8 == 0 ? 8 : 4; }
// wider pencils where the length allows them (nx a multiple of the width)
template <typename R, int N> constexpr int pencil_tx_wide() {
  constexpr bool D = sizeof(R) == 8;
  return N % 32 == 0 ? 32 : N == 24 ? 24 : N == 40 ? 40 : N == 48 ? (D ? 24 : 48) : N == 56 ? (D ? 28 : 56)
         : N == 80 ? 40 : pencil_tx<N>();
}
template <int N> constexpr int xlines_nl() { return N >= 2048 ? 1 : 2048 / N; }

// the xy transform of a forward or inverse pass: planes where they fit, else x lines
template <typename R, int N, int MODE> static void launch_xy(dim3 g, hipStream_t st,
                                                             const PassArgs &a) {
  if constexpr (PlaneShape<R, N>::fits)
    hipLaunchKernelGGL((k_plane<R, N, MODE>), g, dim3(PlaneShape<R, N>::T), 0, st, a);
  else
    hipLaunchKernelGGL((k_xlines<R, N, xlines_nl<N>(), MODE>), g, dim3(NT_FFT), 0, st, a);
}
template <typename R, int N, int TX> static void launch_pencil(dim3 g, hipStream_t st,
                                                               const PassArgs &a) {
  hipLaunchKernelGGL((k_pencil<R, N, TX>), g, dim3(PencilShape<R, N, TX>::T), 0, st, a);
}

template <typename R, int N> struct Kernels {
  static void xy(dim3 g, hipStream_t st, const PassArgs &a) {
    switch (a.mode) {
      case PLANE_FWD: launch_xy<R, N, PLANE_FWD>(g, st, a); break;
      case PLANE_INV_STORE: launch_xy<R, N, PLANE_INV_STORE>(g, st, a); break;
      case PLANE_INV_HPSI: launch_xy<R, N, PLANE_INV_HPSI>(g, st, a); break;
      case PLANE_INV_CHEB: launch_xy<R, N, PLANE_INV_CHEB>(g, st, a); break;
      case PLANE_INV_POISSON: launch_xy<R, N, PLANE_INV_POISSON>(g, st, a); break;
      case PLANE_INV_SPLIT: launch_xy<R, N, PLANE_INV_SPLIT>(g, st, a); break;
    }
  }
  static void ypencil(dim3 g, hipStream_t st, const PassArgs &a) {
    if constexpr (!PlaneShape<R, N>::fits)
      hipLaunchKernelGGL((k_ypencil<R, N, pencil_tx<N>()>), g, dim3(NT_FFT), 0, st, a);
  }
  static void pencil(dim3 g, hipStream_t st, const PassArgs &a) {
    launch_pencil<R, N, pencil_tx<N>()>(g, st, a);
  }
  static void pencil_wide(dim3 g, hipStream_t st, const PassArgs &a) {
    launch_pencil<R, N, pencil_tx_wide<R, N>()>(g, st, a);
  }
};

// the passes that carry the projector gather and its reduction (FP32, planes
// and pencils of at least the gather's four waves; not the planes held to a
// register budget, where the gather spills: 128^3, 4 vectors, 30 filter terms
// 6.15 ms against 5.86 with launches of its own)
template <int N> struct RideKernels {
  static constexpr int TX = pencil_tx_wide<float, N>();
  static constexpr bool plane_ok = PlaneShape<float, N>::fits && PlaneShape<float, N>::T >= NTK &&
                                   PlaneShape<float, N>::WPE == 1;
  static constexpr bool pencil_ok = PencilShape<float, N, TX>::T >= NTK;
  static void plane(int nvec, hipStream_t st, const PassArgs &a, const KbGather<float> &g) {
    if constexpr (plane_ok)
      hipLaunchKernelGGL(k_plane_gather<N>, dim3(g.gx * g.gy + a.nz * nvec),
                         dim3(PlaneShape<float, N>::T), 0, st, a, g, nvec);
  }
  static void pencil(int nvec, hipStream_t st, const PassArgs &a, const KbReduce<float> &r) {
    if constexpr (pencil_ok)
      hipLaunchKernelGGL((k_pencil_reduce<N, TX>),
                         dim3(r.gx * r.nproj + a.nx / TX * a.ny * nvec),
                         dim3(PencilShape<float, N, TX>::T), 0, st, a, r, nvec);
  }
};

struct SizeOps {
  void (*xy)(dim3, hipStream_t, const PassArgs &);
  void (*ypencil)(dim3, hipStream_t, const PassArgs &);
  void (*pencil)(dim3, hipStream_t, const PassArgs &);
  void (*pencil_wide)(dim3, hipStream_t, const PassArgs &);
  bool has_plane;
  int tx, nl, tx_wide;
  // with projector work beside them; nullptr where not built
  void (*plane_kb)(int, hipStream_t, const PassArgs &, const KbGather<float> &) = nullptr;
  void (*pencil_kb)(int, hipStream_t, const PassArgs &, const KbReduce<float> &) = nullptr;
};

template <typename R, int N> SizeOps make_ops() {
  using K = Kernels<R, N>;
  SizeOps o{&K::xy, &K::ypencil, &K::pencil, &K::pencil_wide, PlaneShape<R, N>::fits,
            pencil_tx<N>(), xlines_nl<N>(), pencil_tx_wide<R, N>()};
  if constexpr (sizeof(R) == 4 && N % 8 == 0) {      // projector grids
    if (RideKernels<N>::plane_ok) o.plane_kb = &RideKernels<N>::plane;
    if (RideKernels<N>::pencil_ok) o.pencil_kb = &RideKernels<N>::pencil;
  }
  return o;
}

template <typename R> bool get_ops(int n, SizeOps &o) {
  switch (n) {
#define SGW_SIZE(N) case N: o = make_ops<R, N>(); return true;
    SGW_SIZE(8) SGW_SIZE(12) SGW_SIZE(16) SGW_SIZE(24) SGW_SIZE(32) SGW_SIZE(40)
    SGW_SIZE(48) SGW_SIZE(56) SGW_SIZE(64) SGW_SIZE(80) SGW_SIZE(96) SGW_SIZE(112)
    SGW_SIZE(128) SGW_SIZE(160)
#undef SGW_SIZE
    default: return false;
  }
}

bool fft_size_supported(int n, bool dbl) {
  SizeOps o;
  return dbl ? get_ops<double>(n, o) : get_ops<float>(n, o);
}

// The pencil passes launch (nx / width) workgroups per row of columns, the
// width being that of the pencil length: every column is covered only when
// nx is a multiple of the z pencils' width (and of the y pencils', which
// holds whenever nx == ny).
bool fft_pencils_cover(int nx, int ny, int nz, bool dbl) {
  SizeOps oy, oz;
  const bool ok = dbl ? (get_ops<double>(ny, oy) && get_ops<double>(nz, oz))
                      : (get_ops<float>(ny, oy) && get_ops<float>(nz, oz));
  return ok && nx % oz.tx == 0 && nx % oy.tx == 0;
}

bool fft_carries_kb(const sgw_ctx *ctx) {
  SizeOps o;
  return !ctx->dbl && get_ops<float>(ctx->nx, o) && o.plane_kb && ctx->kb_ly == 3 &&
         ctx->kb_lx == (ctx->nx % 16 == 0 ? 4 : 3);
}

template <typename R>
void fft3d_apply_t(sgw_ctx *ctx, const void *src, void *tmp, void *dst, int64_t nvec,
                   int64_t ld, MulMode mul, double tau, PlaneMode inv_mode,
                   const EpiArgs &epi, int64_t ldt, void *tmp2, bool rev,
                   const KbRide *kb) {
  using C = cplx<R>;
  SizeOps ox, oy, oz;
  SGW_REQUIRE(get_ops<R>(ctx->nx, ox) && get_ops<R>(ctx->ny, oy) && get_ops<R>(ctx->nz, oz),
              SGW_EUNSUPPORTED, "grid size not built");
  const int64_t N = ctx->N;
  const C *tw = ctx->d_tw.as<C>();
  const R *k2 = ctx->d_k2.as<R>();
  PassArgs base;
  base.nx = ctx->nx; base.ny = ctx->ny; base.nz = ctx->nz;
  base.N = N;
  base.invN = 1.0 / (double)N;
  base.tau = tau;
  base.ecut = ctx->ecut;
  base.k2x = k2; base.k2y = k2 + ctx->nx; base.k2z = k2 + ctx->nx + ctx->ny;
  base.e = epi;
  const C *twx = tw, *twy = tw + ctx->nx, *twz = tw + ctx->nx + ctx->ny;
  hipStream_t st = ctx->stream;
  const bool use_plane = ox.has_plane;   // nx == ny (sgw_create refuses others)
  for (int64_t v0 = 0; v0 < nvec; v0 += 65535) {
    const int64_t nv = std::min<int64_t>(65535, nvec - v0);
    const C *srcv = static_cast<const C *>(src) + v0 * ld;
    C *tmpv = static_cast<C *>(tmp) + v0 * ldt;
    C *tmp2v = tmp2 ? static_cast<C *>(tmp2) + v0 * ldt : tmpv;   // z pencils' output
    C *dstv = dst ? static_cast<C *>(dst) + v0 * ld : nullptr;
    PassArgs a = base;
    // shift epilogue vector pointers to this chunk
    if (a.e.x) a.e.x = static_cast<const C *>(a.e.x) + v0 * ld;
    if (a.e.vold) a.e.vold = static_cast<C *>(a.e.vold) + v0 * ld;
    if (a.e.vout) a.e.vout = static_cast<C *>(a.e.vout) + v0 * ld;
    if (a.e.acc) a.e.acc = static_cast<C *>(a.e.acc) + v0 * ld;
    if (a.e.vh0) a.e.vh0 = static_cast<const R *>(a.e.vh0) + v0 * N;
    if (a.e.r0) a.e.r0 = static_cast<R *>(a.e.r0) + v0 * N;
    if (a.e.r1) a.e.r1 = static_cast<R *>(a.e.r1) + v0 * N;
    a.ld_x = ld;
    // forward xy
    PassArgs f = a;
    // successive passes run the vectors in alternate directions, each starting
    // on those the pass before wrote last
    int dir = rev ? 1 : 0;
    const dim3 gxy(use_plane ? ctx->nz : (ctx->ny * ctx->nz + ox.nl - 1) / ox.nl, nv);
    f.src = srcv; f.dst = tmpv; f.ld_src = ld; f.ld_dst = ldt; f.mode = PLANE_FWD; f.inverse = 0;
    f.rev = dir;
    f.tw0 = twx;
    if (kb) ox.plane_kb((int)nv, st, f, kb_ride_gather(ctx, *kb, nv));   // one chunk: kb_rides
    else ox.xy(gxy, st, f);
    if (!use_plane) {
      PassArgs py = a;
      py.dst = tmpv; py.ld_dst = ldt; py.tw0 = twy; py.inverse = 0;
      dir ^= 1;
      py.rev = dir;
      oy.ypencil(dim3((ctx->nx / oy.tx) * ctx->nz, nv), st, py);
    }
    SGW_HIP(hipGetLastError());
    // z: forward, multiply, inverse
    PassArgs pz = a;
    pz.dst = tmp2v; pz.ld_dst = ldt; pz.tw0 = twz; pz.mul = mul;
    if (tmp2) { pz.src = tmpv; pz.ld_src = ldt; }
    dir ^= 1;
    pz.rev = dir;
    // z pencils: rows of 32 complex when the lengths allow it (SGW_FORCE_VARIANT
    // pencil=0 keeps rows of 16); every column is the same 1D transform either way
    const auto fp = ctx->forced.find("pencil");
    const bool wide = oz.tx_wide != oz.tx && ctx->nx % oz.tx_wide == 0 &&
                      (fp == ctx->forced.end() || fp->second != 0);
    const bool ride = kb && oz.pencil_kb && (wide || oz.tx_wide == oz.tx);
    if (kb && !ride) kb_launch_reduce(ctx, kb_ride_reduce(ctx, *kb, nv));
    if (ride)
      oz.pencil_kb((int)nv, st, pz, kb_ride_reduce(ctx, *kb, nv));
    else if (wide)
      oz.pencil_wide(dim3((ctx->nx / oz.tx_wide) * ctx->ny, nv), st, pz);
    else
      oz.pencil(dim3((ctx->nx / oz.tx) * ctx->ny, nv), st, pz);
    SGW_HIP(hipGetLastError());
    // inverse xy with the epilogue
    PassArgs b = a;
    b.src = tmp2v; b.ld_src = ldt; b.dst = dstv; b.ld_dst = ld; b.mode = inv_mode; b.inverse = 1;
    const bool timed = (ctx->ktimer & 1) && inv_mode == PLANE_INV_CHEB && ctx->ns.empty();
    if (!use_plane) {
      PassArgs py = a;
      py.dst = tmp2v; py.ld_dst = ldt; py.tw0 = twy; py.inverse = 1;
      dir ^= 1;
      py.rev = dir;
      oy.ypencil(dim3((ctx->nx / oy.tx) * ctx->nz, nv), st, py);
    }
    dir ^= 1;
    b.rev = dir;
    if (timed) SGW_HIP(hipEventRecord(ctx->kt[0].event(0), st));
    b.tw0 = twx;
    ox.xy(gxy, st, b);
    if (timed) {
      SGW_HIP(hipEventRecord(ctx->kt[0].event(1), st));
      ctx->kt[0].used++;
      ctx->kt[0].points += nv * N;
    }
    SGW_HIP(hipGetLastError());
  }
}

void fft3d_apply(sgw_ctx *ctx, const void *src, void *tmp, void *dst, int64_t nvec,
                 int64_t ld, MulMode mul, double tau, PlaneMode inv_mode,
                 const EpiArgs &epi, int64_t ld_tmp, void *tmp2, bool rev, const KbRide *kb) {
  if (nvec <= 0) return;
  const int64_t ldt = ld_tmp > 0 ? ld_tmp : ctx->N;
  if (ctx->dbl)
    fft3d_apply_t<double>(ctx, src, tmp, dst, nvec, ld, mul, tau, inv_mode, epi, ldt, tmp2, rev,
                          kb);
  else
    fft3d_apply_t<float>(ctx, src, tmp, dst, nvec, ld, mul, tau, inv_mode, epi, ldt, tmp2, rev,
                         kb);
}

}  // namespace sgw
