// Register-resident FFT building blocks (forward sign, exp(-2 pi i jk/N)).
//
// A line of length N = R1 R2 is transformed in two Stockham stages.  A thread
// holds whole butterflies in registers: radix-R1 butterfly j reads x[j + i R2]
// and leaves y[j R1 + i]; radix-R2 butterfly k reads y[k + i R1], multiplies
// by exp(-2 pi i i k/N) and leaves X[k + i R1].  LDS only carries the exchange
// between two stages, so a pass touches it once per stage boundary, and the
// first stage loads from and the last one stores to global memory directly.
// Inverse transforms are taken as conj(FFT(conj(x))).
#pragma once

#include <type_traits>

#include "fft_lds.h"

namespace sgw {

// the two radices of each built length
template <int N> struct Radix {
  static constexpr int R1 = N == 8 ? 4 : N == 12 ? 4 : N == 16 ? 4 : N == 24 ? 6 : N == 32 ? 8
                          : N == 40 ? 8 : N == 48 ? 8 : N == 56 ? 8 : N == 64 ? 8 : N == 80 ? 16
                          : N == 96 ? 12 : N == 112 ? 14 : 16;
  static constexpr int R2 = N / R1;
  static_assert(R1 * R2 == N && R2 >= 2 && R2 <= R1, "length not built");
};

template <int I, int N, typename F> __device__ __forceinline__ void static_for(F &&f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// cos and sin of 2 pi m / R at compile time: reduced to at most pi / 4, then
// the Taylor series
constexpr double taylor_cos(double x) {
  double s = 0, t = 1;
  for (int k = 1; k < 12; ++k) {
    s += t;
    t *= -x * x / ((2 * k - 1) * (2 * k));
  }
  return s;
}
constexpr double taylor_sin(double x) {
  double s = 0, t = x;
  for (int k = 1; k < 12; ++k) {
    s += t;
    t *= -x * x / ((2 * k) * (2 * k + 1));
  }
  return s;
}
constexpr double kTwoPi = 6.283185307179586476925286766559;
constexpr double turn_cos(int m, int R);
constexpr double turn_sin(int m, int R) {    // 0 <= m < R
  return 2 * m > R ? -turn_sin(R - m, R)
       : 4 * m > R ? (8 * m > 3 * R ? taylor_sin(kTwoPi * (R - 2 * m) / (2.0 * R))
                                    : taylor_cos(kTwoPi * (4 * m - R) / (4.0 * R)))
       : 8 * m > R ? taylor_cos(kTwoPi * (R - 4 * m) / (4.0 * R))
                   : taylor_sin(kTwoPi * m / R);
}
constexpr double turn_cos(int m, int R) {
  return 2 * m > R ? turn_cos(R - m, R)
       : 4 * m > R ? (8 * m > 3 * R ? -taylor_cos(kTwoPi * (R - 2 * m) / (2.0 * R))
                                    : -taylor_sin(kTwoPi * (4 * m - R) / (4.0 * R)))
       : 8 * m > R ? taylor_sin(kTwoPi * (R - 4 * m) / (4.0 * R))
                   : taylor_cos(kTwoPi * m / R);
}

// z exp(-2 pi i M / R)
template <int M, int R, typename C> __device__ __forceinline__ C turn(C z) {
  using T = decltype(z.x);
  if constexpr (M == 0) {
    return z;
  } else if constexpr (4 * M == R) {
    return mul_mi(z);
  } else {
    constexpr T c = (T)turn_cos(M, R), s = (T)turn_sin(M, R);
    C r;
    r.x = c * z.x + s * z.y;
    r.y = c * z.y - s * z.x;
    return r;
  }
}

// radix A B from radices A and B: n = n1 B + n2, k = k1 + A k2
template <typename C, int A, int B> struct DFTprod {
  static __device__ __forceinline__ void run(C *a) {
    C t[B][A];
    static_for<0, B>([&](auto n2) {
#pragma unroll
      for (int n1 = 0; n1 < A; ++n1) t[n2][n1] = a[n1 * B + n2];
      DFT<C, A>::run(t[n2]);
      static_for<0, A>([&](auto k1) {
        t[n2][k1] = turn<(int)n2 * (int)k1 % (A * B), A * B>(t[n2][k1]);
      });
    });
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
      C w[B];
#pragma unroll
      for (int n2 = 0; n2 < B; ++n2) w[n2] = t[n2][k1];
      DFT<C, B>::run(w);
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2) a[k1 + A * k2] = w[k2];
    }
  }
};
template <typename C> struct DFT<C, 6> : DFTprod<C, 3, 2> {};
template <typename C> struct DFT<C, 10> : DFTprod<C, 5, 2> {};
template <typename C> struct DFT<C, 12> : DFTprod<C, 4, 3> {};
template <typename C> struct DFT<C, 14> : DFTprod<C, 7, 2> {};
template <typename C> struct DFT<C, 16> : DFTprod<C, 4, 4> {};

// The butterflies of one stage over a workgroup: NB butterflies of radix R,
// butterfly b = tid + q T in slot q.
template <typename C, int R_, int NB_, int T_> struct Stage {
  static constexpr int R = R_, NB = NB_, T = T_, Q = (NB_ + T_ - 1) / T_;
  C v[Q][R];
  // f(q, b) for every butterfly of this thread
  template <typename F> static __device__ __forceinline__ void each(int tid, F &&f) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int b = tid + q * T;
      if (NB % T == 0 || b < NB) f(q, b);
    }
  }
  __device__ __forceinline__ void dft(int tid) {
    each(tid, [&](int q, int) { DFT<C, R>::run(v[q]); });
  }
};

// a's values to LDS at index wi(b, i), barrier, b's from ri(b, i).  SPLIT
// sends real and imaginary parts one after the other through half the LDS.
// `more`: another exchange follows (barrier at the end).
template <bool SPLIT, typename C, typename SA, typename SB, typename W, typename Rd>
__device__ __forceinline__ void exchange(void *lds, int tid, SA &a, SB &b, bool more, W wi,
                                         Rd ri) {
  using T = decltype(a.v[0][0].x);
  if constexpr (SPLIT) {
    T *s = static_cast<T *>(lds);
    SA::each(tid, [&](int q, int j) {
#pragma unroll
      for (int i = 0; i < SA::R; ++i) s[wi(j, i)] = a.v[q][i].x;
    });
    __syncthreads();
    SB::each(tid, [&](int q, int j) {
#pragma unroll
      for (int i = 0; i < SB::R; ++i) b.v[q][i].x = s[ri(j, i)];
    });
    __syncthreads();
    SA::each(tid, [&](int q, int j) {
#pragma unroll
      for (int i = 0; i < SA::R; ++i) s[wi(j, i)] = a.v[q][i].y;
    });
    __syncthreads();
    SB::each(tid, [&](int q, int j) {
#pragma unroll
      for (int i = 0; i < SB::R; ++i) b.v[q][i].y = s[ri(j, i)];
    });
  } else {
    C *s = static_cast<C *>(lds);
    SA::each(tid, [&](int q, int j) {
#pragma unroll
      for (int i = 0; i < SA::R; ++i) s[wi(j, i)] = a.v[q][i];
    });
    __syncthreads();
    SB::each(tid, [&](int q, int j) {
#pragma unroll
      for (int i = 0; i < SB::R; ++i) b.v[q][i] = s[ri(j, i)];
    });
  }
  if (more) __syncthreads();
}

// twiddles exp(-2 pi i i k / N) of radix butterflies whose k is k_of(b)
template <typename C, typename S, typename K>
__device__ __forceinline__ void twiddle(S &a, const C *tw, int tid, K k_of) {
  S::each(tid, [&](int q, int b) {
    const int k = k_of(b);
#pragma unroll
    for (int i = 1; i < S::R; ++i) a.v[q][i] = cmul(a.v[q][i], tw[i * k]);
  });
}

}  // namespace sgw
