// Register-resident FFT building blocks (forward sign, exp(-2 pi i jk/N)).
//
// A line of length N = R1 R2 is transformed in two Stockham stages.  A thread
// holds whole butterflies in registers: radix-R1 butterfly j reads x[j + i R2]
// and leaves y[j R1 + i]; radix-R2 butterfly k reads y[k + i R1], multiplies
// by exp(-2 pi i i k/N) and leaves X[k + i R1].  LDS only carries the exchange
// between two stages, so a pass touches it once per stage boundary, and the
// first stage loads from and the last one stores to global memory directly.
// R1 is 8 (4 for length 12) and an R2 above 8 is taken as two radices inside
// the thread, in the order and with the twiddles of the separate stages of
// lds_fft: the two transforms round every value alike, bit for bit (but for
// the 96-point z lines, see ALT).
// Inverse transforms are taken as conj(FFT(conj(x))).
#pragma once

#include "fft_lds.h"

namespace sgw {

// the two stages of each built length
template <int N> struct Radix {
  static constexpr int R1 = pick_radix(N), R2 = N / R1;
};

template <typename C> struct DFT<C, 1> {
  static __device__ __forceinline__ void run(C *) {}
};

// Keeps the operations that made z from being contracted with, or moved to,
// those that use it (as a store to LDS and back would).
__device__ __forceinline__ void settle(float2 &z) { asm volatile("" : "+v"(z.x), "+v"(z.y)); }
__device__ __forceinline__ void settle(double2 &z) { asm volatile("" : "+v"(z.x), "+v"(z.y)); }

// a t, and the same with the imaginary part's other product rounded first
template <bool ALT, typename C> __device__ __forceinline__ C twist(C a, C t) {
  C r;
  r.x = fma(a.x, t.x, -(a.y * t.y));
  r.y = ALT ? fma(a.x, t.y, a.y * t.x) : fma(a.y, t.x, a.x * t.y);
  return r;
}

// Radix-R butterfly k of a stage whose sub-transforms have length NS, in
// place: twiddles exp(-2 pi i i k/(NS R)) from the table tw of length N, then
// the transform; for R = A B (A = pick_radix(R)) the stages of radix A and B.
// ALT: the radix-A butterflies after the first round their twiddles the other
// way round (96-point z lines).
template <typename C, int N, int R, int NS, bool ALT = false> __device__ __forceinline__ void butterfly(
    C *a, const C *tw, int k) {
  constexpr int A = pick_radix(R), B = R / A;
  if constexpr (R == 1) {
    return;
  } else if constexpr (B == 1) {
    if (NS > 1) {
#pragma unroll
      for (int i = 1; i < R; ++i) a[i] = twist<false>(a[i], tw[i * k * (N / (NS * R))]);
    }
    DFT<C, R>::run(a);
#pragma unroll
    for (int i = 0; i < R; ++i) settle(a[i]);
  } else {
    C t[B][A];
#pragma unroll
    for (int m = 0; m < B; ++m) {
#pragma unroll
      for (int i = 0; i < A; ++i) {
        t[m][i] = a[m + i * B];
        if (NS > 1 && i > 0) {
          const C z = tw[i * k * (N / (NS * A))];
          t[m][i] = ALT && m > 0 ? twist<true>(t[m][i], z) : twist<false>(t[m][i], z);
        }
      }
      DFT<C, A>::run(t[m]);
#pragma unroll
      for (int i = 0; i < A; ++i) settle(t[m][i]);
    }
#pragma unroll
    for (int i = 0; i < A; ++i) {
      C w[B];
#pragma unroll
      for (int m = 0; m < B; ++m) {
        w[m] = t[m][i];
        if (m > 0) w[m] = twist<false>(w[m], tw[m * (k + NS * i) * (N / (NS * R))]);
      }
      DFT<C, B>::run(w);
#pragma unroll
      for (int m = 0; m < B; ++m) {
        settle(w[m]);
        a[i + A * m] = w[m];
      }
    }
  }
}

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
  // butterfly b is number k_of(b) of its sub-transforms (length NS)
  template <int N, int NS, bool ALT = false, typename K>
  __device__ __forceinline__ void run(int tid, const C *tw, K k_of) {
    each(tid, [&](int q, int b) { butterfly<C, N, R, NS, ALT>(v[q], tw, k_of(b)); });
  }
  // f on every value, settled
  template <typename F> __device__ __forceinline__ void map(int tid, F &&f) {
    each(tid, [&](int q, int b) {
#pragma unroll
      for (int i = 0; i < R; ++i) {
        v[q][i] = f(v[q][i], b, i);
        settle(v[q][i]);
      }
    });
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

}  // namespace sgw
