// Device parts of the projector gather and of its reduction, for the kernels
// of kb.hip and for the FFT passes that carry them along for small batches.
#pragma once
#include "common.h"
#include "kernels.h"

namespace sgw {

constexpr int NTK = 256;

// flat grid index of point p of a tile of x extent 2^LX (y extent 8), in
// 32-bit arithmetic (grids below 2^31 points)
template <int LX>
__device__ __forceinline__ int tile_point_c(int base, int p, int nx, int ny) {
  const int x = p & ((1 << LX) - 1), y = (p >> LX) & 7, z = p >> (LX + 3);
  return base + x + nx * (y + ny * z);
}

// operands of the gather (T: operand type of beta) and of the reduction, and
// the grids they run on
template <typename T> struct KbGather {
  const float2 *psi;
  int64_t ld, nvec;
  const int *tile_base, *tile_off;
  const T *beta;
  float2 *partial;
  int nx, ny;
  float dV;
  int ntile, nvb;
  const uint32_t *tile_mask;
  int gx, gy;
};
template <typename R> struct KbReduce {
  const cplx<R> *partial;
  const int *proj_off, *proj_entries;
  const double *ekb;
  int use_e;
  int64_t nvec;
  int lv;                                // 2^lv vectors a workgroup, 3 to 6
  cplx<R> *out;
  int gx, nproj;
};

// out[p][v] = sum of projector p's partial sums (times E_p), FP64.  The
// entries (some 60 to 90) are dealt to KB_SLOTS sums in turn, which are added
// in a tree: an order of the projector alone, so that a vector's result does
// not depend on how many vectors share its launch.  A workgroup holds 2^LV
// vectors of one projector; its threads of a vector share the slots.  Bound by
// the latency of the entry list and the sums behind it: up to 16 loads of a
// thread are in flight (80^3, 24 vectors beside the FFT passes: 9.8 us, 11.9
// with a loop of loads and an order that followed the batch; with 16 slots one
// or two vectors took 1 % longer in all).
constexpr int KB_SLOTS = 32;

template <int LV, typename R>
__device__ __forceinline__ void reduce_slots(const KbReduce<R> &a, int bx, int p, double2 *sh) {
  constexpr int NP = NTK >> LV, SL = KB_SLOTS / NP;   // threads of a vector, slots of a thread
  static_assert(NP * SL == KB_SLOTS, "the threads of a vector share the slots evenly");
  const int vl = threadIdx.x & ((1 << LV) - 1);
  const int part = LV == 6 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> LV) : threadIdx.x >> LV;
  const int64_t v = ((int64_t)bx << LV) + vl;
  double2 s[SL];
#pragma unroll
  for (int j = 0; j < SL; ++j) s[j] = make_double2(0, 0);
  if (v < a.nvec) {
    // IN rounds of the slots are requested before they are added, those past
    // the last entry (a zero then) at the last
    constexpr int IN = SL < 4 ? 4 : 2;
    const int k1 = a.proj_off[p + 1];
    for (int k = a.proj_off[p] + part; k < k1; k += KB_SLOTS * IN) {
      cplx<R> c[IN][SL];
#pragma unroll
      for (int i = 0; i < IN; ++i)
#pragma unroll
        for (int j = 0; j < SL; ++j) {
          const int e = min(k + KB_SLOTS * i + NP * j, k1 - 1);
          c[i][j] = a.partial[(int64_t)a.proj_entries[e] * a.nvec + v];
        }
#pragma unroll
      for (int i = 0; i < IN; ++i)
#pragma unroll
        for (int j = 0; j < SL; ++j) {
          const bool in = k + KB_SLOTS * i + NP * j < k1;
          s[j].x += in ? c[i][j].x : 0;
          s[j].y += in ? c[i][j].y : 0;
        }
    }
  }
#pragma unroll
  for (int h = SL / 2; h > 0; h >>= 1)
#pragma unroll
    for (int j = 0; j < h; ++j) s[j] = make_double2(s[j].x + s[j + h].x, s[j].y + s[j + h].y);
  sh[threadIdx.x] = s[0];
  for (int h = NP / 2; h > 0; h >>= 1) {
    __syncthreads();
    if (part < h) {
      const double2 x = sh[threadIdx.x], y = sh[threadIdx.x + (h << LV)];
      sh[threadIdx.x] = make_double2(x.x + y.x, x.y + y.y);
    }
  }
  if (part > 0 || v >= a.nvec) return;
  double2 t = sh[threadIdx.x];
  if (a.use_e) { t.x *= a.ekb[p]; t.y *= a.ekb[p]; }
  a.out[(int64_t)p * a.nvec + v] = cmake<cplx<R>>(t.x, t.y);
}

template <typename R>
__device__ __forceinline__ void reduce_projector(const KbReduce<R> &a, int bx, int p, double2 *sh) {
  switch (a.lv) {
    case 3: reduce_slots<3>(a, bx, p, sh); break;
    case 4: reduce_slots<4>(a, bx, p, sh); break;
    case 5: reduce_slots<5>(a, bx, p, sh); break;
    default: reduce_slots<6>(a, bx, p, sh); break;
  }
}

// ---------------------------------------------------------------- MFMA
// Per tile the gather is the GEMM  D[e][c] = sum_p beta[e][p] Psi[p][c]
// (M = projector entries, K = 512 points, N = 2 NVB real columns = NVB
// complex vectors) and the scatter  D[p][c] = sum_e beta[e][p] C'[e][c]
// (M = 512 points, K = entries padded to the K group).  The operands are stored in
// FP32 (SGW_C64) or in BF16 rounded to nearest even (SGW_C64_BF16KB; with
// SGW_C64_BF16X2KB the psi / coefficient operand as two BF16 terms); the
// accumulation is FP32 either way.  A lane feeds 16 contiguous bytes of A and
// of B per group of K values:
//   FP32: four v_mfma_f32_16x16x4f32, K group 16, lane l holds the K slots
//         4 (l / 16) + s, s = 0..3, one per instruction;
//   BF16: one v_mfma_f32_16x16x32_bf16, K group 32, lane l holds the K slots
//         8 (l / 16) + s, s = 0..7;
// lane l supplies row l % 16 of A and column l % 16 of B and receives
// D[4 (l / 16) + r][l % 16] in accumulator register r.  Every variant below
// (vectors per workgroup NVB, entry tiles per pass MT) computes each output
// with the same instructions in the same order, so the choice changes the
// speed, not a bit of the result.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// float -> bfloat16 bits, round to nearest even (finite inputs)
__host__ __device__ __forceinline__ uint32_t bf16_bits(float f) {
  uint32_t u;
  __builtin_memcpy(&u, &f, 4);
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

struct OpF32 {
  using T = float;
  static constexpr int GK = 16;
  static constexpr bool SPLIT = false;
  __device__ static void mma(f32x4 &acc, const u32x4 &a, const u32x4 &b) {
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[0]), __uint_as_float(b[0]), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[1]), __uint_as_float(b[1]), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[2]), __uint_as_float(b[2]), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[3]), __uint_as_float(b[3]), acc, 0, 0, 0);
  }
  __device__ static void put2(T *d, float x, float y) {
    *reinterpret_cast<float2 *>(d) = make_float2(x, y);
  }
  __device__ static u32x4 pack(const float *e) {      // 4 values -> one operand
    return u32x4{__float_as_uint(e[0]), __float_as_uint(e[1]), __float_as_uint(e[2]),
                 __float_as_uint(e[3])};
  }
  __device__ static void put1(T *d, float x) { *d = x; }
};

struct OpBF16 {
  using T = uint16_t;
  static constexpr int GK = 32;
  static constexpr bool SPLIT = false;
  __device__ static void mma(f32x4 &acc, const u32x4 &a, const u32x4 &b) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                  __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
  }
  __device__ static void put2(T *d, float x, float y) {
    *reinterpret_cast<uint32_t *>(d) = bf16_bits(x) | (bf16_bits(y) << 16);
  }
  __device__ static void put1(T *d, float x) { *d = (uint16_t)bf16_bits(x); }
  __device__ static u32x4 pack(const float *e) {      // 8 values -> one operand (RNE)
    return u32x4{bf16_bits(e[0]) | (bf16_bits(e[1]) << 16), bf16_bits(e[2]) | (bf16_bits(e[3]) << 16),
                 bf16_bits(e[4]) | (bf16_bits(e[5]) << 16), bf16_bits(e[6]) | (bf16_bits(e[7]) << 16)};
  }
};

__device__ __forceinline__ float bf16_value(uint32_t b) { return __uint_as_float(b << 16); }

// BF16 products with the state-vector operand (psi in the gather, the mixed
// coefficients in the scatter) carried as two BF16 terms hi + lo, hi = RNE(x),
// lo = RNE(x - hi): two MFMAs per operand pair, the split operand exact to
// about 2^-17; beta stays one BF16 term.
struct OpBF16x2 : OpBF16 {
  static constexpr bool SPLIT = true;
  __device__ static void pack2(const float *e, u32x4 &hi, u32x4 &lo) {
    uint32_t h[8], l[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      h[i] = bf16_bits(e[i]);
      l[i] = bf16_bits(e[i] - bf16_value(h[i]));
    }
    hi = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
    lo = u32x4{l[0] | (l[1] << 16), l[2] | (l[3] << 16), l[4] | (l[5] << 16), l[6] | (l[7] << 16)};
  }
  __device__ static void put1x2(T *dhi, T *dlo, float x) {
    const uint32_t h = bf16_bits(x);
    *dhi = (uint16_t)h;
    *dlo = (uint16_t)bf16_bits(x - bf16_value(h));
  }
};

// Workgroup -> (tile, vector block).  Consecutive workgroups go to the 8
// XCDs in turn, so tile t is given to workgroups on XCD t % 8 only, and one
// XCD walks all vector blocks of a tile in a row: the tile's beta rows are
// read from memory once per XCD L2 instead of once per workgroup.
__device__ __forceinline__ bool tile_block(int b, int ntile, int nvb, int &t, int64_t &vb) {
  const int xcd = b & 7, i = b >> 3;
  t = xcd + 8 * (i / nvb);
  vb = i % nvb;
  return t < ntile;
}

inline dim3 tile_grid(int ntile, int64_t nvb) {
  return dim3((unsigned)(8 * ((ntile + 7) / 8) * nvb));
}

template <class T> __device__ __forceinline__ u32x4 ld16(const T *p) {
  return *reinterpret_cast<const u32x4 *>(p);
}

// partial[off + e][v] = dV sum_p beta_e(p) psi_v(p) for the entries e of tile t.
// The B operand of lane (q, col) in K group g is EL consecutive tile points
// (consecutive x, so EL consecutive complex values in memory) of the real
// (col even) or imaginary (col odd) part of vector v0 + 8 n + col / 2: the
// lane reads them straight from memory (lanes col and col ^ 1 read the same
// bytes in the same instruction) -- no staging in LDS.  The tile's x extent
// is 2^LX (y 8).  Lanes of vectors past nvec read the last vector and entry
// rows past ne the last row: both only feed outputs that are never written,
// so the loads need no branch.
template <class Op, int NVB, int MT, int LX>
__device__ __forceinline__ void gather_tile(const KbGather<typename Op::T> &a0, int bx, int by,
                                            int gy, float *red) {
  const float2 *psi = a0.psi;
  const int64_t ld = a0.ld, nvec = a0.nvec;
  const int *tile_base = a0.tile_base, *tile_off = a0.tile_off;
  const typename Op::T *beta = a0.beta;
  float2 *partial = a0.partial;
  const int nx = a0.nx, ny = a0.ny;
  const float dV = a0.dV;
  const uint32_t *__restrict__ tile_mask = a0.tile_mask;
  using T = typename Op::T;
  constexpr int NC = 2 * NVB, NTL = NC / 16;
  constexpr int EL = 16 / (int)sizeof(T);           // operand elements per lane per group
  constexpr int NG = 128 / Op::GK;                  // K groups of one wave (128 points)
  static_assert(Op::GK == 16 || Op::GK == 32, "K group of 16 or 32 points");
  constexpr int NS = Op::SPLIT ? NG : 1, NSN = Op::SPLIT ? NTL : 1;
  int t;
  int64_t vb;
  if (!tile_block(bx, a0.ntile, a0.nvb, t, vb)) return;
  const int64_t v0 = vb * NVB;
  const int base = tile_base[t];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, q = lane >> 4, col = lane & 15;
  const int off = tile_off[t], ne = tile_off[t + 1] - off;
  // the passes over the tile's entries are split over gy workgroups
  // where there are too few vectors to fill the device
  const int mg0 = by * 16 * MT, mstep = gy * 16 * MT;
  if (mg0 >= ne) return;
  // bit g of glive: some point of this wave's K group g (GK consecutive tile
  // points) lies in a projector's support.  A group without one holds only
  // zero beta values: its psi values are not loaded and its products (exact
  // zeros) are not taken.  The condition is uniform over the wave.
  uint32_t glive = 0;
  const int wu = __builtin_amdgcn_readfirstlane(w);   // scalar loads of the four words
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t word = tile_mask[(int64_t)t * (KB_TP / 32) + 4 * wu + i];
    if constexpr (Op::GK == 16)
      glive |= ((word & 0xffffu) ? 1u : 0u) << (2 * i) | ((word >> 16) ? 1u : 0u) << (2 * i + 1);
    else
      glive |= (word ? 1u : 0u) << i;
  }
  glive = __builtin_amdgcn_readfirstlane(glive);
  auto live = [&](int g) { return (glive >> g) & 1u; };
  // B operands of this wave's quarter of K, kept in registers for all entries:
  // every load of a live group is issued first, the lane exchanges follow
  auto load_b = [&](int64_t v0, u32x4 (*b)[NTL], u32x4 (*blo)[NSN]) {
    constexpr int NZ = EL / 4;
    float4 z[NG][NTL][NZ];
    // the lane pair (col, col ^ 1) reads each group of 4 complex values once:
    // the even lane points 0, 1 and the odd lane points 2, 3
    const int od = col & 1;
#pragma unroll
    for (int n = 0; n < NTL; ++n) {
      const int64_t v = min(v0 + 8 * n + (col >> 1), nvec - 1);
      const float2 *src = psi + v * ld;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const int p = 128 * w + g * Op::GK + EL * q;  // EL consecutive points along x
        const float4 *s4 = reinterpret_cast<const float4 *>(src + tile_point_c<LX>(base, p, nx, ny));
#pragma unroll
        for (int i = 0; i < NZ; ++i) z[g][n][i] = live(g) ? s4[2 * i + od] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
    // then they swap the parts the other needs (real parts to the even lane,
    // imaginary parts to the odd lane)
#pragma unroll
    for (int n = 0; n < NTL; ++n)
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        float e[EL];
#pragma unroll
        for (int i = 0; i < NZ; ++i) {
          const float4 zz = z[g][n][i];
          const float g0 = __shfl_xor(od ? zz.x : zz.y, 1, 64);
          const float g1 = __shfl_xor(od ? zz.z : zz.w, 1, 64);
          e[4 * i] = od ? g0 : zz.x;
          e[4 * i + 1] = od ? g1 : zz.z;
          e[4 * i + 2] = od ? zz.y : g0;
          e[4 * i + 3] = od ? zz.w : g1;
        }
        if constexpr (Op::SPLIT) Op::pack2(e, b[g][n], blo[g][n]);
        else b[g][n] = Op::pack(e);
      }
  };
  // A operands (beta rows of MT entry tiles, one K group) alternate between
  // two register sets: group g + 1 is requested before the products of group
  // g (after the last group, the next pass's first one), so one group's loads
  // are in flight behind the products (three in flight, with a ring of four,
  // cost a wave per SIMD in registers and ran 5 % slower).  Entry rows past
  // ne read row ne - 1: in bounds, and their products are never stored.
  constexpr int D = 1, RA = 2;
  static_assert(NG % RA == 0, "the A operands alternate with the K groups");
  auto load_a = [&](int mg, int g, u32x4 *a) {
#pragma unroll
    for (int j = 0; j < MT; ++j) {
      const int e = min(mg + 16 * j + col, ne - 1);   // A row = lane % 16
      a[j] = ld16(beta + (int64_t)(off + e) * KB_TP + 128 * w + g * Op::GK + EL * q);
    }
  };
  u32x4 a[RA][MT];
#pragma unroll
  for (int g = 0; g < D; ++g)
    if (live(g)) load_a(mg0, g, a[g]);
  u32x4 b[NG][NTL], blo[NS][NSN];
  load_b(v0, b, blo);
  for (int mg = mg0; mg < ne; mg += mstep) {
    f32x4 acc[MT][NTL];
#pragma unroll
    for (int j = 0; j < MT; ++j)
#pragma unroll
      for (int n = 0; n < NTL; ++n) acc[j][n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      if (live((g + D) % NG)) load_a(g + D < NG ? mg : mg + mstep, (g + D) % NG, a[(g + D) % RA]);
      if (!live(g)) continue;
#pragma unroll
      for (int j = 0; j < MT; ++j)
        if (mg + 16 * j < ne)
#pragma unroll
          for (int n = 0; n < NTL; ++n) {
            Op::mma(acc[j][n], a[g % RA][j], b[g][n]);
            if constexpr (Op::SPLIT) Op::mma(acc[j][n], a[g % RA][j], blo[g][n]);
          }
    }
    // a barrier between the last products and the LDS writes of their
    // accumulators (without it the <8, 2> instantiation read some
    // accumulators before their last product had landed)
    __syncthreads();
#pragma unroll
    for (int j = 0; j < MT; ++j)
#pragma unroll
      for (int n = 0; n < NTL; ++n)
        *reinterpret_cast<f32x4 *>(red + (((w * MT + j) * NTL + n) * 64 + lane) * 4) = acc[j][n];
    __syncthreads();
    // the four K quarters summed in wave order; one complex (entry, vector) per item
    for (int o = tid; o < MT * 16 * NVB; o += NTK) {
      const int j = o / (16 * NVB), er = (o / NVB) % 16, vl = o % NVB;
      const int e = mg + 16 * j + er;
      const int n = vl >> 3, lre = 16 * (er >> 2) + 2 * (vl & 7), r = er & 3;
      float re = 0.f, im = 0.f;
#pragma unroll
      for (int ww = 0; ww < 4; ++ww) {
        const float *s = red + (((ww * MT + j) * NTL + n) * 64) * 4;
        re += s[lre * 4 + r];
        im += s[(lre + 1) * 4 + r];
      }
      if (e < ne && v0 + vl < nvec)
        partial[(int64_t)(off + e) * nvec + v0 + vl] = make_float2(dV * re, dV * im);
    }
    __syncthreads();
  }
}

// gather by blocks of 8 vectors and passes of 32 entries on 16 x 8 x 4 or 8^3
// tiles (FP32 operands), and its reduction with E_p, as parts of the FFT
// passes of the same product
constexpr int RIDE_NVB = 8, RIDE_MT = 2;
constexpr int RIDE_LDS = 4 * RIDE_MT * (2 * RIDE_NVB / 16) * 256;   // floats
KbGather<float> kb_ride_gather(sgw_ctx *ctx, const KbRide &k, int64_t nvec);
KbReduce<float> kb_ride_reduce(sgw_ctx *ctx, const KbRide &k, int64_t nvec);
void kb_launch_reduce(sgw_ctx *ctx, const KbReduce<float> &r);

}  // namespace sgw
