// Kleinman-Bylander projector contraction (the separable pseudopotential
// part, applied in the paper with atomic adds where neighbouring projector
// spheres overlap, Sec. 3).  Here the work is owned by 512-point grid tiles
// (16 x 8 x 4 where the grid allows it, else 8 x 8 x 8):
//   gather   partial[e][v] = dV sum_{r in tile} beta_e(r) psi_v(r)   per
//            (tile, projector) entry e;
//   reduce   C[p][v] = sum of the partials of projector p, in a fixed order
//            (optionally times E_p);
//   mix      C'[p][v] = sum_q K[p][q] C[q][v]  (dense, for exp(-i tau V_NL));
//   scatter  dst_v(r) += s1 sum_e beta_e(r) C'[p(e)][v] on each tile's own
//            points -- every point is written by exactly one workgroup, so
//            no atomics and bitwise reproducible results.
#include "kb_gather.h"

namespace sgw {

template <typename R>
__global__ __launch_bounds__(NTK) void k_kb_reduce(KbReduce<R> a) {
  __shared__ double2 sh[NTK];
  reduce_projector<R>(a, blockIdx.x, blockIdx.y, sh);
}

template <typename R>
__global__ void k_kb_mix(const cplx<R> *K, const cplx<R> *in, cplx<R> *out, int np,
                         int64_t nvec) {
  const int64_t v = (int64_t)blockIdx.x * NTK + threadIdx.x;
  const int p = blockIdx.y;
  if (v >= nvec) return;
  double sr = 0, si = 0;
  const cplx<R> *k = K + (int64_t)p * np;
  auto add = [&](cplx<R> a, cplx<R> b) {
    sr += (double)a.x * b.x - (double)a.y * b.y;
    si += (double)a.x * b.y + (double)a.y * b.x;
  };
  // the inputs of eight q are requested before they are summed (in order of q)
  int q = 0;
  for (; q + 8 <= np; q += 8) {
    cplx<R> b[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) b[j] = in[(int64_t)(q + j) * nvec + v];
#pragma unroll
    for (int j = 0; j < 8; ++j) add(k[q + j], b[j]);
  }
  for (; q < np; ++q) add(k[q], in[(int64_t)q * nvec + v]);
  out[(int64_t)p * nvec + v] = cmake<cplx<R>>(sr, si);
}

template <class Op, int NVB, int MT, int LX>
__global__ __launch_bounds__(NTK) void k_kb_gather_mma(KbGather<typename Op::T> a) {
  __shared__ __align__(16) float red[4 * MT * (2 * NVB / 16) * 256];   // cross-wave sums
  gather_tile<Op, NVB, MT, LX>(a, blockIdx.x, blockIdx.y, gridDim.y, red);
}

// dst_v(r) += s1 sum_e beta_e(r) C'[p(e)][v] on the points r of tile t (s1 real).
// betaT holds each tile's block transposed, [512 points][nek entries], with the
// entry count nek padded to the K group (16 FP32, 32 BF16; zeros).  The
// coefficient columns sit in dynamic LDS with pitch pe = (largest nek of the
// context) + one 16-byte group, so the LDS a workgroup holds follows the
// projector density of the system, not the 256-entry limit.  A wave
// owns MJ M tiles of 16 points, so a workgroup covers 64 MJ points and a tile
// takes 512 / (64 MJ) workgroups per vector block (fewer registers per wave
// for MJ = 4, more waves per SIMD).  PF (always with one N tile): the old
// destination values are loaded first, so their latency overlaps the
// staging and the products (more registers, fewer waves per SIMD).
template <class Op, int NVB, int MJ, int LX, bool PF>
__device__ __forceinline__ void scatter_mma(
    const float2 *coef, int64_t nvec, const int *tile_base, const int *tile_off,
    const int *tile_offT, const int *entry_proj, const typename Op::T *betaT, float2 *dst,
    int64_t ld, float s1, int nx, int ny, int ntile, int nvb, int pe,
    const uint32_t *tile_mask) {
  using T = typename Op::T;
  constexpr int NC = 2 * NVB, NTL = NC / 16;
  constexpr int EL = 16 / (int)sizeof(T);
  constexpr int NH = KB_TP / (64 * MJ);             // workgroups per tile and vector block
  extern __shared__ __align__(16) unsigned char kb_lds[];
  T *sc = reinterpret_cast<T *>(kb_lds);            // C' [column][entry] (hi, lo), pitch pe
  int t;
  int64_t vbh;
  if (!tile_block(blockIdx.x, ntile, nvb * NH, t, vbh)) return;
  const int64_t vb = vbh / NH;
  const int p0 = (int)(vbh % NH) * 64 * MJ;       // first point of this workgroup
  const int64_t v0 = vb * NVB;
  const int off = tile_off[t], ne = tile_off[t + 1] - off;
  const int offT = tile_offT[t], nek = tile_offT[t + 1] - offT;
  const int base = tile_base[t];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, q = lane >> 4, col = lane & 15;
  // The products are taken transposed, D'[column][point] = sum_e C'[e][column]
  // beta_e(point) (C' from LDS as the A operand, betaT as B): lane l then
  // holds D'[4 (l / 16) + r][l % 16], i.e. the real and imaginary parts of
  // vectors 8 n + 2 (l / 16) (r = 0, 1) and + 1 (r = 2, 3) at point l % 16 of
  // the M tile: two complete complex values, stored without a lane exchange.
  // Lanes of vectors past nvec read the last vector and store nothing.
  const int cg = q;                                 // column group: vectors 2 cg, 2 cg + 1
  int rp[MJ];
#pragma unroll
  for (int j = 0; j < MJ; ++j)
    rp[j] = tile_point_c<LX>(base, p0 + 16 * (MJ * w + j) + col, nx, ny);
  // support bits: M tile j (16 points) with none is skipped by the whole wave
  // (no products, no read or write of psi there: the update is an exact
  // zero).  A live M tile is read and written whole: with 16 x 8 x 4 tiles it
  // is one 128-byte row of each vector, and storing only its supported
  // points would leave partly written cache lines that the next pass over
  // psi pays for.
  uint32_t rowbits[MJ];
  bool live[MJ];
#pragma unroll
  for (int j = 0; j < MJ; ++j) {
    const int pj = p0 + 16 * (MJ * w + j);
    const uint32_t word = __builtin_amdgcn_readfirstlane(
        tile_mask[(int64_t)t * (KB_TP / 32) + (pj >> 5)]);
    rowbits[j] = (word >> (pj & 31)) & 0xffffu;
    live[j] = rowbits[j] != 0u;
  }
  float2 *vrow[NTL][2];
  bool vok[NTL][2];
#pragma unroll
  for (int n = 0; n < NTL; ++n)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int64_t v = v0 + 8 * n + 2 * cg + u;
      vok[n][u] = v < nvec;
      vrow[n][u] = dst + min(v, nvec - 1) * ld;
    }
  // with one N tile, or PF, the old destination values are loaded here, before
  // the staging, so their memory latency overlaps it and the products
  constexpr bool PREFETCH = NTL == 1 || PF;
  float2 o[MJ][NTL][2];
  if constexpr (PREFETCH) {
#pragma unroll
    for (int j = 0; j < MJ; ++j)
#pragma unroll
      for (int n = 0; n < NTL; ++n) {
        o[j][n][0] = live[j] ? vrow[n][0][rp[j]] : make_float2(0.f, 0.f);
        o[j][n][1] = live[j] ? vrow[n][1][rp[j]] : make_float2(0.f, 0.f);
      }
  }
  // betaT rows of this wave's points: the first K group is loaded before the
  // coefficient staging, so its latency overlaps that of the staging loads
  const T *bt =
      betaT + (int64_t)offT * KB_TP + (int64_t)(p0 + 16 * MJ * w + col) * nek + EL * q;
  constexpr int NS = Op::SPLIT ? 2 : 1;            // C' terms (hi, lo)
  u32x4 a_cur[MJ], a_nxt[MJ], b_cur[NS][NTL], b_nxt[NS][NTL];
  if (nek > 0) {
#pragma unroll
    for (int j = 0; j < MJ; ++j) a_cur[j] = ld16(bt + (int64_t)(16 * j) * nek);
  }
  // C' rows of this tile's entries (zero from ne up to nek), four loads in flight
  for (int i0 = 0; i0 < nek * NVB; i0 += 4 * NTK) {
    float2 val[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = i0 + u * NTK + tid, el = idx / NVB, vl = idx % NVB;
      val[u] = make_float2(0.f, 0.f);
      if (el < ne && v0 + vl < nvec) val[u] = coef[(int64_t)entry_proj[off + el] * nvec + v0 + vl];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = i0 + u * NTK + tid, el = idx / NVB, vl = idx % NVB;
      if (el < nek) {
        if constexpr (Op::SPLIT) {
          Op::put1x2(sc + (2 * vl) * pe + el, sc + NC * pe + (2 * vl) * pe + el, val[u].x);
          Op::put1x2(sc + (2 * vl + 1) * pe + el, sc + NC * pe + (2 * vl + 1) * pe + el, val[u].y);
        } else {
          Op::put1(sc + (2 * vl) * pe + el, val[u].x);
          Op::put1(sc + (2 * vl + 1) * pe + el, val[u].y);
        }
      }
    }
  }
  __syncthreads();
  // wave w owns the M tiles (16 points each) MJ w .. MJ w + MJ - 1 from p0
  f32x4 acc[MJ][NTL];
#pragma unroll
  for (int j = 0; j < MJ; ++j)
#pragma unroll
    for (int n = 0; n < NTL; ++n) acc[j][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto load_b = [&](int k0, u32x4 (*b)[NTL]) {
#pragma unroll
    for (int h = 0; h < NS; ++h)
#pragma unroll
      for (int n = 0; n < NTL; ++n)
        b[h][n] = ld16(sc + h * NC * pe + (16 * n + col) * pe + k0 + EL * q);
  };
  auto load_group = [&](int k0, u32x4 *a, u32x4 (*b)[NTL]) {
#pragma unroll
    for (int j = 0; j < MJ; ++j) a[j] = ld16(bt + (int64_t)(16 * j) * nek + k0);
    load_b(k0, b);
  };
  if (nek > 0) load_b(0, b_cur);                  // a_cur holds group 0 already
  for (int k0 = 0; k0 < nek; k0 += Op::GK) {
    if (k0 + Op::GK < nek) load_group(k0 + Op::GK, a_nxt, b_nxt);
#pragma unroll
    for (int j = 0; j < MJ; ++j)
      if (rowbits[j])
#pragma unroll
        for (int n = 0; n < NTL; ++n)
#pragma unroll
          for (int h = 0; h < NS; ++h) Op::mma(acc[j][n], b_cur[h][n], a_cur[j]);
#pragma unroll
    for (int j = 0; j < MJ; ++j) a_cur[j] = a_nxt[j];
#pragma unroll
    for (int h = 0; h < NS; ++h)
#pragma unroll
      for (int n = 0; n < NTL; ++n) b_cur[h][n] = b_nxt[h][n];
  }
  if constexpr (!PREFETCH) {
#pragma unroll
    for (int j = 0; j < MJ; ++j)
#pragma unroll
      for (int n = 0; n < NTL; ++n) {
        o[j][n][0] = live[j] ? vrow[n][0][rp[j]] : make_float2(0.f, 0.f);
        o[j][n][1] = live[j] ? vrow[n][1][rp[j]] : make_float2(0.f, 0.f);
      }
  }
#pragma unroll
  for (int j = 0; j < MJ; ++j)
#pragma unroll
    for (int n = 0; n < NTL; ++n) {
      const f32x4 d = acc[j][n];
      if (live[j] && vok[n][0])
        vrow[n][0][rp[j]] = make_float2(o[j][n][0].x + s1 * d[0], o[j][n][0].y + s1 * d[1]);
      if (live[j] && vok[n][1])
        vrow[n][1][rp[j]] = make_float2(o[j][n][1].x + s1 * d[2], o[j][n][1].y + s1 * d[3]);
    }
}

template <class Op, int NVB, int MJ, int LX, bool PF>
__global__ __launch_bounds__(NTK) void k_kb_scatter_mma(
    const float2 *coef, int64_t nvec, const int *tile_base, const int *tile_off,
    const int *tile_offT, const int *entry_proj, const typename Op::T *betaT, float2 *dst,
    int64_t ld, float s1, int nx, int ny, int ntile, int nvb, int pe,
    const uint32_t *tile_mask) {
  scatter_mma<Op, NVB, MJ, LX, PF>(coef, nvec, tile_base, tile_off, tile_offT, entry_proj, betaT, dst, ld, s1, nx, ny, ntile, nvb, pe, tile_mask);
}

// the same code held to 64 registers per lane, i.e. eight waves per SIMD (the
// accumulators then sit in ordinary vector registers): instantiated for the
// variants of two M tiles per wave, which fit without spilling in FP32 and
// BF16 (the split-BF16 instances spill a few registers; the tuner weighs that)
template <class Op, int NVB, int MJ, int LX, bool PF>
__global__ __launch_bounds__(NTK) __attribute__((amdgpu_waves_per_eu(8, 8))) void
k_kb_scatter_mma_w8(
    const float2 *coef, int64_t nvec, const int *tile_base, const int *tile_off,
    const int *tile_offT, const int *entry_proj, const typename Op::T *betaT, float2 *dst,
    int64_t ld, float s1, int nx, int ny, int ntile, int nvb, int pe,
    const uint32_t *tile_mask) {
  scatter_mma<Op, NVB, MJ, LX, PF>(coef, nvec, tile_base, tile_off, tile_offT, entry_proj, betaT, dst, ld, s1, nx, ny, ntile, nvb, pe, tile_mask);
}

// ---------------------------------------------------------------- FP64
// The same two products in FP64 on v_mfma_f64_16x16x4: lane l supplies A[l %
// 16][l / 16] and B[l / 16][l % 16] and holds D[l / 16 + 4 r][l % 16], r =
// 0..3.  Blocks of 8 vectors (16 real columns).  They are bound by reading
// beta once per vector block and by psi; on the vector ALU the gather's
// cross-lane sums and LDS reads took more time than either.
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int NVB64 = 8;

// As k_kb_gather_mma: a wave's quarter of the tile in 16 K groups of 8 points,
// of which lane (q, col) feeds points 2 q and 2 q + 1, two MFMAs per group;
// column 2 v + part is the real or imaginary part of vector v, the lane pair
// reads one complex value each and swaps halves.  H on 20 vectors of 96^3
// (688 projectors): 265 us on the
// vector ALU, now 94.
template <int MT, int LX>
__global__ __launch_bounds__(NTK) void k_kb_gather_f64(
    const double2 *psi, int64_t ld, int64_t nvec, const int *tile_base, const int *tile_off,
    const double *beta, double2 *partial, int nx, int ny, double dV, int ntile, int nvb,
    const uint32_t *__restrict__ tile_mask) {
  constexpr int NG = 16;
  __shared__ __align__(32) double red[4 * MT * 256];
  int t;
  int64_t vb;
  if (!tile_block(blockIdx.x, ntile, nvb, t, vb)) return;
  const int64_t v0 = vb * NVB64;
  const int base = tile_base[t];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, q = lane >> 4, col = lane & 15;
  const int off = tile_off[t], ne = tile_off[t + 1] - off;
  const int mg0 = blockIdx.y * 16 * MT, mstep = gridDim.y * 16 * MT;
  if (mg0 >= ne) return;
  // bit g: K group g of this wave holds some point of a projector's support
  uint32_t glive = 0;
  const int wu = __builtin_amdgcn_readfirstlane(w);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t word = tile_mask[(int64_t)t * (KB_TP / 32) + 4 * wu + i];
#pragma unroll
    for (int j = 0; j < 4; ++j) glive |= ((word >> (8 * j)) & 0xffu ? 1u : 0u) << (4 * i + j);
  }
  glive = __builtin_amdgcn_readfirstlane(glive);
  auto live = [&](int g) { return (glive >> g) & 1u; };
  const double *bw = beta + 128 * w + 2 * q;
  auto load_a = [&](int mg, int g, double2 *a) {
#pragma unroll
    for (int j = 0; j < MT; ++j) {
      const int e = min(mg + 16 * j + col, ne - 1);   // rows past ne: never stored
      a[j] = *reinterpret_cast<const double2 *>(bw + (int64_t)(off + e) * KB_TP + 8 * g);
    }
  };
  double2 a[2][MT], b[NG];
  if (live(0)) load_a(mg0, 0, a[0]);
  const int od = col & 1;
  const double2 *src = psi + min(v0 + (col >> 1), nvec - 1) * ld + od;
#pragma unroll
  for (int g = 0; g < NG; ++g)
    b[g] = live(g) ? src[tile_point_c<LX>(base, 128 * w + 8 * g + 2 * q, nx, ny)]
                   : make_double2(0, 0);
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    const double got = __shfl_xor(od ? b[g].x : b[g].y, 1, 64);
    b[g] = od ? make_double2(got, b[g].y) : make_double2(b[g].x, got);
  }
  for (int mg = mg0; mg < ne; mg += mstep) {
    f64x4 acc[MT];
#pragma unroll
    for (int j = 0; j < MT; ++j) acc[j] = f64x4{0, 0, 0, 0};
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      if (live((g + 1) % NG)) load_a(g + 1 < NG ? mg : mg + mstep, (g + 1) % NG, a[(g + 1) % 2]);
      if (!live(g)) continue;
#pragma unroll
      for (int j = 0; j < MT; ++j)
        if (mg + 16 * j < ne) {
          acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[g % 2][j].x, b[g].x, acc[j], 0, 0, 0);
          acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[g % 2][j].y, b[g].y, acc[j], 0, 0, 0);
        }
    }
    __syncthreads();                    // the sums of the pass before are read
#pragma unroll
    for (int j = 0; j < MT; ++j)
      *reinterpret_cast<f64x4 *>(red + ((w * MT + j) * 64 + lane) * 4) = acc[j];
    __syncthreads();
    for (int o = tid; o < MT * 16 * NVB64; o += NTK) {
      const int j = o / (16 * NVB64), er = (o / NVB64) % 16, vl = o % NVB64;
      const int e = mg + 16 * j + er, at = (16 * (er & 3) + 2 * vl) * 4 + (er >> 2);
      double re = 0, im = 0;
#pragma unroll
      for (int ww = 0; ww < 4; ++ww) {
        const double *s = red + (ww * MT + j) * 256 + at;
        re += s[0];
        im += s[4];
      }
      if (e < ne && v0 + vl < nvec)
        partial[(int64_t)(off + e) * nvec + v0 + vl] = make_double2(dV * re, dV * im);
    }
  }
}

// dst_v(r) += s1 sum_e beta_e(r) C'[p(e)][v].  A wave owns NP runs of 32 tile
// points: lane column c holds points 2 c and 2 c + 1, one MFMA each per group
// of 4 entries, so beta is read where it lies, 16 bytes a lane, and a lane
// updates two neighbouring complex values.  C' rows are ordered in LDS so that
// the accumulators r = 0, 1 of lane group q are the parts of vector q and r =
// 2, 3 those of vector q + 4.  Runs outside every support are skipped.  Same
// case: 147 us, now 91.
template <int NP, int LX>
__global__ __launch_bounds__(NTK) void k_kb_scatter_f64(
    const double2 *coef, int64_t nvec, const int *tile_base, const int *tile_off,
    const int *entry_proj, const double *beta, double2 *dst, int64_t ld, double s1, int nx,
    int ny, int ntile, int nvb, const uint32_t *tile_mask) {
  constexpr int NH = KB_TP / (128 * NP);            // workgroups per tile and vector block
  extern __shared__ __align__(16) unsigned char kb_lds[];
  double *sc = reinterpret_cast<double *>(kb_lds);  // [entry][16]
  int t;
  int64_t vbh;
  if (!tile_block(blockIdx.x, ntile, nvb * NH, t, vbh)) return;
  const int64_t v0 = vbh / NH * NVB64;
  const int off = tile_off[t], ne = tile_off[t + 1] - off, nek = (ne + 3) / 4 * 4;
  const int base = tile_base[t];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, q = lane >> 4, col = lane & 15;
  const int p0 = (int)(vbh % NH) * 128 * NP + 32 * NP * w;
  bool live[NP];
#pragma unroll
  for (int j = 0; j < NP; ++j)
    live[j] = __builtin_amdgcn_readfirstlane(tile_mask[(int64_t)t * (KB_TP / 32) + p0 / 32 + j]) != 0;
  const double *bt = beta + (int64_t)off * KB_TP + p0 + 2 * col;
  double2 b[2][NP];
  auto load_b = [&](int e0, double2 *x) {
    const double *r = bt + (int64_t)min(e0 + q, ne - 1) * KB_TP;   // past ne: times C' = 0
#pragma unroll
    for (int j = 0; j < NP; ++j)
      if (live[j]) x[j] = *reinterpret_cast<const double2 *>(r + 32 * j);
  };
  load_b(0, b[0]);
  for (int i = tid; i < nek * NVB64; i += NTK) {
    const int el = i / NVB64, vl = i % NVB64;
    double2 c = make_double2(0, 0);
    if (el < ne && v0 + vl < nvec) c = coef[(int64_t)entry_proj[off + el] * nvec + v0 + vl];
    double *d = sc + el * 16 + (vl & 3) + 8 * (vl >> 2);
    d[0] = c.x;
    d[4] = c.y;
  }
  __syncthreads();
  f64x4 acc[NP][2];
#pragma unroll
  for (int j = 0; j < NP; ++j) acc[j][0] = acc[j][1] = f64x4{0, 0, 0, 0};
  auto group = [&](int e0, const double2 *x) {
    const double a = sc[(e0 + q) * 16 + col];
#pragma unroll
    for (int j = 0; j < NP; ++j)
      if (live[j]) {
        acc[j][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, x[j].x, acc[j][0], 0, 0, 0);
        acc[j][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, x[j].y, acc[j][1], 0, 0, 0);
      }
  };
  for (int e0 = 0; e0 < nek; e0 += 8) {
    if (e0 + 4 < nek) load_b(e0 + 4, b[1]);
    group(e0, b[0]);
    if (e0 + 8 < nek) load_b(e0 + 8, b[0]);
    if (e0 + 4 < nek) group(e0 + 4, b[1]);
  }
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    if (!live[j]) continue;
    const int r = tile_point_c<LX>(base, p0 + 32 * j + 2 * col, nx, ny);
    double2 o[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const double2 *d = dst + min(v0 + q + 4 * h, nvec - 1) * ld + r;
      o[h][0] = d[0];
      o[h][1] = d[1];
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t v = v0 + q + 4 * h;
      if (v >= nvec) continue;
      double2 *d = dst + v * ld + r;
#pragma unroll
      for (int u = 0; u < 2; ++u)
        d[u] = make_double2(o[h][u].x + s1 * acc[j][u][2 * h], o[h][u].y + s1 * acc[j][u][2 * h + 1]);
    }
  }
}

// variants (autotuned per context, operand type and batch width)
// (w: the instance held to that many waves per SIMD, 0: the compiler's
// choice; the tuner keeps the first variant within 3 % of the fastest, so a
// held instance comes before its twin)
struct GatherVariant { int nvb, mt; };
static const GatherVariant kGather[] = {{8, 2}, {8, 4}, {16, 2}, {16, 4}};
struct ScatterVariant { int nvb, mj, pf, w; };
static const ScatterVariant kScatter[] = {{8, 8, 0, 0}, {16, 8, 0, 0}, {8, 4, 0, 0},
                                          {16, 4, 0, 0}, {8, 2, 0, 8}, {8, 2, 0, 0},
                                          {16, 2, 0, 8}, {16, 2, 0, 0}, {16, 2, 1, 0}};
constexpr int NGATHER = 4, NSCATTER = 9;

template <class Op>
static void launch_gather_variant(const GatherVariant &v, int lx, hipStream_t st,
                                  const KbGather<typename Op::T> &a) {
  const dim3 g(a.gx, a.gy);
#define SGW_G(A, B, X)                                                                           \
  if (v.nvb == A && v.mt == B && lx == X)                                                        \
    hipLaunchKernelGGL((k_kb_gather_mma<Op, A, B, X>), g, dim3(NTK), 0, st, a);
  SGW_G(8, 2, 4) SGW_G(8, 4, 4) SGW_G(16, 2, 4) SGW_G(16, 4, 4)
  SGW_G(8, 2, 3) SGW_G(8, 4, 3) SGW_G(16, 2, 3) SGW_G(16, 4, 3)
#undef SGW_G
}

template <class Op>
static void launch_scatter_variant(int vi, dim3 g, hipStream_t st, const float2 *coef,
                                   int64_t nvec, const int *tb, const int *to, const int *toT,
                                   const int *ep, const typename Op::T *betaT, float2 *dst,
                                   int64_t ld, float s1, int nx, int ny, int lx, int ntile,
                                   int nvb, int nek_max, const uint32_t *mask) {
  const ScatterVariant v = kScatter[vi];
  constexpr int EL = 16 / (int)sizeof(typename Op::T);
  const int pe = nek_max + EL;
  const size_t lds = (Op::SPLIT ? 2 : 1) * 2 * (size_t)v.nvb * pe * sizeof(typename Op::T);
#define SGW_S(A, B, X, F, W, K)                                                                  \
  if (v.nvb == A && v.mj == B && v.pf == F && v.w == W && lx == X)                               \
    hipLaunchKernelGGL((K<Op, A, B, X, F>), g, dim3(NTK), lds, st, coef, nvec, tb, to, toT, ep, \
                       betaT, dst, ld, s1, nx, ny, ntile, nvb, pe, mask);
  SGW_S(8, 8, 4, 0, 0, k_kb_scatter_mma) SGW_S(16, 8, 4, 0, 0, k_kb_scatter_mma)
  SGW_S(8, 4, 4, 0, 0, k_kb_scatter_mma) SGW_S(16, 4, 4, 0, 0, k_kb_scatter_mma)
  SGW_S(8, 2, 4, 0, 0, k_kb_scatter_mma) SGW_S(16, 2, 4, 0, 0, k_kb_scatter_mma)
  SGW_S(16, 2, 4, 1, 0, k_kb_scatter_mma)
  SGW_S(8, 2, 4, 0, 8, k_kb_scatter_mma_w8) SGW_S(16, 2, 4, 0, 8, k_kb_scatter_mma_w8)
  SGW_S(8, 8, 3, 0, 0, k_kb_scatter_mma) SGW_S(16, 8, 3, 0, 0, k_kb_scatter_mma)
  SGW_S(8, 4, 3, 0, 0, k_kb_scatter_mma) SGW_S(16, 4, 3, 0, 0, k_kb_scatter_mma)
  SGW_S(8, 2, 3, 0, 0, k_kb_scatter_mma) SGW_S(16, 2, 3, 0, 0, k_kb_scatter_mma)
  SGW_S(16, 2, 3, 1, 0, k_kb_scatter_mma)
  SGW_S(8, 2, 3, 0, 8, k_kb_scatter_mma_w8) SGW_S(16, 2, 3, 0, 8, k_kb_scatter_mma_w8)
#undef SGW_S
}

// Operand arrays of the MFMA kernels: beta per entry [entry][512] in the
// operand type (BF16 only; FP32 uses the working-precision copy) and the
// transposed per-tile blocks [512][nek], nek = entries rounded up to the
// scatter's K group.
void kb_upload_operands(sgw_ctx *ctx) {
  const KBHost &kb = ctx->kb;
  auto upload = [](DevBuf &b, const auto *src, size_t n) {
    b.ensure(n * sizeof(*src));
    SGW_HIP(hipMemcpy(b.p, src, n * sizeof(*src), hipMemcpyHostToDevice));
  };
  const int nt = (int)kb.tile_base.size();
  const bool bf = ctx->prec == SGW_C64_BF16KB || ctx->prec == SGW_C64_BF16X2KB;
  const int kg = bf ? OpBF16::GK : OpF32::GK;      // the scatter's K group
  std::vector<int> offT(nt + 1, 0);
  ctx->kb_nek_max = 0;
  for (int t = 0; t < nt; ++t) {
    const int ne = kb.tile_off[t + 1] - kb.tile_off[t];
    offT[t + 1] = offT[t] + (ne + kg - 1) / kg * kg;
    ctx->kb_nek_max = std::max(ctx->kb_nek_max, offT[t + 1] - offT[t]);
  }
  upload(ctx->d_kb_tile_offT, offT.data(), offT.size());
  const size_t nT = (size_t)offT[nt] * KB_TP;
  auto fill_T = [&](auto *out, auto conv) {
    for (int t = 0; t < nt; ++t) {
      const int e0 = kb.tile_off[t], ne = kb.tile_off[t + 1] - e0, nek = offT[t + 1] - offT[t];
      auto *blk = out + (size_t)offT[t] * KB_TP;
      for (int p = 0; p < KB_TP; ++p)
        for (int e = 0; e < ne; ++e) blk[(size_t)p * nek + e] = conv(kb.beta[(size_t)(e0 + e) * KB_TP + p]);
    }
  };
  if (bf) {
    auto conv = [](double v) { return (uint16_t)bf16_bits((float)v); };
    std::vector<uint16_t> t16(nT, 0);
    fill_T(t16.data(), conv);
    upload(ctx->d_kb_betaT, t16.data(), t16.size());
    std::vector<uint16_t> b16(kb.beta.size());
    for (size_t i = 0; i < b16.size(); ++i) b16[i] = conv(kb.beta[i]);
    upload(ctx->d_kb_beta16, b16.data(), b16.size());
  } else {
    std::vector<float> tf(nT, 0.f);
    fill_T(tf.data(), [](double v) { return (float)v; });
    upload(ctx->d_kb_betaT, tf.data(), tf.size());
  }
}

// ---------------------------------------------------------------- launchers
// grid rows over which a gather's passes over entries are split: one pass
// each while there are fewer than four workgroups per CU (40^3, 1 vector:
// 13.5 -> 7.0 us; 64^3, 16 vectors: 24.7 -> 18.5)
static int entry_split(const sgw_ctx *ctx, const dim3 &g, int mt) {
  return g.x < 1024 ? (ctx->kb_ne_max + 16 * mt - 1) / (16 * mt) : 1;
}

// arguments and grid of a gather by blocks of v.nvb vectors
template <typename T>
static KbGather<T> gather_args(const sgw_ctx *ctx, const void *psi, int64_t nvec, int64_t ld,
                               const T *beta, void *partial, const GatherVariant &v) {
  KbGather<T> a;
  a.psi = static_cast<const float2 *>(psi);
  a.ld = ld;
  a.nvec = nvec;
  a.tile_base = ctx->d_kb_tile_base.as<int>();
  a.tile_off = ctx->d_kb_tile_off.as<int>();
  a.beta = beta;
  a.partial = static_cast<float2 *>(partial);
  a.nx = ctx->nx;
  a.ny = ctx->ny;
  a.dV = (float)ctx->dV;
  a.ntile = ctx->kb_ntile;
  a.nvb = (int)((nvec + v.nvb - 1) / v.nvb);
  a.tile_mask = ctx->d_kb_mask.as<uint32_t>();
  const dim3 g = tile_grid(ctx->kb_ntile, a.nvb);
  a.gx = g.x;
  a.gy = entry_split(ctx, g, v.mt);
  return a;
}

template <typename R>
static KbReduce<R> reduce_args(const sgw_ctx *ctx, const void *partial, int64_t nvec, bool use_e,
                               void *out) {
  KbReduce<R> a;
  a.partial = static_cast<const cplx<R> *>(partial);
  a.proj_off = ctx->d_kb_proj_off.as<int>();
  a.proj_entries = ctx->d_kb_proj_entries.as<int>();
  a.ekb = ctx->d_kb_ekb.as<double>();
  a.use_e = use_e ? 1 : 0;
  a.nvec = nvec;
  a.lv = 3;
  while (a.lv < 6 && (int64_t(1) << a.lv) < nvec) ++a.lv;
  a.out = static_cast<cplx<R> *>(out);
  a.gx = (int)((nvec + (1 << a.lv) - 1) >> a.lv);
  a.nproj = ctx->kb.nproj;
  return a;
}

void kb_launch_reduce(sgw_ctx *ctx, const KbReduce<float> &r) {
  hipLaunchKernelGGL(k_kb_reduce<float>, dim3(r.gx, r.nproj), dim3(NTK), 0, ctx->stream, r);
  SGW_HIP(hipGetLastError());
}

int64_t kb_gather_blocks(const sgw_ctx *ctx, int64_t nvec) {
  return 8 * ((ctx->kb_ntile + 7) / 8) * ((nvec + RIDE_NVB - 1) / RIDE_NVB);
}

bool kb_rides(const sgw_ctx *ctx, int64_t nvec, int64_t ld) {
  if (!ctx->has_kb || ctx->prec != SGW_C64 || ld % 2 != 0 || ctx->kb_ntile > 65535) return false;
  if (((ctx->ktimer & 4) && ctx->ns.empty()) || ctx->forced.count("kb_gather")) return false;
  return kb_gather_blocks(ctx, nvec) < 1024 && fft_carries_kb(ctx);
}

static void *partial_buf(sgw_ctx *ctx, int64_t nvec) {
  return ctx->buf("kb_partial", ctx->csize() * (size_t)ctx->kb_nentry * nvec).p;
}

KbGather<float> kb_ride_gather(sgw_ctx *ctx, const KbRide &k, int64_t nvec) {
  return gather_args(ctx, k.psi, nvec, k.ld, ctx->d_kb_beta.as<float>(),
                     k.partial ? k.partial : partial_buf(ctx, nvec),
                     GatherVariant{RIDE_NVB, RIDE_MT});
}

KbReduce<float> kb_ride_reduce(sgw_ctx *ctx, const KbRide &k, int64_t nvec) {
  return reduce_args<float>(ctx, k.partial ? k.partial : partial_buf(ctx, nvec), nvec, true,
                            k.out);
}

template <typename R>
static void gather_t(sgw_ctx *ctx, const void *psi, int64_t nvec, int64_t ld, void *out,
                     bool use_e, void *partial_ext) {
  using C = cplx<R>;
  C *partial = static_cast<C *>(partial_ext ? partial_ext : partial_buf(ctx, nvec));
  SGW_REQUIRE(ctx->kb_ntile <= 65535, SGW_EUNSUPPORTED, "KB gather: too many tiles");
  SGW_REQUIRE(ctx->kb_ly == 3 && (ctx->kb_lx == 3 || ctx->kb_lx == 4), SGW_EUNSUPPORTED,
              "KB tile shape not built");
  if constexpr (sizeof(R) == 4) {
    SGW_REQUIRE(ld % 2 == 0, SGW_EUNSUPPORTED,
                "projectors in complex FP32 need an even leading dimension");
    auto go = [&](auto op, const char *name, const auto *beta) {
      using Op = decltype(op);
      auto run = [&](int vi) {
        launch_gather_variant<Op>(kGather[vi], ctx->kb_lx, ctx->stream,
                                  gather_args(ctx, psi, nvec, ld, beta, partial, kGather[vi]));
      };
      const int vi = ctx->tune(name, nvec, NGATHER, run);   // the gather overwrites: trials are harmless
      const bool timed = (ctx->ktimer & 4) && ctx->ns.empty();
      if (timed) SGW_HIP(hipEventRecord(ctx->kt[2].event(0), ctx->stream));
      run(vi);
      if (timed) {
        SGW_HIP(hipEventRecord(ctx->kt[2].event(1), ctx->stream));
        ctx->kt[2].used++;
        ctx->kt[2].points += (int64_t)ctx->kb_ntile * KB_TP * nvec;
      }
    };
    if (ctx->prec == SGW_C64_BF16KB)
      go(OpBF16{}, "kb_gather_bf16", ctx->d_kb_beta16.as<uint16_t>());
    else if (ctx->prec == SGW_C64_BF16X2KB)
      go(OpBF16x2{}, "kb_gather_bf16x2", ctx->d_kb_beta16.as<uint16_t>());
    else
      go(OpF32{}, "kb_gather", ctx->d_kb_beta.as<float>());
  } else {
    const int64_t nvb = (nvec + NVB64 - 1) / NVB64;
    dim3 g = tile_grid(ctx->kb_ntile, nvb);
    g.y = entry_split(ctx, g, 2);
    const auto k = ctx->kb_lx == 4 ? k_kb_gather_f64<2, 4> : k_kb_gather_f64<2, 3>;
    hipLaunchKernelGGL(k, g, dim3(NTK), 0, ctx->stream, static_cast<const double2 *>(psi), ld,
                       nvec, ctx->d_kb_tile_base.as<int>(), ctx->d_kb_tile_off.as<int>(),
                       ctx->d_kb_beta.as<double>(), reinterpret_cast<double2 *>(partial), ctx->nx,
                       ctx->ny, ctx->dV, ctx->kb_ntile, (int)nvb, ctx->d_kb_mask.as<uint32_t>());
  }
  SGW_HIP(hipGetLastError());
  const KbReduce<R> r = reduce_args<R>(ctx, partial, nvec, use_e, out);
  hipLaunchKernelGGL(k_kb_reduce<R>, dim3(r.gx, r.nproj), dim3(NTK), 0, ctx->stream, r);
  SGW_HIP(hipGetLastError());
}

void kb_gather(sgw_ctx *ctx, const void *psi, int64_t nvec, int64_t ld, void *coef_out) {
  if (ctx->dbl) gather_t<double>(ctx, psi, nvec, ld, coef_out, false, nullptr);
  else gather_t<float>(ctx, psi, nvec, ld, coef_out, false, nullptr);
}

void kb_gather_e(sgw_ctx *ctx, const void *psi, int64_t nvec, int64_t ld, void *coef_out,
                 void *partial) {
  if (ctx->dbl) gather_t<double>(ctx, psi, nvec, ld, coef_out, true, partial);
  else gather_t<float>(ctx, psi, nvec, ld, coef_out, true, partial);
}

size_t kb_partial_bytes_per_vec(const sgw_ctx *ctx) {
  return ctx->csize() * (size_t)ctx->kb_nentry;
}

void kb_mix_dense(sgw_ctx *ctx, const void *K, const void *coef_in, void *coef_out,
                  int64_t nvec) {
  const dim3 g((nvec + NTK - 1) / NTK, ctx->kb.nproj);
  if (ctx->dbl)
    hipLaunchKernelGGL(k_kb_mix<double>, g, dim3(NTK), 0, ctx->stream,
                       static_cast<const double2 *>(K), static_cast<const double2 *>(coef_in),
                       static_cast<double2 *>(coef_out), ctx->kb.nproj, nvec);
  else
    hipLaunchKernelGGL(k_kb_mix<float>, g, dim3(NTK), 0, ctx->stream,
                       static_cast<const float2 *>(K), static_cast<const float2 *>(coef_in),
                       static_cast<float2 *>(coef_out), ctx->kb.nproj, nvec);
  SGW_HIP(hipGetLastError());
}

template <typename R>
static void scatter_t(sgw_ctx *ctx, const void *coef, int64_t nvec, void *dst, int64_t ld,
                      double s1) {
  SGW_REQUIRE(ctx->kb_ntile <= 65535, SGW_EUNSUPPORTED, "KB scatter: too many tiles");
  SGW_REQUIRE(ctx->kb_ly == 3 && (ctx->kb_lx == 3 || ctx->kb_lx == 4), SGW_EUNSUPPORTED,
              "KB tile shape not built");
  if constexpr (sizeof(R) == 4) {
    auto go = [&](auto op, const char *name, const auto *betaT) {
      using Op = decltype(op);
      auto launch = [&](int vi, float s) {
        const ScatterVariant &sv = kScatter[vi];
        const int64_t nvb = (nvec + sv.nvb - 1) / sv.nvb;
        const int64_t nh = KB_TP / (64 * sv.mj);
        launch_scatter_variant<Op>(vi, tile_grid(ctx->kb_ntile, nvb * nh), ctx->stream,
                                   static_cast<const float2 *>(coef), nvec,
                                   ctx->d_kb_tile_base.as<int>(), ctx->d_kb_tile_off.as<int>(),
                                   ctx->d_kb_tile_offT.as<int>(), ctx->d_kb_entry_proj.as<int>(),
                                   betaT, static_cast<float2 *>(dst), ld, s, ctx->nx, ctx->ny,
                                   ctx->kb_lx, ctx->kb_ntile, (int)nvb, ctx->kb_nek_max,
                                   ctx->d_kb_mask.as<uint32_t>());
      };
      // trials add 0 * (B C) to dst, which leaves it unchanged
      const int vi = ctx->tune(name, nvec, NSCATTER, [&](int i) { launch(i, 0.0f); });
      const bool timed = (ctx->ktimer & 2) && ctx->ns.empty();
      if (timed) SGW_HIP(hipEventRecord(ctx->kt[1].event(0), ctx->stream));
      launch(vi, (float)s1);
      if (timed) {
        SGW_HIP(hipEventRecord(ctx->kt[1].event(1), ctx->stream));
        ctx->kt[1].used++;
        ctx->kt[1].points += (int64_t)ctx->kb_ntile * KB_TP * nvec;
      }
    };
    if (ctx->prec == SGW_C64_BF16KB)
      go(OpBF16{}, "kb_scatter_bf16", ctx->d_kb_betaT.as<uint16_t>());
    else if (ctx->prec == SGW_C64_BF16X2KB)
      go(OpBF16x2{}, "kb_scatter_bf16x2", ctx->d_kb_betaT.as<uint16_t>());
    else
      go(OpF32{}, "kb_scatter", ctx->d_kb_betaT.as<float>());
  } else {
    const int64_t nvb = (nvec + NVB64 - 1) / NVB64;
    constexpr int NP = 2, NH = KB_TP / (128 * NP);
    const size_t lds = sizeof(double) * 16 * ((ctx->kb_ne_max + 3) / 4 * 4);
    const auto k = ctx->kb_lx == 4 ? k_kb_scatter_f64<NP, 4> : k_kb_scatter_f64<NP, 3>;
    hipLaunchKernelGGL(k, tile_grid(ctx->kb_ntile, nvb * NH), dim3(NTK), lds, ctx->stream,
                       static_cast<const double2 *>(coef), nvec, ctx->d_kb_tile_base.as<int>(),
                       ctx->d_kb_tile_off.as<int>(), ctx->d_kb_entry_proj.as<int>(),
                       ctx->d_kb_beta.as<double>(), static_cast<double2 *>(dst), ld, s1, ctx->nx,
                       ctx->ny, ctx->kb_ntile, (int)nvb, ctx->d_kb_mask.as<uint32_t>());
  }
  SGW_HIP(hipGetLastError());
}

void kb_scatter(sgw_ctx *ctx, const void *coef, int64_t nvec, void *dst, int64_t ld, double s1) {
  if (ctx->dbl) scatter_t<double>(ctx, coef, nvec, dst, ld, s1);
  else scatter_t<float>(ctx, coef, nvec, dst, ld, s1);
}

}  // namespace sgw
