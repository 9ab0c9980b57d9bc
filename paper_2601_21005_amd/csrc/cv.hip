// Learned control variate for the per-sample self-energy: features of the
// white-noise vectors, a 64 -> 256 -> 256 -> 1 tanh network trained with
// Adam, and the cheap-sample mean of the network's output.  An addition to
// the paper's Monte Carlo average (Sec. 3 averages samples until the QP
// error bar is below 0.03 eV): the control variate lowers the spread of the
// per-sample values without bias when the mean of g is known well.
//
// Every product runs on MFMA with BF16 operands (nearest-even rounding) and
// FP32 accumulation; elementwise work is FP32, sums over samples FP64.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "common.h"
#include "rng.h"

using namespace sgw;

struct sgw_mlp {
  int din = 0, h1 = 0, h2 = 0;
  int64_t nparam = 0;
  hipStream_t stream = nullptr;
  std::string err;
  DevBuf theta, m, v, grad;            // FP32 master parameters, Adam moments, gradient
  DevBuf mean, inv_std;                // standardization of the features (FP32)
  int64_t t = 0;                       // Adam step count
  std::map<std::string, std::unique_ptr<DevBuf>> scratch;
  DevBuf &buf(const std::string &name, size_t bytes) {
    auto &p = scratch[name];
    if (!p) p.reset(new DevBuf());
    p->ensure(bytes);
    return *p;
  }
  // offsets of the parameter blocks in the packed vector
  int64_t oW1() const { return 0; }
  int64_t ob1() const { return (int64_t)h1 * din; }
  int64_t oW2() const { return ob1() + h1; }
  int64_t ob2() const { return oW2() + (int64_t)h2 * h1; }
  int64_t ow3() const { return ob2() + h2; }
  int64_t ob3() const { return ow3() + h2; }
};

namespace {

thread_local std::string g_mlp_error;

template <typename F> sgw_status guard_mlp(sgw_mlp *m, F &&f) {
  try {
    f();
    return SGW_OK;
  } catch (const Error &e) {
    (m ? m->err : g_mlp_error) = e.msg;
    return e.code;
  } catch (const std::bad_alloc &) {
    (m ? m->err : g_mlp_error) = "host allocation failed";
    return SGW_ENOMEM;
  } catch (const std::exception &e) {
    (m ? m->err : g_mlp_error) = e.what();
    return SGW_EINVAL;
  }
}

template <typename F> sgw_status guard_ctx(sgw_ctx *c, F &&f) {
  try {
    f();
    return SGW_OK;
  } catch (const Error &e) {
    c->err = e.msg;
    return e.code;
  } catch (const std::bad_alloc &) {
    c->err = "host allocation failed";
    return SGW_ENOMEM;
  } catch (const std::exception &e) {
    c->err = e.what();
    return SGW_EINVAL;
  }
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// float -> bfloat16 bits, round to nearest even (finite inputs)
__device__ __forceinline__ uint32_t bf16r(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// D += A B on v_mfma_f32_16x16x32_bf16: lane l supplies A[l % 16][8 (l / 16) + s]
// and B[8 (l / 16) + s][l % 16], s = 0..7, and holds D[4 (l / 16) + r][l % 16]
__device__ __forceinline__ void mma(f32x4 &acc, const u32x4 &a, const u32x4 &b) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}

constexpr int NT = 256;

// ---------------------------------------------------------------- features
// phi (FP32 [K][ld]) -> BF16 [rows][N], rows K.. zero, in the order in which
// the feature GEMM takes the points: K slot 8 q + 2 j + h of a 32-point group
// holds point 4 q + j + 16 h, so that the two points of a packed BF16 pair
// have their sign bits 16 apart in the group's 32 random bits.  One thread
// per 8 slots of a row.
__global__ __launch_bounds__(256) void k_phi_bf16(const float *phi, int64_t ld, int K, int64_t N,
                                                  int vec, uint16_t *out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int k = blockIdx.y;
  if (8 * i >= N) return;
  float lo[4] = {0.f, 0.f, 0.f, 0.f}, hi[4] = {0.f, 0.f, 0.f, 0.f};
  if (k < K) {
    const float *p = phi + k * ld + (i >> 2) * 32 + 4 * (i & 3);
    if (vec) {
      const float4 a = *reinterpret_cast<const float4 *>(p);
      const float4 b = *reinterpret_cast<const float4 *>(p + 16);
      lo[0] = a.x; lo[1] = a.y; lo[2] = a.z; lo[3] = a.w;
      hi[0] = b.x; hi[1] = b.y; hi[2] = b.z; hi[3] = b.w;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        lo[j] = p[j];
        hi[j] = p[16 + j];
      }
    }
  }
  u32x4 o;
#pragma unroll
  for (int j = 0; j < 4; ++j) o[j] = bf16r(lo[j]) | bf16r(hi[j]) << 16;
  *reinterpret_cast<u32x4 *>(out + k * N + 8 * i) = o;
}

// rows[t] = the value that lane (16 t + lane % 16) holds, t = 0..3
__device__ __forceinline__ void spread_rows(uint32_t v, uint32_t *rows) {
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);   // rows 0022, 1133
  const auto e = __builtin_amdgcn_permlane32_swap(a[0], a[0], false, false);
  const auto o = __builtin_amdgcn_permlane32_swap(a[1], a[1], false, false);
  rows[0] = e[0];
  rows[1] = o[0];
  rows[2] = e[1];
  rows[3] = o[1];
}

// sum_r phi_k(r) sign_s(r) over part blockIdx.y of the grid (64-point chunks
// c0 .. c0 + cpp - 1): BF16 MFMA GEMM of the state rows (A, MT tiles of 16)
// with the signs of the white-noise vectors (B), bit 0 -> +1.  Workgroup:
// 4 waves x 64 vectors.  The signs never touch memory: per chunk each lane
// draws the 64-bit word of ONE vector (row q of 16 lanes that of vectors
// 16 q .. 16 q + 15) and the four rows exchange them by lane swaps, and with
// the point order of k_phi_bf16 a packed pair of signs is one shift and one
// and-or of the word.  (Every row drawing every word, with bits placed one by
// one, the vector ALU took twice the time of the MFMA pipe.)  The A rows of
// each chunk are staged once per workgroup in LDS, the next chunk's loads in
// flight behind the products.  Parts of the grid fill the chip when there are
// few vectors.  64 states x 64^3 points: 16384 vectors 3250 -> 430 us (16
// parts), 262144 vectors 9.9 -> 7.7 ms (one part): 1.1-1.2 PFLOP/s, the rate
// that a large BF16 matrix product reaches on this device.
// With neta > 0 column c is the occupied-orbital noise vector eta-bar_{c /
// neta, c % neta} (stream kind ETA), else zeta-bar_c.  direct: x[c][k] =
// dV (sum)^2 = |<phi_k|zeta_c>|^2 at rows ldx apart; else the sums go to
// part[blockIdx.y][c][16 MT].
constexpr int FEAT_COLS = 256;                 // vectors per workgroup
constexpr double FEAT_PART_BYTES = 256 << 20;

template <int MT>
__global__ __launch_bounds__(NT) void k_features(const uint16_t *phi16, int64_t N, int K,
                                                 uint64_t seed, int64_t s0, int64_t ncol,
                                                 int64_t cpp, float dV, float *x, int64_t ldx,
                                                 int neta, int direct) {
  constexpr int PA = 72;                           // LDS row pitch (BF16): 64 points + 8
  constexpr int NP = (16 * MT * 8 + NT - 1) / NT;  // 16-byte pieces of a chunk per thread
  __shared__ __align__(16) uint16_t sa[2][16 * MT * PA];
  const int tid = threadIdx.x;
  const int lane = tid & 63, w = tid >> 6, q = lane >> 4, col = lane & 15;
  const int64_t sbase = s0 + (int64_t)blockIdx.x * FEAT_COLS + 64 * w;
  const uint64_t c = (uint64_t)(sbase + 16 * q + col);
  const uint64_t key =
      neta > 0 ? rng_key(seed, rng_stream(RNG_ETA, c / (uint64_t)neta, c % (uint64_t)neta))
               : rng_key(seed, rng_stream(RNG_ZETA, c, 0));
  f32x4 acc[MT][4];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int row0 = tid >> 3, seg = tid & 7;
  auto fetch = [&](int64_t ch, u32x4 *g) {
#pragma unroll
    for (int i = 0; i < NP; ++i)
      if (NP * NT == 16 * MT * 8 || row0 + 32 * i < 16 * MT)
        g[i] = *reinterpret_cast<const u32x4 *>(phi16 + (int64_t)(row0 + 32 * i) * N + 64 * ch + 8 * seg);
  };
  auto stage = [&](int buf, const u32x4 *g) {
#pragma unroll
    for (int i = 0; i < NP; ++i)
      if (NP * NT == 16 * MT * 8 || row0 + 32 * i < 16 * MT)
        *reinterpret_cast<u32x4 *>(&sa[buf][(row0 + 32 * i) * PA + 8 * seg]) = g[i];
  };
  const int64_t c0 = blockIdx.y * cpp, c1 = min(N / 64, c0 + cpp);
  u32x4 gnext[NP];
  fetch(c0, gnext);
  stage(0, gnext);
  __syncthreads();
  int buf = 0;
  const int sh = 12 - 4 * q;
  for (int64_t ch = c0; ch < c1; ++ch) {
    const bool more = ch + 1 < c1;
    if (more) fetch(ch + 1, gnext);
    const uint64_t word = sm64(key + (uint64_t)ch);
    uint32_t bits[2][4];
    spread_rows((uint32_t)word, bits[0]);
    spread_rows((uint32_t)(word >> 32), bits[1]);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      u32x4 a[MT];
#pragma unroll
      for (int m = 0; m < MT; ++m)
        a[m] = *reinterpret_cast<const u32x4 *>(&sa[buf][(16 * m + col) * PA + 32 * half + 8 * q]);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        // points 4 q + j and 4 q + j + 16: bits to positions 15 and 31
        const uint32_t v = bits[half][t] << sh;
        u32x4 b;
#pragma unroll
        for (int j = 0; j < 4; ++j) b[j] = ((v << (3 - j)) & 0x80008000u) | 0x3F803F80u;
#pragma unroll
        for (int m = 0; m < MT; ++m) mma(acc[m][t], a[m], b);
      }
    }
    if (more) stage(buf ^ 1, gnext);
    __syncthreads();
    buf ^= 1;
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int64_t i = sbase + 16 * t + col - s0;
    if (i >= ncol) continue;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      if (direct) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int k = 16 * m + 4 * q + r;
          if (k < K) x[i * ldx + k] = dV * acc[m][t][r] * acc[m][t][r];
        }
      } else {
        *reinterpret_cast<f32x4 *>(x + ((int64_t)blockIdx.y * ncol + i) * (16 * MT) + 16 * m + 4 * q) = acc[m][t];
      }
    }
  }
}

// x[i][k] = (1/neta) sum_l dV (sum_p part[p][i neta + l][k])^2, in order of l
// and p (neta >= 1; part rows are kp floats)
__global__ void k_feature_sums(const float *part, int64_t nsamp, int neta, int np, int kp, int K,
                               float dV, float *x, int64_t ldx) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nsamp * K) return;
  const int64_t s = i / K;
  const int k = (int)(i % K);
  const int64_t step = nsamp * neta * kp;
  float acc = 0.f;
  for (int l = 0; l < neta; ++l) {
    const float *p = part + (s * neta + l) * kp + k;
    float v = 0.f;
#pragma unroll 4
    for (int j = 0; j < np; ++j) v += p[j * step];
    acc += dV * v * v;
  }
  x[s * ldx + k] = acc / (float)neta;
}

// features of nsamp samples from s0 into x (rows ldx apart): zeta-bar
// (neta = 0) or the mean over the sample's neta eta-bar vectors
void features(sgw_ctx *ctx, const float *phi, int K, int64_t ld, uint64_t seed, int64_t s0,
              int64_t nsamp, float *x, int neta = 0, int64_t ldx = 0) {
  const int64_t N = ctx->N;
  if (ldx <= 0) ldx = K;
  const int mt = (K + 15) / 16, kp = 16 * mt;      // state tiles: no products for absent states
  uint16_t *p16 = ctx->buf("cv_phi16", sizeof(uint16_t) * kp * (size_t)N).as<uint16_t>();
  const int vec = ((uintptr_t)phi & 15) == 0 && ld % 4 == 0;
  hipLaunchKernelGGL(k_phi_bf16, dim3((unsigned)((N / 8 + 255) / 256), kp), dim3(256), 0,
                     ctx->stream, phi, ld, K, N, vec, p16);
  SGW_HIP(hipGetLastError());
  const int64_t ncol = neta > 0 ? nsamp * neta : nsamp;
  const int64_t nblk = (ncol + FEAT_COLS - 1) / FEAT_COLS;
  // parts of the grid: about 1024 workgroups (four per CU), at least 16
  // chunks of 64 points each; one part from 1024 blocks of vectors on
  const int64_t nch = N / 64;
  int64_t np = std::max<int64_t>(1, std::min(1024 / nblk, nch / 16));
  const int64_t cpp = (nch + np - 1) / np;
  np = (nch + cpp - 1) / cpp;
  const int direct = np == 1 && neta <= 0;
  // the sums' rows of 16 mt floats take no more than rows of K would, or
  // FEAT_PART_BYTES: past that the samples go in slices (2^20 vectors of 64
  // states in one launch 28 ms, in four 31)
  const double need = 4.0 * np * ncol * kp, most = std::max(FEAT_PART_BYTES, 4.0 * ncol * K);
  const int64_t nslice = direct ? 1 : std::min<int64_t>(nsamp, (int64_t)std::ceil(need / most));
  const int64_t per = (nsamp + nslice - 1) / nslice;
  const int64_t cols = neta > 0 ? per * neta : per;
  float *part = direct ? x
                       : ctx->buf("cv_part_sums", sizeof(float) * (size_t)np * cols * kp).as<float>();
  for (int64_t i = 0; i < nsamp; i += per) {
    const int64_t ns = std::min(per, nsamp - i), nc = neta > 0 ? ns * neta : ns;
    const dim3 g((unsigned)((nc + FEAT_COLS - 1) / FEAT_COLS), (unsigned)np);
    const uint64_t col0 = (uint64_t)(s0 + i) * (neta > 0 ? neta : 1);
#define SGW_F(M)                                                                                \
  case M:                                                                                       \
    hipLaunchKernelGGL(k_features<M>, g, dim3(NT), 0, ctx->stream, p16, N, K, seed,             \
                       (int64_t)col0, nc, cpp, (float)ctx->dV, part, ldx, neta, direct);        \
    break;
    switch (mt) {
      SGW_F(1) SGW_F(2) SGW_F(3) SGW_F(4)
      default: throw Error{SGW_EUNSUPPORTED, "features: K must be in 1..64"};
    }
#undef SGW_F
    SGW_HIP(hipGetLastError());
    if (direct) return;
    hipLaunchKernelGGL(k_feature_sums, dim3((unsigned)((ns * K + NT - 1) / NT)), dim3(NT), 0,
                       ctx->stream, part, ns, std::max(1, neta), (int)np, kp, K, (float)ctx->dV,
                       x + i * ldx, ldx);
    SGW_HIP(hipGetLastError());
  }
}

// ---------------------------------------------------------------- MLP GEMM
// C(m, n) = sum_k A(m, k) B(k, n) for strided FP32 operands (one stride of
// each operand is 1), rounded to BF16 in LDS; a BM x BN output tile per
// workgroup, K in chunks of BK, the next chunk's loads in flight behind the
// current chunk's products.  The network's matrices are small (256 x 256
// weights, a few hundred to a few thousand samples), so what bounds these
// products is the number of workgroups and the round trips to memory one
// after another, not MFMA: 64 x 32 tiles and chunks of 64 for short K, 32 x 32
// tiles with 1024 threads and chunks of 256 for long K (the weight gradients'
// K is the sample count: both products of 1536 samples in one launch of 21
// us, 38 us with 256 threads and chunks of 128, 123 us in two launches of
// 64 x 64 tiles and chunks of 32).  Each output keeps ONE accumulator over
// ascending K groups of 32, so the tile never changes a result: Adam turns
// the last bits of a nearly vanishing gradient into whole steps, which is why
// the products are not split over the samples.  A training step of 1536
// samples took 1400 us in 17 launches, now 70 us in six.
enum Epi { EPI_STORE = 0, EPI_TANH_BIAS = 1, EPI_DTANH = 2 };
// the standardization (b - mean) * inv_std of B, by its K or its N index
enum BStd { BSTD_NONE = 0, BSTD_K = 1, BSTD_N = 2 };

struct GemmArgs {
  const float *a; int64_t sam, sak;
  const float *b; int64_t sbk, sbn;
  float *c; int64_t scm, scn;
  const float *bias;        // EPI_TANH_BIAS: [M]
  const float *aux;         // EPI_DTANH: activation at the strides of C
  const float *mean, *inv_std;   // BSTD_K, BSTD_N
  int M, N, K;
  int avec, bvec, cvec;     // 16-byte accesses allowed (set by finish_args)
};

template <int BM_, int BN_, int BK_, int THREADS_, int NBUF_> struct Tile {
  static constexpr int BM = BM_, BN = BN_, BK = BK_, THREADS = THREADS_, NBUF = NBUF_;
  static constexpr int P = BK + 8;            // LDS pitch (bf16): 16 B reads spread over the banks
  static constexpr int WM = BM / 16 < 4 ? BM / 16 : 4;   // of the four multiplying waves, along M
  static constexpr int NT_W = BN / 16 / (4 / WM);        // 16 x 16 tiles of a wave
  static_assert(WM * 16 == BM && NT_W * 16 * (4 / WM) == BN, "tile does not split over four waves");
  struct Lds {
    __align__(16) uint16_t a[NBUF][BM * P], b[NBUF][BN * P];
  };
  static int count(int M, int N) { return ((N + BN - 1) / BN) * ((M + BM - 1) / BM); }
};
using WideTile = Tile<64, 32, 64, 256, 2>;
using ShortTile = Tile<64, 64, 32, 256, 2>;
using DeepTile = Tile<32, 32, 256, 1024, 1>;
constexpr int DEEP = DeepTile::THREADS;

inline GemmArgs finish_args(GemmArgs g) {
  auto ok = [](const void *p, int64_t s0, int64_t s1) {
    return ((uintptr_t)p & 15) == 0 && (s0 == 1 ? s1 : s0) % 4 == 0;
  };
  g.avec = ok(g.a, g.sam, g.sak);
  g.bvec = ok(g.b, g.sbn, g.sbk);
  g.cvec = g.scm == 1 && ok(g.c, g.scm, g.scn) && (!g.aux || ((uintptr_t)g.aux & 15) == 0);
  return g;
}

// A chunk of ROWS rows x BK K values as 4-value groups along the contiguous
// axis, in registers: along the rows, groups 2 i and 2 i + 1 are the K values 2 kp, 2 kp + 1 of
// one row group, so that a pair of K neighbours is written to LDS at once.
// Values outside the matrix are zero.
template <int ROWS, int BK, int THREADS> struct Chunk {
  static constexpr int NG = ROWS * BK / 4 / THREADS, GP = BK + 8;
  static_assert(NG % 2 == 0, "groups come in pairs");
  float v[NG][4];
  __device__ static void place(bool kc, int i, int tid, int &row, int &k) {
    if (kc) {
      const int idx = tid + THREADS * i;
      row = idx / (BK / 4);
      k = 4 * (idx % (BK / 4));
    } else {
      const int idx = tid + THREADS * (i / 2);
      row = 4 * (idx % (ROWS / 4));
      k = 2 * (idx / (ROWS / 4)) + (i & 1);
    }
  }
  __device__ void load(const float *p, int64_t sr, int64_t sk, bool vec, int r0, int rows, int k0,
                       int kend, int tid) {
    const bool kc = sk == 1;
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      int row, k;
      place(kc, i, tid, row, k);
      const int r = r0 + row, kk = k0 + k;
      const float *q = p + r * sr + kk * sk;
      const bool in = kc ? r < rows && kk + 4 <= kend : kk < kend && r + 4 <= rows;
      if (vec && in) {
        const float4 f = *reinterpret_cast<const float4 *>(q);
        v[i][0] = f.x; v[i][1] = f.y; v[i][2] = f.z; v[i][3] = f.w;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          v[i][e] = (kc ? r < rows && kk + e < kend : kk < kend && r + e < rows)
                        ? q[kc ? (int64_t)e : e * sr] : 0.f;
      }
    }
  }
  template <int STD>
  __device__ void stage(uint16_t *s, bool kc, int tid, int r0, int rows, int k0, int kend,
                        const float *mean, const float *inv_std) {
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      int row, k;
      place(kc, i, tid, row, k);
      if constexpr (STD != BSTD_NONE) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = r0 + row + (kc ? 0 : e), kk = k0 + k + (kc ? e : 0);
          const int j = STD == BSTD_K ? kk : r;
          if (r < rows && kk < kend) v[i][e] = (v[i][e] - mean[j]) * inv_std[j];
        }
      }
      if (kc) {
        const uint2 w = make_uint2(bf16r(v[i][0]) | bf16r(v[i][1]) << 16,
                                   bf16r(v[i][2]) | bf16r(v[i][3]) << 16);
        *reinterpret_cast<uint2 *>(s + row * GP + k) = w;
      } else if (i & 1) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          *reinterpret_cast<uint32_t *>(s + (row + e) * GP + k - 1) =
              bf16r(v[i - 1][e]) | bf16r(v[i][e]) << 16;
      }
    }
  }
};

template <class T, int EPI, int STD>
__device__ __forceinline__ void gemm_tile(const GemmArgs &g, int nb, int mb, typename T::Lds &l) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, q = lane >> 4, col = lane & 15;
  const int m0 = mb * T::BM, n0 = nb * T::BN;
  const int wm = 16 * (w % T::WM), wn = 16 * T::NT_W * (w / T::WM);
  const bool ak = g.sak == 1, bk = g.sbk == 1;
  f32x4 acc[T::NT_W];
#pragma unroll
  for (int t = 0; t < T::NT_W; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  Chunk<T::BM, T::BK, T::THREADS> ca;
  Chunk<T::BN, T::BK, T::THREADS> cb;
  auto load = [&](int k0) {
    ca.load(g.a, g.sam, g.sak, g.avec, m0, g.M, k0, g.K, tid);
    cb.load(g.b, g.sbn, g.sbk, g.bvec, n0, g.N, k0, g.K, tid);
  };
  load(0);
  int buf = 0;
  for (int k0 = 0; k0 < g.K; k0 += T::BK) {
    ca.template stage<BSTD_NONE>(l.a[buf], ak, tid, m0, g.M, k0, g.K, nullptr, nullptr);
    cb.template stage<STD>(l.b[buf], bk, tid, n0, g.N, k0, g.K, g.mean, g.inv_std);
    __syncthreads();
    if (k0 + T::BK < g.K) load(k0 + T::BK);
    if (T::THREADS == 256 || w < 4) {
#pragma unroll
      for (int h = 0; h < T::BK / 32; ++h) {
        const u32x4 a = *reinterpret_cast<const u32x4 *>(l.a[buf] + (wm + col) * T::P + 32 * h + 8 * q);
#pragma unroll
        for (int t = 0; t < T::NT_W; ++t) {
          const u32x4 b = *reinterpret_cast<const u32x4 *>(l.b[buf] + (wn + 16 * t + col) * T::P + 32 * h + 8 * q);
          mma(acc[t], a, b);
        }
      }
    }
    if constexpr (T::NBUF == 2) buf ^= 1;   // the other buffer's readers all passed this chunk's barrier
    else if (k0 + T::BK < g.K) __syncthreads();
  }
  if (T::THREADS > 256 && w >= 4) return;
  const int m = m0 + wm + 4 * q;
  float *c = g.c;
#pragma unroll
  for (int t = 0; t < T::NT_W; ++t) {
    const int n = n0 + wn + 16 * t + col;
    if (n >= g.N || m >= g.M) continue;
    const int64_t o = m * g.scm + n * g.scn;
    const bool vec = g.cvec && m + 4 <= g.M;
    float v[4], x[4];
    if (EPI == EPI_DTANH) {
      if (vec) {
        const float4 f = *reinterpret_cast<const float4 *>(g.aux + o);
        x[0] = f.x; x[1] = f.y; x[2] = f.z; x[3] = f.w;
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = m + r < g.M ? g.aux[o + r * g.scm] : 0.f;
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      v[r] = acc[t][r];
      if (EPI == EPI_TANH_BIAS) v[r] = tanhf(v[r] + (m + r < g.M ? g.bias[m + r] : 0.f));
      if (EPI == EPI_DTANH) v[r] *= 1.f - x[r] * x[r];
    }
    if (vec) {
      *reinterpret_cast<float4 *>(c + o) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (m + r < g.M) c[o + r * g.scm] = v[r];
    }
  }
}

template <class T, int EPI, int STD>
__global__ __launch_bounds__(T::THREADS) void k_gemm(GemmArgs g) {
  __shared__ typename T::Lds l;
  gemm_tile<T, EPI, STD>(g, blockIdx.x, blockIdx.y, l);
}

template <class T, int EPI, int STD> void launch_gemm(hipStream_t st, const GemmArgs &g) {
  hipLaunchKernelGGL((k_gemm<T, EPI, STD>), dim3((g.N + T::BN - 1) / T::BN, (g.M + T::BM - 1) / T::BM),
                     dim3(T::THREADS), 0, st, g);
  SGW_HIP(hipGetLastError());
}

template <int EPI, int STD> void gemm(hipStream_t st, const GemmArgs &a) {
  if (a.M <= 0 || a.N <= 0) return;
  const GemmArgs g = finish_args(a);
  // deep tiles where their chunks of 256 are filled and the launch is at most
  // four workgroups per CU (256 x 256 layer, 1536 samples: 7.8 against 9.4 us;
  // 64 inputs: 14.2 against 7.8, so wide; beyond, wide tiles read less); short
  // tiles where half of a wide tile's chunk would be empty and one workgroup
  // per CU is left (400000 samples through 32-32-32: forward 255 -> 109 us)
  if (g.K > 128 && DeepTile::count(g.M, g.N) <= 1024) launch_gemm<DeepTile, EPI, STD>(st, g);
  else if (g.K <= 32 && ShortTile::count(g.M, g.N) >= 256) launch_gemm<ShortTile, EPI, STD>(st, g);
  else launch_gemm<WideTile, EPI, STD>(st, g);
}

// ---------------------------------------------------------------- output layer
// g = w3 . a2 + b3 (FP32, in order of j) and, in training, the residual's
// dg = 2 (g - y) / n, its square (FP64) and the layer's d2[j] = dg w3[j]
// (1 - a2[j]^2).  S samples per workgroup: their a2 rows are read coalesced
// into LDS, J columns at a time, one thread per sample adds its row (a chain
// of h2 FMAs, 1 us at 256; one thread per sample straight from memory took 33
// us at 1536 samples).  16 samples and 256 columns; 64 and 64 where a row is
// no longer than a wave and the samples fill the chip all the same, or most
// threads would have no column (forward pass of 40000 samples through 9-16-24
// 36.7 us, 22.4 with these and the short GEMM tile; 500 samples 18.7 and 19.7).
template <int S_, int J_> struct OutTile {
  static constexpr int S = S_, J = J_, R = NT / J;   // R rows at a time
};
using OutWide = OutTile<16, 256>;
using OutNarrow = OutTile<64, 64>;

template <class T, bool TRAIN>
__global__ __launch_bounds__(NT) void k_output(const float *a2, const float *w3, const float *b3,
                                               int h2, int64_t n, float *g, const float *y,
                                               float *dg, double *e2, float *d2) {
  constexpr int S = T::S, J = T::J, R = T::R;
  __shared__ float sh[S * (J + 1)], sw[J], sd[S];
  const int64_t s0 = (int64_t)blockIdx.x * S;
  const int tid = threadIdx.x, ns = (int)min((int64_t)S, n - s0);
  const int col = R == 1 ? tid : tid % J, row = R == 1 ? 0 : tid / J;
  float acc = 0.f;
  for (int j0 = 0; j0 < h2; j0 += J) {
    const int nj = min(J, h2 - j0);
    if (col < nj) {
      if (row == 0) sw[col] = w3[j0 + col];
#pragma unroll
      for (int k = 0; k < S / R; ++k) {
        const int i = row + R * k;
        if (i < ns) sh[i * (J + 1) + col] = a2[(s0 + i) * h2 + j0 + col];
      }
    }
    __syncthreads();
    if (tid < ns) {
#pragma unroll 16
      for (int j = 0; j < nj; ++j) acc += sw[j] * sh[tid * (J + 1) + j];
    }
    __syncthreads();
  }
  if (tid < ns) {
    const float gs = acc + b3[0];
    g[s0 + tid] = gs;
    if constexpr (TRAIN) {
      const double r = (double)gs - (double)y[s0 + tid];
      sd[tid] = dg[s0 + tid] = (float)(2.0 * r / (double)n);
      e2[s0 + tid] = r * r;
    }
  }
  if constexpr (TRAIN) {
    __syncthreads();
    for (int j = col; j < h2; j += J) {
      const float w = w3[j];
#pragma unroll
      for (int k = 0; k < S / R; ++k) {
        const int i = row + R * k;
        if (i < ns) {
          const float h = a2[(s0 + i) * h2 + j];
          d2[(s0 + i) * h2 + j] = sd[i] * w * (1.f - h * h);
        }
      }
    }
  }
}

template <bool TRAIN>
void launch_output(hipStream_t st, const float *a2, const float *w3, const float *b3, int h2,
                   int64_t n, float *g, const float *y, float *dg, double *e2, float *d2) {
  auto go = [&](auto t) {
    using T = decltype(t);
    hipLaunchKernelGGL((k_output<T, TRAIN>), dim3((unsigned)((n + T::S - 1) / T::S)), dim3(NT), 0,
                       st, a2, w3, b3, h2, n, g, y, dg, e2, d2);
  };
  if (h2 <= OutNarrow::J && n >= 256 * OutNarrow::S) go(OutNarrow{});
  else go(OutWide{});
  SGW_HIP(hipGetLastError());
}

// ---------------------------------------------------------------- weight gradients
// Everything that is summed over samples, in one launch: dW2 = d2^T a1 and
// dW1 = d1^T xh, and the column sums of d2, a2 dg and d1 and the sums of dg
// and of the squared residuals (FP64) over ranges of samples, which k_grad
// adds in order.  (One thread per column over all samples took 352 us per
// sum at 1536 samples, the two products on 16 and 4 workgroups 60 us each.)
struct WGradArgs {
  GemmArgs w2, w1;
  int tiles2, tiles1, S;           // output tiles of the two products, sample ranges of the sums
  const float *d2, *d1, *a2, *dg;
  const double *e2;
  int h1, h2, chunk;
  int64_t n;
  double *cols;                    // [S][2 h2 + h1 + 2]: d2, a2 dg, d1, dg, e2
};

__global__ __launch_bounds__(DEEP) void k_wgrads(WGradArgs a) {
  __shared__ DeepTile::Lds l;
  int b = blockIdx.x;
  if (b < a.tiles2) {
    const int nbx = (a.w2.N + DeepTile::BN - 1) / DeepTile::BN;
    gemm_tile<DeepTile, EPI_STORE, BSTD_NONE>(a.w2, b % nbx, b / nbx, l);
    return;
  }
  b -= a.tiles2;
  if (b < a.tiles1) {
    const int nbx = (a.w1.N + DeepTile::BN - 1) / DeepTile::BN;
    gemm_tile<DeepTile, EPI_STORE, BSTD_N>(a.w1, b % nbx, b / nbx, l);
    return;
  }
  b -= a.tiles1;
  // sums: four units of 256 threads per workgroup, each one range of samples
  // and one block of columns
  const int c2 = (a.h2 + NT - 1) / NT, c1 = (a.h1 + NT - 1) / NT, per = c2 + c1 + 1;
  const int unit = b * (DEEP / NT) + threadIdx.x / NT, tid = threadIdx.x % NT;
  const int z = unit / per, kind = unit % per;
  if (z >= a.S) return;
  const int64_t s0 = (int64_t)z * a.chunk, s1 = min(a.n, s0 + a.chunk);
  double *out = a.cols + (int64_t)z * (2 * a.h2 + a.h1 + 2);
  if (kind < c2) {
    const int j = kind * NT + tid;
    if (j >= a.h2) return;
    double b2 = 0.0, w3 = 0.0;
#pragma unroll 8
    for (int64_t s = s0; s < s1; ++s) {
      b2 += (double)a.d2[s * a.h2 + j];
      w3 += (double)a.a2[s * a.h2 + j] * (double)a.dg[s];
    }
    out[j] = b2;
    out[a.h2 + j] = w3;
  } else if (kind < c2 + c1) {
    const int j = (kind - c2) * NT + tid;
    if (j >= a.h1) return;
    double b1 = 0.0;
#pragma unroll 8
    for (int64_t s = s0; s < s1; ++s) b1 += (double)a.d1[s * a.h1 + j];
    out[2 * a.h2 + j] = b1;
  } else {
    if (tid >= 64) return;
    double d = 0.0, e = 0.0;
    for (int64_t s = s0 + tid; s < s1; s += 64) {
      d += (double)a.dg[s];
      e += a.e2[s];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      d += __shfl_xor(d, o, 64);
      e += __shfl_xor(e, o, 64);
    }
    if (tid == 0) {
      out[2 * a.h2 + a.h1] = d;
      out[2 * a.h2 + a.h1 + 1] = e;
    }
  }
}

// The bias gradients, dw3 and the loss from the sample ranges' sums, and
// (train) the Adam update with bias-corrected moments, c1 = 1 / (1 - b1^t),
// c2 = 1 / (1 - b2^t); one thread per parameter, one more for the loss.
struct AdamArgs {
  float *theta, *m, *v;
  float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ void adam_update(const AdamArgs &p, int64_t i, float gi) {
  const float mi = p.b1 * p.m[i] + (1.f - p.b1) * gi;
  const float vi = p.b2 * p.v[i] + (1.f - p.b2) * gi * gi;
  p.m[i] = mi;
  p.v[i] = vi;
  p.theta[i] -= p.lr * (mi * p.c1) / (sqrtf(vi * p.c2) + p.eps);
}

template <bool TRAIN>
__global__ __launch_bounds__(NT) void k_grad(const double *cols, int din, int h1, int h2, int S,
                                             float *grad, double *loss, AdamArgs p) {
  const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
  const int64_t n1 = (int64_t)h1 * din, n2 = (int64_t)h2 * h1, nc = 2 * h2 + h1 + 2;
  const int64_t last = n1 + h1 + n2 + 2 * h2 + 1;
  if (i > last) return;
  int64_t j = -1;                                     // column of the sums
  if (i >= n1 && i < n1 + h1) j = 2 * h2 + (i - n1);  // b1
  else if (i >= n1 + h1 + n2) j = i - (n1 + h1 + n2) + (i >= last - 1 ? h1 : 0);   // b2, w3; b3, loss
  float gi;
  if (j >= 0) {
    double acc = 0.0;
#pragma unroll 8
    for (int z = 0; z < S; ++z) acc += cols[z * nc + j];
    if (i == last) {
      *loss = acc;
      return;
    }
    gi = (float)acc;
    grad[i] = gi;
  } else if (TRAIN) {
    gi = grad[i];
  }
  if constexpr (TRAIN) adam_update(p, i, gi);
}

// deterministic FP64 sums: stage 1 per block, stage 2 in block order
template <int POW>
__global__ void k_sum1(const float *x, const double *xd, int64_t n, double *partial) {
  __shared__ double sh[NT];
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT) {
    const double v = x ? (double)x[i] : xd[i];
    acc += POW == 2 ? v * v : v;
  }
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int o = NT / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = sh[0];
}

// one wave: each lane adds every 64th partial, the lanes are added in a tree
__global__ void k_sum2(const double *partial, int nblk, double *out) {
  double acc = 0.0;
  for (int i = threadIdx.x; i < nblk; i += 64) acc += partial[i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if (threadIdx.x == 0) out[0] = acc;
}

constexpr int SUM_BLOCKS = 256;

// out = sum x (POW 1) or sum x^2 (POW 2), left on the device
template <int POW>
void dsum(hipStream_t st, const float *x, const double *xd, int64_t n, double *partial,
          double *out) {
  hipLaunchKernelGGL(k_sum1<POW>, dim3(SUM_BLOCKS), dim3(NT), 0, st, x, xd, n, partial);
  hipLaunchKernelGGL(k_sum2, dim3(1), dim3(64), 0, st, partial, SUM_BLOCKS, out);
  SGW_HIP(hipGetLastError());
}

__global__ void k_adam(AdamArgs p, const float *grad, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) adam_update(p, i, grad[i]);
}

inline unsigned blocks(int64_t n) { return (unsigned)((n + NT - 1) / NT); }

// ---------------------------------------------------------------- network passes
struct Acts {
  float *a1, *a2, *g;
};

Acts activations(sgw_mlp *M, int64_t n) {
  Acts a;
  a.a1 = M->buf("a1", sizeof(float) * n * M->h1).as<float>();
  a.a2 = M->buf("a2", sizeof(float) * n * M->h2).as<float>();
  a.g = M->buf("g", sizeof(float) * n).as<float>();
  return a;
}

// both hidden layers for n samples (x [n][din])
void hidden(sgw_mlp *M, const float *x, int64_t n, const Acts &a) {
  const float *th = M->theta.as<float>();
  hipStream_t st = M->stream;
  GemmArgs g{};
  // a1[s][j] = tanh(sum_k W1[j][k] xh[s][k] + b1[j]), xh standardized as it is loaded
  g.a = th + M->oW1(); g.sam = M->din; g.sak = 1;
  g.b = x; g.sbk = 1; g.sbn = M->din;
  g.mean = M->mean.as<float>(); g.inv_std = M->inv_std.as<float>();
  g.c = a.a1; g.scm = 1; g.scn = M->h1;
  g.bias = th + M->ob1(); g.M = M->h1; g.N = (int)n; g.K = M->din;
  gemm<EPI_TANH_BIAS, BSTD_K>(st, g);
  // a2[s][j] = tanh(sum_k W2[j][k] a1[s][k] + b2[j])
  g.a = th + M->oW2(); g.sam = M->h1; g.sak = 1;
  g.b = a.a1; g.sbk = 1; g.sbn = M->h1;
  g.c = a.a2; g.scm = 1; g.scn = M->h2;
  g.bias = th + M->ob2(); g.M = M->h2; g.K = M->h1;
  gemm<EPI_TANH_BIAS, BSTD_NONE>(st, g);
}

// out = network(x) for n samples (x [n][din]); activations kept in `a`
void forward(sgw_mlp *M, const float *x, int64_t n, const Acts &a, float *out) {
  const float *th = M->theta.as<float>();
  hidden(M, x, n, a);
  launch_output<false>(M->stream, a.a2, th + M->ow3(), th + M->ob3(), M->h2, n, out, nullptr,
                       nullptr, nullptr, nullptr);
}

AdamArgs adam_args(sgw_mlp *M, double lr, double b1, double b2, double eps) {
  M->t += 1;
  AdamArgs p;
  p.theta = M->theta.as<float>(); p.m = M->m.as<float>(); p.v = M->v.as<float>();
  p.lr = (float)lr; p.b1 = (float)b1; p.b2 = (float)b2; p.eps = (float)eps;
  p.c1 = (float)(1.0 / (1.0 - std::pow(b1, (double)M->t)));
  p.c2 = (float)(1.0 / (1.0 - std::pow(b2, (double)M->t)));
  return p;
}

// Forward pass and gradient of L = (1/n) sum (g - y)^2 into M->grad, the sum
// of squares (FP64) into *d_loss; with train, the Adam update too.  Six
// launches a step.
template <bool TRAIN>
void gradient(sgw_mlp *M, const float *x, const float *y, int64_t n, const Acts &a,
              double *d_loss, double lr) {
  const float *th = M->theta.as<float>();
  hipStream_t st = M->stream;
  float *dg = M->buf("dg", sizeof(float) * n).as<float>();
  double *e2 = M->buf("e2", sizeof(double) * n).as<double>();
  float *d2 = M->buf("d2", sizeof(float) * n * M->h2).as<float>();
  float *d1 = M->buf("d1", sizeof(float) * n * M->h1).as<float>();
  hidden(M, x, n, a);
  launch_output<true>(st, a.a2, th + M->ow3(), th + M->ob3(), M->h2, n, a.g, y, dg, e2, d2);
  // d1[s][k] = (sum_j W2[j][k] d2[s][j]) (1 - a1[s][k]^2)
  GemmArgs g{};
  g.a = th + M->oW2(); g.sam = 1; g.sak = M->h1;
  g.b = d2; g.sbk = 1; g.sbn = M->h2;
  g.c = d1; g.scm = 1; g.scn = M->h1;
  g.aux = a.a1; g.M = M->h1; g.N = (int)n; g.K = M->h2;
  gemm<EPI_DTANH, BSTD_NONE>(st, g);
  WGradArgs w{};
  // sums over at most 64 ranges of at least 64 samples each
  const int64_t S = std::max<int64_t>(1, std::min<int64_t>((n + 63) / 64, 64));
  w.chunk = (int)((n + S - 1) / S);
  w.S = (int)((n + w.chunk - 1) / w.chunk);
  w.cols = M->buf("cols", sizeof(double) * w.S * (2 * M->h2 + M->h1 + 2)).as<double>();
  float *gr = M->grad.as<float>();
  // dW2[j][k] = sum_s d2[s][j] a1[s][k] (C transposed: M runs over k, the contiguous index)
  g = GemmArgs{};
  g.a = a.a1; g.sam = 1; g.sak = M->h1;
  g.b = d2; g.sbk = M->h2; g.sbn = 1;
  g.c = gr + M->oW2(); g.scm = 1; g.scn = M->h1;
  g.M = M->h1; g.N = M->h2; g.K = (int)n;
  w.w2 = finish_args(g);
  // dW1[j][k] = sum_s d1[s][j] xh[s][k]
  g.a = d1; g.sam = 1; g.sak = M->h1;
  g.b = x; g.sbk = M->din; g.sbn = 1;
  g.mean = M->mean.as<float>(); g.inv_std = M->inv_std.as<float>();
  g.c = gr + M->oW1(); g.scm = M->din; g.scn = 1;
  g.M = M->h1; g.N = M->din;
  w.w1 = finish_args(g);
  w.tiles2 = DeepTile::count(w.w2.M, w.w2.N);
  w.tiles1 = DeepTile::count(w.w1.M, w.w1.N);
  w.d2 = d2; w.d1 = d1; w.a2 = a.a2; w.dg = dg; w.e2 = e2;
  w.h1 = M->h1; w.h2 = M->h2; w.n = n;
  const int percol = (M->h2 + NT - 1) / NT + (M->h1 + NT - 1) / NT + 1;
  hipLaunchKernelGGL(k_wgrads, dim3(w.tiles2 + w.tiles1 + (w.S * percol + DEEP / NT - 1) / (DEEP / NT)),
                     dim3(DEEP), 0, st, w);
  SGW_HIP(hipGetLastError());
  AdamArgs p{};
  if (TRAIN) p = adam_args(M, lr, 0.9, 0.999, 1e-8);
  hipLaunchKernelGGL(k_grad<TRAIN>, dim3(blocks(M->nparam + 1)), dim3(NT), 0, st, w.cols,
                     M->din, M->h1, M->h2, w.S, gr, d_loss, p);
  SGW_HIP(hipGetLastError());
}

void adam(sgw_mlp *M, double lr, double b1, double b2, double eps) {
  hipLaunchKernelGGL(k_adam, dim3(blocks(M->nparam)), dim3(NT), 0, M->stream,
                     adam_args(M, lr, b1, b2, eps), M->grad.as<float>(), M->nparam);
  SGW_HIP(hipGetLastError());
}

void check_n(int64_t n) {
  SGW_REQUIRE(n > 0 && n <= (int64_t)1 << 30, SGW_EINVAL, "sample count out of range");
}

}  // namespace

// =================================================================== ABI
extern "C" {

const char *sgw_mlp_last_error(const sgw_mlp *m) { return m ? m->err.c_str() : g_mlp_error.c_str(); }

sgw_status sgw_cv_features(sgw_ctx *ctx, const float *phi, int32_t K, int64_t ld_phi,
                           uint64_t seed, int64_t first_sample, int64_t nsamp, float *x) {
  if (!ctx) return SGW_EINVAL;
  return guard_ctx(ctx, [&] {
    SGW_REQUIRE(phi && x, SGW_EINVAL, "NULL argument");
    SGW_REQUIRE(K >= 1 && K <= 64, SGW_EINVAL, "K must be in 1..64");
    SGW_REQUIRE(ld_phi >= ctx->N, SGW_EINVAL, "ld_phi < number of grid points");
    SGW_REQUIRE(nsamp >= 0 && first_sample >= 0 && first_sample + nsamp <= ((int64_t)1 << 20),
                SGW_EINVAL, "sample indices must lie in [0, 2^20)");
    SGW_REQUIRE(ctx->N % 64 == 0, SGW_EUNSUPPORTED, "features need N divisible by 64");
    if (nsamp == 0) return;
    features(ctx, phi, K, ld_phi, seed, first_sample, nsamp, x);
  });
}

sgw_status sgw_cv_features_eta(sgw_ctx *ctx, const float *phi, int32_t K, int64_t ld_phi,
                               uint64_t seed, int64_t first_sample, int64_t nsamp,
                               int32_t n_eta, float *x, int64_t ldx) {
  if (!ctx) return SGW_EINVAL;
  return guard_ctx(ctx, [&] {
    SGW_REQUIRE(phi && x, SGW_EINVAL, "NULL argument");
    SGW_REQUIRE(K >= 1 && K <= 64, SGW_EINVAL, "K must be in 1..64");
    SGW_REQUIRE(n_eta >= 1 && n_eta < (1 << 20), SGW_EINVAL, "n_eta must be in 1..2^20-1");
    SGW_REQUIRE(ldx >= K, SGW_EINVAL, "ldx < K");
    SGW_REQUIRE(ld_phi >= ctx->N, SGW_EINVAL, "ld_phi < number of grid points");
    SGW_REQUIRE(nsamp >= 0 && first_sample >= 0 && first_sample + nsamp <= ((int64_t)1 << 20),
                SGW_EINVAL, "sample indices must lie in [0, 2^20)");
    SGW_REQUIRE(ctx->N % 64 == 0, SGW_EUNSUPPORTED, "features need N divisible by 64");
    if (nsamp == 0) return;
    features(ctx, phi, K, ld_phi, seed, first_sample, nsamp, x, n_eta, ldx);
  });
}

sgw_status sgw_mlp_create(int32_t din, int32_t h1, int32_t h2, const double *theta0,
                          void *hip_stream, sgw_mlp **out) {
  if (out) *out = nullptr;
  sgw_mlp *res = nullptr;
  const sgw_status st = guard_mlp(nullptr, [&] {
    SGW_REQUIRE(out && theta0, SGW_EINVAL, "NULL argument");
    SGW_REQUIRE(din >= 1 && h1 >= 1 && h2 >= 1 && din <= 4096 && h1 <= 4096 && h2 <= 4096,
                SGW_EINVAL, "layer sizes must be in 1..4096");
    std::unique_ptr<sgw_mlp> M(new sgw_mlp());
    M->din = din; M->h1 = h1; M->h2 = h2;
    M->stream = static_cast<hipStream_t>(hip_stream);
    M->nparam = M->ob3() + 1;
    std::vector<float> f(M->nparam);
    for (int64_t i = 0; i < M->nparam; ++i) {
      SGW_REQUIRE(std::isfinite(theta0[i]), SGW_EINVAL, "theta0 has a non-finite value");
      f[i] = (float)theta0[i];
    }
    M->theta.ensure(4 * M->nparam);
    M->m.ensure(4 * M->nparam);
    M->v.ensure(4 * M->nparam);
    M->grad.ensure(4 * M->nparam);
    SGW_HIP(hipMemcpy(M->theta.p, f.data(), 4 * M->nparam, hipMemcpyHostToDevice));
    SGW_HIP(hipMemset(M->m.p, 0, 4 * M->nparam));
    SGW_HIP(hipMemset(M->v.p, 0, 4 * M->nparam));
    SGW_HIP(hipMemset(M->grad.p, 0, 4 * M->nparam));
    std::vector<float> zero(din, 0.f), one(din, 1.f);
    M->mean.ensure(4 * din);
    M->inv_std.ensure(4 * din);
    SGW_HIP(hipMemcpy(M->mean.p, zero.data(), 4 * din, hipMemcpyHostToDevice));
    SGW_HIP(hipMemcpy(M->inv_std.p, one.data(), 4 * din, hipMemcpyHostToDevice));
    res = M.release();
  });
  if (st == SGW_OK) *out = res;
  return st;
}

void sgw_mlp_destroy(sgw_mlp *m) { delete m; }

sgw_status sgw_mlp_set_standardization(sgw_mlp *M, const double *mean, const double *std) {
  if (!M) return SGW_EINVAL;
  return guard_mlp(M, [&] {
    SGW_REQUIRE(mean && std, SGW_EINVAL, "NULL argument");
    std::vector<float> mf(M->din), sf(M->din);
    for (int k = 0; k < M->din; ++k) {
      SGW_REQUIRE(std::isfinite(mean[k]) && std[k] > 0 && std::isfinite(std[k]), SGW_EINVAL,
                  "standardization needs finite means and positive deviations");
      mf[k] = (float)mean[k];
      sf[k] = (float)(1.0 / std[k]);
    }
    SGW_HIP(hipMemcpyAsync(M->mean.p, mf.data(), 4 * M->din, hipMemcpyHostToDevice, M->stream));
    SGW_HIP(hipMemcpyAsync(M->inv_std.p, sf.data(), 4 * M->din, hipMemcpyHostToDevice, M->stream));
    SGW_HIP(hipStreamSynchronize(M->stream));
  });
}

sgw_status sgw_mlp_get_params(sgw_mlp *M, double *theta) {
  if (!M) return SGW_EINVAL;
  return guard_mlp(M, [&] {
    SGW_REQUIRE(theta, SGW_EINVAL, "NULL argument");
    std::vector<float> f(M->nparam);
    SGW_HIP(hipMemcpyAsync(f.data(), M->theta.p, 4 * M->nparam, hipMemcpyDeviceToHost, M->stream));
    SGW_HIP(hipStreamSynchronize(M->stream));
    for (int64_t i = 0; i < M->nparam; ++i) theta[i] = f[i];
  });
}

sgw_status sgw_mlp_forward(sgw_mlp *M, const float *x, int64_t n, float *g) {
  if (!M) return SGW_EINVAL;
  return guard_mlp(M, [&] {
    SGW_REQUIRE(x && g, SGW_EINVAL, "NULL argument");
    check_n(n);
    forward(M, x, n, activations(M, n), g);
  });
}

sgw_status sgw_mlp_gradient(sgw_mlp *M, const float *x, const float *y, int64_t n, double *loss,
                            double *grad) {
  if (!M) return SGW_EINVAL;
  return guard_mlp(M, [&] {
    SGW_REQUIRE(x && y && loss && grad, SGW_EINVAL, "NULL argument");
    check_n(n);
    const Acts a = activations(M, n);
    double *d_loss = M->buf("loss1", sizeof(double)).as<double>();
    gradient<false>(M, x, y, n, a, d_loss, 0.0);
    std::vector<float> f(M->nparam);
    double L = 0;
    SGW_HIP(hipMemcpyAsync(f.data(), M->grad.p, 4 * M->nparam, hipMemcpyDeviceToHost, M->stream));
    SGW_HIP(hipMemcpyAsync(&L, d_loss, sizeof(double), hipMemcpyDeviceToHost, M->stream));
    SGW_HIP(hipStreamSynchronize(M->stream));
    *loss = L / (double)n;
    for (int64_t i = 0; i < M->nparam; ++i) grad[i] = f[i];
  });
}

sgw_status sgw_mlp_adam(sgw_mlp *M, const double *grad, double lr, double b1, double b2,
                        double eps) {
  if (!M) return SGW_EINVAL;
  return guard_mlp(M, [&] {
    SGW_REQUIRE(lr > 0 && b1 >= 0 && b1 < 1 && b2 >= 0 && b2 < 1 && eps > 0, SGW_EINVAL,
                "Adam hyper-parameters out of range");
    if (grad) {
      std::vector<float> f(M->nparam);
      for (int64_t i = 0; i < M->nparam; ++i) f[i] = (float)grad[i];
      SGW_HIP(hipMemcpyAsync(M->grad.p, f.data(), 4 * M->nparam, hipMemcpyHostToDevice,
                             M->stream));
      adam(M, lr, b1, b2, eps);
      SGW_HIP(hipStreamSynchronize(M->stream));
    } else {
      adam(M, lr, b1, b2, eps);
    }
  });
}

sgw_status sgw_mlp_train(sgw_mlp *M, const float *x, const float *y, int64_t n, int32_t steps,
                         double lr, double *loss_hist) {
  if (!M) return SGW_EINVAL;
  return guard_mlp(M, [&] {
    SGW_REQUIRE(x && y, SGW_EINVAL, "NULL argument");
    SGW_REQUIRE(steps >= 0 && lr > 0, SGW_EINVAL, "steps >= 0 and lr > 0 required");
    check_n(n);
    const Acts a = activations(M, n);
    double *d_hist = M->buf("hist", sizeof(double) * std::max(1, (int)steps)).as<double>();
    for (int s = 0; s < steps; ++s) gradient<true>(M, x, y, n, a, d_hist + s, lr);
    if (loss_hist && steps > 0) {
      std::vector<double> h(steps);
      SGW_HIP(hipMemcpyAsync(h.data(), d_hist, sizeof(double) * steps, hipMemcpyDeviceToHost,
                             M->stream));
      SGW_HIP(hipStreamSynchronize(M->stream));
      for (int s = 0; s < steps; ++s) loss_hist[s] = h[s] / (double)n;
    }
  });
}

sgw_status sgw_cv_cheap_moments(sgw_ctx *ctx, sgw_mlp *M, const float *phi, int32_t K,
                                int64_t ld_phi, uint64_t seed, int64_t first_sample, int64_t count,
                                int64_t chunk, double *mean, double *var) {
  if (!ctx || !M) return SGW_EINVAL;
  return guard_ctx(ctx, [&] {
    SGW_REQUIRE(phi && mean && var, SGW_EINVAL, "NULL argument");
    SGW_REQUIRE(K >= 1 && K <= 64, SGW_EINVAL, "K must be in 1..64");
    SGW_REQUIRE(K == M->din, SGW_EINVAL, "K must equal the network's input size");
    SGW_REQUIRE(count >= 2 && chunk >= 1, SGW_EINVAL, "count >= 2 and chunk >= 1 required");
    SGW_REQUIRE(ld_phi >= ctx->N, SGW_EINVAL, "ld_phi < number of grid points");
    SGW_REQUIRE(first_sample >= 0 && first_sample + count <= ((int64_t)1 << 20), SGW_EINVAL,
                "sample indices must lie in [0, 2^20)");
    SGW_REQUIRE(ctx->N % 64 == 0, SGW_EUNSUPPORTED, "features need N divisible by 64");
    SGW_REQUIRE(ctx->stream == M->stream, SGW_EINVAL, "context and network need one stream");
    chunk = std::min(chunk, count);
    float *xf = ctx->buf("cv_x", sizeof(float) * chunk * K).as<float>();
    const Acts a = activations(M, chunk);
    double *part = ctx->buf("cv_part", sizeof(double) * SUM_BLOCKS).as<double>();
    const int64_t nch = (count + chunk - 1) / chunk;
    double *sums = ctx->buf("cv_sums", sizeof(double) * 2 * nch).as<double>();
    for (int64_t c = 0; c < nch; ++c) {
      const int64_t s0 = first_sample + c * chunk, n = std::min(chunk, count - c * chunk);
      features(ctx, phi, K, ld_phi, seed, s0, n, xf);
      forward(M, xf, n, a, a.g);
      dsum<1>(ctx->stream, a.g, nullptr, n, part, sums + 2 * c);
      dsum<2>(ctx->stream, a.g, nullptr, n, part, sums + 2 * c + 1);
    }
    std::vector<double> h(2 * nch);
    SGW_HIP(hipMemcpyAsync(h.data(), sums, sizeof(double) * 2 * nch, hipMemcpyDeviceToHost,
                           ctx->stream));
    SGW_HIP(hipStreamSynchronize(ctx->stream));
    double s1 = 0, s2 = 0;
    for (int64_t c = 0; c < nch; ++c) { s1 += h[2 * c]; s2 += h[2 * c + 1]; }
    const double m = s1 / (double)count;
    *mean = m;
    *var = std::max(0.0, (s2 - (double)count * m * m) / (double)(count - 1));
  });
}

sgw_status sgw_cv_cheap_moments_mixed(sgw_ctx *ctx, sgw_mlp *M, const float *phi_z, int32_t Kz,
                                      const float *phi_e, int32_t Ke, int64_t ld_phi,
                                      uint64_t seed, int32_t n_eta, int64_t first_sample,
                                      int64_t count, int64_t chunk, double *mean, double *var) {
  if (!ctx || !M) return SGW_EINVAL;
  return guard_ctx(ctx, [&] {
    SGW_REQUIRE(mean && var && (Kz == 0 || phi_z) && (Ke == 0 || phi_e), SGW_EINVAL,
                "NULL argument");
    SGW_REQUIRE(Kz >= 0 && Kz <= 64 && Ke >= 0 && Ke <= 64 && Kz + Ke >= 1, SGW_EINVAL,
                "Kz and Ke must be in 0..64, not both 0");
    SGW_REQUIRE(Kz + Ke == M->din, SGW_EINVAL, "Kz + Ke must equal the network's input size");
    SGW_REQUIRE(Ke == 0 || (n_eta >= 1 && n_eta < (1 << 20)), SGW_EINVAL,
                "n_eta must be in 1..2^20-1");
    SGW_REQUIRE(count >= 2 && chunk >= 1, SGW_EINVAL, "count >= 2 and chunk >= 1 required");
    SGW_REQUIRE(ld_phi >= ctx->N, SGW_EINVAL, "ld_phi < number of grid points");
    SGW_REQUIRE(first_sample >= 0 && first_sample + count <= ((int64_t)1 << 20), SGW_EINVAL,
                "sample indices must lie in [0, 2^20)");
    SGW_REQUIRE(ctx->N % 64 == 0, SGW_EUNSUPPORTED, "features need N divisible by 64");
    SGW_REQUIRE(ctx->stream == M->stream, SGW_EINVAL, "context and network need one stream");
    const int K = Kz + Ke;
    chunk = std::min(chunk, count);
    float *xf = ctx->buf("cv_x", sizeof(float) * chunk * K).as<float>();
    const Acts a = activations(M, chunk);
    double *part = ctx->buf("cv_part", sizeof(double) * SUM_BLOCKS).as<double>();
    const int64_t nch = (count + chunk - 1) / chunk;
    double *sums = ctx->buf("cv_sums", sizeof(double) * 2 * nch).as<double>();
    for (int64_t c = 0; c < nch; ++c) {
      const int64_t s0 = first_sample + c * chunk, n = std::min(chunk, count - c * chunk);
      if (Kz > 0) features(ctx, phi_z, Kz, ld_phi, seed, s0, n, xf, 0, K);
      if (Ke > 0) features(ctx, phi_e, Ke, ld_phi, seed, s0, n, xf + Kz, n_eta, K);
      forward(M, xf, n, a, a.g);
      dsum<1>(ctx->stream, a.g, nullptr, n, part, sums + 2 * c);
      dsum<2>(ctx->stream, a.g, nullptr, n, part, sums + 2 * c + 1);
    }
    std::vector<double> h(2 * nch);
    SGW_HIP(hipMemcpyAsync(h.data(), sums, sizeof(double) * 2 * nch, hipMemcpyDeviceToHost,
                           ctx->stream));
    SGW_HIP(hipStreamSynchronize(ctx->stream));
    double s1 = 0, s2 = 0;
    for (int64_t c = 0; c < nch; ++c) { s1 += h[2 * c]; s2 += h[2 * c + 1]; }
    const double m = s1 / (double)count;
    *mean = m;
    *var = std::max(0.0, (s2 - (double)count * m * m) / (double)(count - 1));
  });
}

sgw_status sgw_cv_estimate(const double *yA, const double *gA, int64_t nA, const double *yB,
                           const double *gB, int64_t nB, double gM_mean, double gM_var,
                           int64_t M, sgw_cv_result *out) {
  if (!yA || !gA || !yB || !gB || !out || nA < 2 || nB < 2 || M < 2) return SGW_EINVAL;
  if (!std::isfinite(gM_mean) || !(gM_var >= 0)) return SGW_EINVAL;
  auto mean = [](const double *a, int64_t n) {
    double s = 0; for (int64_t i = 0; i < n; ++i) s += a[i]; return s / (double)n;
  };
  const double my = mean(yA, nA), mg = mean(gA, nA);
  double cyg = 0, vg = 0, vy = 0;
  for (int64_t i = 0; i < nA; ++i) {
    cyg += (yA[i] - my) * (gA[i] - mg);
    vg += (gA[i] - mg) * (gA[i] - mg);
    vy += (yA[i] - my) * (yA[i] - my);
  }
  const double c = vg > 0 ? cyg / vg : 0.0;
  double mr = 0;
  for (int64_t i = 0; i < nB; ++i) mr += yB[i] - c * gB[i];
  mr /= (double)nB;
  double vr = 0;
  for (int64_t i = 0; i < nB; ++i) {
    const double d = yB[i] - c * gB[i] - mr;
    vr += d * d;
  }
  vr /= (double)(nB - 1);
  const double est = mr + c * gM_mean;
  const double var_cv = vr / (double)nB + c * c * gM_var / (double)M;
  double sy = 0;
  for (int64_t i = 0; i < nA; ++i) sy += yA[i];
  for (int64_t i = 0; i < nB; ++i) sy += yB[i];
  const int64_t nt = nA + nB;
  const double plain = sy / (double)nt;
  double vp = 0;
  for (int64_t i = 0; i < nA; ++i) vp += (yA[i] - plain) * (yA[i] - plain);
  for (int64_t i = 0; i < nB; ++i) vp += (yB[i] - plain) * (yB[i] - plain);
  const double var_plain = vp / (double)(nt - 1) / (double)nt;
  out->c = c;
  out->rho2 = (vg > 0 && vy > 0) ? cyg * cyg / (vg * vy) : 0.0;
  out->plain = plain;
  out->sigma_plain = std::sqrt(var_plain);
  out->sigma_cv = std::sqrt(var_cv);
  out->fallback = std::fabs(est - plain) > 3.0 * std::sqrt(var_cv + var_plain) ? 1 : 0;
  out->estimate = out->fallback ? plain : est;
  out->sigma = out->fallback ? out->sigma_plain : out->sigma_cv;
  return SGW_OK;
}

}  // extern "C"
