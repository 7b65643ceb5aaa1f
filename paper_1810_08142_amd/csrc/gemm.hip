// Generic strided FP64 tensor contraction on MFMA (gfx950):
//
//   C(m, n) = alpha * sum_k A(m, k) B(k, n) + beta * C(m, n)
//
// where m, n and k are compound indices: m = (m1, m2), n = (n1, n2),
// k = (k1, k2, k3), each level with its own stride, so a contraction over a
// permuted index pair of a 4-index tensor needs no transposed copy.  Each thread
// walks its k indices with incremental counters (no tables, no divisions in the
// loop).  Contractions with few output tiles and a long k range are split over k
// into partial products that a second kernel sums in a fixed order, so the result
// does not depend on scheduling.
#include <cstdlib>

#include "gemm.h"

namespace ri {
namespace gemm {

typedef double double4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// Arithmetic of the large-tile kernel: FP64 operands on the FP64 MFMA, or operands
// rounded to FP32 on the FP32 MFMA (FP32 accumulation).  Both are 16x16x4 tiles with
// the same operand layout; element r of lane l holds D[drow(r, l)][l % 16].
template <class T>
struct GMma;
template <>
struct GMma<double> {
  typedef double4_t acc_t;
  __device__ static acc_t mma(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ static int drow(int r, int lane) { return 4 * r + (lane >> 4); }
  __device__ static acc_t zero() { return acc_t{0.0, 0.0, 0.0, 0.0}; }
};
template <>
struct GMma<float> {
  typedef f32x4_t acc_t;
  __device__ static acc_t mma(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  __device__ static int drow(int r, int lane) { return 4 * (lane >> 4) + r; }
  __device__ static acc_t zero() { return acc_t{0.f, 0.f, 0.f, 0.f}; }
};

constexpr int BM = 64, BN = 64, KC = 16;

// Quotient by a fixed divisor: for n < 2^31 one multiply-high, an add and a shift (the
// round-up reciprocal of Granlund and Montgomery, PLDI 1994: with s = ceil(log2 d) and
// mul = floor(2^32 (2^s - d) / d) + 1, n / d = (mulhi(n, mul) + n) >> s); 64-bit division
// (about a hundred instructions) only where an extent does not fit.
struct FastDiv {
  uint32_t d, mul, s;
  long wide;  // the divisor where the quotients need 64 bits, else 0
};
static FastDiv fast_div(long d, long max_n) {
  FastDiv f{};
  if (max_n >= (1L << 31)) {
    f.wide = d;
    return f;
  }
  f.d = static_cast<uint32_t>(d);
  while ((1ull << f.s) < static_cast<uint64_t>(d)) ++f.s;
  f.mul = static_cast<uint32_t>(((1ull << 32) * ((1ull << f.s) - static_cast<uint64_t>(d))) / static_cast<uint64_t>(d) + 1);
  return f;
}
__device__ inline void div_mod(const FastDiv& f, long n, long& q, long& r) {
  if (f.wide) {
    q = n / f.wide;
    r = n - q * f.wide;
  } else {
    const uint32_t x = static_cast<uint32_t>(n), y = (__umulhi(x, f.mul) + x) >> f.s;
    q = y;
    r = x - y * f.d;
  }
}

// A contraction as the kernels take it: the description and the divisors of its levels.
struct GemmArgs : GemmDesc {
  FastDiv dM2, dN2, dK2, dK3;
  // offsets of row m of A and C, of column n of B and C
  __device__ long a_row(long m) const {
    long q, r;
    div_mod(dM2, m, q, r);
    return q * am1 + r * am2;
  }
  __device__ long a_row_exchanged(long m) const {
    long q, r;
    div_mod(dM2, m, q, r);
    return r * am1 + q * am2;
  }
  __device__ long c_row(long m) const {
    long q, r;
    div_mod(dM2, m, q, r);
    return q * cm1 + r * cm2;
  }
  __device__ long b_col(long n) const {
    long q, r;
    div_mod(dN2, n, q, r);
    return q * bn1 + r * bn2;
  }
  __device__ long c_col(long n) const {
    long q, r;
    div_mod(dN2, n, q, r);
    return q * cn1 + r * cn2;
  }
};
static GemmArgs make_args(const GemmDesc& g) {
  GemmArgs a;
  static_cast<GemmDesc&>(a) = g;
  a.dM2 = fast_div(g.M2, g.M);
  a.dN2 = fast_div(g.N2, g.N);
  a.dK2 = fast_div(g.K2, g.K);
  a.dK3 = fast_div(g.K3, g.K + 65536);  // positions past the end are stepped through
  return a;
}

// Position of one summed index k in (k2, k3) and its offsets in both operands.
struct KWalk {
  int k2, k3;
  long k, a, b;
};

__device__ inline KWalk kwalk_init(const GemmArgs& g, long k) {
  KWalk w;
  long r, k1, k2, k3;
  div_mod(g.dK3, k, r, k3);
  div_mod(g.dK2, r, k1, k2);
  w.k = k;
  w.k3 = static_cast<int>(k3);
  w.k2 = static_cast<int>(k2);
  w.a = k1 * g.ak1 + k2 * g.ak2 + k3 * g.ak3;
  w.b = k1 * g.bk1 + k2 * g.bk2 + k3 * g.bk3;
  return w;
}

// A fixed step in mixed radix: d2, d3 and the offsets of (d1, d2, d3), so that a walk
// advances by adds and two carries whatever the extents.
struct KStep {
  int n, d2, d3;
  long a, b;
};

__device__ inline KStep kstep_of(const GemmArgs& g, int n) {
  long r, d1, d2, d3;
  div_mod(g.dK3, n, r, d3);
  div_mod(g.dK2, r, d1, d2);
  return KStep{n, static_cast<int>(d2), static_cast<int>(d3), d1 * g.ak1 + d2 * g.ak2 + d3 * g.ak3,
               d1 * g.bk1 + d2 * g.bk2 + d3 * g.bk3};
}

__device__ inline void kwalk_step(KWalk& w, const GemmArgs& g, const KStep& st) {
  w.k += st.n;
  w.k3 += st.d3;
  w.k2 += st.d2;
  w.a += st.a;
  w.b += st.b;
  if (w.k3 >= g.K3) {
    w.k3 -= static_cast<int>(g.K3);
    ++w.k2;
    w.a += g.ak2 - g.K3 * g.ak3;
    w.b += g.bk2 - g.K3 * g.bk3;
  }
  if (w.k2 >= g.K2) {
    w.k2 -= static_cast<int>(g.K2);
    w.a += g.ak1 - g.K2 * g.ak2;
    w.b += g.bk1 - g.K2 * g.bk2;
  }
}

// Result tile element: C at p, or the raw product into the partial sums.
__device__ inline void put(const GemmArgs& g, double* p, double x) {
  const double val = g.alpha * x;
  *p = g.beta == 0.0 ? val : val + g.beta * *p;
}

// A wave's 32 x 32 result from row bm and column bn (element r of a lane: row 4r + kq,
// column l16 of its 16 x 16 tile).
__device__ inline void put_tile(const GemmArgs& g, double* C, double* part, int splits, int zs, long bm, long bn,
                                int kq, int l16, const double4_t (&acc)[2][2]) {
  long n[2], cn[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    n[j] = bn + 16 * j + l16;
    cn[j] = g.c_col(n[j]);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const long m = bm + 16 * i + 4 * r + kq;
      if (m >= g.M) continue;
      double* row = splits > 1 ? part + (zs * g.M + m) * g.N : C + g.c_row(m);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (n[j] >= g.N) continue;
        if (splits > 1)
          row[n[j]] = acc[i][j][r];
        else
          put(g, row + cn[j], acc[i][j][r]);
      }
    }
}

// Small contractions (few or narrow output tiles): bound by latency, so the summed index
// is spread over the waves.  One workgroup computes a 32 x 32 tile; wave w takes the
// chunks of KC summed indices w, w + NW, ... of its split, reads its MFMA operands
// straight from memory (lane l holds A[16i + l%16][4s + l/16], one chunk ahead), and the
// waves' sums are added through LDS in wave order.  There is no barrier in the loop.
// grid (tiles_m * tiles_n, 1, batch * splits); with splits > 1 the raw products of the
// k range z go to part + z * M * N (row-major [M][N]).
// At o=4 v=24 naux=96 the contractions of a residual take 10 us each (24 us with one
// 64 x 64 tile per workgroup walking k chunk by chunk through LDS).
constexpr int SM = 32;
template <int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW == 16 ? 4 : 2))) void gemm_small(GemmArgs g, int tiles_n, int splits, long kper,
                                                      double* __restrict__ part) {
  __shared__ double sR[NW / 2][SM * SM];
  const int t = threadIdx.x, w = t >> 6, lane = t & 63, l16 = lane & 15, kq = lane >> 4;
  const long bm = static_cast<long>(blockIdx.x / tiles_n) * SM, bn = static_cast<long>(blockIdx.x % tiles_n) * SM;
  const int zb = blockIdx.z / splits, zs = blockIdx.z % splits;
  const long k_lo = zs * kper, k_hi = std::min(g.K, k_lo + kper);
  // rows and columns past the edge read the last one; their results are dropped
  const double *Ar[2], *Br[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const long m = std::min(bm + 16 * i + l16, g.M - 1), n = std::min(bn + 16 * i + l16, g.N - 1);
    Ar[i] = g.a + zb * g.a_batch + g.a_row(m);
    Br[i] = g.b + zb * g.b_batch + g.b_col(n);
  }
  const bool two_n = bn + 16 < g.N, two_m = bm + 16 < g.M;  // uniform
  double4_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = double4_t{0.0, 0.0, 0.0, 0.0};
  const long nch = k_hi > k_lo ? (k_hi - k_lo + KC - 1) / KC : 0;
  const KStep st = kstep_of(g, KC * NW);
  KWalk kw[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) kw[s] = kwalk_init(g, std::min(k_lo + w * KC + 4 * s + kq, g.K - 1));
#pragma unroll
  for (int s = 0; s < 4; ++s) kw[s].k = k_lo + w * KC + 4 * s + kq;
  // the next chunk's operands are loaded while one is multiplied; sixteen waves hide the
  // loads from each other and have no registers for a second set
  constexpr int NB = NW == 16 ? 1 : 2;
  double a[NB][2][4], b[NB][2][4];  // [buffer][tile][step]
  bool z[NB][4];                    // past the summed range: the row's first element was read
  auto load = [&](int p) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      z[p][s] = kw[s].k >= k_hi;
      const long ka = z[p][s] ? 0 : kw[s].a, kb = z[p][s] ? 0 : kw[s].b;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[p][i][s] = Ar[i][ka];
        b[p][i][s] = Br[i][kb];
      }
    }
  };
  auto mma = [&](int p) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      double x[2], y[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        x[i] = z[p][s] ? 0.0 : a[p][i][s];
        y[i] = z[p][s] ? 0.0 : b[p][i][s];
      }
      acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[0], y[0], acc[0][0], 0, 0, 0);
      if (two_n) acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[0], y[1], acc[0][1], 0, 0, 0);
      if (two_m) acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[1], y[0], acc[1][0], 0, 0, 0);
      if (two_m && two_n) acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[1], y[1], acc[1][1], 0, 0, 0);
    }
  };
  auto step = [&] {
#pragma unroll
    for (int s = 0; s < 4; ++s) kwalk_step(kw[s], g, st);
  };
  if constexpr (NB == 1) {
    for (long ch = w; ch < nch; ch += NW) {
      load(0);
      step();
      mma(0);
    }
  } else {
    if (w < nch) load(0);
    for (long ch = w; ch < nch; ch += 2 * NW) {
      if (ch + NW < nch) {
        step();
        load(1);
      }
      mma(0);
      if (ch + NW < nch) {
        if (ch + 2 * NW < nch) {
          step();
          load(0);
        }
        mma(1);
      }
    }
  }
  // sum over the waves: the upper half hands its tile to the lower half, NW/2 at a time,
  // element e of a lane at e * 64 + lane
#pragma unroll
  for (int h = NW / 2; h >= 1; h /= 2) {
    if (w >= h && w < 2 * h) {
#pragma unroll
      for (int e = 0; e < 16; ++e) sR[w - h][e * 64 + lane] = acc[e >> 3][(e >> 2) & 1][e & 3];
    }
    __syncthreads();
    if (w < h) {
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[e >> 3][(e >> 2) & 1][e & 3] += sR[w][e * 64 + lane];
    }
    __syncthreads();
  }
  if (w != 0) return;
  double* C = g.c + zb * g.c_batch;
  put_tile(g, C, part, splits, zs, bm, bn, kq, l16, acc);
}

// Tiles of 64 x 64 for the contractions between: two groups of four waves (2 x 2 waves of
// 32 x 32) take alternate chunks of KC summed indices through their own LDS buffers, so
// that every SIMD holds two waves also where the output has one tile per CU; the second
// group's sums are added to the first's through LDS.
// UNI: the chunks run along the innermost summed level alone (its last chunk zero-padded),
// so a chunk's offsets are one wave-uniform base plus a stride; used where the padding is
// small.  Otherwise chunks run over all levels with per-element counters.
// a_kfast / b_kfast choose which index consecutive threads walk when loading.
// grid (ceil(N/64), ceil(M/64), batch * splits); splits as in gemm_small, split z taking
// the chunks [z * cper, (z + 1) * cper).
template <bool UNI>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void gemm_mid(
    GemmArgs g, int a_kfast, int b_kfast, int splits, long cper, double* __restrict__ part) {
  __shared__ double sm[2][2][2][KC][BM + 4];  // [group][buffer][A, B][k][row]
  static_assert(sizeof(sm) >= BM * BN * sizeof(double), "the buffers hold one group's tile");
  const int grp = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  const int t = threadIdx.x & 255, w = t >> 6, lane = t & 63;
  const long bm = static_cast<long>(blockIdx.y) * BM, bn = static_cast<long>(blockIdx.x) * BN;
  const int zb = blockIdx.z / splits, zs = blockIdx.z % splits;
  const double* A = g.a + zb * g.a_batch;
  const double* B = g.b + zb * g.b_batch;
  const int c3n = static_cast<int>((g.K3 + KC - 1) / KC);
  const long total = UNI ? g.K / g.K3 * c3n : (g.K + KC - 1) / KC;
  const long c_lo = zs * cper, c_hi = std::min(total, c_lo + cper);

  // each thread loads one k of a chunk and the rows r0, r0 + 16, + 32, + 48 of each operand,
  // sixteen consecutive lanes walking k or the row, whichever is contiguous
  const int ak = a_kfast ? t & 15 : t >> 4, am = a_kfast ? t >> 4 : t & 15;
  const int bk = b_kfast ? t & 15 : t >> 4, bnn = b_kfast ? t >> 4 : t & 15;
  // rows and columns past the edge read the last one; their results are dropped
  const double *Ap[4], *Bp[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    Ap[r] = A + g.a_row(std::min(bm + am + 16 * r, g.M - 1));
    Bp[r] = B + g.b_col(std::min(bn + bnn + 16 * r, g.N - 1));
  }

  // UNI: position of the group's chunk; otherwise one counter per thread and operand
  int c3 = 0;
  long k2 = 0, k1 = 0;
  KWalk wa{}, wb{};
  KStep st{};
  const long c0 = c_lo + grp;
  if constexpr (UNI) {
    c3 = static_cast<int>(c0 % c3n);
    const long r = c0 / c3n;
    k2 = r % g.K2;
    k1 = r / g.K2;
  } else {
    st = kstep_of(g, 2 * KC);
    wa = kwalk_init(g, c0 * KC + ak);
    wb = kwalk_init(g, c0 * KC + bk);
  }
  // positions past the summed range read the row's first element and are zeroed on the way
  // to LDS, so that the loads carry no branches
  double ra[4], rb[4];
  bool oa, ob;
  auto load = [&](long ch) {  // the group's chunk ch (nothing past c_hi); then advance
    long pa, pb;
    bool ia, ib;
    if constexpr (UNI) {
      const int left = ch < c_hi ? static_cast<int>(g.K3) - c3 * KC : 0;
      ia = ak < left;
      ib = bk < left;
      pa = k1 * g.ak1 + k2 * g.ak2 + (static_cast<long>(c3) * KC + ak) * g.ak3;
      pb = k1 * g.bk1 + k2 * g.bk2 + (static_cast<long>(c3) * KC + bk) * g.bk3;
      c3 += 2;
      while (c3 >= c3n) {
        c3 -= c3n;
        if (++k2 == g.K2) {
          k2 = 0;
          ++k1;
        }
      }
    } else {
      const long k_hi = ch < c_hi ? std::min(g.K, c_hi * KC) : 0;
      ia = wa.k < k_hi;
      ib = wb.k < k_hi;
      pa = wa.a;
      pb = wb.b;
      kwalk_step(wa, g, st);
      kwalk_step(wb, g, st);
    }
    oa = !ia;
    ob = !ib;
    pa = ia ? pa : 0;
    pb = ib ? pb : 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      ra[r] = Ap[r][pa];
      rb[r] = Bp[r][pb];
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      sm[grp][buf][0][ak][am + 16 * r] = oa ? 0.0 : ra[r];
      sm[grp][buf][1][bk][bnn + 16 * r] = ob ? 0.0 : rb[r];
    }
  };
  double4_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = double4_t{0.0, 0.0, 0.0, 0.0};
  const int wm = (w >> 1) * 32, wn = (w & 1) * 32;
  const int l16 = lane & 15, kq = lane >> 4;
  const long iters = c_hi > c_lo ? (c_hi - c_lo + 1) / 2 : 0;  // the same for both groups
  load(c0);
  store(0);
  load(c0 + 2);
  __syncthreads();
  for (long it = 0; it < iters; ++it) {
    const int buf = it & 1;
    if (it + 1 < iters) {
      store(buf ^ 1);
      load(c0 + 2 * it + 4);
    }
#pragma unroll
    for (int s = 0; s < KC / 4; ++s) {
      const int kk = 4 * s + kq;
      double a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = sm[grp][buf][0][kk][wm + 16 * i + l16];
#pragma unroll
      for (int j = 0; j < 2; ++j) b[j] = sm[grp][buf][1][kk][wn + 16 * j + l16];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
  double* sr = &sm[0][0][0][0][0] + w * 1024 + lane;
  if (grp == 1) {
#pragma unroll
    for (int e = 0; e < 16; ++e) sr[e * 64] = acc[e >> 3][(e >> 2) & 1][e & 3];
  }
  __syncthreads();
  if (grp == 1) return;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e >> 3][(e >> 2) & 1][e & 3] += sr[e * 64];
  // D[4r + lane/16][lane%16] in element r
  double* C = g.c + zb * g.c_batch;
  put_tile(g, C, part, splits, zs, bm + wm, bn + wn, kq, l16, acc);
}

// Large tiles for large contractions whose innermost summed extent K3 is a multiple
// of KC: a chunk of KC summed indices then never crosses a level boundary, so its
// offset is one wave-uniform base plus dk * stride.  Tile 128 x 128, four waves in
// a 2 x 2 arrangement, each wave 64 x 64 (4 x 4 MFMA tiles).  grid (ceil(N/128),
// ceil(M/128), batch), no split.
constexpr int BL = 128;
template <class T, int a_kfast, int b_kfast>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_large(GemmArgs g) {
  typedef GMma<T> MF;
  __shared__ T sA[2][KC][BL + 2];
  __shared__ T sB[2][KC][BL + 2];
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  const long bm = static_cast<long>(blockIdx.y) * BL, bn = static_cast<long>(blockIdx.x) * BL;
  const long zb = blockIdx.z;
  const double* A = g.a + zb * g.a_batch;
  const double* B = g.b + zb * g.b_batch;

  // element r of this thread: (row, dk) of the 128 x 16 tile; k-fast operands put
  // 16 consecutive lanes on consecutive k, the others 64 lanes on consecutive rows
  // (row, dk) of element r; recomputed where used rather than kept in registers
#define A_ROW(r) (a_kfast ? (t >> 4) + 16 * (r) : (t & 127))
#define A_K(r) (a_kfast ? (t & 15) : (t >> 7) + 2 * (r))
#define B_ROW(r) (b_kfast ? (t >> 4) + 16 * (r) : (t & 127))
#define B_K(r) (b_kfast ? (t & 15) : (t >> 7) + 2 * (r))
  long aoff[8], boff[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const long m = bm + A_ROW(r), n = bn + B_ROW(r);
    aoff[r] = m < g.M ? g.a_row(m) + A_K(r) * g.ak3 : -1;
    boff[r] = n < g.N ? g.b_col(n) + B_K(r) * g.bk3 : -1;
  }
  // wave-uniform position of the chunk base in (k1, k2, k3) and its offsets
  long k2 = 0, k3 = 0, ka = 0, kb = 0;
  const long nchunks = g.K / KC;

  typename MF::acc_t acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = MF::zero();
  const int wm = (w >> 1) * 64, wn = (w & 1) * 64;
  const int l16 = lane & 15, kq = lane >> 4;
  double ra[8], rb[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    ra[r] = aoff[r] >= 0 ? A[aoff[r]] : 0.0;
    rb[r] = boff[r] >= 0 ? B[boff[r]] : 0.0;
  }
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    sA[0][A_K(r)][A_ROW(r)] = static_cast<T>(ra[r]);
    sB[0][B_K(r)][B_ROW(r)] = static_cast<T>(rb[r]);
  }
  __syncthreads();
  for (long ch = 0; ch < nchunks; ++ch) {
    const int buf = ch & 1;
    const bool more = ch + 1 < nchunks;
    if (more) {
      // advance the base by KC (never past a K3 boundary inside the chunk)
      k3 += KC;
      ka += KC * g.ak3;
      kb += KC * g.bk3;
      if (k3 == g.K3) {
        k3 = 0;
        ka += g.ak2 - g.K3 * g.ak3;
        kb += g.bk2 - g.K3 * g.bk3;
        if (++k2 == g.K2) {
          k2 = 0;
          ka += g.ak1 - g.K2 * g.ak2;
          kb += g.bk1 - g.K2 * g.bk2;
        }
      }
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        ra[r] = aoff[r] >= 0 ? A[aoff[r] + ka] : 0.0;
        rb[r] = boff[r] >= 0 ? B[boff[r] + kb] : 0.0;
      }
    }
#pragma unroll
    for (int s4 = 0; s4 < KC / 4; ++s4) {
      const int kk = 4 * s4 + kq;
      T a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = sA[buf][kk][wm + 16 * i + l16];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = sB[buf][kk][wn + 16 * j + l16];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = MF::mma(a[i], b[j], acc[i][j]);
    }
    if (more) {
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        sA[buf ^ 1][A_K(r)][A_ROW(r)] = static_cast<T>(ra[r]);
        sB[buf ^ 1][B_K(r)][B_ROW(r)] = static_cast<T>(rb[r]);
      }
    }
    __syncthreads();
  }
  // element r of a lane: D[drow(r, lane)][lane % 16]
  double* C = g.c + zb * g.c_batch;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const long n = bn + wn + 16 * j + l16;
    if (n >= g.N) continue;
    double* col = C + g.c_col(n);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const long m = bm + wm + 16 * i + MF::drow(r, lane);
        if (m < g.M) put(g, col + g.c_row(m), static_cast<double>(acc[i][j][r]));
      }
  }
}

#undef A_ROW
#undef A_K
#undef B_ROW
#undef B_K

// One 16-byte global load per lane straight into LDS, lane l of the wave to dst + 16 l bytes
// (dst uniform over the wave); counted by vmcnt alone.
__device__ __forceinline__ void load_lds16(const void* src, void* dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                   (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}

// The FP64 large tiles where both operands come in aligned 16-byte pieces (dma_ok): the
// same 128 x 128 tile, loaded straight to LDS, a chunk ahead.  Every vector instruction
// beside the products takes issue time from the matrix pipe (twelve per FP64 MFMA cost it
// a third of its rate), and staging through registers spent some 120 per 64 products on
// addresses, edge selects and LDS stores; here it is eight loads and their addresses.  A
// k-contiguous operand is kept as rows of 16 k, its 16-byte pieces u at u ^ ((row / 2) & 7)
// (the sixteen rows of one operand read then lie in distinct banks); the other as 16 rows
// of 128.  Rows past the edge read the last one; their results are dropped.  Two buffers,
// one barrier per chunk; the second workgroup of the CU fills the gaps.
// grid (ceil(N/128), ceil(M/128), batch * splits); splits as in gemm_mid.
// PAIR: batch entry z computes C = A1 B1 + A2 B2 with the two levels of A2's rows exchanged
// (row (m1, m2) of A2 at m2 am1 + m1 am2); items: per entry the offsets of A1, B1, A2, B2
// and C.  The summed index runs over the first product, then the second; cper is the number
// of k steps (of 4) that hold anything in each product's last chunk.
// At M = N = K = 16384 (o=32 v=512) 125 ms, 70 TFLOP/s (139 ms through registers).
template <int AK, int BK, bool PAIR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_dma(
    GemmArgs g, const long* __restrict__ items, int splits, long cper, double* __restrict__ part) {
  constexpr int OP = BL * KC;  // doubles of one operand's chunk
  __shared__ double lds[2 * 2 * OP];
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(w);
  const long bm = static_cast<long>(blockIdx.y) * BL, bn = static_cast<long>(blockIdx.x) * BL;
  const long zb = blockIdx.z / splits, zs = blockIdx.z % splits;
  if constexpr (PAIR) items += 5 * zb;
  const double* A = g.a + (PAIR ? items[0] : zb * g.a_batch);
  const double* B = g.b + (PAIR ? items[1] : zb * g.b_batch);
  double* C = g.c + (PAIR ? items[4] : zb * g.c_batch);

  // 16-byte piece t + 256 r of an operand's chunk: k-contiguous: row t/8 + 32 r, piece t%8
  // (the one stored there: t%8 ^ (row/2)&7, which does not depend on r); else rows
  // 2 (t%64), +1 at k = t/64 + 4 r
  const double *pa[4], *pb[4];
  auto set_rows = [&](bool second) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int u = (t & 7) ^ ((t >> 4) & 7), k = (t >> 6) + 4 * r;
      const long ma = AK ? std::min(bm + (t >> 3) + 32 * r, g.M - 1) : std::min(bm + 2 * (t & 63), g.M - 2);
      const long nb = BK ? std::min(bn + (t >> 3) + 32 * r, g.N - 1) : std::min(bn + 2 * (t & 63), g.N - 2);
      pa[r] = A + (PAIR && second ? g.a_row_exchanged(ma) : g.a_row(ma)) + (AK ? 2 * u : k * g.ak3);
      pb[r] = B + g.b_col(nb) + (BK ? 2 * u : k * g.bk3);
    }
  };
  set_rows(false);
  // position of the next chunk to load
  const long c_lo = zs * cper, nchunks = PAIR ? 2 * g.K / KC : std::min(g.K / KC, c_lo + cper) - c_lo;
  long k1, k2, k3;
  div_mod(g.dK3, c_lo * KC, k1, k3);
  div_mod(g.dK2, k1, k1, k2);
  long ka = k1 * g.ak1 + k2 * g.ak2 + k3 * g.ak3, kb = k1 * g.bk1 + k2 * g.bk2 + k3 * g.bk3;
  auto load = [&](int buf) {
    double* d = lds + buf * 2 * OP;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      load_lds16(pa[r] + ka, d + (wv * 64 + 256 * r) * 2);
      load_lds16(pb[r] + kb, d + OP + (wv * 64 + 256 * r) * 2);
    }
    k3 += KC;
    ka += KC * g.ak3;
    kb += KC * g.bk3;
    if (k3 == g.K3) {
      k3 = 0;
      ka += g.ak2 - g.K3 * g.ak3;
      kb += g.bk2 - g.K3 * g.bk3;
      if (++k2 == g.K2) {
        k2 = 0;
        ka += g.ak1 - g.K2 * g.ak2;
        kb += g.bk1 - g.K2 * g.bk2;
      }
    }
  };
  double4_t acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = double4_t{0.0, 0.0, 0.0, 0.0};
  const int wm = (w >> 1) * 64, wn = (w & 1) * 64;
  const int l16 = lane & 15, kq = lane >> 4;
  // operand element (row l16, k = 4 s + kq) of a 16-row tile, relative to the tile
  auto at = [&](int kc, int s) {
    return kc ? l16 * KC + 2 * ((2 * s + (kq >> 1)) ^ (l16 >> 1)) + (kq & 1) : (4 * s + kq) * BL + l16;
  };
  double fa[2][4], fb[2][4];
  auto fread = [&](int q, int buf, int s) {
    const double* sa = lds + buf * 2 * OP + wm * (AK ? KC : 1) + at(AK, s);
    const double* sb = lds + buf * 2 * OP + OP + wn * (BK ? KC : 1) + at(BK, s);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      fa[q][i] = sa[16 * i * (AK ? KC : 1)];
      fb[q][i] = sb[16 * i * (BK ? KC : 1)];
    }
  };
  load(0);
  for (long ch = 0; ch < nchunks; ++ch) {
    const int buf = ch & 1;
    if (PAIR && ch + 1 == g.K / KC) {  // the next chunk is the second product's first
      A = g.a + items[2];
      B = g.b + items[3];
      set_rows(true);
      k2 = k3 = ka = kb = 0;
    }
    // this chunk has landed and every wave is past its reads of the other buffer
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (ch + 1 < nchunks) load(buf ^ 1);
    fread(0, buf, 0);
    // PAIR: the zeros that pad a product's last chunk are skipped by whole steps
    const int steps = PAIR && (ch + 1 == g.K / KC || ch + 1 == nchunks) ? static_cast<int>(cper) : KC / 4;
#pragma unroll
    for (int s = 0; s < KC / 4; ++s) {
      if (PAIR && s >= steps) break;
      if (s + 1 < KC / 4) fread((s + 1) & 1, buf, s + 1);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[s & 1][i], fb[s & 1][j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const long n = bn + wn + 16 * j + l16;
    if (n >= g.N) continue;
    double* col = C + g.c_col(n);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const long m = bm + wm + 16 * i + 4 * r + kq;
        if (m >= g.M) continue;
        if (splits > 1)
          part[(zs * g.M + m) * g.N + n] = acc[i][j][r];
        else
          put(g, col + g.c_row(m), acc[i][j][r]);
      }
  }
}

// Whether every 16-byte piece gemm_dma loads is aligned and inside the operand: pairs run
// along k (k-contiguous: all other strides even) or along the rows (rows contiguous in
// pairs: an even innermost extent, all other strides even).
static bool dma_ok(const void* p, int kfast, long rows2, long r1, long r2, long k1, long k2, long k3, long batch) {
  if (reinterpret_cast<uintptr_t>(p) & 15) return false;
  if ((r1 | k1 | k2 | batch) & 1) return false;
  return kfast ? k3 == 1 && r2 % 2 == 0 : r2 == 1 && rows2 % 2 == 0 && k3 % 2 == 0;
}

static bool dma_ok(const GemmDesc& g, int batch, int a_kfast, int b_kfast) {
  return g.K3 % KC == 0 &&
         dma_ok(g.a, a_kfast, g.M2, g.am1, g.am2, g.ak1, g.ak2, g.ak3, batch > 1 ? g.a_batch : 0) &&
         dma_ok(g.b, b_kfast, g.N2, g.bn1, g.bn2, g.bk1, g.bk2, g.bk3, batch > 1 ? g.b_batch : 0);
}

template <int AK, int BK, bool PAIR = false>
static void launch_dma_k(const GemmArgs& ga, int batch, const long* items, int splits, long cper, double* part,
                         hipStream_t s) {
  const dim3 grid(static_cast<unsigned>((ga.N + BL - 1) / BL), static_cast<unsigned>((ga.M + BL - 1) / BL),
                  static_cast<unsigned>(batch * splits));
  gemm_dma<AK, BK, PAIR><<<grid, 256, 0, s>>>(ga, items, splits, cper, part);
}
static void launch_dma(const GemmArgs& ga, int batch, int a_kfast, int b_kfast, int splits, long cper, double* part,
                       hipStream_t s) {
  if (a_kfast && b_kfast) launch_dma_k<1, 1>(ga, batch, nullptr, splits, cper, part, s);
  else if (a_kfast) launch_dma_k<1, 0>(ga, batch, nullptr, splits, cper, part, s);
  else if (b_kfast) launch_dma_k<0, 1>(ga, batch, nullptr, splits, cper, part, s);
  else launch_dma_k<0, 0>(ga, batch, nullptr, splits, cper, part, s);
}

int run_pairs(const GemmDesc& g, long k_used, int count, const long* items, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || count <= 0) return RI_OK;
  if (g.K <= 0 || k_used > g.K || k_used <= g.K - KC || !dma_ok(g, 1, 1, 1) || g.am1 % 2) {
    set_error("gemm pairs: operands must be k-contiguous and aligned, K a multiple of %d", KC);
    return RI_E_ARG;
  }
  launch_dma_k<1, 1, true>(make_args(g), count, items, 1, (k_used - (g.K - KC) + 3) / 4, nullptr, s);
  return check_launch("gemm_dma");
}

// C(m, n) = alpha * sum_z part[z][m][n] + beta * C(m, n), z in order
__global__ void split_reduce(GemmArgs g, int splits, const double* __restrict__ part) {
  const long idx = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= g.M * g.N) return;
  const long m = idx / g.N, n = idx % g.N;
  double acc = 0.0;
  for (int z = 0; z < splits; ++z) acc += part[z * g.M * g.N + idx];
  put(g, g.c + g.c_row(m) + g.c_col(n), acc);
}

// How a contraction that the large tiles do not take is run.
struct Choice {
  bool small;   // gemm_small (nw waves per tile), else
  bool dma;     // gemm_dma split over k, else gemm_mid
  bool uni;     // gemm_mid's chunks run along the innermost summed level
  int nw, splits;
  long per;     // per split: summed indices (small) or chunks (dma, mid)
  int a_kfast, b_kfast;
};

// Small tiles where 64 x 64 ones, split over k or not, would not give every CU one, or
// would be mostly padding.  The waves per small tile fill the chip first (about two per SIMD), then k is
// split over workgroups while a wave keeps at least four chunks.  The mid tiles are split
// to one round of two workgroups per CU, at least 16 chunks each, unless they give most
// CUs a tile as they are (1000 x 1000 x 1000: 74 us whole, 64 us in two splits and 14 us
// to add them).  Partials take at most 2^26 doubles.  The contractions of a residual at
// o=10 v=100 naux=300 take 1.09 ms (1.67 ms with 64 x 64 tiles of four waves throughout).
// The 128 x 128 tiles loaded straight to LDS come first where splitting k gives them a
// workgroup per CU, at least 32 chunks each (1024 x 1024 over 262144 summed indices: 14.2 ms
// in 64 x 64 tiles, 8.5 ms so).
static Choice choose(const GemmDesc& g, int batch) {
  Choice c{};
  // consecutive threads walk k when the innermost k stride is 1 and the m/n stride is not
  c.a_kfast = (g.ak3 == 1 && g.K3 >= 4 && g.am2 != 1) ? 1 : 0;
  c.b_kfast = (g.bk3 == 1 && g.K3 >= 4 && g.bn2 != 1) ? 1 : 0;
  const long tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  const long tiles_s = ((g.M + SM - 1) / SM) * ((g.N + SM - 1) / SM) * batch;
  const long cap = std::max(1L, (1L << 26) / (g.M * g.N));
  const long tiles_l = ((g.M + BL - 1) / BL) * ((g.N + BL - 1) / BL);
  const long z_l = std::min({512 / tiles_l, g.K / (32 * KC), cap});
  if (batch == 1 && std::min(g.M, g.N) >= BL && tiles_l * z_l >= 256 && dma_ok(g, 1, c.a_kfast, c.b_kfast)) {
    c.dma = true;
    c.per = (g.K / KC + z_l - 1) / z_l;
    c.splits = static_cast<int>((g.K / KC + c.per - 1) / c.per);
    return c;
  }
  const long full = 16L * KC;  // the least k range of a mid split
  c.small = tiles * batch * std::max(1L, batch > 1 ? 1 : std::min(g.K / full, cap)) < 256 || std::min(g.M, g.N) <= SM;
  if (c.small) {
    const long chunks = (g.K + KC - 1) / KC;
    c.nw = tiles_s <= 128 && chunks >= 16 ? 16 : tiles_s <= 256 && chunks >= 8 ? 8 : 4;
    long z = std::min(2048 / (tiles_s * c.nw), chunks / (4 * c.nw));
    z = batch > 1 ? 1 : std::max(1L, std::min(z, cap));
    c.per = ((g.K + z - 1) / z + KC - 1) / KC * KC;
    c.splits = static_cast<int>((g.K + c.per - 1) / c.per);
  } else {
    const long c3n = (g.K3 + KC - 1) / KC;
    c.uni = c3n * KC * 7 <= g.K3 * 8;  // at most 1/7 padding
    const long chunks = c.uni ? g.K / g.K3 * c3n : (g.K + KC - 1) / KC;
    long z = tiles > 192 ? 1 : std::min(512 / tiles, chunks / 16);
    z = batch > 1 ? 1 : std::max(1L, std::min(z, cap));
    c.per = (chunks + z - 1) / z;
    c.splits = static_cast<int>((chunks + c.per - 1) / c.per);
  }
  return c;
}

// Large tiles, whole, when they still give the chip a few workgroups per CU
// (RI_GEMM_LARGE_MIN_TILES overrides the threshold, e.g. to test the path at small sizes).
static bool large_tiles(const GemmDesc& g, int batch) {
  const char* env = getenv("RI_GEMM_LARGE_MIN_TILES");
  const long env_tiles = env ? strtol(env, nullptr, 10) : 0;
  const long min_tiles = env_tiles > 0 ? env_tiles : 256;
  return g.K3 % KC == 0 && ((g.M + BL - 1) / BL) * ((g.N + BL - 1) / BL) * batch >= min_tiles;
}

size_t scratch_doubles(const GemmDesc& g, int batch) {
  if (g.M <= 0 || g.N <= 0 || g.K <= 0 || batch <= 0 || large_tiles(g, batch)) return 0;
  const Choice c = choose(g, batch);
  return c.splits > 1 ? static_cast<size_t>(c.splits) * g.M * g.N : 0;
}

int run(const GemmDesc& g, int batch, double* scratch, size_t scratch_len, hipStream_t s, int prec) {
  if (g.M <= 0 || g.N <= 0 || batch <= 0) return RI_OK;
  if (g.K <= 0) {
    set_error("gemm: K must be positive");
    return RI_E_ARG;
  }
  const GemmArgs ga = make_args(g);
  Choice c = choose(g, batch);
  const int a_kfast = c.a_kfast, b_kfast = c.b_kfast;
  if (large_tiles(g, batch)) {
    dim3 grid(static_cast<unsigned>((g.N + BL - 1) / BL), static_cast<unsigned>((g.M + BL - 1) / BL),
              static_cast<unsigned>(batch));
    if (prec == RI_PREC_FP32) {
      if (a_kfast && b_kfast) gemm_large<float, 1, 1><<<grid, 256, 0, s>>>(ga);
      else if (a_kfast) gemm_large<float, 1, 0><<<grid, 256, 0, s>>>(ga);
      else if (b_kfast) gemm_large<float, 0, 1><<<grid, 256, 0, s>>>(ga);
      else gemm_large<float, 0, 0><<<grid, 256, 0, s>>>(ga);
    } else if (dma_ok(g, batch, a_kfast, b_kfast)) {
      launch_dma(ga, batch, a_kfast, b_kfast, 1, g.K / KC, nullptr, s);
    } else {
      if (a_kfast && b_kfast) gemm_large<double, 1, 1><<<grid, 256, 0, s>>>(ga);
      else if (a_kfast) gemm_large<double, 1, 0><<<grid, 256, 0, s>>>(ga);
      else if (b_kfast) gemm_large<double, 0, 1><<<grid, 256, 0, s>>>(ga);
      else gemm_large<double, 0, 0><<<grid, 256, 0, s>>>(ga);
    }
    return check_launch("gemm_large");
  }
  if (c.splits > 1 && !(scratch && scratch_len >= static_cast<size_t>(c.splits) * g.M * g.N)) {
    c.splits = 1;
    c.per = g.K;  // at least as many chunks
  }
  const int splits = c.splits;
  if (c.dma) {
    launch_dma(ga, 1, a_kfast, b_kfast, splits, c.per, scratch, s);
  } else if (c.small) {
    const long tm = (g.M + SM - 1) / SM, tn = (g.N + SM - 1) / SM;
    const dim3 grid(static_cast<unsigned>(tm * tn), 1, static_cast<unsigned>(batch * splits));
    if (c.nw == 16) gemm_small<16><<<grid, 1024, 0, s>>>(ga, static_cast<int>(tn), splits, c.per, scratch);
    else if (c.nw == 8) gemm_small<8><<<grid, 512, 0, s>>>(ga, static_cast<int>(tn), splits, c.per, scratch);
    else gemm_small<4><<<grid, 256, 0, s>>>(ga, static_cast<int>(tn), splits, c.per, scratch);
  } else {
    const dim3 grid(static_cast<unsigned>((g.N + BN - 1) / BN), static_cast<unsigned>((g.M + BM - 1) / BM),
                    static_cast<unsigned>(batch * splits));
    if (c.uni) gemm_mid<true><<<grid, 512, 0, s>>>(ga, a_kfast, b_kfast, splits, c.per, scratch);
    else gemm_mid<false><<<grid, 512, 0, s>>>(ga, a_kfast, b_kfast, splits, c.per, scratch);
  }
  RI_TRY(check_launch("gemm_f64"));
  if (splits > 1) {
    const long n = g.M * g.N;
    split_reduce<<<static_cast<unsigned>((n + 255) / 256), 256, 0, s>>>(ga, splits, scratch);
    RI_TRY(check_launch("split_reduce"));
  }
  return RI_OK;
}

}  // namespace gemm
}  // namespace ri
